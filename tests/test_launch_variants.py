"""Host-only: every lattice-kernel variant the criterion entry points can dispatch to, every form of the train
step's shared gradient launch, and every kernel that an fp32 convolution takes over haloed operands, is the variant of at least one GPU parity case (tests/variant_cases.py).  The set of
reachable variants is found by asking the library's launch-configuration query for every size it accepts (gradients:
for layers all over the range)."""
import random

import paper_1812_07625_amd as P
from variant_cases import ASG_CASES, BWD_CASES, CTC_CASES, F32_CASES, asg_variant, bwd_variant, ctc_variant, f32_variants


def _reachable(query, classes, lmax_max):
    seen = {}
    for C in classes:
        for L in range(1, lmax_max + 1):
            try:
                v = query(P, C, L)
            except P.W2LError:
                continue
            seen.setdefault(v, (C, L))
    return seen


def test_ctc_cases_cover_every_reachable_variant():
    reach = _reachable(ctc_variant, list(range(1, 260)) + [300, 600, 1000, 4096], 3000)
    assert len(reach) == 24, sorted(reach)          # 3 pair counts x 2 block lengths x 4 table depths
    covered = {ctc_variant(P, c, l) for c, l in CTC_CASES}
    missing = {v: eg for v, eg in reach.items() if v not in covered}
    assert not missing, "variants (pairs per lane, table values, block) with no parity case; e.g. (C, Lmax): %r" % missing


def test_asg_cases_cover_every_reachable_variant():
    reach = _reachable(asg_variant, range(1, 65), 3000)
    covered = {asg_variant(P, c, l) for c, l in ASG_CASES}
    missing = {v: eg for v, eg in reach.items() if v not in covered}
    assert not missing, "variants (positions, class lanes, max threads, block, row values) with no parity case: %r" % missing


def test_gradient_cases_cover_every_reachable_form():
    rng, reach = random.Random(4), {}
    for _ in range(60000):
        unit = rng.choice((64, 64, 16, 8))
        case = (rng.choice((1, 2, 3, 4, 6, 8, 12, 16)), int(2 ** rng.uniform(5, 10.7)), rng.choice((1, 1, 3, 5, 7, 9, 11, 13)),
                max(64, int(2 ** rng.uniform(6, 10.7) / unit) * unit), int(2 ** rng.uniform(6, 11.2) / 64) * 64)
        reach.setdefault(bwd_variant(P, *case), case)
    assert set(reach) == {(0, 0)} | {(d, t) for d in range(1, 7) for t in range(4)}, sorted(reach)
    covered = {bwd_variant(P, *c) for c in BWD_CASES}
    missing = {v: eg for v, eg in reach.items() if v not in covered and v != (0, 0)}
    assert not missing, "forms (data gradient, weight tile) of the shared launch with no parity case; e.g. (B, T, k, cin, cout): %r" % missing


def test_fp32_cases_cover_every_kernel():
    rng, reach = random.Random(6), {}
    for _ in range(12000):
        unit = rng.choice((32, 32, 4))
        wide = lambda most: max(unit, int(2 ** rng.uniform(5.1, most) / unit) * unit)
        case = (int(2 ** rng.uniform(0, 5.3)), int(2 ** rng.uniform(0, 10.7)), wide(10.5), wide(11), rng.choice((1, 3, 5, 7, 9, 11, 13)))
        for p, v in enumerate(f32_variants(P, *case)):
            if v:
                reach.setdefault((p,) + v, case)
    assert set(reach) == {(p, rows, terms, split) for p in (0, 1, 2) for rows, terms in ((64, 0), (64, 1), (128, 1)) for split in (False, True)}, sorted(reach)
    covered = {(p,) + v for c in F32_CASES for p, v in enumerate(f32_variants(P, *c)) if v}
    missing = {v: eg for v, eg in reach.items() if v not in covered}
    assert not missing, "kernels (pass, rows, terms, split) with no parity case; e.g. (B, T, Cin, Cout, k): %r" % missing


def test_launch_config_rejects_what_the_entry_points_reject():
    import pytest
    for bad in ((0, 10), (5000, 10), (29, 0), (29, 3001)):
        with pytest.raises(P.W2LError):
            P.w2l_ctc_launch_config(*bad)
    for bad in ((0, 10), (65, 10), (28, 0), (28, 3001)):
        with pytest.raises(P.W2LError):
            P.w2l_asg_launch_config(*bad)
    net = [dict(k=3, stride=1, cin=16, cout=64, glu=1), dict(k=1, stride=1, cin=32, cout=29, glu=0)]
    for B, T, dtype, layer in ((0, 10, 1, 0), (2, 10, 7, 0), (2, 10, 1, 2), (2, 10, 1, -1)):
        with pytest.raises(P.W2LError):
            P.w2l_train_step_launch_config(net, B, T, dtype, layer)
