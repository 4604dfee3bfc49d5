// One training step of the conv-GLU network with the CTC or ASG criterion, ordered by the caller's
// stream with no host synchronisation (paper Sec. 2.3: network forward, criterion,
// backward; the optimiser update is a separate stage of the paper's loop, Sec. 2.4).
//
//   forward   for each layer: conv1d(+bias) -> [GLU]      (pre-GLU and post-GLU kept)
//   criterion log-softmax + CTC, or ASG, on the fp32 logits; yields d loss / d logits directly
//   backward  for each layer, last to first: [GLU bwd] -> wgrad(+dbias) and dgrad, in one launch where their tiles
//             pack, else dgrad on the caller's stream and most wgrads on a helper stream that it waits for
//             (dgrad is skipped for layer 0: the features need no gradient)
#include <mutex>
#include <vector>
#include "common.h"

namespace w2l {
namespace {

// Activations that feed a convolution (GLU outputs h_i, and the gradients dy_i that feed
// dgrad/wgrad) are kept with HALO zero frames around every utterance and SLACK zero frames
// after the last one, so the convolution kernels can read every window as plain memory.
// Tensors only read elementwise (pre-GLU outputs y_i, gradients dh_i) stay dense.
constexpr int HALO = LAYOUT_HALO;
constexpr int SLACK = LAYOUT_SLACK;            // allocated after the last utterance
constexpr int SLACK_ZERO = LAYOUT_SLACK_ZERO;  // of which kept zero

// A helper stream (default priority) for the weight gradients that neither share a launch with their layer's data
// gradient (conv_bwd) nor are shorter than its events (main_wgrad): wgrad of layer i needs
// only dy_i and h_{i-1}, nothing downstream needs it before the step ends, and neither wgrad
// nor dgrad fills all 256 CUs with its tile grid alone -- side by side they do.  Created once
// per device on first use; no device memory is allocated.
struct SideStream {
    hipStream_t stream = nullptr;
    std::vector<hipEvent_t> ready, done;  // per layer: dy_i written (main) / wgrad_i finished (side)
    bool ok = false;
};
SideStream* side_stream(int n_layers)
{
    static std::mutex mu;
    static SideStream per_device[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    SideStream& s = per_device[dev];
    if (!s.stream) {
        if (hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) != hipSuccess) { s.stream = nullptr; return nullptr; }
        s.ok = true;
    }
    while (s.ok && (int)s.ready.size() < n_layers) {
        hipEvent_t a, b;
        if (hipEventCreateWithFlags(&a, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&b, hipEventDisableTiming) != hipSuccess) { s.ok = false; break; }
        s.ready.push_back(a);
        s.done.push_back(b);
    }
    return s.ok ? &s : nullptr;
}

enum { CRIT_CTC = 0, CRIT_ASG = 1 };

struct Plan {
    int n = 0, C = 0, Tlast = 0, tot_stride = 1;
    std::vector<int> Tin, Tout, outch;
    std::vector<int> live;          // channels behind a layer's GLU that the caller's network has (widen)
    std::vector<size_t> pre, post;  // workspace offsets of conv output (dense) and GLU output (haloed) per layer
    size_t dlogits = 0, gdy[3] = {0, 0, 0}, gdh[2] = {0, 0}, ctc = 0, conv = 0, conv0 = 0, dbias = 0, dgs = 0, part = 0, total = 0;
    size_t ctc_bytes = 0, conv_bytes = 0, conv0_bytes = 0, dgs_bytes = 0, part_bytes = 0;  // part: sums of split reductions on the caller's stream
    size_t xfold = 0;      // haloed copy of x with the first layer's stride folded into the channels (0 bytes if unused)
    bool fold0 = false;
    bool cls_glu = false;  // the last layer's data gradient and the GLU backward below it share a launch (class_bwd_glu)
    size_t cls = 0;        // otherwise: operands of that data gradient prepared for the MFMA kernels (its dy is fp32)
    DgradPrep cls_prep;
    std::vector<ConvBwdPlan> bwd;  // per layer: both gradients in one launch, where that can be done
    bool crowded = false;
    bool long_wgrad = false;  // a weight gradient that is worth the helper stream
    int status = W2L_OK;
};

size_t max_of(size_t a, size_t b) { return a > b ? a : b; }
size_t haloed_bytes(int B, int frames, int ch, size_t es) { return ((size_t)B * (frames + 2 * HALO) + SLACK) * ch * es; }

// Geometry of layer i's forward pass (its input is the caller's dense x, i = 0, or the haloed h_{i-1}) and of its
// gradients (dy haloed too where the layer has a GLU).  p.Tin and p.Tout of the layer have to be known.
ConvDesc layer_desc(const Plan& p, const w2l_layer* L, int B, int i)
{
    ConvDesc d = dense_desc(B, p.Tin[i], L[i].cin, L[i].cout, L[i].k, L[i].stride);
    if (i > 0) { d.x_pitch = p.Tin[i] + 2 * HALO; d.x_halo = HALO; d.slack = SLACK; d.x_live = p.live[i - 1]; }
    d.h_live = p.live[i];
    return d;
}
ConvDesc layer_bwd_desc(const Plan& p, const w2l_layer* L, int B, int i)
{
    ConvDesc d = layer_desc(p, L, B, i);
    d.slack = 0;  // a dense dy: nothing may be read past its end
    if (L[i].glu) { d.y_pitch = p.Tout[i] + 2 * HALO; d.y_halo = HALO; d.slack = SLACK; }
    return d;
}
// whether the last layer's data gradient and the GLU backward below it share a launch (class_bwd_glu)
bool class_layer_fused(const Plan& p, const w2l_layer* L, int B, int i, int dtype)
{
    return L[i].k == 1 && L[i].stride == 1 && L[i - 1].glu && class_bwd_glu_ok(B, p.Tin[i] + 2 * HALO, SLACK_ZERO, L[i].cout, L[i].cin, dtype);
}
// A strided bf16 first layer whose weight gradient runs over folded frames, x copied into the haloed layout of its dy: f, its
// geometry.  Only where the matrix kernels take that: the others know nothing of a folded row's end (w_cols).
bool folded_first(const Plan& p, const w2l_layer* L, int n, int B, int dtype, ConvDesc& f)
{
    if (dtype != W2L_BF16 || n < 2 || !L[0].glu || !fold_stride(dense_desc(B, p.Tin[0], L[0].cin, L[0].cout, L[0].k, L[0].stride), f)) return false;
    f.x_pitch = f.y_pitch = p.Tout[0] + 2 * HALO;
    f.x_halo = f.y_halo = HALO;
    f.slack = SLACK;
    return f.p <= HALO && conv_wgrad_mfma_takes_dbias(f);
}
size_t planes_bytes(int parts, size_t values) { return parts > 1 ? parts * values * 4 : 0; }

// Layer 0 has no data gradient to run beside, and the weight gradients of narrow outputs and of little work are shorter
// than the events that a second stream takes (on the device, and on the host, which a small step waits for): these stay
// on the caller's stream (unless the second stream is there anyway: beside a body of 0.57 GFLOP, a head of 0.22 on the
// caller's stream 242 -> 255).  Steps of fp32 networks with four equal body layers, us,
// with their weight gradients on the second stream and on the caller's: 0.13 GFLOP a layer (4 x 100 frames, k = 5,
// 128 -> 256) 235 and 196, 0.26 212..239 and 211, 0.58 250..261 and 260, 1.2 304 and 327; the tiny network (0.016) 94..100 and 85..88.
constexpr double SHORT_WGRAD = 3e8;
bool short_wgrad(const Plan& p, const w2l_layer& l, int i, int B) { return 2.0 * B * p.Tout[i] * l.k * l.cin * l.cout <= SHORT_WGRAD; }
bool main_wgrad(const Plan& p, const w2l_layer& l, int i, int B)
{
    return i == 0 || (!p.crowded && (l.cout <= 32 || (!p.long_wgrad && short_wgrad(p, l, i, B))));
}
// whether a weight gradient may cut its reduction
Runs wgrad_runs(const Plan& p, int dydt) { return p.crowded && dydt == W2L_BF16 ? Runs::WHOLE : Runs::IN_STEP; }
bool same_layer(const w2l_layer& a, const w2l_layer& b) { return a.k == b.k && a.stride == b.stride && a.cin == b.cin && a.cout == b.cout && a.glu == b.glu; }

// real: the caller's layers, of which L may be wider ones (widen)
Plan make_plan(const w2l_layer* L, const w2l_layer* real, int n, int B, int T, int Lmax, int dtype, int criterion)
{
    Plan p;
    p.n = n;
    if (!L) { p.status = W2L_ERR_NULL; return p; }
    if (n <= 0 || n > 1024 || B <= 0 || T <= 0 || Lmax <= 0) { p.status = W2L_ERR_SHAPE; return p; }
    if (!valid_dtype(dtype)) { p.status = W2L_ERR_DTYPE; return p; }
    const size_t es = dtype_size(dtype);
    size_t off = 0, dymax = 0, dhmax = 0;
    int t = T;
    for (int i = 0; i < n; ++i) {
        const w2l_layer& l = L[i];
        if (l.k <= 0 || (l.k & 1) == 0 || l.stride <= 0 || l.cin <= 0 || l.cout <= 0) { p.status = W2L_ERR_SHAPE; return p; }
        if (l.glu && (l.cout & 1)) { p.status = W2L_ERR_SHAPE; return p; }
        if (i == n - 1 && l.glu) { p.status = W2L_ERR_SHAPE; return p; }
        if (i > 0 && l.cin != p.outch[i - 1]) { p.status = W2L_ERR_SHAPE; return p; }
        const int to = out_len(t, l.stride);
        p.Tin.push_back(t);
        p.Tout.push_back(to);
        p.outch.push_back(l.glu ? l.cout / 2 : l.cout);
        p.live.push_back(l.glu ? real[i].cout / 2 : 0);
        p.tot_stride *= l.stride;
        const size_t oes = (i == n - 1) ? 4 : es;  // logits are fp32
        p.pre.push_back(off);
        off += round_up((size_t)B * to * l.cout * oes, 256);
        if (l.glu) {
            p.post.push_back(off);
            off += round_up(haloed_bytes(B, to, l.cout / 2, es), 256);
            const size_t g1 = haloed_bytes(B, to, l.cout, es);
            dymax = g1 > dymax ? g1 : dymax;
        } else if (i < n - 1) {
            // a layer without GLU that feeds another layer: its output is copied into the haloed layout too
            p.post.push_back(off);
            off += round_up(haloed_bytes(B, to, l.cout, es), 256);
        } else {
            p.post.push_back(p.pre.back());
        }
        const size_t g2 = (size_t)B * t * l.cin * es;
        dhmax = g2 > dhmax ? g2 : dhmax;
        ConvDesc dd = dense_desc(B, t, l.cin, l.cout, l.k, l.stride);
        if (i > 0) { dd.x_pitch = t + 2 * HALO; dd.x_halo = HALO; dd.slack = SLACK; }
        if (l.glu) { dd.y_pitch = to + 2 * HALO; dd.y_halo = HALO; dd.slack = SLACK; }
        // sums of split reductions: the geometries that the step's passes will have
        const ConvDesc fd = layer_desc(p, L, B, i), bd = layer_bwd_desc(p, L, B, i);
        p.part_bytes = max_of(p.part_bytes, l.glu ? planes_bytes(conv_fwd_parts(fd, dtype), (size_t)B * to * l.cout) : conv_fwd_scratch(fd, dtype));
        if (i > 0 && i == n - 1) p.cls_glu = class_layer_fused(p, L, B, i, dtype);
        if (i > 0 && !p.cls_glu) {
            const int dydt = i == n - 1 ? W2L_F32 : dtype;
            p.part_bytes = max_of(p.part_bytes, L[i - 1].glu ? planes_bytes(conv_dgrad_parts(bd, dtype, dydt), (size_t)B * t * l.cin)
                                                             : conv_dgrad_scratch(bd, dtype, dydt));
        }
        const bool as_above = i > 1 && same_layer(l, L[i - 1]) && L[i - 2].glu && p.Tin[i] == p.Tin[i - 1];
        p.bwd.push_back(as_above ? p.bwd.back()
                        : i > 0 && i < n - 1 && l.glu && L[i - 1].glu && dtype == W2L_BF16 ? conv_bwd_plan(bd) : ConvBwdPlan{});
        p.crowded = p.crowded || p.bwd.back().crowded;
        // a data gradient of two workgroups per tile: its tickets and the sums of both
        if (i > 0 && L[i - 1].glu) p.dgs_bytes = max_of(p.dgs_bytes, conv_dgrad_pair_bytes(bd));
        t = to;
    }
    // A network with layers whose gradients fill the chip from two streams keeps those streams for all of them, and cuts no
    // bf16 weight gradient: their workgroups take turns with the other stream's as it is (105M step, 8 x 1500 frames, mixed with shared launches and cut: 1.3 % slower).
    if (p.crowded) p.bwd.assign(n, ConvBwdPlan{});
    for (int i = 1; i < n; ++i) p.long_wgrad = p.long_wgrad || (!p.bwd[i].ok && L[i].cout > 32 && !short_wgrad(p, L[i], i, B));
    // scratch of the weight gradients: on the caller's stream, or on the helper stream beside it
    for (int i = 0; i < n; ++i) {
        const w2l_layer& l = L[i];
        const ConvDesc d = i ? layer_bwd_desc(p, L, B, i) : dense_desc(B, T, l.cin, l.cout, l.k, l.stride);
        size_t& bytes = p.bwd[i].ok || main_wgrad(p, l, i, B) ? p.conv0_bytes : p.conv_bytes;
        const int dydt = i == n - 1 ? W2L_F32 : dtype;
        bytes = max_of(bytes, p.bwd[i].ok ? p.bwd[i].wscratch : conv_wgrad_scratch_bytes(d, dtype, dydt, wgrad_runs(p, dydt)));
    }
    p.Tlast = t;
    p.C = L[n - 1].cout;
    p.dlogits = off; off += round_up((size_t)B * p.Tlast * p.C * 4, 256);
    for (int q = 0; q < 3; ++q) { p.gdy[q] = off; off += round_up(dymax, 256); }
    for (int q = 0; q < 2; ++q) { p.gdh[q] = off; off += round_up(dhmax, 256); }
    p.ctc_bytes = criterion == CRIT_ASG ? w2l_asg_workspace_bytes(B, p.Tlast, p.C, Lmax) : w2l_ctc_workspace_bytes(B, p.Tlast, p.C, Lmax);
    if (p.ctc_bytes == 0) { p.status = W2L_ERR_SHAPE; return p; }  // more classes or labels than the criterion takes
    p.ctc = off; off += round_up(p.ctc_bytes, 256);
    p.conv = off; off += round_up(p.conv_bytes, 256);
    // weight gradients on the caller's stream (layer 0's, and those that share a launch with the data gradient) run next
    // to the helper stream's launches: their own scratch
    p.conv0 = off;
    off += round_up(p.conv0_bytes, 256);
    int cmax = 0;
    for (int i = 0; i < n; ++i) cmax = L[i].cout > cmax ? L[i].cout : cmax;
    p.dbias = off; off += round_up((size_t)DBIAS_CHUNKS * cmax * 4, 256);
    p.dgs = off; off += round_up(p.dgs_bytes, 256);
    p.part = off; off += round_up(p.part_bytes, 256);
    {
        // a strided first layer with GLU (its dy is haloed): the weight gradient reads x folded and haloed
        ConvDesc f0;
        p.fold0 = folded_first(p, L, n, B, dtype, f0);
        p.xfold = off;
        if (p.fold0) off += round_up(haloed_bytes(B, f0.T, f0.Cin, es), 256);
    }
    if (n > 1 && !p.cls_glu) {
        // (it rounds the criterion's fp32 gradient to bf16, so only a layer that takes it at the caller's own width does)
        const w2l_layer& ll = L[n - 1];
        if (dgrad_prep(B, p.Tin[n - 1], real[n - 1].cin, ll.cout, ll.k, ll.stride, dtype).ok)
            p.cls_prep = dgrad_prep(B, p.Tin[n - 1], ll.cin, ll.cout, ll.k, ll.stride, dtype);
        p.cls = off;
        if (p.cls_prep.ok) off += round_up(p.cls_prep.total(), 256);
    }
    p.total = off;
    return p;
}

// ---- widths that the matrix kernels do not take --------------------------------------
// The bf16 kernels want whole blocks of 64 output channels for a data gradient and whole chunks of 8 input channels for
// any pass; a network of other widths ran its passes on the fp32 matrix instruction, a sixteenth of the rate.  Such a
// network is stepped as one of wider layers: the halves of those gated layers are rounded up, the weights and biases copied
// with zeros in the new places, and the gradients of the real ones copied out at the end.  Behind every GLU and every GLU
// backward the new channels hold zeros (written as such: 0 times an infinity of a real channel is none), so the real ones'
// sums gain zeros and nothing else.
// Steps, us, k = 7, four layers, 16 x 1600 frames at stride 2: width 40 527 -> 318, 100 559 -> 248, 240 548 -> 300, 500 3853 -> 418,
// 1000 11649 -> 1047; 4 x 800: 40 204 -> 181, 100 230 -> 189, 240 270 -> 198, 500 785 -> 242, 1000 1526 -> 349.
// It is done where the passes that leave the kernels for any shape save more than the two copying launches, their host calls
// and the larger tensors take: 6 us a pass (9 a data gradient) and 15 a GFLOP against 17 us and some room for the error of
// these, from 600 networks of 1 .. 7 layers and widths of 8 .. 1300 (three of which it makes slower, by 2, 3 and 7 %).  Below it:
// two layers of width 100, 4 x 800 frames, 87 -> 91; widths 24 and three of 512, 8 x 1200, 320 -> 326; four of 64 and one of
// 200, 4 x 800, 212 -> 216; tensors beyond the kernels' 32-bit offsets.  Networks with halves below 64 are quick on the other
// kernels, where their data gradients stay (four of width 24, 16 x 1600, 240 -> 318; of 32, k = 13, 284 -> 358; seven of 36,
// 10 x 141, 277 -> 309), so they may take 2.7 times the products (four of 36: 2.57, 570 -> 385; the three named: 5.1, 3.1, 2.8).
// And below 0.2 GFLOP the copies cost more than they give: 1 x 100 frames of width 240 (and too few frames for the kernels)
// 166 -> 170, of 132 (0.03) 117 -> 133.
constexpr double WIDEN_FLOPS = 2e8, WIDEN_PASS = 6.0, WIDEN_DGRAD = 9.0, WIDEN_FLOP = 15e-9, WIDEN_COST = 24.0, WIDEN_MOST = 2.7;
constexpr long long WIDEN_FRAMES = 128;  // what the matrix kernels ask for (conv_fwd_mfma_ok, conv_dgrad_mfma_ok)
struct Widened {
    std::vector<w2l_layer> L;                // empty: nothing to widen
    std::vector<size_t> w, b, dw, db;        // offsets of the copies, for layers that change
    std::vector<char> changed;
    size_t total = 0;
    bool any() const { return !L.empty(); }
};
// Halves of 32 channels more make whole blocks of 64; of 64, also rows of weights that panels divide whatever the taps
// (FAST addressing in the forward pass), which is worth it up to a seventh more channels.
int wide_half(int h)
{
    const int a = (h + 31) / 32 * 32, b = (h + 63) / 64 * 64;
    return b * 7 <= a * 8 ? b : a;
}
// a bf16 step's products, and what its passes on the kernels for any shape count for (us)
struct StepWork { double flops = 0, any = 0; };
StepWork step_work(const w2l_layer* L, const w2l_layer* real, int n, int B, int T)
{
    StepWork v;
    Plan p;
    for (int i = 0, t = T; i < n; ++i) {
        p.Tin.push_back(t);
        p.Tout.push_back(t = out_len(t, L[i].stride));
        p.live.push_back(L[i].glu ? real[i].cout / 2 : 0);
        const double f = 2.0 * B * t * L[i].k * L[i].cin * L[i].cout;
        auto add = [&](bool any, double pass) { v.flops += f; v.any += any ? pass + WIDEN_FLOP * f : 0; };
        const ConvDesc d = layer_desc(p, L, B, i), b = layer_bwd_desc(p, L, B, i);
        const bool last = i == n - 1;
        add(conv_fwd_is_generic(d, W2L_BF16), WIDEN_PASS);
        add(conv_wgrad_is_generic(b, W2L_BF16, last ? W2L_F32 : W2L_BF16), WIDEN_PASS);
        if (i == 0) continue;
        add(last ? !class_layer_fused(p, L, B, i, W2L_BF16) && !dgrad_prep(B, p.Tin[i], real[i].cin, L[i].cout, L[i].k, L[i].stride, W2L_BF16).ok
                 : conv_dgrad_is_generic(b, W2L_BF16, W2L_BF16), WIDEN_DGRAD);
    }
    return v;
}
Widened widen(const w2l_layer* L, int n, int B, int T, int dtype)
{
    Widened v;
    if (!L || n < 2 || n > 1024 || B <= 0 || T <= 0 || dtype != W2L_BF16) return v;
    bool wanted = false;
    double flops = 0;
    int t = T;
    for (int i = 0; i < n; ++i) {
        const w2l_layer& l = L[i];
        if (l.k <= 0 || (l.k & 1) == 0 || l.stride <= 0 || l.cin <= 0 || l.cout <= 0 || l.cout > 1 << 20 || l.cin > 1 << 20) return v;
        if (i < n - 1 ? !l.glu || (l.cout & 1) : l.glu) return v;  // (layers without GLU keep their widths)
        if (i > 0 && l.cin != L[i - 1].cout / 2) return v;
        if (i < n - 1) wanted = wanted || l.cout / 2 % 8 || (i > 0 && l.cout % 64);
        t = out_len(t, l.stride);
        flops += 6.0 * B * t * l.k * l.cin * l.cout;
    }
    if (!wanted || flops < WIDEN_FLOPS || (long long)B * t < WIDEN_FRAMES || L[0].cin % 4) return v;
    std::vector<w2l_layer> wide(L, L + n);
    bool narrow = false;
    for (int i = 0; i < n - 1; ++i) {
        if (L[i].cout % 64) wide[i].cout = 2 * wide_half(L[i].cout / 2);
        wide[i + 1].cin = wide[i].cout / 2;
        narrow = narrow || wide[i].cout < 128;
    }
    const StepWork now = step_work(L, L, n, B, T), then = step_work(wide.data(), L, n, B, T);
    if ((narrow && then.flops > WIDEN_MOST * now.flops) || now.any - then.any < WIDEN_COST) return v;
    v.L = wide;
    for (int i = 0; i < n; ++i) {
        const w2l_layer& l = v.L[i];
        v.changed.push_back(l.cout != L[i].cout || l.cin != L[i].cin);
        const size_t m = (size_t)l.cout * l.k * l.cin;
        auto take = [&](size_t bytes) { const size_t o = v.total; v.total += v.changed[i] ? round_up(bytes, 256) : 0; return o; };
        v.w.push_back(take(m * 2));
        v.b.push_back(take((size_t)l.cout * 4));
        v.dw.push_back(take(m * 4));
        v.db.push_back(take((size_t)l.cout * 4));
    }
    return v;
}

struct WideJob {  // one layer; half = 0: no halves (the classes), all rows stay where they are
    const bf16_t* w; bf16_t* ww; const float* b; float* wb;
    const float* wdw; float* dw; const float* wdb; float* db;
    int cout, half, wcout, whalf, k, cin, wcin, vec;
    unsigned first;  // block of the launch that begins the layer
};
constexpr int WIDE_JOBS = 24, WIDE_ITEMS = 4;  // layers a launch; items of a thread, whose loads are in flight together
struct WideJobs { WideJob j[WIDE_JOBS]; int n; };
__device__ __forceinline__ int wide_row(int co, int half, int whalf) { return co < half || !half ? co : co - half + whalf; }
// row of the layer that row co of the wide one is, or -1
__device__ __forceinline__ int real_row(int co, const WideJob& j)
{
    if (!j.half) return co;
    return co < j.whalf ? (co < j.half ? co : -1) : (co - j.whalf < j.half ? co - j.whalf + j.half : -1);
}
__device__ __forceinline__ const WideJob& wide_job(const WideJobs& a)
{
    int q = 0;
    while (q + 1 < a.n && blockIdx.x >= a.j[q + 1].first) ++q;
    return a.j[q];
}
// Bound by memory: a layer's weights read and the wide ones written (the gradients, the other way), four channels a
// thread and turn where rows start on whole groups of four, one otherwise.
__global__ __launch_bounds__(256) void widen_k(WideJobs a)
{
    const WideJob& j = wide_job(a);
    const unsigned blk = blockIdx.x - j.first;
    if (blk == 0 && j.b)
        for (int c = threadIdx.x; c < j.wcout; c += 256) {
            const int r = real_row(c, j);
            j.wb[c] = r >= 0 ? j.b[r] : 0.f;
        }
    const long long cols = j.wcin / 4, items = (long long)j.wcout * j.k * cols;  // (wcin is a multiple of 4)
#pragma unroll
    for (int u = 0; u < WIDE_ITEMS; ++u) {
        const long long e = ((long long)blk * WIDE_ITEMS + u) * 256 + threadIdx.x;
        if (e >= items) continue;
        const long long line = e / cols;
        const int c = (int)(e - line * cols) * 4, co = (int)(line / j.k), tap = (int)(line - (long long)co * j.k), r = real_row(co, j);
        bf16_t v[4] = {0, 0, 0, 0};
        if (r >= 0) {
            const bf16_t* const src = j.w + ((long long)r * j.k + tap) * j.cin;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (c + q < j.cin) v[q] = src[c + q];
        }
        *reinterpret_cast<uint2*>(j.ww + line * j.wcin + c) =
            make_uint2((unsigned)v[0] | ((unsigned)v[1] << 16), (unsigned)v[2] | ((unsigned)v[3] << 16));
    }
}
__global__ __launch_bounds__(256) void narrow_k(WideJobs a)
{
    const WideJob& j = wide_job(a);
    const unsigned blk = blockIdx.x - j.first;
    if (blk == 0 && j.db)
        for (int c = threadIdx.x; c < j.cout; c += 256) j.db[c] = j.wdb[wide_row(c, j.half, j.whalf)];
    const long long cols = j.cin / j.vec, items = (long long)j.cout * j.k * cols;
#pragma unroll
    for (int u = 0; u < WIDE_ITEMS; ++u) {
        const long long e = ((long long)blk * WIDE_ITEMS + u) * 256 + threadIdx.x;
        if (e >= items) continue;
        const long long line = e / cols;
        const int c = (int)(e - line * cols) * j.vec, co = (int)(line / j.k), tap = (int)(line - (long long)co * j.k);
        const float* const src = j.wdw + ((long long)wide_row(co, j.half, j.whalf) * j.k + tap) * j.wcin + c;
        float* const dst = j.dw + line * j.cin + c;
        if (j.vec == 4) *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(src);
        else *dst = *src;
    }
}
// the layers that change, some to a launch: their weights widened, or their gradients copied out
int launch_wide(bool out, const Widened& v, const w2l_layer* L, int n, const void* const* weights, const float* const* biases,
                float* const* dweights, float* const* dbiases, unsigned char* ws, hipStream_t st)
{
    WideJobs a;
    a.n = 0;
    unsigned blocks = 0;
    for (int i = 0; i <= n; ++i) {
        if (a.n && (i == n || a.n == WIDE_JOBS)) {
            if (out) hipLaunchKernelGGL(narrow_k, dim3(blocks), dim3(256), 0, st, a);
            else hipLaunchKernelGGL(widen_k, dim3(blocks), dim3(256), 0, st, a);
            const int rc = launch_status();
            if (rc) return rc;
            a.n = 0;
            blocks = 0;
        }
        if (i == n || !v.changed[i]) continue;
        WideJob& j = a.j[a.n++];
        j.w = (const bf16_t*)weights[i]; j.ww = (bf16_t*)(ws + v.w[i]);
        j.b = biases[i]; j.wb = (float*)(ws + v.b[i]);
        j.wdw = (const float*)(ws + v.dw[i]); j.dw = dweights[i];
        j.wdb = (const float*)(ws + v.db[i]); j.db = dbiases[i];
        j.cout = L[i].cout; j.half = L[i].glu ? L[i].cout / 2 : 0;
        j.wcout = v.L[i].cout; j.whalf = v.L[i].glu ? v.L[i].cout / 2 : 0;
        j.k = L[i].k; j.cin = L[i].cin; j.wcin = v.L[i].cin;
        j.vec = j.cin % 4 == 0 && aligned16(j.dw) ? 4 : 1;
        j.first = blocks;
        const long long items = out ? (long long)j.cout * j.k * (j.cin / j.vec) : (long long)j.wcout * j.k * (j.wcin / 4);
        blocks += (unsigned)((items + 256 * WIDE_ITEMS - 1) / (256 * WIDE_ITEMS));
    }
    return W2L_OK;
}

}  // namespace
}  // namespace w2l

using namespace w2l;

static size_t step_bytes(const w2l_layer* layers, int n_layers, int B, int T, int Lmax, int dtype, int criterion)
{
    const Widened v = widen(layers, n_layers, B, T, dtype);
    const Plan p = make_plan(v.any() ? v.L.data() : layers, layers, n_layers, B, T, Lmax, dtype, criterion);
    return p.status == W2L_OK ? p.total + v.total : 0;
}

extern "C" size_t w2l_train_step_workspace_bytes(const w2l_layer* layers, int n_layers, int B, int T, int Lmax,
                                                 int dtype)
{
    return step_bytes(layers, n_layers, B, T, Lmax, dtype, CRIT_CTC);
}

extern "C" size_t w2l_train_step_asg_workspace_bytes(const w2l_layer* layers, int n_layers, int B, int T, int Lmax,
                                                     int dtype)
{
    return step_bytes(layers, n_layers, B, T, Lmax, dtype, CRIT_ASG);
}

extern "C" int w2l_train_step_launch_config(const w2l_layer* layers, int n_layers, int B, int T, int dtype, int layer, int* data_form, int* data_runs,
                                            int* weight_tile, int* weight_runs)
{
    if (!layers || !data_form || !data_runs || !weight_tile || !weight_runs) return W2L_ERR_NULL;
    const Widened v = widen(layers, n_layers, B, T, dtype);
    const Plan p = make_plan(v.any() ? v.L.data() : layers, layers, n_layers, B, T, 1, dtype, CRIT_CTC);
    if (p.status) return p.status;
    if (layer < 0 || layer >= n_layers) return W2L_ERR_SHAPE;
    const ConvBwdPlan& b = p.bwd[layer];
    *data_form = b.ok ? 1 + b.dkind : 0;
    *data_runs = b.ok ? b.dparts : 0;
    *weight_tile = b.ok ? b.wtile : 0;
    *weight_runs = b.ok ? b.wsplits : 0;
    return W2L_OK;
}

extern "C" int w2l_train_step_layer_config(const w2l_layer* layers, int n_layers, int B, int T, int dtype, int layer, int* cin, int* cout, int* helper)
{
    if (!layers || !cin || !cout || !helper) return W2L_ERR_NULL;
    const Widened v = widen(layers, n_layers, B, T, dtype);
    const w2l_layer* const L = v.any() ? v.L.data() : layers;
    const Plan p = make_plan(L, layers, n_layers, B, T, 1, dtype, CRIT_CTC);
    if (p.status) return p.status;
    if (layer < 0 || layer >= n_layers) return W2L_ERR_SHAPE;
    *cin = L[layer].cin;
    *cout = L[layer].cout;
    *helper = !p.bwd[layer].ok && !main_wgrad(p, L[layer], layer, B);
    return W2L_OK;
}

// network forward, criterion (CTC on the log-softmax of the output, or ASG on the output itself), backward; arguments checked
static int run_step(const Plan& p, int criterion, const w2l_layer* layers, int n_layers, const void* const* weights, const float* const* biases,
                    float* const* dweights, float* const* dbiases, const void* x, const int* in_len, const int* targets,
                    const int* tgt_len, const float* trans, float* dtrans, float* loss, float* logits, int B, int T, int Lmax, int blank,
                    int dtype, float grad_scale, void* workspace, void* stream)
{
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    hipStream_t st = (hipStream_t)stream;
    const int n = n_layers;
    int rc;

    // the last layer writes the caller's logits where it can (the entry points' alignment), and the criterion reads them there
    float* const z = logits && aligned16(logits) ? logits : reinterpret_cast<float*>(ws + p.pre[n - 1]);

    // ---- network forward: y_i = conv(h_{i-1}) + bias (dense), h_i = GLU(y_i) (haloed)
    const void* h = x;
    for (int i = 0; i < n; ++i) {
        const w2l_layer& l = layers[i];
        const int ydt = (i == n - 1) ? W2L_F32 : dtype;
        const ConvDesc fd = layer_desc(p, layers, B, i);
        float* const part = reinterpret_cast<float*>(ws + p.part);
        const int parts = l.glu ? conv_fwd_parts(fd, dtype) : 1;
        if (parts > 1) {
            rc = conv_fwd_partial(fd, h, weights[i], dtype, part, st);  // the GLU pass adds the parts up
            if (rc) return rc;
            rc = finish_glu_fwd(part, parts, biases[i], ws + p.pre[i], ws + p.post[i], B, p.Tout[i], l.cout, dtype,
                                p.Tout[i] + 2 * HALO, HALO, SLACK_ZERO, st, p.live[i]);
            if (rc) return rc;
            h = ws + p.post[i];
            continue;
        }
        if (l.glu && dtype == W2L_BF16 && conv_fwd_glu_ok(fd)) {
            rc = conv_fwd_glu(fd, h, weights[i], biases[i], ws + p.pre[i], ws + p.post[i], st);  // GLU in the epilogue
            if (rc) return rc;
            h = ws + p.post[i];
            continue;
        }
        rc = conv_fwd(fd, h, weights[i], biases[i], i == n - 1 ? (void*)z : ws + p.pre[i], dtype, ydt, st, part, p.part_bytes);
        if (rc) return rc;
        if (l.glu) {
            rc = glu_fwd_layout(ws + p.pre[i], ws + p.post[i], B, p.Tout[i], l.cout, dtype, p.Tout[i] + 2 * HALO, HALO,
                                SLACK_ZERO, st, p.live[i]);
            if (rc) return rc;
        } else if (i < n - 1) {
            rc = pad_layout(ws + p.pre[i], ws + p.post[i], B, p.Tout[i], l.cout, dtype, p.Tout[i] + 2 * HALO, HALO,
                            SLACK_ZERO, st);
            if (rc) return rc;
        }
        h = ws + p.post[i];
    }
    if (logits && z != logits) {
        hipError_t e = hipMemcpyAsync(logits, z, (size_t)B * p.Tlast * p.C * 4, hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) { note_hip_error(e); return W2L_ERR_LAUNCH; }
    }

    // ---- criterion: frames seen = ceil(in_len / total stride)
    float* dz = reinterpret_cast<float*>(ws + p.dlogits);
    if (criterion == CRIT_ASG) {
        rc = asg_fwd_bwd_strided(z, trans, targets, in_len, tgt_len, loss, dz, dtrans, B, p.Tlast, p.C, Lmax, grad_scale,
                                 ws + p.ctc, p.ctc_bytes, stream, p.tot_stride);
    } else {
        rc = ctc_fwd_bwd_strided(z, 1, targets, in_len, tgt_len, loss, dz, B, p.Tlast, p.C, Lmax, blank, grad_scale,
                                 ws + p.ctc, p.ctc_bytes, stream, p.tot_stride);
    }
    if (rc) return rc;

    // ---- backward.  dh = gradient wrt layer i's output (dense); dy = gradient wrt its conv
    // output: the haloed result of the GLU backward, or dh itself for a layer without GLU.
    // Caller's stream: the dgrad chain.  Where the shapes allow, the data gradient of layer i applies
    // the GLU backward of layer i-1 in its epilogue or in the pass that adds its planes, and writes dy_{i-1} directly;
    // otherwise dh goes to memory and a GLU-backward kernel follows.  A layer's weight gradient (+dbias) is one of
    //   part of that launch     (p.bwd[i].ok and the bias gradient wanted): no event,
    //   on the caller's stream  (main_wgrad): no event,
    //   on the helper stream    (the others): started by ready[i] as soon as its dy exists, done[i] recorded behind it
    //                           and helped[i] set.
    // dy buffers rotate over three slots, so the writer of dy_i only has to wait for the weight gradient of layer i+3,
    // if that one is on the helper stream.
    SideStream* side = side_stream(n);
    auto hip_ok = [&](hipError_t e) { if (e != hipSuccess) { note_hip_error(e); return false; } return true; };
    int on_helper = n;                  // layers n - 1 .. on_helper have a weight gradient on the helper stream, some of them
    std::vector<char> helped(n, 0);     // (these)
    auto wait_wgrad = [&](int layer) {  // main stream waits until that layer's weight gradient has read its dy
        if (layer >= n || !helped[layer]) return true;
        return hip_ok(hipStreamWaitEvent(st, side->done[layer], 0));
    };
    // dh tensors that go to memory alternate between two buffers: a layer without GLU takes dh itself as its dy,
    // so its data gradient must not write the buffer it reads, nor one the helper stream's weight gradient
    // of the layer above still reads (gdh_reader: that layer, or -1)
    void* const gdhb[2] = {ws + p.gdh[0], ws + p.gdh[1]};
    int gdh_reader[2] = {-1, -1};
    int cur = -1;  // the buffer that holds dh; -1: dh is the criterion's gradient
    const void* dh = dz;
    int dh_dt = W2L_F32;
    bool dy_ready = false;  // dy of the current layer was already written by the layer above
    bool tickets = false;   // of the split data gradients: zeroed
    for (int i = n - 1; i >= 0; --i) {
        const w2l_layer& l = layers[i];
        ConvDesc d = layer_bwd_desc(p, layers, B, i);
        const void* dy = dh;
        int dy_dt = dh_dt;
        if (l.glu) {
            void* gdy = ws + p.gdy[i % 3];
            if (!dy_ready) {
                if (!wait_wgrad(i + 3)) return W2L_ERR_LAUNCH;
                rc = glu_bwd_layout(ws + p.pre[i], dh, gdy, B, p.Tout[i], l.cout, dtype, p.Tout[i] + 2 * HALO, HALO,
                                    SLACK_ZERO, st, p.live[i]);
                if (rc) return rc;
            }
            dy = gdy;
            dy_dt = dtype;
        } else if (side && i > 0 && cur >= 0) {
            gdh_reader[cur] = i;
        }
        dy_ready = false;
        const void* xin = (i == 0) ? x : (const void*)(ws + p.post[i - 1]);
        const ConvBwdPlan& both = p.bwd[i];
        if (both.ok && dbiases[i]) {
            // both gradients in one launch: no other stream, nothing to wait for but the last reader of what it writes
            if (both.fused() && !tickets && p.dgs_bytes) {
                rc = zero_dgrad_tickets(reinterpret_cast<int*>(ws + p.dgs), st);
                if (rc) return rc;
            }
            tickets = tickets || both.fused();
            const bool planes = both.dparts > 1, below = both.fused() || planes;
            const int q = (cur == 0) ? 1 : 0;
            if (below ? !wait_wgrad(i + 2) : (gdh_reader[q] >= 0 && !wait_wgrad(gdh_reader[q]))) return W2L_ERR_LAUNCH;
            if (!below) gdh_reader[q] = -1;
            void* const dyb = ws + p.gdy[(i + 2) % 3];
            rc = conv_bwd(both, d, dy, weights[i], xin, ws + p.pre[i - 1], below ? dyb : gdhb[q], dweights[i], dbiases[i],
                          ws + (planes ? p.part : p.dgs), ws + p.conv0, st);
            if (rc) return rc;
            if (planes) {
                rc = finish_glu_bwd(reinterpret_cast<float*>(ws + p.part), both.dparts, ws + p.pre[i - 1], dyb, B, p.Tout[i - 1],
                                    layers[i - 1].cout, dtype, p.Tout[i - 1] + 2 * HALO, HALO, SLACK_ZERO, st, p.live[i - 1]);
                if (rc) return rc;
            }
            dy_ready = below;
            if (!below) {
                dh = gdhb[q];
                cur = q;
                dh_dt = dtype;
            }
            continue;
        }
        // (layer 0's takes the caller's stream next to the helper stream's last launch instead of queueing behind it)
        const bool on_main = main_wgrad(p, l, i, B), on_side = side && !on_main;
        hipStream_t wst = on_side ? side->stream : st;
        if (on_side) {
            if (!hip_ok(hipEventRecord(side->ready[i], st)) || !hip_ok(hipStreamWaitEvent(wst, side->ready[i], 0)))
                return W2L_ERR_LAUNCH;
        }
        if (i == 0 && p.fold0) {
            // the strided first layer as a stride-1 layer over folded frames: x copied (2 MB) into the haloed time
            // layout of dy_0, then the same dense weight-gradient kernel as every other layer, bias gradient included
            ConvDesc f;
            folded_first(p, layers, n, B, dtype, f);
            rc = pad_layout_bf16(x, ws + p.xfold, B, f.T, f.Cin, f.x_pitch, HALO, SLACK_ZERO, st);
            if (rc) return rc;
            d = f;
            xin = ws + p.xfold;
        }
        // The bias gradient comes out of the same launch, except of bf16 layers whose reduction does not walk through
        // haloed frames: there it is a (small, bandwidth-bound) column sum that stays on the caller's stream, which has
        // the shorter chain
        const bool fused_dbias = dbiases[i] && conv_wgrad_fuses_dbias(d, dtype, dy_dt);
        rc = conv_wgrad(d, xin, dy, dweights[i], (fused_dbias || !side) ? dbiases[i] : nullptr, dtype, dy_dt, 0,
                        ws + (on_main ? p.conv0 : p.conv), on_main ? p.conv0_bytes : p.conv_bytes, wst, wgrad_runs(p, dy_dt));
        if (rc) return rc;
        if (on_side) {
            if (!hip_ok(hipEventRecord(side->done[i], wst))) return W2L_ERR_LAUNCH;
            helped[i] = 1;
            on_helper = i;
        }
        if (side && dbiases[i] && !fused_dbias) {
            // halo frames hold zeros, so summing every frame of the allocation is the same sum
            rc = dbias_reduce(dy, dbiases[i], (long long)d.B * d.y_pitch, d.Cout, 0,
                              reinterpret_cast<float*>(ws + p.dbias), st);
            if (rc) return rc;
        }
        if (i > 0 && i == n - 1 && p.cls_glu) {
            rc = class_bwd_glu(dz, weights[i], ws + p.pre[i - 1], ws + p.gdy[(i - 1) % 3], B, p.Tout[i - 1], l.cout, l.cin, dtype,
                               p.Tout[i - 1] + 2 * HALO, HALO, SLACK_ZERO, st, p.live[i - 1]);
            if (rc) return rc;
            dy_ready = true;
            continue;
        }
        if (i > 0) {
            const bool prepared = i == n - 1 && dy_dt == W2L_F32 && p.cls_prep.ok;
            const int parts = layers[i - 1].glu && !prepared ? conv_dgrad_parts(d, dtype, dy_dt) : 1;
            if (parts > 1) {
                float* const part = reinterpret_cast<float*>(ws + p.part);
                if (!wait_wgrad(i + 2)) return W2L_ERR_LAUNCH;  // last reader of the slot dy_{i-1} goes into
                rc = conv_dgrad_partial(d, dy, weights[i], dtype, dy_dt, part, st);
                if (rc) return rc;
                rc = finish_glu_bwd(part, parts, ws + p.pre[i - 1], ws + p.gdy[(i - 1) % 3], B, p.Tout[i - 1],
                                    layers[i - 1].cout, dtype, p.Tout[i - 1] + 2 * HALO, HALO, SLACK_ZERO, st, p.live[i - 1]);
                if (rc) return rc;
                dy_ready = true;
                continue;
            }
            if (layers[i - 1].glu && dtype == W2L_BF16 && dy_dt == W2L_BF16 && conv_dgrad_glu_ok(d)) {
                if (!tickets && p.dgs_bytes) {
                    rc = zero_dgrad_tickets(reinterpret_cast<int*>(ws + p.dgs), st);
                    if (rc) return rc;
                }
                tickets = true;
                if (!wait_wgrad(i + 2)) return W2L_ERR_LAUNCH;
                rc = conv_dgrad_glu(d, dy, weights[i], ws + p.pre[i - 1], ws + p.gdy[(i - 1) % 3], ws + p.dgs, p.dgs_bytes, st);
                if (rc) return rc;
                dy_ready = true;
                continue;
            }
            ConvDesc dd = d;   // dx = dh_{i-1} is written dense
            dd.x_pitch = p.Tin[i];
            dd.x_halo = 0;
            const int q = (cur == 0) ? 1 : 0;
            if (gdh_reader[q] >= 0) {
                if (!wait_wgrad(gdh_reader[q])) return W2L_ERR_LAUNCH;
                gdh_reader[q] = -1;
            }
            if (prepared)  // the criterion's fp32 gradient: cast, pad, MFMA
                rc = conv_dgrad_prepared(p.cls_prep, dy, dy_dt, weights[i], gdhb[q], ws + p.cls, p.cls_prep.total(), st);
            else
                rc = conv_dgrad(dd, dy, weights[i], gdhb[q], dtype, dy_dt, st, ws + p.part, p.part_bytes);
            if (rc) return rc;
            dh = gdhb[q];
            cur = q;
            dh_dt = dtype;
        }
    }
    // join: the side stream is in order, so its last event covers every weight gradient
    if (on_helper < n && !hip_ok(hipStreamWaitEvent(st, side->done[on_helper], 0))) return W2L_ERR_LAUNCH;
    return W2L_OK;
}

static int train_step_impl(int criterion, const w2l_layer* layers, int n_layers, const void* const* weights,
                           const float* const* biases, float* const* dweights, float* const* dbiases, const void* x,
                           const int* in_len, const int* targets, const int* tgt_len, const float* trans, float* dtrans,
                           float* loss, float* logits, int B, int T, int Lmax, int blank, int dtype, float grad_scale,
                           void* workspace, size_t ws_bytes, void* stream)
{
    if (!layers || !weights || !biases || !dweights || !dbiases || !x || !in_len || !targets || !tgt_len || !loss)
        return W2L_ERR_NULL;
    if (criterion == CRIT_ASG && !trans) return W2L_ERR_NULL;
    const Widened v = widen(layers, n_layers, B, T, dtype);
    const w2l_layer* const L = v.any() ? v.L.data() : layers;
    const Plan p = make_plan(L, layers, n_layers, B, T, Lmax, dtype, criterion);
    if (p.status) return p.status;
    if (criterion == CRIT_CTC && (blank < 0 || blank >= p.C)) return W2L_ERR_SHAPE;
    for (int i = 0; i < n_layers; ++i)
        if (!weights[i] || !dweights[i]) return W2L_ERR_NULL;
    if (!workspace || ws_bytes < p.total + v.total || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return W2L_ERR_WORKSPACE;
    if (!aligned16(x)) return W2L_ERR_ALIGN;
    if (!v.any())
        return run_step(p, criterion, L, n_layers, weights, biases, dweights, dbiases, x, in_len, targets, tgt_len, trans, dtrans, loss, logits,
                        B, T, Lmax, blank, dtype, grad_scale, workspace, stream);
    unsigned char* const wide = static_cast<unsigned char*>(workspace) + p.total;
    std::vector<const void*> w(weights, weights + n_layers);
    std::vector<const float*> b(biases, biases + n_layers);
    std::vector<float*> dw(dweights, dweights + n_layers), db(dbiases, dbiases + n_layers);
    for (int i = 0; i < n_layers; ++i) {
        if (!v.changed[i]) continue;
        w[i] = wide + v.w[i];
        dw[i] = reinterpret_cast<float*>(wide + v.dw[i]);
        if (b[i]) b[i] = reinterpret_cast<float*>(wide + v.b[i]);
        if (db[i]) db[i] = reinterpret_cast<float*>(wide + v.db[i]);
    }
    hipStream_t st = (hipStream_t)stream;
    int rc = launch_wide(false, v, layers, n_layers, weights, biases, dweights, dbiases, wide, st);
    if (rc) return rc;
    rc = run_step(p, criterion, L, n_layers, w.data(), b.data(), dw.data(), db.data(), x, in_len, targets, tgt_len, trans, dtrans, loss, logits,
                  B, T, Lmax, blank, dtype, grad_scale, workspace, stream);
    if (rc) return rc;
    return launch_wide(true, v, layers, n_layers, weights, biases, dweights, dbiases, wide, st);
}

extern "C" int w2l_train_step(const w2l_layer* layers, int n_layers, const void* const* weights,
                              const float* const* biases, float* const* dweights, float* const* dbiases,
                              const void* x, const int* in_len, const int* targets, const int* tgt_len,
                              float* loss, float* logits, int B, int T, int Lmax, int blank, int dtype,
                              float grad_scale, void* workspace, size_t ws_bytes, void* stream)
{
    return train_step_impl(CRIT_CTC, layers, n_layers, weights, biases, dweights, dbiases, x, in_len, targets, tgt_len,
                           nullptr, nullptr, loss, logits, B, T, Lmax, blank, dtype, grad_scale, workspace, ws_bytes, stream);
}

extern "C" int w2l_train_step_asg(const w2l_layer* layers, int n_layers, const void* const* weights,
                                  const float* const* biases, float* const* dweights, float* const* dbiases,
                                  const void* x, const int* in_len, const int* targets, const int* tgt_len,
                                  const float* trans, float* dtrans, float* loss, float* logits, int B, int T, int Lmax,
                                  int dtype, float grad_scale, void* workspace, size_t ws_bytes, void* stream)
{
    return train_step_impl(CRIT_ASG, layers, n_layers, weights, biases, dweights, dbiases, x, in_len, targets, tgt_len,
                           trans, dtrans, loss, logits, B, T, Lmax, 0, dtype, grad_scale, workspace, ws_bytes, stream);
}
