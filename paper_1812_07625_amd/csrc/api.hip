// C-ABI entry points for the temporal convolution and the library's bookkeeping calls.
// Argument checks happen here, on the host, before any launch; the kernels assume
// the shapes they are given.
#include "common.h"

namespace w2l {
static thread_local int g_last_hip_error = 0;
void note_hip_error(hipError_t e) { g_last_hip_error = (int)e; }
}  // namespace w2l

using namespace w2l;

extern "C" int w2l_version(void) { return 100; }

extern "C" int w2l_last_hip_error(void) { return g_last_hip_error; }

extern "C" const char* w2l_status_str(int s)
{
    switch (s) {
        case W2L_OK: return "ok";
        case W2L_ERR_NULL: return "null pointer";
        case W2L_ERR_SHAPE: return "bad shape";
        case W2L_ERR_DTYPE: return "bad dtype";
        case W2L_ERR_ALIGN: return "pointer not 16-byte aligned";
        case W2L_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case W2L_ERR_TARGET: return "bad target label or length";
        case W2L_ERR_LAUNCH: return "HIP launch failed";
        default: return "unknown status";
    }
}

namespace {
int check_conv_shape(int B, int T, int Cin, int Cout, int k, int s)
{
    if (B <= 0 || T <= 0 || Cin <= 0 || Cout <= 0 || k <= 0 || s <= 0) return W2L_ERR_SHAPE;
    if ((k & 1) == 0) return W2L_ERR_SHAPE;
    if ((long long)B * T > (1LL << 30) || (long long)k * Cin > (1LL << 30) || (long long)k * Cout > (1LL << 30))
        return W2L_ERR_SHAPE;
    return W2L_OK;
}
bool ws_ok(void* ws, size_t have, size_t need)
{
    if (need == 0) return true;
    return ws && have >= need && (reinterpret_cast<uintptr_t>(ws) & 255u) == 0;
}
}  // namespace

namespace w2l {

bool conv_fwd_is_generic(const ConvDesc& d, int dt) { return !(dt == W2L_BF16 && conv_fwd_mfma_ok(d)); }
bool conv_dgrad_is_generic(const ConvDesc& d, int dt, int dydt) { return !(dt == W2L_BF16 && dydt == W2L_BF16 && conv_dgrad_mfma_ok(d)); }
bool conv_wgrad_is_generic(const ConvDesc& d, int dt, int dydt)
{
    return d.Cout > 32 && !(dt == W2L_BF16 && dydt == W2L_BF16 && conv_wgrad_mfma_ok(d));
}

int conv_fwd(const ConvDesc& d, const void* x, const void* w, const float* bias, void* y, int dt, int ydt,
             hipStream_t st, void* scratch, size_t scratch_bytes)
{
    if (!conv_fwd_is_generic(d, dt)) return conv_fwd_mfma(d, x, w, bias, y, ydt, st, scratch, scratch_bytes);
    return conv_fwd_generic(d, x, w, bias, y, dt, ydt, st, scratch, scratch_bytes);
}

int conv_dgrad(const ConvDesc& d, const void* dy, const void* w, void* dx, int dt, int dydt, hipStream_t st,
               void* scratch, size_t scratch_bytes)
{
    if (!conv_dgrad_is_generic(d, dt, dydt)) return conv_dgrad_mfma(d, dy, w, dx, scratch, scratch_bytes, st);
    return conv_dgrad_generic(d, dy, w, dx, dt, dydt, st, scratch, scratch_bytes);
}

int conv_fwd_parts(const ConvDesc& d, int dt) { return conv_fwd_is_generic(d, dt) ? conv_fwd_generic_parts(d, dt) : conv_fwd_mfma_parts(d); }
int conv_dgrad_parts(const ConvDesc& d, int dt, int dydt)
{
    return conv_dgrad_is_generic(d, dt, dydt) ? conv_dgrad_generic_parts(d, dt) : conv_dgrad_mfma_parts(d);
}
int conv_fwd_partial(const ConvDesc& d, const void* x, const void* w, int dt, float* part, hipStream_t st)
{
    return conv_fwd_is_generic(d, dt) ? conv_fwd_generic_partial(d, x, w, dt, part, st) : conv_fwd_mfma_partial(d, x, w, part, st);
}
int conv_dgrad_partial(const ConvDesc& d, const void* dy, const void* w, int dt, int dydt, float* part, hipStream_t st)
{
    return conv_dgrad_is_generic(d, dt, dydt) ? conv_dgrad_generic_partial(d, dy, w, dt, dydt, part, st) : conv_dgrad_mfma_partial(d, dy, w, part, st);
}
size_t conv_fwd_scratch(const ConvDesc& d, int dt) { return conv_fwd_is_generic(d, dt) ? conv_fwd_generic_scratch(d, dt) : conv_fwd_mfma_scratch(d); }
size_t conv_dgrad_scratch(const ConvDesc& d, int dt, int dydt)
{
    return conv_dgrad_is_generic(d, dt, dydt) ? conv_dgrad_generic_scratch(d, dt) : conv_dgrad_scratch_bytes(d);
}

// scratch of a weight gradient: column sums (in the 256 bytes a channel that a workspace has to have at least: the sums
// take 64), then what the kernel of the shape needs
static size_t wgrad_dbias_scratch(const ConvDesc& d) { return d.Cout <= 32 ? 0 : (size_t)256 * d.Cout; }
size_t conv_wgrad_scratch_bytes(const ConvDesc& d, int dt, int dydt, Runs runs)
{
    const size_t rest = d.Cout <= 32                    ? conv_wgrad_skinny_scratch(d.Cin, d.Cout, d.k)
                        : runs == Runs::WHOLE           ? 0
                        : conv_wgrad_is_generic(d, dt, dydt) ? conv_wgrad_generic_scratch(d, dt, runs == Runs::ALONE)
                                                        : conv_wgrad_mfma_scratch(d);
    return wgrad_dbias_scratch(d) + rest;
}

bool conv_wgrad_fuses_dbias(const ConvDesc& d, int dt, int dydt)
{
    return d.Cout <= 32 || conv_wgrad_is_generic(d, dt, dydt) ||
           (dt == W2L_BF16 && dydt == W2L_BF16 && conv_wgrad_mfma_takes_dbias(d));
}

int conv_wgrad(const ConvDesc& d, const void* x, const void* dy, float* dw, float* dbias, int dt, int dydt,
               int accumulate, void* scratch, size_t scratch_bytes, hipStream_t st, Runs runs)
{
    float* dbias_scratch = static_cast<float*>(scratch);
    unsigned char* rest = static_cast<unsigned char*>(scratch) + wgrad_dbias_scratch(d);
    const size_t rest_bytes = runs != Runs::WHOLE && scratch_bytes > wgrad_dbias_scratch(d) ? scratch_bytes - wgrad_dbias_scratch(d) : 0;
    if (conv_wgrad_is_generic(d, dt, dydt))
        return conv_wgrad_generic(d, x, dy, dw, dbias, dt, dydt, accumulate, st, rest, rest_bytes, runs == Runs::ALONE);
    if (d.Cout <= 32) return conv_wgrad_skinny(d, x, dy, dw, dbias, dt, dydt, accumulate, reinterpret_cast<float*>(rest), st);
    if (dbias && conv_wgrad_fuses_dbias(d, dt, dydt)) return conv_wgrad_mfma(d, x, dy, dw, dbias, accumulate, st, rest, rest_bytes);
    if (dbias) {
        // halo frames hold zeros, so summing every frame of the allocation is the same sum
        const int rc = dbias_reduce(dy, dbias, (long long)d.B * d.y_pitch, d.Cout, accumulate, dbias_scratch, st);
        if (rc) return rc;
    }
    return conv_wgrad_mfma(d, x, dy, dw, nullptr, accumulate, st, rest, rest_bytes);
}

}  // namespace w2l

namespace {
// The C ABI takes dense tensors; the MFMA kernels run fastest on tensors with a zero halo
// around every utterance.  Given workspace, the entry points first copy the window-read
// operand(s) into that layout (one bandwidth-bound pass, a few percent of the GEMM).
constexpr int ABI_HALO = LAYOUT_HALO, ABI_SLACK = LAYOUT_SLACK, ABI_SLACK_ZERO = LAYOUT_SLACK_ZERO;
size_t haloed_bytes(int B, int frames, int C) { return round_up(((size_t)B * (frames + 2 * ABI_HALO) + ABI_SLACK) * C * 2, 256); }
bool stage_fwd(int Cin, int Cout, int k, int s, int dt) { return dt == W2L_BF16 && k > 1 && (k - 1) / 2 <= ABI_HALO && Cin % 64 == 0 && Cout >= 16 && s >= 1; }
bool stage_wgrad(int Cin, int Cout, int k, int s, int dt) { return dt == W2L_BF16 && s == 1 && (k - 1) / 2 <= ABI_HALO && Cin % 8 == 0 && Cout % 8 == 0 && Cout >= 64 && (long long)k * Cin >= 64; }
// The same for fp32, for the kernels of conv_generic.hip: a copy of 16-byte chunks, i.e. of twice the channels in bf16
bool stage_f32(int k, int s, int dt) { return dt == W2L_F32 && k > 1 && (k - 1) / 2 <= ABI_HALO && s == 1; }
bool stage_fwd_f32(int Cin, int k, int s, int dt) { return stage_f32(k, s, dt) && k * Cin % 32 == 0 && Cin % 4 == 0; }
bool stage_dgrad_f32(int Cin, int Cout, int k, int s, int dt) { return stage_f32(k, s, dt) && Cout % 32 == 0 && Cin % 4 == 0; }
bool stage_wgrad_f32(int Cin, int Cout, int k, int s, int dt) { return stage_f32(k, s, dt) && Cin % 4 == 0 && Cout % 4 == 0 && Cout > 32; }
// the geometry that staged operands have
void staged_x(ConvDesc& d) { d.x_pitch = d.T + 2 * ABI_HALO; d.x_halo = ABI_HALO; d.slack = ABI_SLACK; }
void staged_y(ConvDesc& d) { d.y_pitch = d.Tp + 2 * ABI_HALO; d.y_halo = ABI_HALO; d.slack = ABI_SLACK; }
// a strided layer whose stride folds into the channels (fold_stride) is staged as the stride-1 layer it folds to
bool stage_wgrad_folded(int B, int T, int Cin, int Cout, int k, int s, int dt, ConvDesc& f)
{
    if (s <= 1 || !fold_stride(dense_desc(B, T, Cin, Cout, k, s), f) || !stage_wgrad(f.Cin, Cout, f.k, 1, dt)) return false;
    ConvDesc g = f;  // (kernels for any shape know nothing of a folded row's end)
    staged_x(g);
    staged_y(g);
    return conv_wgrad_mfma_takes_dbias(g);
}
}  // namespace

extern "C" size_t w2l_conv1d_fwd_workspace_bytes(int B, int T, int Cin, int Cout, int k, int stride, int dtype)
{
    if (check_conv_shape(B, T, Cin, Cout, k, stride)) return 0;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    if (!valid_dtype(dtype)) return 0;
    const bool f32 = stage_fwd_f32(Cin, k, stride, dtype);
    if (f32) staged_x(d);  // (the layout decides on the kernel, and that on the runs of its reduction)
    return (f32 || stage_fwd(Cin, Cout, k, stride, dtype) ? haloed_bytes(B, T, f32 ? 2 * Cin : Cin) : 0) + conv_fwd_scratch(d, dtype);
}

extern "C" int w2l_conv1d_fwd(const void* x, const void* w, const float* bias, void* y, int B, int T, int Cin,
                              int Cout, int k, int stride, int dtype, int y_dtype, void* workspace,
                              size_t ws_bytes, void* stream)
{
    if (!x || !w || !y) return W2L_ERR_NULL;
    int rc = check_conv_shape(B, T, Cin, Cout, k, stride);
    if (rc) return rc;
    if (!valid_dtype(dtype) || !valid_dtype(y_dtype) || (dtype == W2L_F32 && y_dtype != W2L_F32))
        return W2L_ERR_DTYPE;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y) || (bias && !aligned16(bias))) return W2L_ERR_ALIGN;
    // given a workspace, a bf16 layer takes its haloed copy; a split reduction and an fp32 layer's copy where there is
    // room for all of it
    const bool bf16 = stage_fwd(Cin, Cout, k, stride, dtype), f32 = stage_fwd_f32(Cin, k, stride, dtype);
    const size_t need = w2l_conv1d_fwd_workspace_bytes(B, T, Cin, Cout, k, stride, dtype), least = bf16 ? haloed_bytes(B, T, Cin) : 0;
    const bool all = workspace && ws_ok(workspace, ws_bytes, need);
    if (workspace && !all && !ws_ok(workspace, ws_bytes, least)) return W2L_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    if (workspace && (bf16 || (all && f32))) {
        const int C = f32 ? 2 * Cin : Cin;
        rc = pad_layout_bf16(x, workspace, B, T, C, T + 2 * ABI_HALO, ABI_HALO, ABI_SLACK_ZERO, st);
        if (rc) return rc;
        staged_x(d);
        const size_t copy = haloed_bytes(B, T, C);
        return conv_fwd(d, workspace, w, bias, y, dtype, y_dtype, st, static_cast<unsigned char*>(workspace) + copy, all ? need - copy : 0);
    }
    return conv_fwd(d, x, w, bias, y, dtype, y_dtype, st, all ? workspace : nullptr, all ? need : 0);
}

namespace w2l {
DgradPrep dgrad_prep(int B, int T, int Cin, int Cout, int k, int s, int dt)
{
    DgradPrep p;
    p.Cout = Cout; p.k = k; p.Cin = Cin; p.s = s;
    if (dt != W2L_BF16) return p;
    ConvDesc f = dense_desc(B, T, Cin, Cout, k, s);
    if (s > 1 && !fold_stride(dense_desc(B, T, Cin, Cout, k, s), f)) return p;   // a stride that does not fold
    f.w_cols = 0;
    const int Cp = (Cout + 63) / 64 * 64;
    p.copy_w = s > 1 || Cp != Cout;
    f.Cout = Cp;
    if (f.p > ABI_HALO) return p;
    f.y_pitch = f.Tp + 2 * ABI_HALO;
    f.y_halo = ABI_HALO;
    f.slack = ABI_SLACK;
    if (!conv_dgrad_mfma_ok(f)) return p;
    p.ok = true;
    p.d = f;
    p.dy_bytes = haloed_bytes(B, f.Tp, Cp);
    p.w_bytes = p.copy_w ? round_up((size_t)Cp * f.k * f.Cin * 2, 256) : 0;
    p.split_bytes = round_up(conv_dgrad_scratch_bytes(f), 256);
    p.pair_bytes = round_up(conv_dgrad_pair_bytes(f), 256);
    return p;
}

int conv_dgrad_prepared(const DgradPrep& prep, const void* dy, int dydt, const void* w, void* dx, void* ws, size_t ws_bytes, hipStream_t st)
{
    if (!prep.ok) return W2L_ERR_SHAPE;
    const ConvDesc& f = prep.d;
    unsigned char* base = static_cast<unsigned char*>(ws);
    const size_t split_bytes = ws_bytes >= prep.total() ? prep.split_bytes : prep.pair_bytes;
    // the staging launch also zeroes the split reduction's tickets (the head of its scratch)
    int* const tickets = split_bytes ? reinterpret_cast<int*>(base + prep.dy_bytes + prep.w_bytes) : nullptr;
    int rc = prep_dgrad_dy(dy, dydt, base, f.B, f.Tp, prep.Cout, f.Cout, f.y_pitch, f.y_halo, ABI_SLACK_ZERO, st, tickets,
                           tickets ? (int)(DGRAD_TICKET_BYTES / 4) : 0);
    if (rc) return rc;
    const void* wp = w;
    if (prep.copy_w) {
        rc = prep_dgrad_w(w, base + prep.dy_bytes, prep.Cout, prep.k, prep.Cin, f.Cout, f.k, prep.s, st);
        if (rc) return rc;
        wp = base + prep.dy_bytes;
    }
    return conv_dgrad_mfma(f, base, wp, dx, tickets, split_bytes, st, tickets != nullptr);
}
}  // namespace w2l

extern "C" size_t w2l_conv1d_bwd_data_workspace_bytes(int B, int T, int Cin, int Cout, int k, int stride, int dtype)
{
    if (check_conv_shape(B, T, Cin, Cout, k, stride)) return 0;
    const DgradPrep p = dgrad_prep(B, T, Cin, Cout, k, stride, dtype);
    if (p.ok) return p.total();
    if (!valid_dtype(dtype)) return 0;
    const size_t copy = stage_dgrad_f32(Cin, Cout, k, stride, dtype) ? haloed_bytes(B, T, 2 * Cout) : 0;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    if (copy) staged_y(d);
    const size_t a = conv_dgrad_scratch(d, dtype, dtype), b = dtype == W2L_F32 ? a : conv_dgrad_scratch(d, dtype, W2L_F32);
    return copy + (a > b ? a : b);
}

extern "C" int w2l_conv1d_bwd_data(const void* dy, const void* w, void* dx, int B, int T, int Cin, int Cout,
                                   int k, int stride, int dtype, int dy_dtype, void* workspace, size_t ws_bytes,
                                   void* stream)
{
    if (!dy || !w || !dx) return W2L_ERR_NULL;
    int rc = check_conv_shape(B, T, Cin, Cout, k, stride);
    if (rc) return rc;
    if (!valid_dtype(dtype) || !valid_dtype(dy_dtype) || (dtype == W2L_F32 && dy_dtype != W2L_F32))
        return W2L_ERR_DTYPE;
    if (!aligned16(dy) || !aligned16(w) || !aligned16(dx)) return W2L_ERR_ALIGN;
    const DgradPrep p = dgrad_prep(B, T, Cin, Cout, k, stride, dtype);
    const size_t need = w2l_conv1d_bwd_data_workspace_bytes(B, T, Cin, Cout, k, stride, dtype);
    const bool all = workspace && ws_ok(workspace, ws_bytes, need);
    if (workspace && !all && !ws_ok(workspace, ws_bytes, p.ok ? p.least() : 0)) return W2L_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    // dy staged as bf16 into the haloed layout (channels padded to whole blocks of 64), weights copied padded /
    // with the stride folded where the layer needs it: every bf16 shape the MFMA kernels can be brought to.
    // (A 1x1 layer with bf16 dy and whole channel blocks needs none of it: the kernels read its dense dy as it is.)
    const bool plain_1x1 = k == 1 && stride == 1 && dy_dtype == W2L_BF16 && !p.copy_w;
    if (workspace && p.ok && !plain_1x1) return conv_dgrad_prepared(p, dy, dy_dtype, w, dx, workspace, all ? need : p.least(), st);
    if (all && !p.ok && stage_dgrad_f32(Cin, Cout, k, stride, dtype)) {
        rc = pad_layout_bf16(dy, workspace, B, T, 2 * Cout, T + 2 * ABI_HALO, ABI_HALO, ABI_SLACK_ZERO, st);
        if (rc) return rc;
        staged_y(d);
        const size_t copy = haloed_bytes(B, T, 2 * Cout);
        return conv_dgrad(d, workspace, w, dx, dtype, dy_dtype, st, static_cast<unsigned char*>(workspace) + copy, need - copy);
    }
    return conv_dgrad(d, dy, w, dx, dtype, dy_dtype, st, all ? workspace : nullptr, all ? need : 0);
}

// haloed copies of a bf16 weight gradient's operands
static size_t wgrad_copies(int B, int T, int Cin, int Cout, int k, int stride, int dtype)
{
    ConvDesc f;
    if (stage_wgrad(Cin, Cout, k, stride, dtype)) return haloed_bytes(B, T, Cin) + haloed_bytes(B, T, Cout);
    return stage_wgrad_folded(B, T, Cin, Cout, k, stride, dtype, f) ? haloed_bytes(B, f.T, f.Cin) + haloed_bytes(B, f.T, Cout) : 0;
}

// and an fp32 one's, which are taken where there is room for them
static size_t wgrad_all_copies(int B, int T, int Cin, int Cout, int k, int stride, int dtype)
{
    return wgrad_copies(B, T, Cin, Cout, k, stride, dtype) +
           (stage_wgrad_f32(Cin, Cout, k, stride, dtype) ? haloed_bytes(B, T, 2 * Cin) + haloed_bytes(B, T, 2 * Cout) : 0);
}

// scratch of the kernels: fp32 layers in the layout of their copies
static size_t wgrad_split_scratch(int B, int T, int Cin, int Cout, int k, int stride, int dtype)
{
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    if (stage_wgrad_f32(Cin, Cout, k, stride, dtype)) { staged_x(d); staged_y(d); }
    return conv_wgrad_scratch_bytes(d, dtype, dtype, Runs::ALONE);
}

extern "C" size_t w2l_conv1d_bwd_weight_workspace_bytes(int B, int T, int Cin, int Cout, int k, int stride,
                                                        int dtype)
{
    if (check_conv_shape(B, T, Cin, Cout, k, stride)) return 0;
    if (!valid_dtype(dtype)) return 0;
    return wgrad_split_scratch(B, T, Cin, Cout, k, stride, dtype) + wgrad_all_copies(B, T, Cin, Cout, k, stride, dtype);
}

extern "C" int w2l_conv1d_bwd_weight(const void* x, const void* dy, float* dw, float* dbias, int B, int T,
                                     int Cin, int Cout, int k, int stride, int dtype, int dy_dtype,
                                     int accumulate, void* workspace, size_t ws_bytes, void* stream)
{
    if (!x || !dy || !dw) return W2L_ERR_NULL;
    int rc = check_conv_shape(B, T, Cin, Cout, k, stride);
    if (rc) return rc;
    if (!valid_dtype(dtype) || !valid_dtype(dy_dtype) || (dtype == W2L_F32 && dy_dtype != W2L_F32))
        return W2L_ERR_DTYPE;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dw) || (dbias && !aligned16(dbias))) return W2L_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    // room for the bf16 copies and the bias sums has to be there; a split reduction and fp32 copies where there is room
    // for all of it (an fp32 dy of bf16 operands splits as far as the scratch of a bf16 one takes it)
    const size_t split = wgrad_split_scratch(B, T, Cin, Cout, k, stride, dtype), least = Cout <= 32 ? split : wgrad_dbias_scratch(d);
    const bool all = ws_ok(workspace, ws_bytes, split + wgrad_all_copies(B, T, Cin, Cout, k, stride, dtype));
    const size_t scratch = all ? split : least;
    if (!all && !ws_ok(workspace, ws_bytes, least + wgrad_copies(B, T, Cin, Cout, k, stride, dtype))) return W2L_ERR_WORKSPACE;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    ConvDesc f;
    if (dy_dtype == W2L_BF16 && stage_wgrad_folded(B, T, Cin, Cout, k, stride, dtype, f)) {
        unsigned char* xp = ws + scratch;
        unsigned char* dyp = xp + haloed_bytes(B, f.T, f.Cin);
        rc = pad_layout2_bf16(x, xp, f.Cin, dy, dyp, Cout, B, f.T, f.T + 2 * ABI_HALO, ABI_HALO, ABI_SLACK_ZERO, st);
        if (rc) return rc;
        staged_x(f);
        staged_y(f);
        return conv_wgrad(f, xp, dyp, dw, dbias, dtype, dy_dtype, accumulate, workspace, scratch, st, Runs::ALONE);
    }
    const bool f32 = all && stage_wgrad_f32(Cin, Cout, k, stride, dtype);
    if (f32 || (dy_dtype == W2L_BF16 && stage_wgrad(Cin, Cout, k, stride, dtype))) {
        const int e = f32 ? 2 : 1;
        unsigned char* xp = ws + scratch;
        unsigned char* dyp = xp + haloed_bytes(B, T, e * Cin);
        rc = pad_layout2_bf16(x, xp, e * Cin, dy, dyp, e * Cout, B, T, T + 2 * ABI_HALO, ABI_HALO, ABI_SLACK_ZERO, st);
        if (rc) return rc;
        staged_x(d);
        staged_y(d);
        x = xp;
        dy = dyp;
    }
    return conv_wgrad(d, x, dy, dw, dbias, dtype, dy_dtype, accumulate, workspace, scratch, st, Runs::ALONE);
}

// what a pass launches; rows and terms of the kernels for any shape
static int launch_form(int pass, int B, int T, int Cin, int Cout, int k, int stride, int dtype, int with_workspace, ConvForm* form)
{
    const int rc = check_conv_shape(B, T, Cin, Cout, k, stride);
    if (rc) return rc;
    if (!valid_dtype(dtype)) return W2L_ERR_DTYPE;
    ConvDesc d = dense_desc(B, T, Cin, Cout, k, stride);
    *form = ConvForm{CONV_BF16, 0, 0, 0};
    if (pass == 0) {
        if (!conv_fwd_is_generic(d, dtype)) return W2L_OK;
        if (with_workspace && stage_fwd_f32(Cin, k, stride, dtype)) staged_x(d);
        const size_t scratch = with_workspace ? conv_fwd_scratch(d, dtype) : 0;
        return conv_fwd_generic_form(d, dtype, scratch, form);
    }
    if (pass == 1) {
        if ((with_workspace && dgrad_prep(B, T, Cin, Cout, k, stride, dtype).ok) || !conv_dgrad_is_generic(d, dtype, dtype)) return W2L_OK;
        if (with_workspace && stage_dgrad_f32(Cin, Cout, k, stride, dtype)) staged_y(d);
        const size_t scratch = with_workspace ? conv_dgrad_scratch(d, dtype, dtype) : 0;
        return conv_dgrad_generic_form(d, dtype, scratch, form);
    }
    if (pass != 2) return W2L_ERR_SHAPE;
    if (Cout <= 32) { *form = ConvForm{CONV_NARROW, SKINNY_CHUNKS, 0, 0}; return W2L_OK; }
    if (!conv_wgrad_is_generic(d, dtype, dtype)) return W2L_OK;
    if (stage_wgrad_f32(Cin, Cout, k, stride, dtype)) { staged_x(d); staged_y(d); }
    return conv_wgrad_generic_form(d, dtype, form);
}

extern "C" int w2l_conv1d_launch_config(int pass, int B, int T, int Cin, int Cout, int k, int stride, int dtype, int with_workspace, int* form,
                                        int* splits)
{
    if (!form || !splits) return W2L_ERR_NULL;
    ConvForm f{0, 0, 0, 0};
    const int rc = launch_form(pass, B, T, Cin, Cout, k, stride, dtype, with_workspace, &f);
    if (rc) return rc;
    *form = f.form;
    *splits = f.splits;
    return W2L_OK;
}

extern "C" int w2l_conv1d_launch_tile(int pass, int B, int T, int Cin, int Cout, int k, int stride, int dtype, int with_workspace, int* rows,
                                      int* terms)
{
    if (!rows || !terms) return W2L_ERR_NULL;
    ConvForm f{0, 0, 0, 0};
    const int rc = launch_form(pass, B, T, Cin, Cout, k, stride, dtype, with_workspace, &f);
    if (rc) return rc;
    *rows = f.rows;
    *terms = f.terms;
    return W2L_OK;
}

// ---- measurement aid: what the matrix pipe sustains with nothing else going on -----------
namespace {
typedef __attribute__((ext_vector_type(8))) __bf16 probe_bf16x8;
typedef __attribute__((ext_vector_type(16))) float probe_f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned probe_u32x4;
// RANDOM: operands with random sign and mantissa bits (what real activations look like to the multipliers);
// otherwise small integers.  The part is power-limited, and the power of the matrix pipe depends on how many
// operand bits toggle: the two settings sustain different clocks.
template <bool RANDOM>
__global__ __launch_bounds__(256) void mfma_probe_k(float* out, int iters)
{
    probe_f32x16 acc[8];
    for (int i = 0; i < 8; ++i)
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    probe_u32x4 a[4], b[4];
    unsigned h = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
    for (int q = 0; q < 4; ++q)
        for (int e = 0; e < 4; ++e) {
            h = h * 1664525u + 1013904223u;
            unsigned va = h;
            h = h * 1664525u + 1013904223u;
            unsigned vb = h;
            if (RANDOM) {  // two bf16 per word: random sign and mantissa, magnitude in [0.5, 1)
                va = (va & 0x807f807fu) | 0x3f003f00u;
                vb = (vb & 0x807f807fu) | 0x3f003f00u;
            } else {       // 1.0 and 2.0 everywhere
                va = 0x3f803f80u;
                vb = 0x40004000u;
            }
            a[q][e] = va;
            b[q][e] = vb;
        }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(probe_bf16x8, a[i & 3]),
                                                             __builtin_bit_cast(probe_bf16x8, b[(i + it) & 3]), acc[i], 0, 0, 0);
    }
    float s = 0.f;
    for (int i = 0; i < 8; ++i)
        for (int r = 0; r < 16; ++r) s += acc[i][r];
    out[(size_t)blockIdx.x * 256 + threadIdx.x] = s;
}
}  // namespace

extern "C" int w2l_probe_mfma(float* out, int blocks, int iters, int random_operands, void* stream)
{
    if (!out) return W2L_ERR_NULL;
    if (blocks <= 0 || blocks > 65535 || iters <= 0) return W2L_ERR_SHAPE;
    if (random_operands) hipLaunchKernelGGL(mfma_probe_k<true>, dim3(blocks), dim3(256), 0, (hipStream_t)stream, out, iters);
    else hipLaunchKernelGGL(mfma_probe_k<false>, dim3(blocks), dim3(256), 0, (hipStream_t)stream, out, iters);
    return launch_status();
}
