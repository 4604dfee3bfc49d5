// Temporal-convolution kernels for any shape and type, on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation).
//
// (fp32 tensors in the train step's layout: their exact split into bf16 values, gemm_split_k.)
//
// These take every problem that the bf16 kernels do not: fp32 tensors, channel counts that are not multiples of 8,
// strides that do not fold, calls without workspace.  bf16 operands are widened on their way into LDS, so their
// products stay exact.  Each of the three passes is the GEMM C[m,n] = sum_r A(m,r) * B(r,n) over the convolution's
// own tensors -- no unfolded copy of the input is made:
//   fwd   y[b,t',co]  = bias[co] + sum_{j,ci} w[co,j,ci] * x[b, s t' + j - p, ci]
//   dgrad dx[b,t,ci]  = sum_{j,co} w[co,j,ci] * dy[b,(t+p-j)/s,co]   (divisible, in range)
//   wgrad dw[co,j,ci] = sum_{b,t'} dy[b,t',co] * x[b, s t' + j - p, ci]
// (the paper names the op in Sec. 2.3 without a formula).
//
// What bounds them: the fp32 matrix pipe, 256 FLOP per cycle and CU, a sixteenth of the bf16 rate.  A wavefront
// multiplies for 64 cycles on one dword per lane of either operand, so the operands' way costs little as long as it
// costs no vector instructions (fp32 matrix instructions run on the vector units), and what is worth something is
// work for all 1024 SIMDs: the reduction is split over workgroups (any_plan) whose fp32 sums a finishing pass adds in
// a fixed order -- inside the train step that pass is the layer's GLU, which would be launched anyway.
// Measured inside the train step of the 10M-parameter network in fp32 (4 x 400 frames, k = 11, 256 -> 512, 4.6 GFLOP
// a pass; 30 us at the pipe's rate), before (64 x 64 tiles of scalar FMAs, one workgroup per tile) and now: forward
// 476 -> 47 us, data gradient 1190 -> 64, weight gradient 325 -> 66 (the last two side by side), step 11.4 -> 1.00 ms,
// and 0.86 ms with gemm_split_k.
#include <type_traits>
#include "common.h"

namespace w2l {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4a __attribute__((ext_vector_type(4)));

constexpr int TILE = 64, PANEL = 32;  // a workgroup's outputs in either direction; steps of the reduction per panel

// ---- operands ------------------------------------------------------------------------
// A line is a run of memory: element c of line i is base[off + c], real where lo <= c < hi and zero elsewhere.
// K_LINES: the lines are the rows (columns) of the output and c runs along the reduction; otherwise the lines are
// the steps of the reduction and c runs along the output.
struct Line { long long off; int lo, hi; };
__device__ __forceinline__ Line no_line() { return Line{0, 0, 0}; }

// What an unpredicated panel (DmaPanel, FAST) needs of an operand's lines beyond whole chunks: a lane keeps its offset
// from the first line of its tile or panel in 32 bits of bytes, so they have to lie within 2 GB of each other.
inline bool near_lines(long long elements) { return elements < (1LL << 29) - TILE; }
// Frames between the first and the last of a tile's rows at most; row r: frame step * (r % count) of utterance r / count
inline long long row_reach(int count, int step, int pitch, int rows = TILE)
{
    const long long cross = (rows - 2LL + count) / count, gap = pitch - (long long)count * step;  // utterance ends met, and what each adds
    const long long a = (rows - 1LL) * step + cross * (gap > 0 ? gap : 0), b = cross * pitch + (count - 1LL) * step;
    return a < b ? a : b;
}

template <typename T>
struct XWindow {  // fwd A: m = (b,t') -> x[b, s t' - p ..], r = (j,ci)
    static constexpr bool K_LINES = true, PHASED = false;
    typedef T type;
    const T* base; int M, T_, Tp, Cin, k, s, p, pitch, halo;
    // every line starts and ends on a 16-byte chunk of fp32
    bool chunks() const { return aligned16(base) && Cin % 4 == 0; }
    bool fast() const { return chunks() && k * Cin % 32 == 0 && (p == 0 || halo >= p) && near_lines(row_reach(Tp, s, pitch) * Cin); }
    bool tall() const { return near_lines(row_reach(Tp, s, pitch, 2 * TILE) * Cin + 2 * TILE); }  // as near over 128 rows
    __device__ __forceinline__ long long fast_line(int m) const { return line(m < M ? m : M - 1).off; }
    __device__ __forceinline__ Line line(int m) const
    {
        if (m >= M) return no_line();
        const int b = (unsigned)m / (unsigned)Tp, t0 = s * (m - b * Tp) - p, last = T_ - t0;
        return Line{((long long)b * pitch + halo + t0) * Cin, (t0 < 0 ? -t0 : 0) * Cin, (last < k ? last : k) * Cin};
    }
};
template <typename T>
struct WRows {  // fwd B: n = co -> w[co], r = (j,ci)
    static constexpr bool K_LINES = true;
    typedef T type;
    const T* base; int N, KC;
    bool chunks() const { return aligned16(base) && KC % 4 == 0; }
    bool fast() const { return chunks() && KC % 32 == 0 && near_lines((TILE - 1LL) * KC); }
    __device__ __forceinline__ long long fast_line(int n) const { return (long long)(n < N ? n : N - 1) * KC; }
    __device__ __forceinline__ Line line(int n) const { return n < N ? Line{(long long)n * KC, 0, KC} : no_line(); }
};
// The frames t of the data gradient with the same (t + p) mod s = ph meet the same taps j = ph, ph + s, .. (taps of
// them) and read taps consecutive frames of dy, the last tap first: each such phase is a stride-1 problem of its own.
// One launch takes all of them, a phase per index of grid.z (phase f: the frames f, f + s, ..; phases without taps store
// zeros), however wide the stride.
struct Phase { int ph, taps, first, count; };  // first frame of the phase, frames per utterance
__host__ __device__ inline Phase phase_of(int ph, int T, int k, int s, int p)
{
    Phase q;
    q.ph = ph;
    q.taps = ph < k ? (k - ph + s - 1) / s : 0;
    q.first = ((ph - p) % s + s) % s;
    q.count = q.first < T ? (T - q.first + s - 1) / s : 0;
    return q;
}
template <typename T>
struct DyWindow {  // dgrad A: m = (b, frame of the phase) -> its dy frames, r = (q,co), q-th frame <-> tap ph + s (taps-1-q)
    static constexpr bool K_LINES = true, PHASED = true;
    typedef T type;
    const T* base; int B, T_, Tp, Cout, k, s, p, pitch, halo, f0; Phase q;  // f0: phase of grid.z = 0
    static __host__ __device__ Phase phase(int f, int T_, int k, int s, int p) { return phase_of((int)(((long long)f + p) % s), T_, k, s, p); }
    bool chunks() const { return aligned16(base) && Cout % 4 == 0; }
    bool fast() const { return chunks() && s == 1 && Cout % 32 == 0 && (p == 0 || halo >= p) && near_lines(row_reach(q.count, 1, pitch) * Cout); }
    bool tall() const { return near_lines(row_reach(q.count, 1, pitch, 2 * TILE) * Cout + 2 * TILE); }
    __device__ __forceinline__ long long fast_line(int m) const { return line(m < B * q.count ? m : B * q.count - 1).off; }
    __device__ __forceinline__ Line line(int m) const
    {
        if (m >= B * q.count) return no_line();
        const int b = (unsigned)m / (unsigned)q.count, t = q.first + s * (m - b * q.count);
        const int u0 = (t + p - q.ph) / s - q.taps + 1, last = Tp - u0;
        return Line{((long long)b * pitch + halo + u0) * Cout, (u0 < 0 ? -u0 : 0) * Cout, (last < q.taps ? last : q.taps) * Cout};
    }
};
template <typename T>
struct WCols {  // dgrad B: r = (q,co) -> w[co, tap], n = ci
    static constexpr bool K_LINES = false;
    typedef T type;
    const T* base; int Cin, Cout, k, s; Phase q;
    // every line starts and ends on a 16-byte chunk of fp32
    bool chunks() const { return aligned16(base) && Cin % 4 == 0; }
    // (the 32 lines of a panel lie in one tap)
    bool fast() const { return chunks() && s == 1 && Cout % 32 == 0 && near_lines((PANEL - 1LL) * k * Cin); }
    __device__ __forceinline__ long long fast_base(int r) const { return line(r).off; }
    __device__ __forceinline__ int fast_pitch() const { return k * Cin; }
    __device__ __forceinline__ int width() const { return Cin; }
    __device__ __forceinline__ Line line(int r) const
    {
        const int t = (unsigned)r / (unsigned)Cout, co = r - t * Cout;
        return Line{((long long)co * k + q.ph + s * (q.taps - 1 - t)) * Cin, 0, Cin};
    }
};
template <typename T>
struct DyT {  // wgrad A: r = (b,t') -> dy[b,t'], m = co
    static constexpr bool K_LINES = false, PHASED = false;
    typedef T type;
    const T* base; int Tp, Cout, pitch, halo;
    bool chunks() const { return aligned16(base) && Cout % 4 == 0; }
    // (the walk of wgrad_t through the frames of a haloed layout; a grid holds fewer than 2^22 rows of dw, so these lines
    // are near)
    bool fast() const { return chunks(); }
    bool tall() const { return true; }
    __device__ __forceinline__ long long fast_base(int r) const { return (long long)(halo + r) * Cout; }
    __device__ __forceinline__ int fast_pitch() const { return Cout; }
    __device__ __forceinline__ int width() const { return Cout; }
    __device__ __forceinline__ Line line(int r) const
    {
        const int b = (unsigned)r / (unsigned)Tp, tp = r - b * Tp;
        return Line{((long long)b * pitch + halo + tp) * Cout, 0, Cout};
    }
};
template <typename T>
struct XShift {  // wgrad B: r = (b,t') -> x[b, s t' - p ..], n = (j,ci)
    static constexpr bool K_LINES = false;
    typedef T type;
    const T* base; int T_, Tp, Cin, k, s, p, pitch, halo;
    // every line starts and ends on a 16-byte chunk of fp32
    bool chunks() const { return aligned16(base) && Cin % 4 == 0; }
    bool fast() const { return chunks() && near_lines((PANEL - 1LL) * Cin); }
    __device__ __forceinline__ long long fast_base(int r) const { return (long long)(halo - p + r) * Cin; }
    __device__ __forceinline__ int fast_pitch() const { return Cin; }
    __device__ __forceinline__ int width() const { return k * Cin; }
    __device__ __forceinline__ Line line(int r) const
    {
        const int b = (unsigned)r / (unsigned)Tp, t0 = s * (r - b * Tp) - p, last = T_ - t0;
        return Line{((long long)b * pitch + halo + t0) * Cin, (t0 < 0 ? -t0 : 0) * Cin, (last < k ? last : k) * Cin};
    }
};

// ---- outputs -------------------------------------------------------------------------
// row(m) = element offset of output row m; sums of split z go one plane further each
template <typename T>
struct StoreRows {  // m = (b, i): frame first + step * i of utterance b
    T* y; const float* bias; int N, count, first, step, pitch, halo; long long plane;
    __device__ __forceinline__ long long row(int m) const
    {
        const int b = (unsigned)m / (unsigned)count;
        return ((long long)b * pitch + halo + first + (long long)step * (m - b * count)) * N;
    }
    __device__ __forceinline__ float add(int n) const { return bias ? bias[n] : 0.f; }
    __device__ __forceinline__ void store(long long i, float v, int split) const { Elem<T>::store(y + split * plane, (size_t)i, v); }
};
struct StoreAcc {
    float* d; int N, accumulate; long long plane;
    __device__ __forceinline__ long long row(int m) const { return (long long)m * N; }
    __device__ __forceinline__ float add(int) const { return 0.f; }
    __device__ __forceinline__ void store(long long i, float v, int split) const
    {
        float* q = d + split * plane + i;
        *q = accumulate ? *q + v : v;
    }
};

// the phase of a strided data gradient that the workgroup belongs to: its operands, rows and reduction
template <class OA, class OB, class EP>
__device__ __forceinline__ void take_phase(OA& oa, OB& ob, EP& ep, int z, int& M, int& R)
{
    if constexpr (OA::PHASED) {
        if (oa.s > 1) {
            const Phase q = OA::phase(oa.f0 + z, oa.T_, oa.k, oa.s, oa.p);
            oa.q = q;
            ob.q = q;
            ep.first = q.first;
            ep.count = q.count;
            M = oa.B * q.count;
            R = q.taps * oa.Cout;
        }
    }
}

// four consecutive elements from c on
template <typename T>
__device__ __forceinline__ void load4(const T* base, const Line& l, int c, float (&v)[4])
{
    const T* q = base + l.off + c;
    if (c >= l.lo && c + 4 <= l.hi) {
        if constexpr (sizeof(T) == 4) {
            const f32x4u u = *reinterpret_cast<const f32x4u*>(q);  // lines start at any element: dword alignment
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = u[e];
        } else {
            if ((reinterpret_cast<uintptr_t>(q) & 7) == 0) {
                const uint2 u = *reinterpret_cast<const uint2*>(q);
                v[0] = __uint_as_float(u.x << 16);
                v[1] = __uint_as_float(u.x & 0xffff0000u);
                v[2] = __uint_as_float(u.y << 16);
                v[3] = __uint_as_float(u.y & 0xffff0000u);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = Elem<T>::load(q, e);
            }
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (c + e >= l.lo && c + e < l.hi) ? Elem<T>::load(q, e) : 0.f;
    }
}

// One operand's share of a panel: W rows of the output by BK steps of the reduction.
template <class OP, int W, int BK>
struct AnyPanel {
    static constexpr bool KL = OP::K_LINES;
    // LDS image: [W][BK + 4] (a row pitch of 36 dwords starts 16 consecutive rows on distinct banks) or
    // [BK][W + 8] (the two halves of a wavefront read lines four apart: 32 banks apart)
    static constexpr int PITCH = KL ? BK + 4 : W + 8;
    static constexpr int FLOATS = KL ? W * PITCH : BK * PITCH;
    static constexpr int CPL = (KL ? BK : W) / 4;  // 4-element chunks per line
    static constexpr int LPP = 256 / CPL;          // lines that the workgroup's threads cover at once
    static constexpr int NC = W * BK / 1024;       // chunks per thread
    static_assert(W * BK % 1024 == 0 && 256 % CPL == 0, "a panel splits evenly over 256 threads");
    Line ln[KL ? NC : 1];
    float v[NC][4];
    static __device__ __forceinline__ int l_of(int i) { return threadIdx.x / CPL + i * LPP; }
    static __device__ __forceinline__ int c_of() { return threadIdx.x % CPL * 4; }
    __device__ __forceinline__ void init(const OP& op, int w0, int r_end)
    {
        if constexpr (KL) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                ln[i] = op.line(w0 + l_of(i));
                if (ln[i].hi > r_end) ln[i].hi = r_end;
            }
        }
    }
    __device__ __forceinline__ void load(const OP& op, int w0, int r0, int r_end)
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            if constexpr (KL) load4(op.base, ln[i], r0 + c_of(), v[i]);
            else {
                const int r = r0 + l_of(i);
                const Line l = r < r_end ? op.line(r) : no_line();
                load4(op.base, l, w0 + c_of(), v[i]);
            }
        }
    }
    __device__ __forceinline__ void store(float* lds) const
    {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const f32x4a u = {v[i][0], v[i][1], v[i][2], v[i][3]};
            *reinterpret_cast<f32x4a*>(lds + l_of(i) * PITCH + c_of()) = u;
        }
    }
    // Operand registers of the 32 rows from row w on, for the four instructions of reduction steps r .. r + 7:
    // instruction q takes step r + q from lanes 0..31 and step r + 4 + q from lanes 32..63, so that a lane's four values
    // are consecutive in a [W][BK] image.
    static __device__ __forceinline__ void frags(const float* lds, int w, int r, int lane, float (&f)[4])
    {
        const int c = lane & 31, h = lane >> 5;
        if constexpr (KL) {
            const f32x4a u = *reinterpret_cast<const f32x4a*>(lds + (w + c) * PITCH + r + 4 * h);
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = u[q];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = lds[(r + 4 * h + q) * PITCH + w + c];
        }
    }
};

// TILE x TILE outputs per workgroup of four wavefronts (2 x 2), 32 x 32 each.  grid.z = phases * splits.  colsum (A by
// reduction lines, i.e. the weight gradient): the sums of A over the reduction -- the bias gradient -- from the values
// that pass through the first column of workgroups anyway.
template <class OA, class OB, class EP>
__global__ __launch_bounds__(256, 4) void gemm_any_k(OA oa, OB ob, EP ep, int M, int N, int R, int per, int splits, float* colsum, int colsum_acc)
{
    constexpr int BM = TILE, BN = TILE, BK = PANEL;
    using PA = AnyPanel<OA, BM, BK>;
    using PB = AnyPanel<OB, BN, BK>;
    constexpr int STAGE = PA::FLOATS + PB::FLOATS;
    __shared__ __align__(16) float lds[2 * STAGE];
    const int split = blockIdx.z % splits;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    take_phase(oa, ob, ep, blockIdx.z / splits, M, R);
    if (OA::PHASED && m0 >= M) return;  // (phases differ by a frame per utterance)
    const int r_begin = split * per, r_end = R < r_begin + per ? R : r_begin + per;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
    const bool sum_a = !PA::KL && colsum && blockIdx.x == 0;
    PA pa;
    PB pb;
    pa.init(oa, m0, r_end);
    pb.init(ob, n0, r_end);
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    float asum[4] = {0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int r0) {
        pa.load(oa, m0, r0, r_end);
        pb.load(ob, n0, r0, r_end);
    };
    auto put = [&](float* q) {
        pa.store(q);
        pb.store(q + PA::FLOATS);
        if (sum_a) {
#pragma unroll
            for (int i = 0; i < PA::NC; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) asum[e] += pa.v[i][e];
        }
    };
    const int steps = r_end > r_begin ? (r_end - r_begin + BK - 1) / BK : 0;
    if (steps > 0) {
        fetch(r_begin);
        put(lds);
    }
    __syncthreads();
    for (int st = 0; st < steps; ++st) {
        if (st + 1 < steps) fetch(r_begin + (st + 1) * BK);
        const float* la = lds + (st & 1) * STAGE;
        const float* lb = la + PA::FLOATS;
#pragma unroll
        for (int r = 0; r < BK; r += 8) {
            float fa[4], fb[4];
            PA::frags(la, wm, r, lane, fa);
            PB::frags(lb, wn, r, lane, fb);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q], fb[q], acc, 0, 0, 0);
        }
        if (st + 1 < steps) put(lds + ((st + 1) & 1) * STAGE);
        __syncthreads();
    }
    const int n = n0 + wn + (lane & 31);
    const float addn = n < N ? ep.add(n) : 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int m = m0 + wm + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (m < M && n < N) ep.store(ep.row(m) + n, acc[e] + addn, split);
    }
    if (sum_a) {  // thread (line, column chunk) partial sums, added over the lines in order
        float* red = lds;  // every wavefront is past its last read of the panels
#pragma unroll
        for (int e = 0; e < 4; ++e) red[PA::l_of(0) * BM + PA::c_of() + e] = asum[e];
        __syncthreads();
        for (int c = threadIdx.x; c < BM; c += 256) {
            float v = 0.f;
            for (int l = 0; l < PA::LPP; ++l) v += red[l * BM + c];
            const int m = m0 + c;
            if (m < M) {
                float* q = colsum + (long long)split * M + m;
                *q = colsum_acc ? *q + v : v;
            }
        }
    }
}

// ---- fp32 operands in 16-byte chunks: global -> LDS directly -------------------------
// Where every line starts and ends on a multiple of four elements, a panel needs no registers on its way: each lane
// asks for its 16-byte chunk (or for a block of zeros), the chunk lands in LDS at 16 bytes times the lane.  The loads
// of a panel and the LDS reads of the next eight steps are placed between the matrix instructions (64 cycles each,
// so a dozen other instructions pass in the shadow of one): a wavefront alone on its SIMD keeps the pipe busy.
// FAST: tensors in the haloed time layout (the train step's, and what the entry points stage).  Every window is then
// plain memory: a lane's offset from the first line of its panel never changes and the loads cost no vector
// instruction at all, which counts, because fp32 matrix instructions run on the vector units (the two do not overlap).
// (The weight gradient then walks through the frames between two utterances as well: dy is zero there, and the x that
// it would meet is taken for zero too -- in the panels that hold such frames -- or an infinite x near an utterance's
// end would turn up as a NaN in taps that never see it.)
__device__ __align__(16) const float g_zero_chunk[4] = {0.f, 0.f, 0.f, 0.f};
typedef __attribute__((address_space(3))) unsigned char lds_byte;

__device__ __forceinline__ void dma16(const void* g, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_addr) : "memory");
}

// address = uniform 64-bit base + per-lane 32-bit byte offset
__device__ __forceinline__ void dma16s(unsigned voff, const void* sbase, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

template <class OP, int W, bool FAST>
struct DmaPanel {
    static constexpr int BK = PANEL;
    static constexpr bool KL = OP::K_LINES;
    // [W][32] with the 16-byte chunks of a row permuted (16 consecutive rows read at one chunk index lie on all
    // banks), or [32][W]: a half wavefront reads consecutive columns of one line, nothing to permute
    static constexpr int FLOATS = W * BK;
    static constexpr int CPL = (KL ? BK : W) / 4;     // chunks per line
    static constexpr int NI = FLOATS * 4 / 1024 / 4;  // 1 KB load instructions per wavefront
    Line ln[KL && !FAST ? NI : 1];
    unsigned voff[FAST ? NI : 1];
    const typename OP::type* sbase;
    static __device__ __forceinline__ int swz(int row) { return KL ? (row & 7) ^ ((row >> 3) & 1) : 0; }
    static __device__ __forceinline__ int chunk(int i) { return ((threadIdx.x >> 6) + 4 * i) * 64 + (threadIdx.x & 63); }
    static __device__ __forceinline__ int l_of(int i) { return chunk(i) / CPL; }
    static __device__ __forceinline__ int c_of(int i) { return ((chunk(i) % CPL) ^ swz(l_of(i))) * 4; }
    __device__ __forceinline__ void init(const OP& op, int w0, int r_end)
    {
        if constexpr (FAST && KL) {
            const long long first = op.fast_line(w0);
            sbase = op.base + first;
#pragma unroll
            for (int i = 0; i < NI; ++i) voff[i] = (unsigned)((op.fast_line(w0 + l_of(i)) - first + c_of(i)) * 4);
        } else if constexpr (FAST) {
            sbase = op.base + w0;
            const int cols = op.width() - w0;  // columns past the end read the first ones: outputs nobody stores
#pragma unroll
            for (int i = 0; i < NI; ++i) voff[i] = (unsigned)((l_of(i) * op.fast_pitch() + (c_of(i) < cols ? c_of(i) : 0)) * 4);
        } else if constexpr (KL) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                ln[i] = op.line(w0 + l_of(i));
                if (ln[i].hi > r_end) ln[i].hi = r_end;
            }
        }
    }
    __device__ __forceinline__ void issue(const OP& op, int i, int w0, int r0, int r_end, unsigned lds_panel) const
    {
        const unsigned dst = __builtin_amdgcn_readfirstlane(lds_panel + (threadIdx.x >> 6) * 1024) + i * 4096;
        if constexpr (FAST) {
            if constexpr (KL) dma16s(voff[i], sbase + r0, dst);
            else dma16s(voff[i], sbase + op.fast_base(r0), dst);
            return;
        }
        Line l;
        int c;
        if constexpr (KL) {
            l = ln[i];
            c = r0 + c_of(i);
        } else {
            const int r = r0 + l_of(i);
            l = r < r_end ? op.line(r) : no_line();
            c = w0 + c_of(i);
        }
        dma16(c >= l.lo && c < l.hi ? (const void*)(op.base + l.off + c) : (const void*)g_zero_chunk, dst);
    }
    // as AnyPanel::frags
    static __device__ __forceinline__ void frags(const float* lds, int w, int r, int lane, float (&f)[4])
    {
        const int c = lane & 31, h = lane >> 5;
        if constexpr (KL) {
            const int row = w + c;
            const f32x4a u = *reinterpret_cast<const f32x4a*>(lds + row * BK + (((r >> 2) + h) ^ swz(row)) * 4);
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = u[q];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = lds[(r + 4 * h + q) * W + w + c];
        }
    }
};

// Same tiles, splits and results as gemm_any_k.  The next panel is requested under the first matrix instructions of a
// panel, into the other of two slots; before the last eight steps every wavefront waits for its share of it and the
// barrier makes it everybody's, so that its first operands are read under those last instructions.  (Three slots are
// no faster for 64 x 64 tiles -- 2.33 against 2.18 ms for the forward pass of 16 x 1600 frames, k = 11, 512 -> 1024 --
// because their 48 KB leave room for three workgroups on a CU instead of four.)
template <class OA, class OB, class EP, bool FAST>
__global__ __launch_bounds__(256, 4) void gemm_f32_k(OA oa, OB ob, EP ep, int M, int N, int R, int per, int splits,
                                                                   float* colsum, int colsum_acc)
{
    constexpr int BM = TILE, BN = TILE, BK = PANEL;
    using PA = DmaPanel<OA, BM, FAST>;
    using PB = DmaPanel<OB, BN, FAST>;
    constexpr int STAGE = PA::FLOATS + PB::FLOATS, NL = PA::NI + PB::NI;
    constexpr int GROUPS = BK / 8;                           // of eight steps, four matrix instructions
    static_assert(NL <= (GROUPS - 1) * 4, "a load after every instruction: all of them before the hand-over");
    __shared__ __align__(1024) float lds[2 * STAGE];
    const int split = blockIdx.z % splits;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    take_phase(oa, ob, ep, blockIdx.z / splits, M, R);
    if (OA::PHASED && m0 >= M) return;  // (phases differ by a frame per utterance)
    const int r_begin = split * per, r_end = R < r_begin + per ? R : r_begin + per;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
    const bool sum_a = !PA::KL && colsum && blockIdx.x == 0;
    const unsigned lds0 = (unsigned)(size_t)(lds_byte*)lds;
    PA pa;
    PB pb;
    pa.init(oa, m0, r_end);
    pb.init(ob, n0, r_end);
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    float asum = 0.f;
    const int steps = r_end > r_begin ? (r_end - r_begin + BK - 1) / BK : 0;
    // (past the last panel the loads fetch zeros, or that panel again: the number in flight never changes)
    auto issue = [&](int i, int st) {
        const unsigned dst = lds0 + (st & 1) * (STAGE * 4);
        const int r0 = r_begin + (FAST && st >= steps ? steps - 1 : st) * BK;
        if (i < PA::NI) pa.issue(oa, i, m0, r0, r_end, dst);
        else pb.issue(ob, i - PA::NI, n0, r0, r_end, dst + PA::FLOATS * 4);
    };
    constexpr bool WALK = FAST && !PA::KL;  // the weight gradient
    int walk0 = 0;                          // WALK: the panel's first frame, counted from its utterance's first one
    if constexpr (WALK) walk0 = r_begin % oa.pitch;
    float fa[2][4], fb[2][4];
    if (steps > 0) {
#pragma unroll
        for (int i = 0; i < NL; ++i) issue(i, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        PA::frags(lds, wm, 0, lane, fa[0]);
        PB::frags(lds + PA::FLOATS, wn, 0, lane, fb[0]);
    }
    for (int st = 0; st < steps; ++st) {
        const float* cur = lds + (st & 1) * STAGE;
        const float* nxt = lds + ((st + 1) & 1) * STAGE;
        bool between = false;  // some of the panel's frames lie behind an utterance
        int left = 0;          // frames up to the end of the run
        if constexpr (WALK) {
            left = r_end - r_begin - st * BK;
            between = walk0 + BK > oa.Tp || left < BK;
        }
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            const int u = g & 1;
            const float* src = g + 1 < GROUPS ? cur : nxt;
            if (g + 1 == GROUPS) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // my share of panel st + 1
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            PA::frags(src, wm, (g + 1) % GROUPS * 8, lane, fa[1 - u]);
            PB::frags(src + PA::FLOATS, wn, (g + 1) % GROUPS * 8, lane, fb[1 - u]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (WALK) {
                if (between) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int l = g * 8 + 4 * (lane >> 5) + q;
                        unsigned t = walk0 + l;
                        t = min(t, t - oa.pitch);  // a panel may reach into the utterance after the next one, no further:
                        t = min(t, t - oa.pitch);  // wgrad_walks
                        fb[u][q] = t < (unsigned)oa.Tp && l < left ? fb[u][q] : 0.f;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u][q], fb[u][q], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (g * 4 + q < NL) issue(g * 4 + q, st + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (sum_a) {
                asm volatile("");  // a branch: without it every workgroup would add, and select
                asum += (fa[u][0] + fa[u][1]) + (fa[u][2] + fa[u][3]);
            }
        }
        if constexpr (WALK) {
            walk0 += BK;
            walk0 = min((unsigned)walk0, (unsigned)(walk0 - oa.pitch));
            walk0 = min((unsigned)walk0, (unsigned)(walk0 - oa.pitch));
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may land in LDS once it is used otherwise
    const int n = n0 + wn + (lane & 31);
    const float addn = n < N ? ep.add(n) : 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int m = m0 + wm + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (m < M && n < N) ep.store(ep.row(m) + n, acc[e] + addn, split);
    }
    if (sum_a && (wave & 1) == 0) {  // the two wavefronts of a row of the tile hold the same values: one writes
        const float v = asum + __shfl_xor(asum, 32, 64);  // lanes 0..31 and 32..63 took different steps
        const int m = m0 + wm + (lane & 31);
        if (lane < 32 && m < M) {
            float* q = colsum + (long long)split * M + m;
            *q = colsum_acc ? *q + v : v;
        }
    }
}

// ---- fp32 products on the bf16 matrix instruction -------------------------------------
// A float is the sum of three bf16 values, exactly: its rounding h, the rounding m of the rest x - h, and l = x - h - m, at
// most eight significant bits (of a float below 2^-109, to within 2^-134: bf16 values are multiples of 2^-133).  Of the nine products of
// two such sums six are taken; the others, m l', l m' and l l', stay below 2^-25 of the product, and a sum over 16 products
// is rounded six times with v_mfma_f32_32x32x16_bf16, eight times with the fp32 instruction.  Those roundings all go down,
// towards minus infinity, 5e-8 of the result's rms in its mean, which adds up where many outputs are summed (a bias
// gradient over the frames came out at twice its distance from 64 bits): so one wavefront of a pair adds up the products
// and the other one their negatives, and the difference of the two sums has the mean error of the fp32 instruction (1e-9).
// Distance from 64 bits against that instruction: 28 layers 0.47 to 1.00 of it (a single pass up to 1.014), 8 steps 0.60 to 0.96.
//
// Six of these instructions take 192 cycles where the fp32 ones take 512 for the same 16 steps; what bounds the kernel is the
// vector instructions of the splits, 5.5 an element, beside them.  So every wavefront takes 64 rows (two operand blocks of A to
// one or two of B) and half of a panel's steps: its neighbour's sums meet its own through LDS at the end.  128 rows: fewer
// splits and LDS reads per product, where there are enough tiles (any_plan); 128 x 128 was no faster (16 x 800 frames, k = 11,
// 256 -> 512: the three passes 779 against 776 us).
// The workgroup starts over with the fp32 instruction where the terms do not carry its operands:
//  - An operand that is not finite, or that rounds to infinity, makes a NaN of the split; so does a sum that overflows: sums that
//    are not finite in the end.
//  - Operands below 2^-109 lose up to 2^-134 each, a sum of K products K 2^-133 M at most, M the largest operand of the tile:
//    a sum below 2^24 times that, but not zero.  (The loss stays below 2^-24 of any other.)
//  - Some row or column whose operands are all below 2^-108, but not all zero.  (So where a sum is zero the loss stays below
//    K 2^-26 of the largest operand of its row times that of its column.)
// The look at the magnitudes, one instruction for two operands in one of the wavefronts that split them, costs 3 % (the
// 10M-parameter network's step 889 -> 914 us); a test of every third term for bits below the smallest bf16 cost 5 %.
// Panels and outputs as gemm_f32_k's over FAST lines.  Measured, layers of 256 -> 512, k = 11, forward and backward, this
// kernel against gemm_f32_k over the same lines: 4 x 400 frames 162 -> 160 us, 16 x 800 973 -> 847; 512 -> 1024, k = 3, 8 x 501
// frames 354 -> 330; the 10M-parameter network's step 1006 -> 892 (996 .. 1006 -> 874 .. 918 by box).
// The method -- an fp32 operand as three bf16 ones, the smallest products left out -- is Henry, Tang and Heinecke's ("Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019).
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
struct Split8 { bf16x8 h, m, l; };
// of sign * v, flip: the sign bits of two bf16 values, set where sign is -1; most (or null): the largest magnitude so far
__device__ __forceinline__ Split8 split8(const float (&v)[8], float* most, float sign = 1.f, unsigned flip = 0)
{
    u32x4 h, m, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a = v[2 * q], b = v[2 * q + 1];
        if (most) *most = fmaxf(fmaxf(*most, fabsf(a)), fabsf(b));
        auto round2 = [&] { return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2)); };
        h[q] = round2() ^ flip;
        a = __builtin_fmaf(a, sign, -__uint_as_float(h[q] << 16));
        b = __builtin_fmaf(b, sign, -__uint_as_float(h[q] & 0xffff0000u));
        m[q] = round2();
        a -= __uint_as_float(m[q] << 16);
        b -= __uint_as_float(m[q] & 0xffff0000u);
        l[q] = round2();
    }
    return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// the largest of a wavefront's magnitudes (their bits are in the same order)
__device__ __forceinline__ unsigned wave_most(float v)
{
    unsigned u = __float_as_uint(v);
    u = max(u, (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0xb1 /* quad_perm 1 0 3 2 */, 0xf, 0xf, true));
    u = max(u, (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x4e /* quad_perm 2 3 0 1 */, 0xf, 0xf, true));
    u = max(u, (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x141 /* row_half_mirror */, 0xf, 0xf, true));
    u = max(u, (unsigned)__builtin_amdgcn_update_dpp(0, (int)u, 0x140 /* row_mirror */, 0xf, 0xf, true));
    auto row = [&](int l) { return (unsigned)__builtin_amdgcn_readlane((int)u, l); };
    return max(max(row(0), row(16)), max(row(32), row(48)));
}

template <class OA, class OB, class EP, int BM>
__global__ __launch_bounds__(256, BM == TILE ? 4 : OA::K_LINES ? 3 : 2) void gemm_split_k(OA oa, OB ob, EP ep, int M, int N, int R, int per,
                                                                                          int splits, float* colsum, int colsum_acc)
{
    constexpr int BN = TILE, BK = PANEL, NB = BM / 64;  // operand blocks of B a wavefront takes, to two of A
    using PA = DmaPanel<OA, BM, true>;
    using PB = DmaPanel<OB, BN, true>;
    constexpr int STAGE = PA::FLOATS + PB::FLOATS;
    __shared__ __align__(1024) float lds[2 * STAGE];
    __shared__ float colsums[2 * BM];
    __shared__ unsigned largest[4];
    const int split = blockIdx.z % splits;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    take_phase(oa, ob, ep, blockIdx.z / splits, M, R);
    if (OA::PHASED && m0 >= M) return;  // (phases differ by a frame per utterance)
    const int r_begin = split * per, r_end = R < r_begin + per ? R : r_begin + per;
    // wavefront: 64 rows from wm and 32 NB columns from wn of the tile, steps kh .. kh + 15 of every panel.  Two wavefronts take the
    // same rows (128 rows: the same columns), each begins with another 32 of them (xa, xb) and looks at the magnitudes of these
    const int lane = threadIdx.x & 63, half = lane >> 5, wave = threadIdx.x >> 6;
    const int wm = BM == 128 ? (wave & 1) * 64 : 0, wn = BM == 128 ? 0 : (wave & 1) * 32;
    const int xa = BM == 128 ? 0 : (wave & 1) * 32, xb = BM == 128 ? (wave & 1) * 32 : 0, kh = __builtin_amdgcn_readfirstlane((wave >> 1) * 16);
    const bool sum_a = !PA::KL && colsum && blockIdx.x == 0;
    const unsigned lds0 = (unsigned)(size_t)(lds_byte*)lds;
    PA pa;
    PB pb;
    pa.init(oa, m0, r_end);
    pb.init(ob, n0, r_end);
    f32x16 acc[2][NB];
    float asum[2], most[3] = {0.f, 0.f, 0.f};  // most: of a row or column of A's blocks and B's first
    const int steps = r_end > r_begin ? (r_end - r_begin + BK - 1) / BK : 0;
    auto request = [&](int st) {  // (past the last panel: that panel again)
        const unsigned dst = lds0 + (st & 1) * (STAGE * 4);
        const int r0 = r_begin + (st >= steps ? steps - 1 : st) * BK;
#pragma unroll
        for (int i = 0; i < PA::NI; ++i) pa.issue(oa, i, m0, r0, r_end, dst);
#pragma unroll
        for (int i = 0; i < PB::NI; ++i) pb.issue(ob, i, n0, r0, r_end, dst + PA::FLOATS * 4);
    };
    auto arrived = [] {  // my share of the panel in flight, then everybody's
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    constexpr bool WALK = !PA::KL;  // the weight gradient
    const float sign = kh ? -1.f : 1.f;  // of this wavefront's sums, in bf16
    const unsigned flip = kh ? 0x80008000u : 0u;
    auto run = [&](auto exact) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            asum[i] = 0.f;
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][n][e] = 0.f;
        }
        int walk0 = 0;  // WALK: the panel's first frame, counted from its utterance's first one
        if constexpr (WALK) walk0 = r_begin % oa.pitch;
        if (steps > 0) {
            request(0);
            arrived();
        }
        for (int st = 0; st < steps; ++st) {
            const float* cur = lds + (st & 1) * STAGE;
            request(st + 1);  // into the slot that every wavefront had read before the last barrier
            float fa[2][8], fb[NB][8];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float f[4];
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    PB::frags(cur + PA::FLOATS, wn + (32 * n ^ xb), kh + 8 * u, lane, f);
#pragma unroll
                    for (int q = 0; q < 4; ++q) fb[n][4 * u + q] = f[q];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    PA::frags(cur, wm + (32 * i ^ xa), kh + 8 * u, lane, f);
#pragma unroll
                    for (int q = 0; q < 4; ++q) fa[i][4 * u + q] = f[q];
                }
            }
            if constexpr (WALK) {
                const int left = r_end - r_begin - st * BK;       // frames up to the end of the run
                if (walk0 + BK > oa.Tp || left < BK) {            // some of the panel's frames lie behind an utterance
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int l = kh + 8 * (e >> 2) + 4 * half + (e & 3);
                        unsigned t = walk0 + l;
                        t = min(t, t - oa.pitch);  // a panel may reach into the utterance after the next one, no further:
                        t = min(t, t - oa.pitch);  // wgrad_walks
#pragma unroll
                        for (int n = 0; n < NB; ++n) fb[n][e] = t < (unsigned)oa.Tp && l < left ? fb[n][e] : 0.f;
                    }
                }
                walk0 += BK;
                walk0 = min((unsigned)walk0, (unsigned)(walk0 - oa.pitch));
                walk0 = min((unsigned)walk0, (unsigned)(walk0 - oa.pitch));
            }
            if constexpr (decltype(exact)::value) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int n = 0; n < NB; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[n][e], acc[i][n], 0, 0, 0);
            } else {
                Split8 b[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) b[n] = split8(fb[n], n ? nullptr : &most[2], sign, flip);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const Split8 a = split8(fa[i], BM == 128 || i == 0 ? &most[i] : nullptr);
                    auto add = [&](const bf16x8& x, bf16x8 Split8::*y) {
#pragma unroll
                        for (int n = 0; n < NB; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b[n].*y, acc[i][n], 0, 0, 0);
                    };
                    add(a.l, &Split8::h);
                    add(a.h, &Split8::l);
                    add(a.m, &Split8::m);
                    add(a.m, &Split8::h);
                    add(a.h, &Split8::m);
                    add(a.h, &Split8::h);
                }
            }
            if (sum_a) {
                asm volatile("");  // a branch: without it every workgroup would add, and select
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float(&f)[8] = fa[i];
                    asum[i] += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // the wait stays behind the matrix instructions
            arrived();
        }
        if constexpr (!decltype(exact)::value) {
            const unsigned u = wave_most(fmaxf(fmaxf(most[0], most[1]), most[2]));
            if (lane == 0) largest[wave] = u;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may land in LDS once it is used otherwise
        __syncthreads();
    };
    run(std::false_type{});
    bool redo = false;
#pragma unroll
    for (int i = 0; i < 3; ++i) redo |= most[i] > 0.f && most[i] < 0x1p-108f;
    const float least = __uint_as_float(max(max(largest[0], largest[1]), max(largest[2], largest[3]))) * 0x1p-109f * (float)(16 * steps);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = fabsf(acc[i][n][e]);
                redo |= !(v <= 3.402823466e38f) | (v != 0.f & v < least);
            }
    if (__syncthreads_or(redo)) {
        run(std::true_type{});
    } else if (kh) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][n][e] = -acc[i][n][e];
    }
    // the two wavefronts of a part of the tile: each finishes one of its two blocks of rows, with the other's sums of it
    constexpr int EXCH = NB * 1024;
    float* const mine = lds + wave * EXCH;
    const int keep = wave >> 1;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) mine[(n * 16 + e) * 64 + lane] = keep ? acc[0][n][e] : acc[1][n][e];
    if (sum_a) {
#pragma unroll
        for (int i = 0; i < 2; ++i) asum[i] += __shfl_xor(asum[i], 32, 64);  // lanes 0..31 and 32..63 took different steps
        if ((BM == 128 || (wave & 1) == 0) && lane < 32) {  // (64 rows: the two wavefronts of a half of the steps have the same sums)
            colsums[keep * BM + wm + xa + lane] = asum[0];
            colsums[keep * BM + wm + (32 ^ xa) + lane] = asum[1];
        }
    }
    __syncthreads();
    const float* const other = lds + (wave ^ 2) * EXCH;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = n0 + wn + (32 * nb ^ xb) + (lane & 31);
        const float addn = n < N ? ep.add(n) : 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int m = m0 + wm + (32 * keep ^ xa) + 8 * (e >> 2) + 4 * half + (e & 3);
            const float own = keep ? acc[1][nb][e] : acc[0][nb][e], far = other[(nb * 16 + e) * 64 + lane];
            if (m < M && n < N) ep.store(ep.row(m) + n, (own + far) + addn, split);
        }
    }
    if (sum_a && threadIdx.x < BM && m0 + (int)threadIdx.x < M) {
        float* const q = colsum + (long long)split * M + m0 + threadIdx.x;
        const float v = colsums[threadIdx.x] + colsums[BM + threadIdx.x];
        *q = colsum_acc ? *q + v : v;
    }
}

// How many workgroups share the reduction of an M x N x R problem's tiles.  The candidates' times are added up from
// cycles: panels at 16 instructions of 64 cycles, one after the other for the workgroups that share a CU (at 0.67 of
// the rate if there is one, 0.76 from three on: measured, 4 x 400 frames, k = 11, 256 -> 512, forward: 200 workgroups
// of 88 panels 61 us, 1000 of 18 panels 46 us), about 12000 to fill and to drain, and for a split the partial sums'
// way to memory and back (2500 bytes per cycle) plus the finishing launch.  64 x 64 outputs per workgroup with the fp32
// instruction: 128 x 128 was slower on the largest problems as well (16 x 1600 frames, k = 11, 512 -> 1024: forward 2.30 against
// 2.18 ms, data gradient 2.69 against 2.38, weight gradient 3.06 against 2.45), four small workgroups on a CU
// covering each other's barriers better than two large ones.
// fp32 operands in haloed tensors choose between gemm_f32_k and gemm_split_k's tiles of 64 or 128 rows: 800 and 1470 cycles a
// panel for the matrix instructions and the splits, the rates and what is added (the exchange of sums, the look at the
// magnitudes, the longer code) fitted twice.  Inside a train step the passes before and behind, and the other gradient on
// its second stream, cover a launch's ends.  A pass called by itself has them in the open, and short runs keep the fp32
// instruction.  250 layers of up to 27 GFLOP a pass, each pass by either kernel in every split that the rule may pick, times of the
// whole layer: by the step's figures 72 of 750 passes cost their layer more than 2 % against the fp32 instruction (up to 6.4 %) and the
// mean layer gains 0.1 % a pass; by those for passes alone 4 (up to 4 %), and 0.7 %.  The steps of 25 networks the other way round: by
// the figures for passes alone 9 are more than 2 % slower than by their own (up to 9 %), none is more than 2 % faster.
struct AnyPlan { int splits, per, rows; bool terms; };  // rows: of a tile; terms: gemm_split_k
struct TileCost { int rows; double cycles, fill[3], fixed; };  // of a panel; the rate with one, two, or more workgroups on a CU
constexpr TileCost TILES[2][3] = {{{64, 1024, {0.67, 0.72, 0.76}, 12000}, {64, 800, {0.62, 0.70, 0.76}, 14400}, {128, 1470, {0.50, 0.62, 0.78}, 14400}},
                                  {{64, 1024, {0.67, 0.72, 0.76}, 12000}, {64, 800, {0.53, 0.73, 0.75}, 23000}, {128, 1470, {0.54, 0.81, 0.84}, 27000}}};
// values: of a plane; problems: that share a launch, each M x N x R (the phases of a stride); alone: not part of a train step.
// Every call plans its passes, so the search leaves out what cannot be the best: with all CUs at work to the last panel,
// a tile shape takes `least` (less the rounding of sums), and whatever adds to that adds more with every further run.
AnyPlan any_plan(long long M, long long N, long long R, size_t budget, double finish_cycles, long long values, int problems, bool f32, bool alone)
{
    AnyPlan best{1, 0, TILE, false};
    double best_t = -1;
    const long long columns = problems * ((N + TILE - 1) / TILE), panels = (R + PANEL - 1) / PANEL;
    for (int v = 0; v < (f32 ? 3 : 1); ++v) {
        const TileCost& c = TILES[alone][v];
        const long long tiles = columns * ((M + c.rows - 1) / c.rows);
        const double least = (double)tiles * panels / 256 * c.cycles / c.fill[2] * (1 - 1e-9) + c.fixed;
        for (int s = 1; s <= 16; ++s) {
            const double planes = s > 1 ? 8.0 * s * values / 2500 + finish_cycles : 0;
            if (best_t >= 0 && least + planes >= best_t) break;
            const long long per = s > 1 ? (panels + s - 1) / s : panels;
            if (s > 1 && (per < 2 || (size_t)s * values * 4 > budget)) break;
            if (s > 1 && per * (s - 1) >= panels) continue;
            const long long load = (tiles * s + 255) / 256;
            double t = load * per * c.cycles / c.fill[load > 2 ? 2 : load > 1 ? 1 : 0] + c.fixed;
            if (s > 1) t += planes;
            if (best_t < 0 || t < best_t) {
                best_t = t;
                best = AnyPlan{s, (int)(per * PANEL), c.rows, v > 0};
            }
        }
    }
    return best;
}

template <class OA, class OB, class EP>
int launch_any(const AnyPlan& pl, OA oa, OB ob, EP ep, long long M, long long N, long long R, hipStream_t st, float* colsum = nullptr,
               int colsum_acc = 0, bool fast = false, ConvForm* form = nullptr, int phases = 1)
{
    constexpr bool f32 = std::is_same<typename OA::type, float>::value && std::is_same<typename OB::type, float>::value;
    const bool tall = f32 && fast && pl.rows > TILE && oa.tall();
    const int rows = tall ? 2 * TILE : TILE;
    const long long gy = (M + rows - 1) / rows, gx = (N + TILE - 1) / TILE;
    if (M > 2147483647LL || R > 2147483647LL - 4096 || gy > 65535 || gx > 2147483647LL) return W2L_ERR_SHAPE;
    if (M <= 0) return W2L_OK;
    const bool chunks = f32 && oa.chunks() && ob.chunks();
    if (form) {  // asked which kernel it is
        *form = ConvForm{!chunks ? CONV_REGISTERS : fast ? CONV_PLAIN : CONV_CHUNKS, pl.splits, rows, chunks && fast && pl.terms};
        return W2L_OK;
    }
    const dim3 g((unsigned)gx, (unsigned)gy, (unsigned)(phases * pl.splits));
#define W2L_ANY(KERN) hipLaunchKernelGGL(KERN, g, dim3(256), 0, st, oa, ob, ep, (int)M, (int)N, (int)R, pl.per, pl.splits, colsum, colsum_acc)
    if constexpr (f32) {
        if (chunks) {
            if (tall) W2L_ANY((gemm_split_k<OA, OB, EP, 2 * TILE>));
            else if (fast && pl.terms) W2L_ANY((gemm_split_k<OA, OB, EP, TILE>));
            else if (fast) W2L_ANY((gemm_f32_k<OA, OB, EP, true>));
            else W2L_ANY((gemm_f32_k<OA, OB, EP, false>));
            return launch_status();
        }
    }
    W2L_ANY((gemm_any_k<OA, OB, EP>));
#undef W2L_ANY
    return launch_status();
}

// the operands of the three passes
template <typename T> XWindow<T> fwd_a(const ConvDesc& d, const void* x) { return {(const T*)x, (int)((long long)d.B * d.Tp), d.T, d.Tp, d.Cin, d.k, d.s, d.p, d.x_pitch, d.x_halo}; }
template <typename T> WRows<T> fwd_b(const ConvDesc& d, const void* w) { return {(const T*)w, d.Cout, d.k * d.Cin}; }
template <typename T> DyWindow<T> dgrad_a(const ConvDesc& d, const void* dy, int f, Phase q) { return {(const T*)dy, d.B, d.T, d.Tp, d.Cout, d.k, d.s, d.p, d.y_pitch, d.y_halo, f, q}; }
template <typename T> WCols<T> dgrad_b(const ConvDesc& d, const void* w, Phase q) { return {(const T*)w, d.Cin, d.Cout, d.k, d.s, q}; }
template <typename T> DyT<T> wgrad_a(const ConvDesc& d, const void* dy) { return {(const T*)dy, d.Tp, d.Cout, d.y_pitch, d.y_halo}; }
template <typename T> XShift<T> wgrad_b(const ConvDesc& d, const void* x) { return {(const T*)x, d.T, d.Tp, d.Cin, d.k, d.s, d.p, d.x_pitch, d.x_halo}; }

bool wgrad_walks(const ConvDesc& d)
{
    return d.s == 1 && d.x_pitch == d.y_pitch && d.x_halo == d.y_halo && d.x_halo >= d.p && d.slack >= 64 && d.x_pitch >= PANEL / 2 &&
           (d.B == 1 || d.x_halo > 0 || d.p == 0);
}

template <typename TI, typename TO>
int fwd_t(const ConvDesc& d, const AnyPlan& pl, const void* x, const void* w, const float* bias, TO* y, int pitch, int halo,
          long long plane, hipStream_t st, ConvForm* form = nullptr)
{
    const long long M = (long long)d.B * d.Tp;
    const XWindow<TI> a = fwd_a<TI>(d, x);
    const WRows<TI> b = fwd_b<TI>(d, w);
    StoreRows<TO> ep{y, bias, d.Cout, d.Tp, 0, 1, pitch, halo, plane};
    return launch_any(pl, a, b, ep, M, d.Cout, (long long)d.k * d.Cin, st, nullptr, 0, a.fast() && b.fast(), form);
}
template <typename TW, typename TDY, typename TO>
int dgrad_t(const ConvDesc& d, const AnyPlan& pl, const void* dy, const void* w, TO* dx, int pitch, int halo, long long plane, hipStream_t st,
            ConvForm* form = nullptr)
{
    const int phases = d.s < d.T ? d.s : d.T, most = 65535 / pl.splits;  // (that have frames; that a grid takes)
    for (int f = 0; f < phases; f += most) {
        const Phase q = DyWindow<TDY>::phase(f, d.T, d.k, d.s, d.p);  // of the launch, the one with the most frames
        const DyWindow<TDY> a = dgrad_a<TDY>(d, dy, f, q);
        const WCols<TW> b = dgrad_b<TW>(d, w, q);
        StoreRows<TO> ep{dx, nullptr, d.Cin, q.count, q.first, d.s, pitch, halo, plane};
        const int rc = launch_any(pl, a, b, ep, (long long)d.B * q.count, d.Cin, (long long)q.taps * d.Cout, st, nullptr, 0, a.fast() && b.fast(),
                                  form, phases - f < most ? phases - f : most);
        if (rc || form) return rc;
    }
    return W2L_OK;
}
template <typename TX, typename TDY>
int wgrad_t(const ConvDesc& d, const AnyPlan& pl, const void* x, const void* dy, float* dw, float* dbias, int accumulate, long long plane,
            hipStream_t st, ConvForm* form = nullptr)
{
    const DyT<TDY> a = wgrad_a<TDY>(d, dy);
    const XShift<TX> b = wgrad_b<TX>(d, x);
    StoreAcc ep{dw, d.k * d.Cin, accumulate, plane};
    // with x and dy in one haloed layout the reduction runs straight through its frames: dy is zero in the halo
    // frames, and in the slack that the last panel reads into
    const long long walk = (long long)(d.B - 1) * d.y_pitch + d.Tp;
    // (only the kernel that launch_any takes for fp32 operands in whole chunks walks; the others count real frames)
    const bool fast = std::is_same<TX, float>::value && std::is_same<TDY, float>::value && a.fast() && b.fast() && wgrad_walks(d) &&
                      walk <= (long long)pl.per * pl.splits;
    const long long R = fast ? walk : (long long)d.B * d.Tp;
    return launch_any(pl, a, b, ep, d.Cout, (long long)d.k * d.Cin, R, st, dbias, accumulate, fast, form);
}

// ---- weight gradient for narrow outputs (Cout <= 32, e.g. the 29 grapheme classes) ---------
// dw[co, n=(j,ci)] = sum_{r=(b,t')} dy[r,co] * x[b, s t' + j - p, ci].  A 64-wide tile would be half empty and there are
// few of them: the reduction is cut into SKINNY_CHUNKS ranges of frames (grid.y), and a second pass adds the chunks in a
// fixed order.
// N1 columns: the N of the weights and, for the bias gradient, one more that meets ones instead of x.
// v_mfma_f32_32x32x2_f32 straight from memory: 32 classes by 2 x 32 columns a wavefront, two frames an instruction (one
// in lanes 0..31, the next in lanes 32..63), SKINNY_AHEAD instructions' operands requested together; what bounds it is
// the issue of their loads, one element a lane.  The four wavefronts of a workgroup interleave the chunk's frames and
// add up through LDS.  16 x 800 frames, 512 -> 29: 18 us, where scalar FMAs over frames staged in LDS took 31 and the
// bias gradient 20 more.
constexpr int SKINNY_AHEAD = 16;

template <typename TX, typename TDY>
__global__ __launch_bounds__(256) void wgrad_skinny_stage1(const TX* __restrict__ x, const TDY* __restrict__ dy,
                                                           float* __restrict__ part, ConvDesc d, int N1)
{
    __shared__ float red[3][32][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 31, half = lane >> 5;
    const int N = d.k * d.Cin, R = d.B * d.Tp;
    const int per = (R + gridDim.y - 1) / gridDim.y;
    const int r_begin = per * blockIdx.y < R ? per * blockIdx.y : R, r_end = (r_begin + per < R) ? r_begin + per : R;
    int j[2], ci[2];
    bool real[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int n = blockIdx.x * 64 + 32 * q + c;
        real[q] = n < N;  // (columns past the end meet ones: the first of them is the bias gradient)
        j[q] = real[q] ? n / d.Cin : 0;
        ci[q] = real[q] ? n - j[q] * d.Cin : 0;
    }
    f32x16 acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    // this lane's frame, and where its dy row and (tap 0, channel 0) of its window lie: from frame to frame by addition
    int r = r_begin + 2 * wave + half, tp = r % d.Tp, t0 = d.s * tp - d.p;
    const long long b0 = r / d.Tp, xstep = 8LL * d.s * d.Cin, ystep = 8LL * d.Cout;
    const long long xwrap = ((long long)d.x_pitch - (long long)d.s * d.Tp) * d.Cin, ywrap = (long long)(d.y_pitch - d.Tp) * d.Cout;
    const TDY* py = dy + (b0 * d.y_pitch + d.y_halo + tp) * d.Cout + (c < d.Cout ? c : 0);
    const TX* px = x + (b0 * d.x_pitch + d.x_halo + t0) * d.Cin;
    const int xo[2] = {j[0] * d.Cin + ci[0], j[1] * d.Cin + ci[1]};
    const int steps = r_end > r_begin ? (r_end - r_begin + 7) / 8 : 0;  // of eight frames, two a wavefront
    for (int st = 0; st < steps; st += SKINNY_AHEAD) {
        float dv[SKINNY_AHEAD], xv[SKINNY_AHEAD][2];
#pragma unroll
        for (int u = 0; u < SKINNY_AHEAD; ++u) {
            const bool ok = r < r_end;  // (frames past the chunk read element 0 and count 0)
            const float v = Elem<TDY>::load(ok ? py : dy, 0);
            dv[u] = ok && c < d.Cout ? v : 0.f;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const bool in = ok && (unsigned)(t0 + j[q]) < (unsigned)d.T;
                const float xe = Elem<TX>::load(in ? px + xo[q] : x, 0);
                xv[u][q] = real[q] ? (in ? xe : 0.f) : 1.f;
            }
            r += 8;
            tp += 8;
            t0 += 8 * d.s;
            px += xstep;
            py += ystep;
            while (tp >= d.Tp) { tp -= d.Tp; t0 -= d.s * d.Tp; px += xwrap; py += ywrap; }
        }
#pragma unroll
        for (int u = 0; u < SKINNY_AHEAD; ++u)
#pragma unroll
            for (int q = 0; q < 2; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(dv[u], xv[u][q], acc[q], 0, 0, 0);
    }
    if (wave > 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 16; ++e) red[wave - 1][8 * (e >> 2) + 4 * half + (e & 3)][32 * q + c] = acc[q][e];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int n = blockIdx.x * 64 + 32 * q + c;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = 8 * (e >> 2) + 4 * half + (e & 3);
                if (m < d.Cout && n < N1)
                    part[((size_t)blockIdx.y * d.Cout + m) * N1 + n] = ((acc[q][e] + red[0][m][32 * q + c]) + red[1][m][32 * q + c]) + red[2][m][32 * q + c];
            }
        }
    }
}
__global__ __launch_bounds__(256) void wgrad_skinny_stage2(const float* __restrict__ part, float* __restrict__ dw, float* __restrict__ dbias,
                                                           int N, int N1, int total, int accumulate)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    float acc = 0.f, v[SKINNY_CHUNKS];
#pragma unroll
    for (int c = 0; c < SKINNY_CHUNKS; ++c) v[c] = part[(size_t)c * total + i];  // independent loads, added in order
#pragma unroll
    for (int c = 0; c < SKINNY_CHUNKS; ++c) acc += v[c];
    const int co = i / N1, n = i - co * N1;
    float* const q = n < N ? dw + (size_t)co * N + n : dbias + co;
    *q = accumulate ? *q + acc : acc;
}

// ---- dbias: deterministic two-stage column sum -------------------------------------
// bf16, Cout % 8 == 0.  A workgroup owns 32 columns (4 lanes x 16-byte loads) of one of
// DBIAS_CHUNKS row ranges, 64 row lanes each; the 64 partial sums per column are added in a
// fixed tree through LDS; colsum_stage2 then adds the chunks in order.
__global__ __launch_bounds__(256) void colsum_bf16_stage1(const bf16_t* __restrict__ dy, float* __restrict__ part,
                                                          long long rows, int Cout)
{
    const int cg = threadIdx.x & 3, rl = threadIdx.x >> 2;
    const int c0 = blockIdx.x * 32 + cg * 8;
    const long long per = (rows + gridDim.y - 1) / gridDim.y;
    const long long r0 = per * blockIdx.y, r1 = (r0 + per < rows) ? r0 + per : rows;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    if (c0 < Cout)
        for (long long r = r0 + rl; r < r1; r += 64) {
            const uint4 v = *reinterpret_cast<const uint4*>(dy + r * Cout + c0);
            const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] += __uint_as_float(u[j] << 16);
                acc[2 * j + 1] += __uint_as_float(u[j] & 0xffff0000u);
            }
        }
    __shared__ float sm[64][33];
#pragma unroll
    for (int j = 0; j < 8; ++j) sm[rl][cg * 8 + j] = acc[j];
    __syncthreads();
    for (int half = 32; half > 0; half >>= 1) {
        for (int e = threadIdx.x; e < half * 32; e += 256) {
            const int r = e >> 5, c = e & 31;
            sm[r][c] += sm[r + half][c];
        }
        __syncthreads();
    }
    if (threadIdx.x < 32) {
        const int c = blockIdx.x * 32 + threadIdx.x;
        if (c < Cout) part[(size_t)blockIdx.y * Cout + c] = sm[0][threadIdx.x];
    }
}
__global__ void colsum_stage2(const float* part, float* dbias, int chunks, int Cout, int accumulate)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= Cout) return;
    float acc = 0.f;
    for (int i0 = 0; i0 < chunks; i0 += 16) {
        float v[16];  // independent loads, then added in order
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = (i0 + u < chunks) ? part[(size_t)(i0 + u) * Cout + c] : 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += v[u];
    }
    dbias[c] = accumulate ? dbias[c] + acc : acc;
}

}  // namespace

namespace {
// a finishing launch of its own costs about 5 us; inside the train step it is the layer's GLU, launched in any case
constexpr double FINISH_OWN = 12000, FINISH_FREE = 2000;
AnyPlan fwd_plan(const ConvDesc& d, size_t budget, double fin, bool f32)
{
    const long long M = (long long)d.B * d.Tp;
    return any_plan(M, d.Cout, (long long)d.k * d.Cin, budget, fin, M * d.Cout, 1, f32, fin == FINISH_OWN);
}
AnyPlan dgrad_plan(const ConvDesc& d, size_t budget, double fin, bool f32)
{
    // of a stride's phases, the one with the most taps, as often as there are any with taps; a plane takes all of them
    const int phases = d.s < d.k ? d.s : d.k;
    return any_plan((long long)d.B * ((d.T + d.s - 1) / d.s), d.Cin, (long long)((d.k + d.s - 1) / d.s) * d.Cout, budget, fin,
                    (long long)d.B * d.T * d.Cin, phases < d.T ? phases : d.T, f32, fin == FINISH_OWN);
}
constexpr long long MOST_WALK = 1LL << 30;
long long walk_frames(const ConvDesc& d) { return (long long)d.B * (d.Tp + 2 * LAYOUT_HALO); }
AnyPlan wgrad_plan(const ConvDesc& d, size_t budget, bool f32, bool alone)
{
    // the reduction as long as the walk through the haloed layout makes it (where that is no more frames than an entry
    // point takes: a run's end has to stay below 2^31)
    const long long walk = walk_frames(d);
    return any_plan(d.Cout, (long long)d.k * d.Cin, walk <= MOST_WALK ? walk : (long long)d.B * d.Tp, budget, FINISH_OWN,
                    (long long)d.Cout * d.k * d.Cin, 1, f32, alone);
}
// Passes that gemm_split_k may take: fp32, every window plain memory in the layout at hand (operands aligned: the entry
// points ask for that).  The others are planned by the costs of the fp32 instruction, which they run on (13 x 1063 frames at a stride
// of 2, k = 5, 512 -> 256: 107.5 us with the runs that gemm_split_k would take, 3, and 102.0 with 4).
bool fwd_splits(const ConvDesc& d, int dt) { return dt == W2L_F32 && fwd_a<float>(d, nullptr).fast() && fwd_b<float>(d, nullptr).fast(); }
bool dgrad_splits(const ConvDesc& d, int dt)
{
    const Phase q = DyWindow<float>::phase(0, d.T, d.k, d.s, d.p);
    return dt == W2L_F32 && dgrad_a<float>(d, nullptr, 0, q).fast() && dgrad_b<float>(d, nullptr, q).fast();
}
bool wgrad_splits(const ConvDesc& d, int dt)
{
    return dt == W2L_F32 && wgrad_a<float>(d, nullptr).fast() && wgrad_b<float>(d, nullptr).fast() && wgrad_walks(d) && walk_frames(d) <= MOST_WALK;
}
size_t part_bytes(int splits, long long rows, long long cols) { return splits > 1 ? round_up((size_t)splits * rows * cols * 4, 256) : 0; }
}  // namespace

size_t conv_fwd_generic_scratch(const ConvDesc& d, int dt)
{
    return part_bytes(fwd_plan(d, MAX_PARTIALS, FINISH_OWN, fwd_splits(d, dt)).splits, (long long)d.B * d.Tp, d.Cout);
}
size_t conv_dgrad_generic_scratch(const ConvDesc& d, int dt)
{
    return part_bytes(dgrad_plan(d, MAX_PARTIALS, FINISH_OWN, dgrad_splits(d, dt)).splits, (long long)d.B * d.T, d.Cin);
}
size_t conv_wgrad_generic_scratch(const ConvDesc& d, int dt, bool alone)
{
    return part_bytes(wgrad_plan(d, MAX_PARTIALS, wgrad_splits(d, dt), alone).splits, d.Cout, (long long)d.k * d.Cin + 1);
}
int conv_fwd_generic_parts(const ConvDesc& d, int dt) { return fwd_plan(d, MAX_PARTIALS, FINISH_FREE, fwd_splits(d, dt)).splits; }
int conv_dgrad_generic_parts(const ConvDesc& d, int dt) { return dgrad_plan(d, MAX_PARTIALS, FINISH_FREE, dgrad_splits(d, dt)).splits; }

int conv_fwd_generic_partial(const ConvDesc& d, const void* x, const void* w, int dt, float* part, hipStream_t st)
{
    const AnyPlan pl = fwd_plan(d, MAX_PARTIALS, FINISH_FREE, fwd_splits(d, dt));
    const long long plane = (long long)d.B * d.Tp * d.Cout;
    if (dt == W2L_F32) return fwd_t<float, float>(d, pl, x, w, nullptr, part, d.Tp, 0, plane, st);
    return fwd_t<bf16_t, float>(d, pl, x, w, nullptr, part, d.Tp, 0, plane, st);
}
int conv_dgrad_generic_partial(const ConvDesc& d, const void* dy, const void* w, int dt, int dydt, float* part, hipStream_t st)
{
    const AnyPlan pl = dgrad_plan(d, MAX_PARTIALS, FINISH_FREE, dgrad_splits(d, dt));
    const long long plane = (long long)d.B * d.T * d.Cin;
    if (dt == W2L_F32) return dgrad_t<float, float, float>(d, pl, dy, w, part, d.T, 0, plane, st);
    if (dydt == W2L_BF16) return dgrad_t<bf16_t, bf16_t, float>(d, pl, dy, w, part, d.T, 0, plane, st);
    return dgrad_t<bf16_t, float, float>(d, pl, dy, w, part, d.T, 0, plane, st);
}

int conv_fwd_generic(const ConvDesc& d, const void* x, const void* w, const float* bias, void* y, int dt, int ydt,
                     hipStream_t st, void* scratch, size_t scratch_bytes)
{
    if (dt == W2L_F32 && ydt != W2L_F32) return W2L_ERR_DTYPE;
    const AnyPlan pl = fwd_plan(d, scratch ? (scratch_bytes < MAX_PARTIALS ? scratch_bytes : MAX_PARTIALS) : 0, FINISH_OWN, fwd_splits(d, dt));
    if (pl.splits > 1) {
        float* part = static_cast<float*>(scratch);
        const long long rows = (long long)d.B * d.Tp, plane = rows * d.Cout;
        const int rc = dt == W2L_F32 ? fwd_t<float, float>(d, pl, x, w, nullptr, part, d.Tp, 0, plane, st)
                                     : fwd_t<bf16_t, float>(d, pl, x, w, nullptr, part, d.Tp, 0, plane, st);
        return rc ? rc : finish_rows(part, pl.splits, bias, y, ydt, d.B, d.Tp, d.Cout, d.y_pitch, d.y_halo, st);
    }
    if (dt == W2L_F32) return fwd_t<float, float>(d, pl, x, w, bias, (float*)y, d.y_pitch, d.y_halo, 0, st);
    if (ydt == W2L_BF16) return fwd_t<bf16_t, bf16_t>(d, pl, x, w, bias, (bf16_t*)y, d.y_pitch, d.y_halo, 0, st);
    return fwd_t<bf16_t, float>(d, pl, x, w, bias, (float*)y, d.y_pitch, d.y_halo, 0, st);
}
int conv_dgrad_generic(const ConvDesc& d, const void* dy, const void* w, void* dx, int dt, int dydt, hipStream_t st, void* scratch,
                       size_t scratch_bytes)
{
    if (dt == W2L_F32 && dydt != W2L_F32) return W2L_ERR_DTYPE;
    const AnyPlan pl = dgrad_plan(d, scratch ? (scratch_bytes < MAX_PARTIALS ? scratch_bytes : MAX_PARTIALS) : 0, FINISH_OWN, dgrad_splits(d, dt));
    if (pl.splits > 1) {
        float* part = static_cast<float*>(scratch);
        const long long plane = (long long)d.B * d.T * d.Cin;
        int rc;
        if (dt == W2L_F32) rc = dgrad_t<float, float, float>(d, pl, dy, w, part, d.T, 0, plane, st);
        else if (dydt == W2L_BF16) rc = dgrad_t<bf16_t, bf16_t, float>(d, pl, dy, w, part, d.T, 0, plane, st);
        else rc = dgrad_t<bf16_t, float, float>(d, pl, dy, w, part, d.T, 0, plane, st);
        return rc ? rc : finish_rows(part, pl.splits, nullptr, dx, dt, d.B, d.T, d.Cin, d.x_pitch, d.x_halo, st);
    }
    if (dt == W2L_F32) return dgrad_t<float, float, float>(d, pl, dy, w, (float*)dx, d.x_pitch, d.x_halo, 0, st);
    if (dydt == W2L_BF16) return dgrad_t<bf16_t, bf16_t, bf16_t>(d, pl, dy, w, (bf16_t*)dx, d.x_pitch, d.x_halo, 0, st);
    return dgrad_t<bf16_t, float, bf16_t>(d, pl, dy, w, (bf16_t*)dx, d.x_pitch, d.x_halo, 0, st);
}
int conv_wgrad_generic(const ConvDesc& d, const void* x, const void* dy, float* dw, float* dbias, int dt, int dydt, int accumulate,
                       hipStream_t st, void* scratch, size_t scratch_bytes, bool alone)
{
    if (dt == W2L_F32 && dydt != W2L_F32) return W2L_ERR_DTYPE;
    // (the bias sums of the splits lie behind the weight sums: one more column)
    const long long n = (long long)d.k * d.Cin, plane = d.Cout * n;
    AnyPlan pl = wgrad_plan(d, MAX_PARTIALS, wgrad_splits(d, dt), alone);
    if (!scratch || scratch_bytes < part_bytes(pl.splits, d.Cout, n + 1)) {
        const size_t bias = (size_t)17 * d.Cout * 4;  // (room for the bias sums of 16 splits, rounded up)
        pl = wgrad_plan(d, scratch && scratch_bytes > bias ? scratch_bytes - bias : 0, wgrad_splits(d, dt), alone);
    }
    float* part = static_cast<float*>(scratch);
    const bool split = pl.splits > 1;
    float* const out = split ? part : dw;
    float* const bout = !dbias ? nullptr : split ? part + pl.splits * plane : dbias;
    const int acc = split ? 0 : accumulate;
    int rc;
    if (dt == W2L_F32) rc = wgrad_t<float, float>(d, pl, x, dy, out, bout, acc, plane, st);
    else if (dydt == W2L_BF16) rc = wgrad_t<bf16_t, bf16_t>(d, pl, x, dy, out, bout, acc, plane, st);
    else rc = wgrad_t<bf16_t, float>(d, pl, x, dy, out, bout, acc, plane, st);
    if (rc || !split) return rc;
    return finish_sums(part, pl.splits, plane, dw, bout, d.Cout, dbias, accumulate, st);
}
// Which kernel the calls below would take and into how many runs the reduction goes (operands aligned; nothing is launched)
int conv_fwd_generic_form(const ConvDesc& d, int dt, size_t scratch_bytes, ConvForm* form)
{
    const AnyPlan pl = fwd_plan(d, scratch_bytes < MAX_PARTIALS ? scratch_bytes : MAX_PARTIALS, FINISH_OWN, fwd_splits(d, dt));
    float* const y = nullptr;
    if (dt == W2L_F32) return fwd_t<float, float>(d, pl, nullptr, nullptr, nullptr, y, d.y_pitch, d.y_halo, 0, nullptr, form);
    return fwd_t<bf16_t, float>(d, pl, nullptr, nullptr, nullptr, y, d.y_pitch, d.y_halo, 0, nullptr, form);
}
int conv_dgrad_generic_form(const ConvDesc& d, int dt, size_t scratch_bytes, ConvForm* form)
{
    const AnyPlan pl = dgrad_plan(d, scratch_bytes < MAX_PARTIALS ? scratch_bytes : MAX_PARTIALS, FINISH_OWN, dgrad_splits(d, dt));
    float* const dx = nullptr;
    if (dt == W2L_F32) return dgrad_t<float, float, float>(d, pl, nullptr, nullptr, dx, d.x_pitch, d.x_halo, 0, nullptr, form);
    return dgrad_t<bf16_t, bf16_t, float>(d, pl, nullptr, nullptr, dx, d.x_pitch, d.x_halo, 0, nullptr, form);
}
int conv_wgrad_generic_form(const ConvDesc& d, int dt, ConvForm* form)
{
    const AnyPlan pl = wgrad_plan(d, MAX_PARTIALS, wgrad_splits(d, dt), true);
    if (dt == W2L_F32) return wgrad_t<float, float>(d, pl, nullptr, nullptr, nullptr, nullptr, 0, 0, nullptr, form);
    return wgrad_t<bf16_t, bf16_t>(d, pl, nullptr, nullptr, nullptr, nullptr, 0, 0, nullptr, form);
}

size_t conv_wgrad_skinny_scratch(int Cin, int Cout, int k)
{
    return Cout <= 32 ? round_up((size_t)SKINNY_CHUNKS * Cout * ((size_t)k * Cin + 1) * 4, 256) : 0;
}
int conv_wgrad_skinny(const ConvDesc& d, const void* x, const void* dy, float* dw, float* dbias, int dt, int dydt, int accumulate,
                      float* scratch, hipStream_t st)
{
    const long long N = (long long)d.k * d.Cin, N1 = N + (dbias ? 1 : 0), total = d.Cout * N1;
    if (total > 2147483647LL - 256) return W2L_ERR_SHAPE;
    const dim3 g1((unsigned)((N1 + 63) / 64), SKINNY_CHUNKS);
    if (dt == W2L_F32 && dydt == W2L_F32)
        hipLaunchKernelGGL((wgrad_skinny_stage1<float, float>), g1, dim3(256), 0, st, (const float*)x, (const float*)dy, scratch, d, (int)N1);
    else if (dt == W2L_BF16 && dydt == W2L_BF16)
        hipLaunchKernelGGL((wgrad_skinny_stage1<bf16_t, bf16_t>), g1, dim3(256), 0, st, (const bf16_t*)x, (const bf16_t*)dy, scratch, d, (int)N1);
    else if (dt == W2L_BF16 && dydt == W2L_F32)
        hipLaunchKernelGGL((wgrad_skinny_stage1<bf16_t, float>), g1, dim3(256), 0, st, (const bf16_t*)x, (const float*)dy, scratch, d, (int)N1);
    else
        return W2L_ERR_DTYPE;
    int rc = launch_status();
    if (rc) return rc;
    hipLaunchKernelGGL(wgrad_skinny_stage2, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, scratch, dw, dbias, (int)N, (int)N1,
                       (int)total, accumulate);
    return launch_status();
}
int dbias_reduce(const void* dy, float* dbias, long long rows, int Cout, int accumulate, float* scratch, hipStream_t st)
{
    hipLaunchKernelGGL(colsum_bf16_stage1, dim3((Cout + 31) / 32, DBIAS_CHUNKS), dim3(256), 0, st, (const bf16_t*)dy, scratch, rows, Cout);
    const int rc = launch_status();
    if (rc) return rc;
    hipLaunchKernelGGL(colsum_stage2, dim3((Cout + 255) / 256), dim3(256), 0, st, scratch, dbias, (int)DBIAS_CHUNKS, Cout, accumulate);
    return launch_status();
}

}  // namespace w2l
