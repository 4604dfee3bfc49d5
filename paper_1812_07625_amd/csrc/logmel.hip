// Log-mel filterbank features on the GPU (paper Sec. 2.2 lists log-mels among the feature types
// computed on the fly before every network evaluation, Sec. 4.1 uses them as the network input;
// the paper computes them on host threads and fixes no constant -- the recipe is this library's
// reading: frames wholly inside the signal, Hamming window, zero-padded DFT, power spectrum,
// triangular filters equally spaced on the mel scale m = 2595 log10(1 + f/700), natural log).
//
// logmel_k, any size: one wavefront per frame, four frames in flight per workgroup, a workgroup covers a run of consecutive
// frames of one utterance (their samples overlap, so they come from L2 / the same cache lines).
// The DFT of the real, zero-padded frame is taken as a complex FFT of half the size on
// z[n] = x[2n] + i x[2n+1], followed by the usual split into the spectrum of x.  The FFT is a
// radix-4 Stockham (self-sorting, out-of-place) transform between two LDS buffers owned by the
// wavefront, with one radix-2 pass when the size is not a power of four: for nfft = 512 that is
// four passes of 64 butterflies, one per lane, and no workgroup barrier.  Twiddle factors, the
// window, the mel points and the band weights are computed once per workgroup (sincospi / cospi
// on exact binary fractions; the mel points in double) -- there is no table in memory.  A lane
// then owns mel bands (lane, lane + 64, ...) and adds its weighted bins in ascending order, so the
// result does not depend on scheduling.  logmel512_k below takes the usual transform size.
#include <cmath>
#include "common.h"

namespace w2l {
namespace {


struct LogmelDims {
    int B, Nmax, Tmax, F, sr, win, hop, nfft;
    int fpw;  // of a workgroup: frames, a multiple of 4 (logmel_k), or groups of four frames (logmel512_k)
    float fmin, fmax, floor;
    double mlo, mhi;  // the mel scale's ends
    int chunks;       // logmel512_k: room for the band weights
};

template <typename T> __device__ __forceinline__ void store_as(T* p, float v) { Elem<T>::store(p, 0, v); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

// LDS layout (floats unless noted), shared by the kernel and the host-side size
struct LogmelLds {
    int tw, window, pts, k0, off, wgt, bufs, power, total;  // offsets in bytes
};
__host__ __device__ inline LogmelLds logmel_lds(int nfft, int win, int F)
{
    auto up8 = [](int v) { return (v + 7) & ~7; };
    LogmelLds l;
    int o = 0;
    l.tw = o;     o += up8((3 * nfft / 4 + 1) * 8);          // float2 exp(-2 pi i k / nfft), k <= 3 nfft / 4
    l.window = o; o += up8(win * 4);
    l.pts = o;    o += up8((F + 2) * 4);                     // mel points in Hz
    l.k0 = o;     o += up8(F * 4);                           // int: first bin of a band
    l.off = o;    o += up8((F + 1) * 4);                     // int: start of a band's weights in wgt
    l.wgt = o;    o += up8((nfft + 2 + 4 * F) * 4);          // band weights, band after band
    l.bufs = o;   o += 4 * 2 * (nfft / 2) * 8;               // per wavefront: two float2 buffers of nfft/2
    l.power = o;  o += up8(4 * (nfft / 2 + 1) * 4);          // per wavefront: nfft/2 + 1
    l.total = o;
    return l;
}

template <typename TO>
__global__ __launch_bounds__(256) void logmel_k(const float* __restrict__ wav, const int* __restrict__ wav_len,
                                                TO* __restrict__ feat, int* __restrict__ feat_len, LogmelDims d)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.y, t0 = blockIdx.x * d.fpw;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = d.nfft, M = N / 2;
    const LogmelLds L = logmel_lds(N, d.win, d.F);
    float2* tw = reinterpret_cast<float2*>(smem + L.tw);
    float* window = reinterpret_cast<float*>(smem + L.window);
    float* pts = reinterpret_cast<float*>(smem + L.pts);
    int* bk0 = reinterpret_cast<int*>(smem + L.k0);
    int* boff = reinterpret_cast<int*>(smem + L.off);
    float* bw = reinterpret_cast<float*>(smem + L.wgt);
    float2* x = reinterpret_cast<float2*>(smem + L.bufs) + (size_t)wave * 2 * M;
    float2* y = x + M;
    float* power = reinterpret_cast<float*>(smem + L.power) + (size_t)wave * (M + 1);

    int n = wav_len[b];
    n = n < 0 ? 0 : (n > d.Nmax ? d.Nmax : n);
    int T = n < d.win ? 0 : 1 + (n - d.win) / d.hop;
    T = T > d.Tmax ? d.Tmax : T;
    if (blockIdx.x == 0 && tid == 0) feat_len[b] = T;
    TO* fb = feat + (size_t)b * d.Tmax * d.F;
    if (t0 >= T) {  // nothing but padding in this workgroup's frames
        for (int e = tid; e < d.fpw * d.F; e += 256) {
            const int t = t0 + e / d.F;
            if (t < d.Tmax) store_as(fb + (size_t)t0 * d.F + e, 0.f);
        }
        return;
    }
    // a frame's samples, two a lane and register: the first frame's on their way during the set-up, every next frame's
    // during the frame before
    const float* wb = wav + (size_t)b * d.Nmax;
    constexpr int MOST = 8;  // nfft <= 1024
    float2 pre[MOST];
    auto fetch = [&](int t) {
        const float* seg = wb + (size_t)t * d.hop;
#pragma unroll
        for (int q = 0; q < MOST; ++q) {
            const int e = 2 * (lane + 64 * q);
            pre[q] = make_float2(e < d.win ? seg[e] : 0.f, e + 1 < d.win ? seg[e + 1] : 0.f);
        }
    };
    if (t0 + wave < T) fetch(t0 + wave);
    // ---- per workgroup: twiddles, window, mel points, band weights.  It lasts about as long as two frames' passes, all
    // of it latency, so every part is spread over the threads: the points (a double-precision power each) start from the
    // last thread, the table entries from the first.
    for (int i = 255 - tid; i < d.F + 2; i += 256) {
        const double m = d.mlo + (d.mhi - d.mlo) * (double)i / (double)(d.F + 1);
        pts[i] = (float)(700.0 * (pow(10.0, m / 2595.0) - 1.0));
    }
    for (int k = tid; k <= 3 * N / 4; k += 256) {
        float s, c;
        sincospif(2.f * (float)k / (float)N, &s, &c);  // the argument is an exact binary fraction
        tw[k] = make_float2(c, -s);
    }
    for (int i = tid; i < d.win; i += 256) window[i] = 0.54f - 0.46f * cospif(2.f * (float)i / (float)(d.win - 1));
    __syncthreads();
    const float bin_hz = (float)d.sr / (float)N;
    // bins of a band: a superset of those with a positive weight; thread f takes band f (F <= 255) and the start of its
    // weights is the sum of the counts before it
    int cnt_f = 0;
    if (tid < d.F) {
        int k0 = (int)(pts[tid] / bin_hz), k1 = (int)(pts[tid + 2] / bin_hz) + 1;
        k0 = k0 < 0 ? 0 : k0;
        k1 = k1 > M ? M : k1;
        bk0[tid] = k0;
        cnt_f = k1 - k0 + 1;
    }
    int sum = cnt_f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(sum, o, 64);
        if (lane >= o) sum += v;
    }
    __shared__ int wave_sum[4];
    if (lane == 63) wave_sum[wave] = sum;
    __syncthreads();
    for (int q = 0; q < wave; ++q) sum += wave_sum[q];
    if (tid < d.F) boff[tid + 1] = sum;
    if (tid == 0) boff[0] = 0;
    __syncthreads();
    const int share = 256 / d.F;  // threads per band
    for (int f = tid / share, i0 = tid % share; f < d.F; f += 256) {
        const float lo = pts[f], ce = pts[f + 1], hi = pts[f + 2];
        const float ru = 1.f / (ce - lo), rd = 1.f / (hi - ce);
        const int k0 = bk0[f], cnt = boff[f + 1] - boff[f];
        for (int i = i0; i < cnt; i += share) {
            const float fr = (float)(k0 + i) * bin_hz;
            bw[boff[f] + i] = fmaxf(0.f, fminf((fr - lo) * ru, (hi - fr) * rd));
        }
    }
    __syncthreads();

    for (int t = t0 + wave; t < t0 + d.fpw && t < d.Tmax; t += 4) {
        TO* out = fb + (size_t)t * d.F;
        if (t >= T) {
            for (int f = lane; f < d.F; f += 64) store_as(out + f, 0.f);
            continue;
        }
#pragma unroll
        for (int q = 0; q < MOST; ++q) {
            const int i = lane + 64 * q, e = 2 * i;
            if (i < M) x[i] = make_float2(e < d.win ? pre[q].x * window[e] : 0.f, e + 1 < d.win ? pre[q].y * window[e + 1] : 0.f);
        }
        if (t + 4 < t0 + d.fpw && t + 4 < T) fetch(t + 4);
        __builtin_amdgcn_wave_barrier();
        // Stockham radix-4, decimation in frequency, on M points: at a pass the sequence length is
        // len = M / s; butterfly (p, q), p < len/4, q < s, takes src[q + s (p + r len/4)], r = 0..3,
        // and writes dst[q + s (4p + r)] with the factors exp(-2 pi i r p / len) = tw[2 r p s].
        float2* src = x;
        float2* dst = y;
        int len = M, s = 1, ls = 0;
        for (; len >= 4; len >>= 2, s <<= 2, ls += 2) {
            const int m = len >> 2;
            for (int j = lane; j < (M >> 2); j += 64) {
                const int p = j >> ls, q = j & (s - 1);
                const float2* in = src + q + s * p;
                const float2 a = in[0], bb = in[s * m], c = in[2 * s * m], dd = in[3 * s * m];
                const int ti = 2 * p * s;
                const float2 apc = cadd(a, c), amc = csub(a, c), bpd = cadd(bb, dd), bmd = csub(bb, dd);
                const float2 jbmd = make_float2(-bmd.y, bmd.x);  // i (b - d)
                float2* o = dst + q + s * 4 * p;
                o[0] = cadd(apc, bpd);
                o[s] = cmul(tw[ti], csub(amc, jbmd));
                o[2 * s] = cmul(tw[2 * ti], csub(apc, bpd));
                o[3 * s] = cmul(tw[3 * ti], cadd(amc, jbmd));
            }
            __builtin_amdgcn_wave_barrier();
            float2* tmp = src; src = dst; dst = tmp;
        }
        if (len == 2) {  // one radix-2 pass: s = M / 2
            for (int q = lane; q < s; q += 64) {
                const float2 a = src[q], c = src[q + s];
                dst[q] = cadd(a, c);
                dst[q + s] = csub(a, c);
            }
            __builtin_amdgcn_wave_barrier();
            float2* tmp = src; src = dst; dst = tmp;
        }
        // spectrum of the real frame from the spectrum Z of the packed one:
        //   X[k] = (Z[k] + conj Z[M-k]) / 2 - (i / 2) exp(-2 pi i k / N) (Z[k] - conj Z[M-k]),  k = 0..M
        for (int k = lane; k <= M; k += 64) {
            const float2 zk = src[k & (M - 1)], zm = src[(M - k) & (M - 1)];
            const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
            const float2 o = make_float2(0.5f * (zk.x - zm.x), 0.5f * (zk.y + zm.y));
            const float2 r = cmul(tw[k], make_float2(o.y, -o.x));  // (-i) o, turned by the twiddle
            const float re = e.x + r.x, im = e.y + r.y;
            power[k] = re * re + im * im;
        }
        __builtin_amdgcn_wave_barrier();
        for (int f = lane; f < d.F; f += 64) {
            const int k0 = bk0[f], o0 = boff[f], cnt = boff[f + 1] - o0;
            float acc = 0.f;
#pragma unroll 8
            for (int i = 0; i < cnt; ++i) acc = fmaf(bw[o0 + i], power[k0 + i], acc);
            store_as(out + f, logf(fmaxf(acc, d.floor)));
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- nfft = 512, the usual transform (25 ms at 16 kHz): four frames a wavefront, sixteen lanes a frame.
// Bound by instruction issue, so the transform stays in registers: 256 = 16 x 16 points, a lane takes a 16-point DFT over
// z[16 n1 + r] (r = its place in the frame's sixteen lanes), turns the results by exp(-2 pi i r k1 / 256), trades them for
// the other index through LDS -- the transform's one round trip -- and takes a second 16-point DFT: lane r then holds
// Z[r + 16 k2].  The partner Z[256 - k] that the spectrum of the real frame needs is in lane 16 - r, two DPP moves away,
// and gives the bins k and 256 - k together.  About 250 instructions a frame against 1000 of logmel_k.
// One workgroup of 16 wavefronts a CU shares the tables; its last wavefront makes the band weights (a double-precision
// power per mel point) while the others transform their first frames, and takes frames itself after that.
// 8 x 1500 frames x 80 bands, bf16, a call among others: 22.3 -> 11.6 us; 32 x 2000 frames: 89.3 -> 29.9.
constexpr int WAVES512 = 16, PITCH512 = 17, FRAME512 = 16 * PITCH512;  // float2 of a frame: 16 rows, one of padding each

struct Logmel512Lds { int twa, twb, win, pts, k0, steps, bufs, wgt, total; };  // offsets in bytes
__host__ __device__ inline Logmel512Lds logmel512_lds(int F, int chunks)
{
    Logmel512Lds l;
    int o = 0;
    l.twa = o;   o += 256 * 8;                          // float2 exp(-2 pi i r k1 / 256) at [k1][r]
    l.twb = o;   o += 128 * 8;                          // float2 exp(-2 pi i k / 512)
    l.win = o;   o += 256 * 8;                          // the window, two values an entry, zeros behind it
    l.bufs = o;  o += WAVES512 * 4 * FRAME512 * 8;
    l.wgt = o;   o += chunks * 256;                     // four weights for each of sixteen bands a chunk
    l.pts = o;   o += (F + 2) * 4;
    l.k0 = o;    o += F * 4;                            // int: first bin of a band, a multiple of four
    l.steps = o; o += 17 * 4;                           // int: chunks before the sixteen bands 16 i ..
    l.total = o;
    return l;
}

// a, b, c, d -> their 4-point DFT in order
__device__ __forceinline__ void dft4(float2& a, float2& b, float2& c, float2& d)
{
    const float2 s = cadd(a, c), m = csub(a, c), u = cadd(b, d), v = csub(b, d);
    a = cadd(s, u);
    b = make_float2(m.x + v.y, m.y - v.x);
    c = csub(s, u);
    d = make_float2(m.x - v.y, m.y + v.x);
}
// 16-point DFT; bin k comes out at v[at16(k)]
__device__ constexpr int at16(int k) { return 4 * (k & 3) + (k >> 2); }
__device__ __forceinline__ void dft16(float2 (&v)[16])
{
    constexpr float C1 = 0.92387953251128674f, S1 = 0.38268343236508977f, R = 0.70710678118654752f;  // cos, sin of pi/8; 1/sqrt 2
#pragma unroll
    for (int n = 0; n < 4; ++n) dft4(v[n], v[4 + n], v[8 + n], v[12 + n]);
    auto turn = [](float2 z, float c, float s) { return make_float2(z.x * c + z.y * s, z.y * c - z.x * s); };  // z exp(-i phi)
    auto eighth = [](float2 z) { return make_float2((z.x + z.y) * R, (z.y - z.x) * R); };                     // z exp(-i pi/4)
    v[5] = turn(v[5], C1, S1);
    v[6] = eighth(v[6]);
    v[7] = turn(v[7], S1, C1);
    v[9] = eighth(v[9]);
    v[10] = make_float2(v[10].y, -v[10].x);
    v[11] = make_float2((v[11].y - v[11].x) * R, -(v[11].x + v[11].y) * R);
    v[13] = turn(v[13], S1, C1);
    v[14] = make_float2((v[14].y - v[14].x) * R, -(v[14].x + v[14].y) * R);
    v[15] = turn(v[15], -C1, -S1);
#pragma unroll
    for (int k = 0; k < 4; ++k) dft4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
}
// the value of lane (16 - r) % 16 of the same sixteen lanes
__device__ __forceinline__ float from_partner(float v)
{
    const int m = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140 /* row_mirror */, 0xf, 0xf, true);
    return __int_as_float(__builtin_amdgcn_update_dpp(0, m, 0x121 /* row_ror:1 */, 0xf, 0xf, true));
}
struct __attribute__((packed, aligned(4))) Pair { float x, y; };  // two samples: frames start at any sample

template <typename TO>
__global__ __launch_bounds__(64 * WAVES512) void logmel512_k(const float* __restrict__ wav, const int* __restrict__ wav_len,
                                                             TO* __restrict__ feat, int* __restrict__ feat_len, LogmelDims d)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int next;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, sub = lane >> 4;
    constexpr int M = 256;
    const Logmel512Lds L = logmel512_lds(d.F, d.chunks);
    float2* const twa = reinterpret_cast<float2*>(smem + L.twa);
    float2* const twb = reinterpret_cast<float2*>(smem + L.twb);
    float2* const win2 = reinterpret_cast<float2*>(smem + L.win);
    float* const pts = reinterpret_cast<float*>(smem + L.pts);
    int* const bk0 = reinterpret_cast<int*>(smem + L.k0);
    int* const step = reinterpret_cast<int*>(smem + L.steps);
    float4* const bw = reinterpret_cast<float4*>(smem + L.wgt);
    float2* const z = reinterpret_cast<float2*>(smem + L.bufs) + (size_t)(4 * wave + sub) * FRAME512;  // this lane's frame
    float* const power = reinterpret_cast<float*>(z);  // takes the place of what the second DFT has read

    // the workgroup's groups of four frames; a group lies within one utterance
    const int gpu = (d.Tmax + 3) / 4;  // groups of an utterance
    const int g0 = blockIdx.x * d.fpw, g1 = min(g0 + d.fpw, d.B * gpu);
    struct Frame { int b, t, T; };
    auto frame_of = [&](int g) {
        const int b = g / gpu, t = 4 * (g - b * gpu) + sub;
        int n = wav_len[b];
        n = n < 0 ? 0 : (n > d.Nmax ? d.Nmax : n);
        const int T = n < d.win ? 0 : 1 + (n - d.win) / d.hop;
        return Frame{b, t, min(T, d.Tmax)};
    };
    float2 v[16];
    // Rows of 32 samples.  What lies behind the window repeats its last two samples (the window's zeros drop them), so no
    // lane is masked; frames behind the last of their utterance repeat it (their bands are zeroed below), and a group
    // without any frame is not transformed at all.
    auto fetch = [&](const Frame& f) {
        const float* seg = wav + (size_t)f.b * d.Nmax + (size_t)min(f.t, f.T - 1) * d.hop;
        auto edge = [&](int q) {
            const int e = 32 * q + 2 * r;
            const Pair p = *reinterpret_cast<const Pair*>(seg + min(e, d.win - 2));
            v[q] = make_float2(e == d.win - 1 ? p.y : p.x, p.y);
        };
        if (d.win >= 384) {
#pragma unroll
            for (int q = 0; q < 12; ++q) {
                const Pair p = *reinterpret_cast<const Pair*>(seg + 32 * q + 2 * r);
                v[q] = make_float2(p.x, p.y);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 12; ++q) edge(q);
        }
#pragma unroll
        for (int q = 12; q < 16; ++q) edge(q);
    };
    // everything between the samples and a group's powers in LDS
    auto transform = [&]() {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const float2 w = win2[16 * q + r];
            v[q].x *= w.x;
            v[q].y *= w.y;
        }
        dft16(v);
#pragma unroll
        for (int k = 0; k < 16; ++k) z[k * PITCH512 + r] = k ? cmul(twa[16 * k + r], v[at16(k)]) : v[0];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n = 0; n < 16; ++n) v[n] = z[r * PITCH512 + n];
        __builtin_amdgcn_wave_barrier();
        dft16(v);
        // X[k] = e + w, X[256 - k] = conj(e - w) with e = (Z[k] + conj Z[256-k]) / 2 and
        // w = -(i / 2) exp(-2 pi i k / 512) (Z[k] - conj Z[256-k]).  Lanes r > 0 find Z[256 - k] of k = r + 16 k2 as the
        // partner's bin 15 - k2, lane 0 as its own bin 16 - k2 (bin 0 for k = 0).
#pragma unroll
        for (int k2 = 0; k2 < 8; ++k2) {
            const float2 zk = v[at16(k2)], own = v[at16((16 - k2) & 15)], far = v[at16(15 - k2)];
            const float px = from_partner(far.x), py = from_partner(far.y);
            const float2 zm = r ? make_float2(px, py) : own;
            const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
            const float2 o = make_float2(0.5f * (zk.x - zm.x), 0.5f * (zk.y + zm.y));
            const float2 w = cmul(twb[16 * k2 + r], make_float2(o.y, -o.x));
            const float re = e.x + w.x, im = e.y + w.y, re2 = e.x - w.x, im2 = e.y - w.y;
            power[16 * k2 + r] = re * re + im * im;
            power[M - 16 * k2 - r] = re2 * re2 + im2 * im2;
        }
        if (r == 0) {  // k = 128 is its own partner: X = conj Z
            const float2 zk = v[at16(8)];
            power[128] = zk.x * zk.x + zk.y * zk.y;
        }
        if (r < 15) power[M + 1 + r] = 0.f;  // met by the zero weights behind a band's last bin
        __builtin_amdgcn_wave_barrier();
    };
    // Lane r adds up the bands r, r + 16, ..: in ascending order of the bins, four at a time from a multiple of four on.
    // Sixteen bands take as many steps as the widest of them (zero weights behind the others' last bins), so the loop
    // is uniform.
    auto bands = [&](const Frame& f) {
        if (f.t == 0 && r == 0) feat_len[f.b] = f.T;
        TO* out = feat + ((size_t)f.b * d.Tmax + f.t) * d.F;
        for (int c = r, i = 0; i * 16 < d.F; c += 16, ++i) {
            const int ch = __builtin_amdgcn_readfirstlane(step[i]), n = __builtin_amdgcn_readfirstlane(step[i + 1]) - ch;
            const float4 *p = reinterpret_cast<const float4*>(power + bk0[min(c, d.F - 1)]), *w = bw + ch * 16 + r;
            float acc = 0.f;
#pragma unroll 2
            for (int k = 0; k < n; ++k) {
                const float4 wk = w[16 * k], q = p[k];
                acc = fmaf(wk.w, q.w, fmaf(wk.z, q.z, fmaf(wk.y, q.y, fmaf(wk.x, q.x, acc))));
            }
            if (__builtin_expect(__any(acc != acc), 0)) {  // a power beyond fp32 met a zero weight: the bands' own bins alone
                acc = 0.f;
#pragma unroll 1
                for (int k = 0; k < 4 * n; ++k) {
                    const float wk = reinterpret_cast<const float*>(w + 16 * (k >> 2))[k & 3];
                    acc = wk > 0.f ? fmaf(wk, reinterpret_cast<const float*>(p)[k], acc) : acc;
                }
            }
            if (c < d.F && f.t < d.Tmax) store_as(out + c, f.t < f.T ? logf(fmaxf(acc, d.floor)) : 0.f);
        }
        __builtin_amdgcn_wave_barrier();
    };

    constexpr int FIRST = WAVES512 - 1;  // wavefronts that start with frames
    const bool helper = wave == FIRST;
    Frame f{0, 0, 0};
    int g = g0 + wave;
    const bool work = !helper && g < g1;
    if (work) f = frame_of(g);
    const bool any = __any(f.t < f.T);
    if (any) fetch(f);
    if (tid == 0) next = g0 + FIRST;
    for (int i = tid; i < 640; i += 64 * FIRST) {
        if (helper) break;
        if (i < 384) {  // arguments are exact binary fractions
            const int k = i - 256;
            float s, c;
            sincospif(i < 256 ? (float)((i >> 4) * (i & 15)) / 128.f : (float)k / 256.f, &s, &c);
            twa[i] = make_float2(c, -s);  // twb follows twa
        } else {
            const int e = 2 * (i - 384);
            const float den = (float)(d.win - 1);
            win2[i - 384] = make_float2(e < d.win ? 0.54f - 0.46f * cospif(2.f * (float)e / den) : 0.f,
                                        e + 1 < d.win ? 0.54f - 0.46f * cospif(2.f * (float)(e + 1) / den) : 0.f);
        }
    }
    __syncthreads();
    if (any) transform();
    if (helper) {
        for (int i = lane; i < d.F + 2; i += 64) {
            const double m = d.mlo + (d.mhi - d.mlo) * (double)i / (double)(d.F + 1);
            pts[i] = (float)(700.0 * (pow(10.0, m / 2595.0) - 1.0));
        }
        __builtin_amdgcn_wave_barrier();
        // bins of a band: a superset of those with a positive weight
        const float bin_hz = (float)d.sr / 512.f;
        int base = 0;
        for (int c0 = 0; c0 < d.F; c0 += 64) {
            const int c = c0 + lane;
            int k0 = 0, n = 1;  // sixteen bands have a step at least
            float lo = 0.f, ce = 0.f, hi = 0.f;
            if (c < d.F) {
                lo = pts[c], ce = pts[c + 1], hi = pts[c + 2];
                k0 = (int)(lo / bin_hz);
                int k1 = (int)(hi / bin_hz) + 1;
                k0 = (k0 < 0 ? 0 : k0) & ~3;
                k1 = k1 > M ? M : k1;
                n = (k1 - k0 + 4) >> 2;
                bk0[c] = k0;
            }
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) n = max(n, __shfl_xor(n, o, 64));
            int at = base;  // chunks before this lane's sixteen bands
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int nq = __shfl(n, 16 * q, 64);
                if (q < sub) at += nq;
                base += nq;
            }
            if (r == 0 && c < d.F) {
                step[c >> 4] = at;
                step[(c >> 4) + 1] = at + n;
            }
            const float ru = 1.f / (ce - lo), rd = 1.f / (hi - ce);
            if (c < ((d.F + 15) & ~15)) {
                for (int i = 0; i < n; ++i) {
                    float4 w;
                    float* const wp = &w.x;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int k = k0 + 4 * i + u;
                        const float fr = (float)k * bin_hz;
                        wp[u] = c < d.F && k <= M ? fmaxf(0.f, fminf((fr - lo) * ru, (hi - fr) * rd)) : 0.f;
                    }
                    bw[(at + i) * 16 + r] = w;
                }
            }
        }
    }
    __syncthreads();
    if (work) bands(f);
    for (;;) {
        int mine = 0;
        if (lane == 0) mine = atomicAdd(&next, 1);
        g = __builtin_amdgcn_readfirstlane(mine);
        if (g >= g1) break;
        f = frame_of(g);
        if (__any(f.t < f.T)) {
            fetch(f);
            transform();
        }
        bands(f);
    }
}

}  // namespace
}  // namespace w2l

using namespace w2l;

extern "C" int w2l_logmel_num_frames(int n_samples, int win, int hop)
{
    if (win <= 0 || hop <= 0 || n_samples < win) return 0;
    return 1 + (n_samples - win) / hop;
}

extern "C" int w2l_logmel_fwd(const float* wav, const int* wav_len, void* feat, int* feat_len, int B, int Nmax, int Tmax,
                              int n_mels, int sample_rate, int win, int hop, int nfft, float fmin, float fmax, float floor,
                              int dtype, void* stream)
{
    if (!wav || !wav_len || !feat || !feat_len) return W2L_ERR_NULL;
    if (B <= 0 || B > 65535 || Nmax <= 0 || Tmax <= 0 || n_mels <= 0 || n_mels > 255 || sample_rate <= 0 || win < 2 ||
        hop <= 0 || nfft < 128 || nfft > 1024 || (nfft & (nfft - 1)) || win > nfft || !(fmin >= 0.f) || !(fmax > fmin) ||
        fmax > 0.5f * (float)sample_rate || !(floor > 0.f))
        return W2L_ERR_SHAPE;
    if (!valid_dtype(dtype)) return W2L_ERR_DTYPE;
    LogmelDims d{B, Nmax, Tmax, n_mels, sample_rate, win, hop, nfft, 0, fmin, fmax, floor,
                 2595.0 * std::log10(1.0 + (double)fmin / 700.0), 2595.0 * std::log10(1.0 + (double)fmax / 700.0), 0};
    hipStream_t st = (hipStream_t)stream;
    bool fast = false;
    size_t lds;
    dim3 grid, block;
    if (nfft == 512) {
        // Room for the band weights of logmel512_k: the widest of sixteen neighbouring bands spans two intervals of the mel
        // points, no more than an eighth of the sixteen intervals after it (they grow) or, for the last two sixteens, than
        // the last two; and at most seven bins of slack, in whole fours.
        const double bins = ((double)fmax - (double)fmin) * nfft / sample_rate;
        const double last = ((double)fmax + 700.0) * nfft / sample_rate * (1.0 - std::pow(10.0, -2.0 * (d.mhi - d.mlo) / ((n_mels + 1) * 2595.0)));
        const int sixteens = (n_mels + 15) / 16;
        d.chunks = (int)((bins / 8 + 2 * std::fmin(last, bins)) / 4) + 1 + (sixteens * 11 + 3) / 4;
        lds = (size_t)logmel512_lds(n_mels, d.chunks).total;
        // (few bands spread over the whole spectrum ask for more than a CU has: logmel_k takes them)
        fast = lds <= 159 * 1024 && (long long)B * ((Tmax + 3) / 4) <= 0x7fffffffll - 4096;
    }
    if (fast) {
        // a group of four frames for each of a workgroup's wavefronts once the chip has a workgroup a CU
        const long long groups = (long long)B * ((Tmax + 3) / 4);
        d.fpw = (int)((groups + 255) / 256);
        grid = dim3((unsigned)((groups + d.fpw - 1) / d.fpw));
        block = dim3(64 * WAVES512);
    } else {
        // the per-workgroup set-up is shared by fpw frames; about a thousand workgroups keep four of them
        // (sixteen wavefronts) on every CU, which is what hides the LDS round trips of the FFT passes
        long long fpw = ((long long)B * Tmax + 999) / 1000;
        fpw = fpw < 4 ? 4 : (fpw > 256 ? 256 : fpw);
        d.fpw = (int)((fpw + 3) / 4 * 4);
        lds = (size_t)logmel_lds(nfft, win, n_mels).total;
        grid = dim3((Tmax + d.fpw - 1) / d.fpw, B);
        block = dim3(256);
    }
    const bool bf = dtype == W2L_BF16;
    const void* fn = fast ? (bf ? (const void*)logmel512_k<bf16_t> : (const void*)logmel512_k<float>)
                          : (bf ? (const void*)logmel_k<bf16_t> : (const void*)logmel_k<float>);
    if (lds > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) { note_hip_error(e); return W2L_ERR_LAUNCH; }
    }
    if (fast && bf) hipLaunchKernelGGL(logmel512_k<bf16_t>, grid, block, lds, st, wav, wav_len, (bf16_t*)feat, feat_len, d);
    else if (fast) hipLaunchKernelGGL(logmel512_k<float>, grid, block, lds, st, wav, wav_len, (float*)feat, feat_len, d);
    else if (bf) hipLaunchKernelGGL(logmel_k<bf16_t>, grid, block, lds, st, wav, wav_len, (bf16_t*)feat, feat_len, d);
    else hipLaunchKernelGGL(logmel_k<float>, grid, block, lds, st, wav, wav_len, (float*)feat, feat_len, d);
    return launch_status();
}
