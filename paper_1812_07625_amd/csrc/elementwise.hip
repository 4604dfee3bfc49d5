// Bandwidth-bound kernels of the network: gated linear unit and per-frame log-softmax.
// (The paper's tensor library fuses such chains of simple ops into one kernel, Sec. 2.1;
// here each is one hand-fused pass: every input read once, every output written once.)
#include "common.h"

namespace w2l {
namespace {


// ---- GLU ---------------------------------------------------------------------------
// Vector path: 8 channels per thread (16-byte bf16 loads, 2x16-byte fp32 loads).
struct alignas(16) bf16x8 { bf16_t v[8]; };
struct alignas(16) f32x4 { float v[4]; };

template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> {
    static __device__ __forceinline__ void load(const bf16_t* p, float* o) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        // plain load: the producer kernel has usually just written these values and they are still in the memory-side cache
        const u4 r = *reinterpret_cast<const u4*>(p);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[2 * i] = bf16_to_f32((bf16_t)(r[i] & 0xffffu));
            o[2 * i + 1] = bf16_to_f32((bf16_t)(r[i] >> 16));
        }
    }
    static __device__ __forceinline__ void store(bf16_t* p, const float* o) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        u4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (unsigned)f32_to_bf16(o[2 * i]) | ((unsigned)f32_to_bf16(o[2 * i + 1]) << 16);
        __builtin_nontemporal_store(r, reinterpret_cast<u4*>(p));
    }
};
template <> struct Vec8<float> {
    static __device__ __forceinline__ void load(const float* p, float* o) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 a = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p)), b = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p) + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) { o[i] = a[i]; o[4 + i] = b[i]; }
    }
    static __device__ __forceinline__ void store(float* p, const float* o) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        f4 a, b;
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[i] = o[i]; b[i] = o[4 + i]; }
        __builtin_nontemporal_store(a, reinterpret_cast<f4*>(p));
        __builtin_nontemporal_store(b, reinterpret_cast<f4*>(p) + 1);
    }
};

// Output rows run over every frame of the output allocation: B*pitch + slack frames.  Frame f
// belongs to utterance b = f / pitch at time t = f % pitch - halo; it is real iff 0 <= t < Tp
// (then its dense source row is b*Tp + t), otherwise it is a halo/slack frame and gets zeros.
struct RowMap {
    int Tp, pitch, halo;
    long long real_frames;  // B * pitch
    int live = 1 << 30;     // channels behind the GLU that are there; the others are written as zeros
    // v, values of channels c .., with zeros in those that are not there.  (Rows that have such channels are whole vectors: kernels
    // of one channel a thread go without: 0.4 us of the 81 of a layer of 3 x 731 frames, 200 -> 440, pass by pass.)
    template <int V>
    __device__ __forceinline__ void clear(int c, float (&v)[V]) const
    {
        if (V == 1 || c + V <= live) return;
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = c + j < live ? v[j] : 0.f;
    }
    // IDX: long long, or unsigned where every frame index fits (the 64-bit division is slow)
    template <typename IDX>
    __device__ __forceinline__ long long src(IDX f) const
    {
        if (pitch == Tp) return (long long)f < real_frames ? (long long)f : -1;
        if ((long long)f >= real_frames) return -1;
        const IDX b = f / (IDX)pitch;
        const int t = (int)(f - b * (IDX)pitch) - halo;
        return (t >= 0 && t < Tp) ? (long long)b * Tp + t : -1;
    }
};

// IDX: the type of the flat element index -- unsigned where the element count fits 32 bits (the launchers
// choose): a 64-bit division per element costs more than the rest of the element's work
template <typename T, int V, typename IDX>  // V = 8 (vector path, H % 8 == 0) or 1
__global__ __launch_bounds__(256) void glu_fwd_k(const T* __restrict__ y, T* __restrict__ h, long long out_rows,
                                                 int H, RowMap map)
{
    const int hv = H / V;
    const IDX total = (IDX)(out_rows * hv);
    for (IDX i = blockIdx.x * (IDX)blockDim.x + threadIdx.x; i < total; i += (IDX)gridDim.x * blockDim.x) {
        const IDX f = i / (IDX)hv;
        const int c = (int)(i - f * hv) * V;
        const long long r = map.src(f);
        float o[V];
        if (r >= 0) {
            float a[V], g[V];
            if (V == 8) {
                Vec8<T>::load(y + r * 2 * H + c, a);
                Vec8<T>::load(y + r * 2 * H + H + c, g);
            } else {
                a[0] = Elem<T>::load(y, r * 2 * H + c);
                g[0] = Elem<T>::load(y, r * 2 * H + H + c);
            }
#pragma unroll
            for (int j = 0; j < V; ++j) o[j] = a[j] * sigmoidf_(g[j]);
            map.clear(c, o);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) o[j] = 0.f;
        }
        if (V == 8) Vec8<T>::store(h + (size_t)f * H + c, o);
        else Elem<T>::store(h, (size_t)f * H + c, o[0]);
    }
}

template <typename T, int V, typename IDX>
__global__ __launch_bounds__(256) void glu_bwd_k(const T* __restrict__ y, const T* __restrict__ dh,
                                                 T* __restrict__ dy, long long out_rows, int H, RowMap map)
{
    const int hv = H / V;
    const IDX total = (IDX)(out_rows * hv);
    for (IDX i = blockIdx.x * (IDX)blockDim.x + threadIdx.x; i < total; i += (IDX)gridDim.x * blockDim.x) {
        const IDX f = i / (IDX)hv;
        const int c = (int)(i - f * hv) * V;
        const long long r = map.src(f);
        float da[V], dg[V];
        if (r >= 0) {
            float a[V], g[V], d[V];
            if (V == 8) {
                Vec8<T>::load(y + r * 2 * H + c, a);
                Vec8<T>::load(y + r * 2 * H + H + c, g);
                Vec8<T>::load(dh + r * H + c, d);
            } else {
                a[0] = Elem<T>::load(y, r * 2 * H + c);
                g[0] = Elem<T>::load(y, r * 2 * H + H + c);
                d[0] = Elem<T>::load(dh, r * H + c);
            }
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float sg = sigmoidf_(g[j]);
                da[j] = d[j] * sg;
                dg[j] = d[j] * a[j] * sg * (1.f - sg);
            }
            map.clear(c, da);
            map.clear(c, dg);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) { da[j] = 0.f; dg[j] = 0.f; }
        }
        if (V == 8) {
            Vec8<T>::store(dy + (size_t)f * 2 * H + c, da);
            Vec8<T>::store(dy + (size_t)f * 2 * H + H + c, dg);
        } else {
            Elem<T>::store(dy, (size_t)f * 2 * H + c, da[0]);
            Elem<T>::store(dy, (size_t)f * 2 * H + H + c, dg[0]);
        }
    }
}

// ---- finishing passes of a split reduction --------------------------------------------
// A convolution whose tiles do not fill the chip is cut along its reduction (conv_generic.hip, conv_mfma.hip); the
// planes of fp32 sums are added here, in order, by the pass that would have read the result next.  V consecutive
// values a thread (4 where the row length allows: 16-byte loads); the planes were written by the launch before and
// mostly still lie in the memory-side cache, so what bounds these is the number of loads in flight: a thread's loads
// of up to four planes are issued together.
template <int V> struct FVec { float v[V]; };
template <int V>
__device__ __forceinline__ FVec<V> sum_parts(const float* __restrict__ q, long long plane, int parts)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    FVec<V> o;
#pragma unroll
    for (int j = 0; j < V; ++j) o.v[j] = 0.f;
    int p = 0;
    for (; p + 4 <= parts; p += 4) {
        vec u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = *reinterpret_cast<const vec*>(q + (p + e) * plane);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < V; ++j) o.v[j] += u[e][j];
    }
    for (; p < parts; ++p) {
        const vec u = *reinterpret_cast<const vec*>(q + p * plane);
#pragma unroll
        for (int j = 0; j < V; ++j) o.v[j] += u[j];
    }
    return o;
}
// v rounded to T and back
template <typename T> __device__ __forceinline__ float as_stored(float v) { return v; }
template <> __device__ __forceinline__ float as_stored<bf16_t>(float v) { return bf16_to_f32(f32_to_bf16(v)); }
template <typename T, int V>
__device__ __forceinline__ void store_vec(T* p, const float (&v)[V])
{
    if constexpr (V == 1) Elem<T>::store(p, 0, v[0]);
    else if constexpr (sizeof(T) == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    else *reinterpret_cast<uint2*>(p) = make_uint2((unsigned)f32_to_bf16(v[0]) | ((unsigned)f32_to_bf16(v[1]) << 16),
                                                   (unsigned)f32_to_bf16(v[2]) | ((unsigned)f32_to_bf16(v[3]) << 16));
}
template <typename T, int V>
__device__ __forceinline__ void load_vec(const T* p, float (&v)[V])
{
    if constexpr (V == 1) v[0] = Elem<T>::load(p, 0);
    else if constexpr (sizeof(T) == 4) {
        const float4 u = *reinterpret_cast<const float4*>(p);
        v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
    } else {
        const uint2 u = *reinterpret_cast<const uint2*>(p);
        v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
        v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
    }
}

template <typename T, int V>
__global__ __launch_bounds__(256) void finish_rows_k(const float* __restrict__ part, int parts, const float* __restrict__ bias,
                                                     T* __restrict__ y, unsigned rows, int N, int frames, int pitch, int halo)
{
    const unsigned nv = N / V, total = rows * nv;
    const long long plane = (long long)rows * N;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned r = i / nv, b = r / (unsigned)frames;
        const int c = (int)(i - r * nv) * V;
        FVec<V> s = sum_parts<V>(part + (long long)r * N + c, plane, parts);
        if (bias) {
#pragma unroll
            for (int j = 0; j < V; ++j) s.v[j] += bias[c + j];
        }
        store_vec<T, V>(y + ((long long)b * pitch + halo + (r - b * frames)) * N + c, s.v);
    }
}
template <typename T, int V>
__global__ __launch_bounds__(256) void finish_glu_fwd_k(const float* __restrict__ part, int parts, const float* __restrict__ bias,
                                                        T* __restrict__ y, T* __restrict__ h, unsigned out_rows, int H, RowMap map,
                                                        long long plane)
{
    const unsigned hv = H / V, total = out_rows * hv;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned f = i / hv;
        const int c = (int)(i - f * hv) * V;
        const long long r = map.src(f);
        float o[V];
        if (r >= 0) {
            FVec<V> a = sum_parts<V>(part + r * 2 * H + c, plane, parts), g = sum_parts<V>(part + r * 2 * H + H + c, plane, parts);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                if (bias) { a.v[j] += bias[c + j]; g.v[j] += bias[H + c + j]; }
                o[j] = as_stored<T>(a.v[j]) * sigmoidf_(as_stored<T>(g.v[j]));
            }
            map.clear(c, o);
            store_vec<T, V>(y + r * 2 * H + c, a.v);
            store_vec<T, V>(y + r * 2 * H + H + c, g.v);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) o[j] = 0.f;
        }
        store_vec<T, V>(h + (size_t)f * H + c, o);
    }
}
template <typename T, int V>
__global__ __launch_bounds__(256) void finish_glu_bwd_k(const float* __restrict__ part, int parts, const T* __restrict__ y,
                                                        T* __restrict__ dy, unsigned out_rows, int H, RowMap map, long long plane)
{
    const unsigned hv = H / V, total = out_rows * hv;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const unsigned f = i / hv;
        const int c = (int)(i - f * hv) * V;
        const long long r = map.src(f);
        float da[V], dg[V];
        if (r >= 0) {
            const FVec<V> s = sum_parts<V>(part + r * H + c, plane, parts);
            float a[V], g[V];
            load_vec<T, V>(y + r * 2 * H + c, a);
            load_vec<T, V>(y + r * 2 * H + H + c, g);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float d = as_stored<T>(s.v[j]), sg = sigmoidf_(g[j]);
                da[j] = d * sg;
                dg[j] = d * a[j] * sg * (1.f - sg);
            }
            map.clear(c, da);
            map.clear(c, dg);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) { da[j] = 0.f; dg[j] = 0.f; }
        }
        store_vec<T, V>(dy + (size_t)f * 2 * H + c, da);
        store_vec<T, V>(dy + (size_t)f * 2 * H + H + c, dg);
    }
}
// Data gradient of a narrow 1x1 layer and the GLU backward of the layer below it, in one pass: the classes' layer of a
// network, whose reduction is too short for matrix tiles.  dh[r][c] = sum_q dz[r][q] w[q][c] over C <= 64 outputs, in fp32,
// then dy as in glu_bwd_k.  Bound: the bytes of y and dy (C = 29: 30 multiply-adds a value of dh, about as long as they
// take).  A thread holds four frames of 16 bytes of channels, so that a step of the sum costs two 16-byte LDS reads (dz:
// the same for the frames' threads) for 16 or 32 multiply-adds.  As four launches (dz cast and padded, w padded, matrix
// product, GLU) it took 20 us for 4 x 619 frames of 512 channels, 30 for 16 x 800; now 9
// and 19 (the last: 10 for the bytes, 6 for the products, which a chip full of workgroups that started together takes in
// turn).  (What it costs at 8 to 64 classes: class_bwd_glu_ok.)
template <typename T, int V, int CS>  // CS channel groups of V channels (16 bytes) and 256 / CS groups of four frames
__global__ __launch_bounds__(256) void class_bwd_glu_k(const float* __restrict__ dz, const T* __restrict__ w, const T* __restrict__ y,
                                                       T* __restrict__ dy, unsigned out_rows, int H, int C, RowMap map)
{
    constexpr int R = 4, FR = 256 / CS * R, DP = FR + 4;  // (rows of dz 16 bytes apart from a multiple of all banks)
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* const sz = reinterpret_cast<float*>(smem_raw);                      // [C][DP]
    uint4* const sw = reinterpret_cast<uint4*>(smem_raw + (size_t)C * DP * 4);  // [C][CS]
    const int tid = threadIdx.x, tx = tid % CS, ty = tid / CS;
    const unsigned f0 = blockIdx.x * FR;
    const int c0 = blockIdx.y * CS * V, c = c0 + tx * V;
    const bool live = c < H;
    long long r[R];
    uint4 ya[R], yg[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const unsigned f = f0 + ty * R + u;
        r[u] = f < out_rows ? map.src(f) : -1;
        ya[u] = yg[u] = make_uint4(0, 0, 0, 0);
        if (live && r[u] >= 0) {
            ya[u] = *reinterpret_cast<const uint4*>(y + r[u] * 2 * H + c);
            yg[u] = *reinterpret_cast<const uint4*>(y + r[u] * 2 * H + H + c);
        }
    }
    // dz and w on their way into LDS: all of a thread's loads in flight together
    constexpr int TPR = 256 / FR, NZ = 64 / TPR, NW = 64 * CS / 256;
    const bool wide = (reinterpret_cast<uintptr_t>(w) & 15) == 0;  // (the caller's weights may lie anywhere)
    const int fr = tid / TPR, q0 = tid % TPR;
    const long long row = f0 + fr < out_rows ? map.src(f0 + fr) : -1;
    float z[NZ];
    uint4 wr[NW];
#pragma unroll
    for (int i = 0; i < NZ; ++i) z[i] = row >= 0 && q0 + TPR * i < C ? dz[row * C + q0 + TPR * i] : 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int e = tid + 256 * i, ch = c0 + e % CS * V;
        const T* const src = w + (size_t)(e / CS) * H + ch;
        wr[i] = make_uint4(0, 0, 0, 0);
        if (e < C * CS && ch < H) {
            if (wide) wr[i] = *reinterpret_cast<const uint4*>(src);
            else {
                T t[V];
#pragma unroll
                for (int j = 0; j < V; ++j) t[j] = src[j];
                __builtin_memcpy(&wr[i], t, 16);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NZ; ++i)
        if (q0 + TPR * i < C) sz[(q0 + TPR * i) * DP + fr] = z[i];
#pragma unroll
    for (int i = 0; i < NW; ++i)
        if (tid + 256 * i < C * CS) sw[tid + 256 * i] = wr[i];
    __syncthreads();
    auto widen = [](const uint4& q, float (&o)[V]) {
        const unsigned* b = &q.x;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            if constexpr (sizeof(T) == 4) o[j] = __uint_as_float(b[j]);
            else o[j] = __uint_as_float((j & 1) ? b[j / 2] & 0xffff0000u : b[j / 2] << 16);
        }
    };
    float acc[R][V];
#pragma unroll
    for (int u = 0; u < R; ++u)
#pragma unroll
        for (int j = 0; j < V; ++j) acc[u][j] = 0.f;
#pragma unroll 4
    for (int q = 0; q < C; ++q) {
        const float4 d4 = *reinterpret_cast<const float4*>(sz + q * DP + ty * R);
        const float* const d = &d4.x;
        float wv[V];
        widen(sw[q * CS + tx], wv);
#pragma unroll
        for (int u = 0; u < R; ++u)
#pragma unroll
            for (int j = 0; j < V; ++j) acc[u][j] = __builtin_fmaf(d[u], wv[j], acc[u][j]);
    }
    if (!live) return;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const unsigned f = f0 + ty * R + u;
        if (f >= out_rows) continue;
        float a[V], g[V], da[V], dg[V];
        widen(ya[u], a);
        widen(yg[u], g);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float sg = sigmoidf_(g[j]);
            da[j] = r[u] >= 0 ? acc[u][j] * sg : 0.f;
            dg[j] = r[u] >= 0 ? acc[u][j] * a[j] * sg * (1.f - sg) : 0.f;
        }
        map.clear(c, da);
        map.clear(c, dg);
        auto narrow = [](const float (&v)[V]) {
            uint4 q;
            unsigned* const b = &q.x;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (sizeof(T) == 4) b[j] = __float_as_uint(v[j]);
                else b[j] = (unsigned)f32_to_bf16(v[2 * j]) | ((unsigned)f32_to_bf16(v[2 * j + 1]) << 16);
            }
            return q;
        };
        T* const o = dy + (size_t)f * 2 * H + c;
        *reinterpret_cast<uint4*>(o) = narrow(da);
        *reinterpret_cast<uint4*>(o + H) = narrow(dg);
    }
}
template <int V>
__global__ __launch_bounds__(256) void finish_sums_k(const float* __restrict__ part, int parts, long long n, float* __restrict__ out,
                                                     const float* __restrict__ bpart, int nb, float* __restrict__ bout, int accumulate)
{
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x, nv = n / V;
    if (t < nv) {
        FVec<V> s = sum_parts<V>(part + t * V, n, parts);
        if (accumulate) {
#pragma unroll
            for (int j = 0; j < V; ++j) s.v[j] += out[t * V + j];
        }
        store_vec<float, V>(out + t * V, s.v);
    } else if (bout && t - nv < nb) {
        const int c = (int)(t - nv);
        const FVec<1> s = sum_parts<1>(bpart + c, nb, parts);
        bout[c] = accumulate ? bout[c] + s.v[0] : s.v[0];
    }
}

// dense [B*Tp, C] -> haloed layout (zeros in halo and slack frames); C % 8 == 0, bf16
__global__ __launch_bounds__(256) void pad_layout_k(const bf16_t* __restrict__ src, bf16_t* __restrict__ dst,
                                                    long long out_rows, int C, RowMap map, int* __restrict__ clear,
                                                    int nclear)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nclear; i += blockDim.x) clear[i] = 0;
    const int cv = C / 8;
    const long long total = out_rows * cv;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long f = i / cv;
        const int c = (int)(i - f * cv) * 8;
        const long long r = map.src(f);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r >= 0) v = *reinterpret_cast<const uint4*>(src + r * C + c);
        *reinterpret_cast<uint4*>(dst + f * C + c) = v;
    }
}

// two tensors with the same time layout in one launch (the weight gradient stages x and dy)
__global__ __launch_bounds__(256) void pad_layout2_k(const bf16_t* __restrict__ src0, bf16_t* __restrict__ dst0, int C0,
                                                     const bf16_t* __restrict__ src1, bf16_t* __restrict__ dst1, int C1,
                                                     long long out_rows, RowMap map)
{
    const int cv0 = C0 / 8, cv1 = C1 / 8;
    const long long n0 = out_rows * cv0, total = n0 + out_rows * cv1;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const bool second = i >= n0;
        const long long e = second ? i - n0 : i;
        const int cv = second ? cv1 : cv0, C = second ? C1 : C0;
        const bf16_t* src = second ? src1 : src0;
        bf16_t* dst = second ? dst1 : dst0;
        const long long f = e / cv;
        const int c = (int)(e - f * cv) * 8;
        const long long r = map.src(f);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r >= 0) v = *reinterpret_cast<const uint4*>(src + r * C + c);
        *reinterpret_cast<uint4*>(dst + f * C + c) = v;
    }
}

// the same for any dtype and channel count, one element per thread
template <typename T>
__global__ __launch_bounds__(256) void pad_layout_any_k(const T* __restrict__ src, T* __restrict__ dst, long long out_rows,
                                                        int C, RowMap map)
{
    const long long total = out_rows * C;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long f = i / C;
        const long long r = map.src(f);
        dst[i] = r >= 0 ? src[r * C + (i - f * C)] : T(0);
    }
}

// Operand preparation for data gradients the MFMA kernels do not take as they come (fp32 dy, a channel count that
// is not a multiple of 64, a strided layer): dy -> bf16, haloed, channels padded with zeros to Cp.
template <typename T>
__global__ __launch_bounds__(256) void prep_dy_k(const T* __restrict__ src, bf16_t* __restrict__ dst, long long out_rows,
                                                 int C, int Cp, RowMap map, int* __restrict__ clear, int nclear)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nclear; i += blockDim.x) clear[i] = 0;
    // one thread writes 8 channels (16 bytes); Cp is a multiple of 64
    const int cv = Cp / 8;
    const long long total = out_rows * cv;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long f = i / cv;
        const int c = (int)(i - f * cv) * 8;
        const long long r = map.src(f);
        bf16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = (r >= 0 && c + e < C) ? f32_to_bf16(Elem<T>::load(src, r * C + c + e)) : (bf16_t)0;
        *reinterpret_cast<uint4*>(dst + f * Cp + c) = *reinterpret_cast<const uint4*>(v);
    }
}
// w[Cout][k][Cin] -> w'[Cp][kf][s * Cin]: w'[co][jj][ph * Cin + ci] = w[co][s * jj + ph][ci], zero where the tap
// s * jj + ph does not exist or co >= Cout (s = 1: a copy with zero rows appended).
// (A folded row w'[co] is w[co] as it lies in memory with zeros behind: s jj + ph is the tap.)  Bound by its latency: 16 bytes
// a thread, where source rows start on them; an element a thread took 5.6 us for 440 x 13 x 200 weights, now 3.1.
__global__ __launch_bounds__(256) void prep_w_k(const bf16_t* __restrict__ w, bf16_t* __restrict__ dst, int Cout, int row, int Cp, int out_row)
{
    const unsigned cv = out_row / 8, total = (unsigned)Cp * cv;  // (out_row is a multiple of 8; fewer than 2^30 values)
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        const int co = (int)(i / cv), e = (int)(i - co * cv) * 8, left = co < Cout ? row - e : 0;
        const bf16_t* const src = w + (size_t)co * row + e;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (left >= 8 && (reinterpret_cast<uintptr_t>(src) & 15) == 0) v = *reinterpret_cast<const uint4*>(src);
        else {
            unsigned* const q = &v.x;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u < left) q[u / 2] |= (unsigned)src[u] << (16 * (u & 1));
        }
        *reinterpret_cast<uint4*>(dst + (size_t)i * 8) = v;
    }
}

inline unsigned grid_for(long long items)
{
    long long b = (items + 255) / 256;
    const long long cap = 256 * 16;  // 16 workgroups per CU keep enough loads in flight
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// ---- log-softmax: one wavefront per row ----------------------------------------------
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T>
__global__ __launch_bounds__(256) void logsoftmax_fwd_k(const T* __restrict__ z, float* __restrict__ lp,
                                                        long long rows, int C)
{
    const int lane = threadIdx.x & 63;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
    const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
    for (long long r = wave; r < rows; r += nwaves) {
        const T* zr = z + r * C;
        float m = -INFINITY;
        for (int c = lane; c < C; c += 64) m = fmaxf(m, Elem<T>::load(zr, c));
        m = wave_max(m);
        float s = 0.f;
        for (int c = lane; c < C; c += 64) s += expf(Elem<T>::load(zr, c) - m);
        s = wave_sum(s);
        const float lse = m + logf(s);
        for (int c = lane; c < C; c += 64) lp[r * C + c] = Elem<T>::load(zr, c) - lse;
    }
}
__global__ __launch_bounds__(256) void logsoftmax_bwd_k(const float* __restrict__ lp,
                                                        const float* __restrict__ dlp,
                                                        float* __restrict__ dz, long long rows, int C)
{
    const int lane = threadIdx.x & 63;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
    const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
    for (long long r = wave; r < rows; r += nwaves) {
        float s = 0.f;
        for (int c = lane; c < C; c += 64) s += dlp[r * C + c];
        s = wave_sum(s);
        for (int c = lane; c < C; c += 64) dz[r * C + c] = dlp[r * C + c] - expf(lp[r * C + c]) * s;
    }
}

// Rows of up to 64 classes: sixteen lanes a row, up to four values each.  A wavefront per row is bound by latency -- 24000 rows
// of 29 are three rounds of what the chip holds -- and most of its lanes have nothing to load.
// 24000 x 29 by the launch's trace: forward 7.6 -> 4.3 us, backward 6.2 -> 4.3; 750 x 29: 3.1 -> 2.9, 2.9 -> 3.0 (the floor).
constexpr int ROW_LANES = 16, ROW_VALUES = 4;
__device__ __forceinline__ float row16_max(float v)
{
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, ROW_LANES));
    return v;
}
__device__ __forceinline__ float row16_sum(float v)
{
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, ROW_LANES);
    return v;
}
template <typename T>
__global__ __launch_bounds__(256) void logsoftmax_fwd_narrow_k(const T* __restrict__ z, float* __restrict__ lp, long long rows, int C)
{
    const int l = threadIdx.x % ROW_LANES;
    const long long stride = (long long)gridDim.x * (256 / ROW_LANES);
    for (long long r = blockIdx.x * (long long)(256 / ROW_LANES) + threadIdx.x / ROW_LANES; r < rows; r += stride) {
        float v[ROW_VALUES], m = -INFINITY, s = 0.f;
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q) v[q] = l + ROW_LANES * q < C ? Elem<T>::load(z + r * C, l + ROW_LANES * q) : -INFINITY;
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q) m = fmaxf(m, v[q]);
        m = row16_max(m);
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q) s += l + ROW_LANES * q < C ? expf(v[q] - m) : 0.f;
        const float lse = m + logf(row16_sum(s));
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q)
            if (l + ROW_LANES * q < C) lp[r * C + l + ROW_LANES * q] = v[q] - lse;
    }
}
__global__ __launch_bounds__(256) void logsoftmax_bwd_narrow_k(const float* __restrict__ lp, const float* __restrict__ dlp, float* __restrict__ dz,
                                                               long long rows, int C)
{
    const int l = threadIdx.x % ROW_LANES;
    const long long stride = (long long)gridDim.x * (256 / ROW_LANES);
    for (long long r = blockIdx.x * (long long)(256 / ROW_LANES) + threadIdx.x / ROW_LANES; r < rows; r += stride) {
        float g[ROW_VALUES], p[ROW_VALUES], s = 0.f;
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q) {
            const bool on = l + ROW_LANES * q < C;
            g[q] = on ? dlp[r * C + l + ROW_LANES * q] : 0.f;
            p[q] = on ? lp[r * C + l + ROW_LANES * q] : 0.f;
            s += g[q];
        }
        s = row16_sum(s);
#pragma unroll
        for (int q = 0; q < ROW_VALUES; ++q)
            if (l + ROW_LANES * q < C) dz[r * C + l + ROW_LANES * q] = g[q] - expf(p[q]) * s;
    }
}

}  // namespace
}  // namespace w2l

using namespace w2l;

namespace w2l {

namespace {
template <typename T, int V, typename IDX>
void launch_glu_fwd(dim3 g, hipStream_t st, const void* y, void* h, long long out_rows, int H, const RowMap& map)
{
    hipLaunchKernelGGL((glu_fwd_k<T, V, IDX>), g, dim3(256), 0, st, (const T*)y, (T*)h, out_rows, H, map);
}
template <typename T, int V, typename IDX>
void launch_glu_bwd(dim3 g, hipStream_t st, const void* y, const void* dh, void* dy, long long out_rows, int H, const RowMap& map)
{
    hipLaunchKernelGGL((glu_bwd_k<T, V, IDX>), g, dim3(256), 0, st, (const T*)y, (const T*)dh, (T*)dy, out_rows, H, map);
}
}  // namespace

int glu_fwd_layout(const void* y, void* h, int B, int Tp, int Cout, int dtype, int pitch, int halo, int slack,
                   hipStream_t st, int live)
{
    const int H = Cout / 2;
    const bool vec = (H % 8) == 0;
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch, live > 0 ? live : H};
    const long long items = vec ? out_rows * (H / 8) : out_rows * H;
    const dim3 g(grid_for(items));
    const bool small = items < (1LL << 31);  // 32-bit element indices
#define W2L_GLU(T_, V_)                                                                    \
    {                                                                                      \
        if (small) launch_glu_fwd<T_, V_, unsigned>(g, st, y, h, out_rows, H, map);        \
        else launch_glu_fwd<T_, V_, long long>(g, st, y, h, out_rows, H, map);             \
    }
    if (dtype == W2L_BF16) {
        if (vec) W2L_GLU(bf16_t, 8) else W2L_GLU(bf16_t, 1)
    } else {
        if (vec) W2L_GLU(float, 8) else W2L_GLU(float, 1)
    }
#undef W2L_GLU
    return launch_status();
}

int glu_bwd_layout(const void* y, const void* dh, void* dy, int B, int Tp, int Cout, int dtype, int pitch, int halo,
                   int slack, hipStream_t st, int live)
{
    const int H = Cout / 2;
    const bool vec = (H % 8) == 0;
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch, live > 0 ? live : H};
    const long long items = vec ? out_rows * (H / 8) : out_rows * H;
    const dim3 g(grid_for(items));
    const bool small = items < (1LL << 31);
#define W2L_GLU(T_, V_)                                                                    \
    {                                                                                      \
        if (small) launch_glu_bwd<T_, V_, unsigned>(g, st, y, dh, dy, out_rows, H, map);   \
        else launch_glu_bwd<T_, V_, long long>(g, st, y, dh, dy, out_rows, H, map);        \
    }
    if (dtype == W2L_BF16) {
        if (vec) W2L_GLU(bf16_t, 8) else W2L_GLU(bf16_t, 1)
    } else {
        if (vec) W2L_GLU(float, 8) else W2L_GLU(float, 1)
    }
#undef W2L_GLU
    return launch_status();
}

}  // namespace w2l

namespace w2l {
int finish_rows(const float* part, int parts, const float* bias, void* y, int dtype, int B, int frames, int N, int pitch, int halo,
                hipStream_t st)
{
    const unsigned rows = (unsigned)B * frames;
    const bool vec = N % 4 == 0;
    const dim3 g(grid_for((long long)rows * (vec ? N / 4 : N))), b(256);
#define W2L_FIN(T_, V_) hipLaunchKernelGGL((finish_rows_k<T_, V_>), g, b, 0, st, part, parts, bias, (T_*)y, rows, N, frames, pitch, halo)
    if (dtype == W2L_BF16) { if (vec) W2L_FIN(bf16_t, 4); else W2L_FIN(bf16_t, 1); }
    else { if (vec) W2L_FIN(float, 4); else W2L_FIN(float, 1); }
#undef W2L_FIN
    return launch_status();
}
int finish_glu_fwd(const float* part, int parts, const float* bias, void* y, void* h, int B, int Tp, int Cout, int dtype, int pitch,
                   int halo, int slack, hipStream_t st, int live)
{
    const int H = Cout / 2;
    const bool vec = H % 4 == 0;
    const unsigned out_rows = (unsigned)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch, live > 0 ? live : H};
    const long long plane = (long long)B * Tp * Cout;
    const dim3 g(grid_for((long long)out_rows * (vec ? H / 4 : H))), b(256);
#define W2L_FIN(T_, V_) hipLaunchKernelGGL((finish_glu_fwd_k<T_, V_>), g, b, 0, st, part, parts, bias, (T_*)y, (T_*)h, out_rows, H, map, plane)
    if (dtype == W2L_BF16) { if (vec) W2L_FIN(bf16_t, 4); else W2L_FIN(bf16_t, 1); }
    else { if (vec) W2L_FIN(float, 4); else W2L_FIN(float, 1); }
#undef W2L_FIN
    return launch_status();
}
int finish_glu_bwd(const float* part, int parts, const void* y, void* dy, int B, int Tp, int Cout, int dtype, int pitch, int halo,
                   int slack, hipStream_t st, int live)
{
    const int H = Cout / 2;
    const bool vec = H % 4 == 0;
    const unsigned out_rows = (unsigned)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch, live > 0 ? live : H};
    const long long plane = (long long)B * Tp * H;
    const dim3 g(grid_for((long long)out_rows * (vec ? H / 4 : H))), b(256);
#define W2L_FIN(T_, V_) hipLaunchKernelGGL((finish_glu_bwd_k<T_, V_>), g, b, 0, st, part, parts, (const T_*)y, (T_*)dy, out_rows, H, map, plane)
    if (dtype == W2L_BF16) { if (vec) W2L_FIN(bf16_t, 4); else W2L_FIN(bf16_t, 1); }
    else { if (vec) W2L_FIN(float, 4); else W2L_FIN(float, 1); }
#undef W2L_FIN
    return launch_status();
}
// Up to 64 classes; beyond, the matrix kernels (conv_dgrad) are for it.  Steps of a network of one 1x1 layer, us, as launches of
// their own and as one, 200 / 1600 / 12800 frames: bf16, H = 256, 8 classes 82 -> 74, 98 -> 90, 205 -> 189; 64 classes 78 -> 77, 91 -> 90,
// 207 -> 197; H = 2048 82 -> 81, 135 -> 132, 429 -> 417.  fp32, H = 256, 48 classes 64 -> 64, 86 -> 85, 184 -> 175; 64 classes 64 -> 65,
// 85 -> 87, 183 -> 180; H = 1024 64 -> 65, 104 -> 102, 350 -> 321; H = 64, 51200 frames 431 -> 442: of fp32, beyond 48 classes, only
// where there is enough of dh.  (A launch has fewer than 2^32 threads: 8 a frame of out_rows.)
bool class_bwd_glu_ok(int B, int pitch, int slack, int C, int H, int dtype)
{
    const bool bf16 = dtype == W2L_BF16;
    const long long rows = (long long)B * pitch;
    return C <= 64 && (bf16 || C <= 48 || (H >= 128 && rows * H >= 1 << 20)) && H % (bf16 ? 8 : 4) == 0 && rows + slack <= (1LL << 29) - 32;
}
int class_bwd_glu(const float* dz, const void* w, const void* y, void* dy, int B, int Tp, int C, int H, int dtype, int pitch, int halo, int slack,
                  hipStream_t st, int live)
{
    if (!class_bwd_glu_ok(B, pitch, slack, C, H, dtype)) return W2L_ERR_SHAPE;
    const unsigned out_rows = (unsigned)((long long)B * pitch + slack);
    const RowMap map{Tp, pitch, halo, (long long)B * pitch, live > 0 ? live : H};
    const bool bf16 = dtype == W2L_BF16;
    const int groups = H / (bf16 ? 8 : 4);
    // 32 groups of channels and 32 frames a workgroup, or 16 and 64 where a row has fewer
#define W2L_CLS(T_, V_, CS_)                                                                                                    \
    {                                                                                                                           \
        constexpr int FR = 256 / CS_ * 4;                                                                                       \
        const dim3 g((out_rows + FR - 1) / FR, (unsigned)((groups + CS_ - 1) / CS_));                                           \
        hipLaunchKernelGGL((class_bwd_glu_k<T_, V_, CS_>), g, dim3(256), (size_t)C * ((FR + 4) * 4 + CS_ * 16), st, dz,         \
                           (const T_*)w, (const T_*)y, (T_*)dy, out_rows, H, C, map);                                           \
    }
    if (bf16) { if (groups > 16) W2L_CLS(bf16_t, 8, 32) else W2L_CLS(bf16_t, 8, 16) }
    else { if (groups > 16) W2L_CLS(float, 4, 32) else W2L_CLS(float, 4, 16) }
#undef W2L_CLS
    return launch_status();
}
int finish_sums(const float* part, int parts, long long n, float* out, const float* bpart, int nb, float* bout, int accumulate,
                hipStream_t st)
{
    if (!bout) nb = 0;
    const bool vec = n % 4 == 0;
    const long long items = (vec ? n / 4 : n) + nb, blocks = (items + 255) / 256;
    if (blocks > 2147483647LL) return W2L_ERR_SHAPE;
    if (vec) hipLaunchKernelGGL(finish_sums_k<4>, dim3((unsigned)blocks), dim3(256), 0, st, part, parts, n, out, bpart, nb, bout, accumulate);
    else hipLaunchKernelGGL(finish_sums_k<1>, dim3((unsigned)blocks), dim3(256), 0, st, part, parts, n, out, bpart, nb, bout, accumulate);
    return launch_status();
}

int pad_layout_bf16(const void* src, void* dst, int B, int Tp, int C, int pitch, int halo, int slack, hipStream_t st,
                    int* clear, int nclear)
{
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch};
    hipLaunchKernelGGL(pad_layout_k, dim3(grid_for(out_rows * (C / 8))), dim3(256), 0, st, (const bf16_t*)src,
                       (bf16_t*)dst, out_rows, C, map, clear, nclear);
    return launch_status();
}

int pad_layout(const void* src, void* dst, int B, int Tp, int C, int dtype, int pitch, int halo, int slack, hipStream_t st)
{
    if (dtype == W2L_BF16 && C % 8 == 0) return pad_layout_bf16(src, dst, B, Tp, C, pitch, halo, slack, st);
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch};
    const dim3 g(grid_for(out_rows * C)), b(256);
    if (dtype == W2L_BF16)
        hipLaunchKernelGGL(pad_layout_any_k<bf16_t>, g, b, 0, st, (const bf16_t*)src, (bf16_t*)dst, out_rows, C, map);
    else
        hipLaunchKernelGGL(pad_layout_any_k<float>, g, b, 0, st, (const float*)src, (float*)dst, out_rows, C, map);
    return launch_status();
}

int prep_dgrad_dy(const void* src, int src_dtype, void* dst, int B, int Tp, int C, int Cp, int pitch, int halo, int slack,
                  hipStream_t st, int* clear, int nclear)
{
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch};
    if (src_dtype == W2L_BF16 && C == Cp) return pad_layout_bf16(src, dst, B, Tp, C, pitch, halo, slack, st, clear, nclear);
    const dim3 g(grid_for(out_rows * (Cp / 8))), b(256);
    if (src_dtype == W2L_BF16)
        hipLaunchKernelGGL(prep_dy_k<bf16_t>, g, b, 0, st, (const bf16_t*)src, (bf16_t*)dst, out_rows, C, Cp, map, clear, nclear);
    else
        hipLaunchKernelGGL(prep_dy_k<float>, g, b, 0, st, (const float*)src, (bf16_t*)dst, out_rows, C, Cp, map, clear, nclear);
    return launch_status();
}

int prep_dgrad_w(const void* w, void* dst, int Cout, int k, int Cin, int Cp, int kf, int s, hipStream_t st)
{
    const int out_row = kf * s * Cin;
    if (out_row % 8 || kf * s < k) return W2L_ERR_SHAPE;
    hipLaunchKernelGGL(prep_w_k, dim3(grid_for((long long)Cp * (out_row / 8))), dim3(256), 0, st, (const bf16_t*)w, (bf16_t*)dst, Cout, k * Cin,
                       Cp, out_row);
    return launch_status();
}

int pad_layout2_bf16(const void* src0, void* dst0, int C0, const void* src1, void* dst1, int C1, int B, int Tp, int pitch,
                     int halo, int slack, hipStream_t st)
{
    if (C0 % 8 || C1 % 8) return W2L_ERR_SHAPE;
    const long long out_rows = (long long)B * pitch + slack;
    const RowMap map{Tp, pitch, halo, (long long)B * pitch};
    hipLaunchKernelGGL(pad_layout2_k, dim3(grid_for(out_rows * ((C0 + C1) / 8))), dim3(256), 0, st, (const bf16_t*)src0,
                       (bf16_t*)dst0, C0, (const bf16_t*)src1, (bf16_t*)dst1, C1, out_rows, map);
    return launch_status();
}
}  // namespace w2l

extern "C" int w2l_glu_fwd(const void* y, void* h, long long rows, int Cout, int dtype, void* stream)
{
    if (!y || !h) return W2L_ERR_NULL;
    if (rows <= 0 || rows > 2147483647LL || Cout <= 0 || (Cout & 1)) return W2L_ERR_SHAPE;
    if (!valid_dtype(dtype)) return W2L_ERR_DTYPE;
    if (!aligned16(y) || !aligned16(h)) return W2L_ERR_ALIGN;
    return glu_fwd_layout(y, h, 1, (int)rows, Cout, dtype, (int)rows, 0, 0, (hipStream_t)stream);
}

extern "C" int w2l_glu_bwd(const void* y, const void* dh, void* dy, long long rows, int Cout, int dtype,
                           void* stream)
{
    if (!y || !dh || !dy) return W2L_ERR_NULL;
    if (rows <= 0 || rows > 2147483647LL || Cout <= 0 || (Cout & 1)) return W2L_ERR_SHAPE;
    if (!valid_dtype(dtype)) return W2L_ERR_DTYPE;
    if (!aligned16(y) || !aligned16(dh) || !aligned16(dy)) return W2L_ERR_ALIGN;
    return glu_bwd_layout(y, dh, dy, 1, (int)rows, Cout, dtype, (int)rows, 0, 0, (hipStream_t)stream);
}

extern "C" int w2l_logsoftmax_fwd(const void* z, float* lp, long long rows, int C, int z_dtype, void* stream)
{
    if (!z || !lp) return W2L_ERR_NULL;
    if (rows <= 0 || C <= 0 || C > 4096) return W2L_ERR_SHAPE;
    if (!valid_dtype(z_dtype)) return W2L_ERR_DTYPE;
    if (!aligned16(z) || !aligned16(lp)) return W2L_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    const bool narrow = C <= ROW_LANES * ROW_VALUES;
    const dim3 g(grid_for(rows * (narrow ? ROW_LANES : 64))), b(256);
    if (narrow && z_dtype == W2L_BF16)
        hipLaunchKernelGGL(logsoftmax_fwd_narrow_k<bf16_t>, g, b, 0, st, (const bf16_t*)z, lp, rows, C);
    else if (narrow)
        hipLaunchKernelGGL(logsoftmax_fwd_narrow_k<float>, g, b, 0, st, (const float*)z, lp, rows, C);
    else if (z_dtype == W2L_BF16)
        hipLaunchKernelGGL(logsoftmax_fwd_k<bf16_t>, g, b, 0, st, (const bf16_t*)z, lp, rows, C);
    else
        hipLaunchKernelGGL(logsoftmax_fwd_k<float>, g, b, 0, st, (const float*)z, lp, rows, C);
    return launch_status();
}

extern "C" int w2l_logsoftmax_bwd(const float* lp, const float* dlp, float* dz, long long rows, int C,
                                  void* stream)
{
    if (!lp || !dlp || !dz) return W2L_ERR_NULL;
    if (rows <= 0 || C <= 0 || C > 4096) return W2L_ERR_SHAPE;
    if (!aligned16(lp) || !aligned16(dlp) || !aligned16(dz)) return W2L_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    if (C <= ROW_LANES * ROW_VALUES)
        hipLaunchKernelGGL(logsoftmax_bwd_narrow_k, dim3(grid_for(rows * ROW_LANES)), dim3(256), 0, st, lp, dlp, dz, rows, C);
    else
        hipLaunchKernelGGL(logsoftmax_bwd_k, dim3(grid_for(rows * 64)), dim3(256), 0, st, lp, dlp, dz, rows, C);
    return launch_status();
}

// ---- SGD with momentum ----------------------------------------------------------------
// 22 bytes of HBM traffic per parameter (read w, v, grad; write w, v and the bf16 copy): 16-byte accesses, two
// groups of four parameters per thread (a whole grid apart, all six loads issued before the first use) and a grid
// that covers the tensor in one pass.  A wavefront that loads, computes, stores and ends keeps more of the memory
// system busy than one that loops: 6.4 TB/s against 4.6 for a grid-stride loop over a grid capped at 4096 blocks.
namespace {
constexpr int SGD_PER_THREAD = 2;
__global__ __launch_bounds__(256) void sgd_momentum_k(float* __restrict__ w, float* __restrict__ v,
                                                      const float* __restrict__ g, w2l::bf16_t* __restrict__ lowp,
                                                      long long n, float lr, float mu, float wd)
{
    const long long n4 = n / 4;
    // every value is touched exactly once: streaming (non-temporal) loads and stores keep it out of the caches
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const long long t0 = blockIdx.x * (long long)blockDim.x + threadIdx.x, stride = (long long)gridDim.x * blockDim.x;
    f4 wv[SGD_PER_THREAD], vv[SGD_PER_THREAD], gv[SGD_PER_THREAD];
#pragma unroll
    for (int u = 0; u < SGD_PER_THREAD; ++u) {
        const long long i = t0 + u * stride;
        if (i < n4) {
            wv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(w) + i);
            vv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(v) + i);
            gv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g) + i);
        }
    }
#pragma unroll
    for (int u = 0; u < SGD_PER_THREAD; ++u) {
        const long long i = t0 + u * stride;
        if (i < n4) {
            f4 &wq = wv[u], &vq = vv[u];
            const f4 gq = gv[u];
            vq.x = mu * vq.x + (gq.x + wd * wq.x); wq.x -= lr * vq.x;
            vq.y = mu * vq.y + (gq.y + wd * wq.y); wq.y -= lr * vq.y;
            vq.z = mu * vq.z + (gq.z + wd * wq.z); wq.z -= lr * vq.z;
            vq.w = mu * vq.w + (gq.w + wd * wq.w); wq.w -= lr * vq.w;
            __builtin_nontemporal_store(wq, reinterpret_cast<f4*>(w) + i);
            __builtin_nontemporal_store(vq, reinterpret_cast<f4*>(v) + i);
            if (lowp) {
                u2 o;
                o.x = (unsigned)w2l::f32_to_bf16(wq.x) | ((unsigned)w2l::f32_to_bf16(wq.y) << 16);
                o.y = (unsigned)w2l::f32_to_bf16(wq.z) | ((unsigned)w2l::f32_to_bf16(wq.w) << 16);
                __builtin_nontemporal_store(o, reinterpret_cast<u2*>(lowp) + i);
            }
        }
    }
    // tail (n % 4 values)
    const long long t = n4 * 4 + t0;
    if (t < n) {
        const float vn = mu * v[t] + (g[t] + wd * w[t]);
        const float wn = w[t] - lr * vn;
        v[t] = vn;
        w[t] = wn;
        if (lowp) lowp[t] = w2l::f32_to_bf16(wn);
    }
}
}  // namespace

extern "C" int w2l_sgd_momentum_step(float* w, float* v, const float* grad, void* w_lowp, long long n, float lr,
                                     float momentum, float weight_decay, void* stream)
{
    using namespace w2l;
    if (!w || !v || !grad) return W2L_ERR_NULL;
    if (n < 0) return W2L_ERR_SHAPE;
    if (!aligned16(w) || !aligned16(v) || !aligned16(grad) || (w_lowp && !aligned16(w_lowp))) return W2L_ERR_ALIGN;
    if (n == 0) return W2L_OK;
    const long long n4 = n / 4 > 0 ? n / 4 : 1;
    const long long blocks = (n4 + 256 * SGD_PER_THREAD - 1) / (256 * SGD_PER_THREAD);
    if (blocks > 2147483647LL) return W2L_ERR_SHAPE;
    hipLaunchKernelGGL(sgd_momentum_k, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, w, v, grad,
                       static_cast<bf16_t*>(w_lowp), n, lr, momentum, weight_decay);
    return launch_status();
}
