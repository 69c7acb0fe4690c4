// gfx950 (CDNA4, wave64) kernels of the self-speculative decoding hot path.
//
// Single-row path (draft model of Section 3 and vanilla decoding): weight-streaming GEMV kernels for
// bf16 / fp16 / fp32 weights -- every lane issues 128-bit loads along K, fp32 FMAs against the
// activation vector held in LDS, wave-shuffle reduction; RMSNorm is fused into the prologue, rotary
// embedding + KV-cache write / residual add / SwiGLU into the epilogues.  Attention over the cache
// runs out of registers on ranges of ~128 positions; the output projection folds the range partials.
// Multi-row path (verification of k+1 rows, prompt rows, per-layer confidence rows): the same
// weight stream, staged through LDS, feeds 16x16x32 MFMA tiles; activations enter as an exact hi+lo
// split of their fp32 values in the weights' 16-bit type, and RMSNorm is folded into the epilogue
// of the producing and the consuming projection.  Models whose shapes do not fit the MFMA tiling
// (and fp32 models) take a plain FMA path with separate norm / rotary kernels.
#include "ssd_kernels.h"
#include "ssd_rules.h"

#include <hip/hip_ext.h>

#include <math.h>

#include <algorithm>
#include <atomic>
#include <mutex>

namespace ssdk {

// ---------------------------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);   // round to nearest even; gfx950 converts in hardware
}

template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int VEC = 4;  // elements per 128-bit load
    __device__ static __forceinline__ void load(const float* p, float (&o)[4])
    {
        float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
    __device__ static __forceinline__ float get(const float* p, size_t i) { return p[i]; }
    __device__ static __forceinline__ void put(float* p, size_t i, float v) { p[i] = v; }
};
template <> struct Elem<uint16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ void load(const uint16_t* p, float (&o)[8])
    {
        uint4 v = *reinterpret_cast<const uint4*>(p);
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
        o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xffff0000u);
        o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xffff0000u);
    }
    __device__ static __forceinline__ float get(const uint16_t* p, size_t i) { return bf16_bits_to_f32(p[i]); }
    __device__ static __forceinline__ void put(uint16_t* p, size_t i, float v) { p[i] = f32_to_bf16_bits(v); }
};

typedef _Float16 f16_t;   // IEEE binary16 storage (weights and cache of fp16 models)
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
template <> struct Elem<f16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ void load(const f16_t* p, float (&o)[8])
    {
        const f16x8_t v = *reinterpret_cast<const f16x8_t*>(p);
#pragma unroll
        for (int i = 0; i < 8; i++) o[i] = (float)v[i];
    }
    __device__ static __forceinline__ float get(const f16_t* p, size_t i) { return (float)p[i]; }
    __device__ static __forceinline__ void put(f16_t* p, size_t i, float v) { p[i] = (f16_t)v; }  // round to nearest even
};
template <typename T> struct IsF16 { static constexpr bool value = false; };
template <> struct IsF16<f16_t> { static constexpr bool value = true; };

// one 16-bit storage element (bf16 or fp16 bit pattern) from an fp32 value
__device__ __forceinline__ uint16_t f32_to_h16_bits(float v, bool f16)
{
    if (f16) return __builtin_bit_cast(uint16_t, (f16_t)v);
    return f32_to_bf16_bits(v);
}
__device__ __forceinline__ float h16_bits_to_f32(uint16_t h, bool f16)
{
    if (f16) return (float)__builtin_bit_cast(f16_t, h);
    return bf16_bits_to_f32(h);
}

// one KV-cache element of type kt (WeightType code) from an fp32 value, round to nearest even
__device__ __forceinline__ void kv_put(void* base, size_t i, float v, int kt)
{
    if (kt == WT_F32) reinterpret_cast<float*>(base)[i] = v;
    else if (kt == WT_F16) reinterpret_cast<f16_t*>(base)[i] = (f16_t)v;
    else reinterpret_cast<uint16_t*>(base)[i] = f32_to_bf16_bits(v);
}

__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// v summed over the 16 lanes of a DPP row (rotations by 8, 4, 2, 1); every lane of the row gets the sum
template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_sum(float v)
{
    v = dpp_add<0x128>(v);  // row_ror:8
    v = dpp_add<0x124>(v);  // row_ror:4
    v = dpp_add<0x122>(v);  // row_ror:2
    return dpp_add<0x121>(v);  // row_ror:1
}
template <int CTRL> __device__ __forceinline__ float dpp_max(float v)
{
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ float row16_max(float v)
{
    v = dpp_max<0x128>(v);
    v = dpp_max<0x124>(v);
    v = dpp_max<0x122>(v);
    return dpp_max<0x121>(v);
}

// exchanges between the 16-lane rows of a wave without the LDS crossbar: sum / max over rows 0 + 1 and 2 + 3, over both halves
__device__ __forceinline__ float rows_swap_sum(float v)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float rows_swap_max(float v)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float wave_sum_fast(float v) { return rows_swap_sum(row16_sum(v)); }
// maximum of a wave, and of the integers of its lanes the least one, without the LDS crossbar; every lane gets them
__device__ __forceinline__ float wave_max_fast(float v) { return rows_swap_max(row16_max(v)); }
template <int CTRL> __device__ __forceinline__ int dpp_min_i(int v) { return min(v, __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false)); }
__device__ __forceinline__ int wave_min_fast(int v)
{
    v = dpp_min_i<0x121>(dpp_min_i<0x122>(dpp_min_i<0x124>(dpp_min_i<0x128>(v))));
    auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = min((int)r[0], (int)r[1]);
    r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return min((int)r[0], (int)r[1]);
}

// Block-wide sum for blocks of NW waves; red must hold NW values. All threads get the result.
template <int NW, typename T>
__device__ __forceinline__ T block_sum(T v, T* red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    T t = 0;
#pragma unroll
    for (int i = 0; i < NW; i++) t += red[i];
    return t;
}

// Block barrier for data exchanged through LDS only: waits for this wave's LDS operations and then for the other
// waves.  __syncthreads() also carries a fence that waits for every global load in flight (loads and stores share
// one counter on this architecture), which would drain a register prefetch at every staging step; a loaded register
// is still protected by the wait the compiler places before its first use.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------------------------
// embedding gather
// ---------------------------------------------------------------------------------------------
// The rotary row of a single-row step's position is copied to a fixed place by whatever starts the step, so that the QKV
// launches of its layers do not have to fetch the position before they can fetch the row.
struct RopeRow {
    const float* table; const int* pos_dev; int pos_off; int hd; int rows; float* out;   // out null: nothing to copy; rows of the table
    __device__ __forceinline__ void copy(int t) const { out[t] = table[(size_t)min(pos_dev[0] + pos_off, rows - 1) * hd + t]; }
};

__device__ __forceinline__ int token_of(const Tokens& t, int r) { return r == 0 && t.first ? t.first[0] : t.ids[r]; }

template <typename WT>
__global__ void embed_kernel(const WT* __restrict__ E, Tokens tok, int d, int V, float* __restrict__ x, RopeRow rr)
{
    int r = blockIdx.y;
    if (rr.out && blockIdx.x == 0 && r == 0 && (int)threadIdx.x < rr.hd) rr.copy(threadIdx.x);
    const size_t row = embed_row(token_of(tok, r), V) * d;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < d; i += gridDim.x * blockDim.x)
        x[(size_t)r * d + i] = Elem<WT>::get(E, row + i);
}

hipError_t embed_rows(const Dims& D, const void* embed, Tokens tok, int M, float* x, hipStream_t s, const float* rope,
                      const int* pos_dev, int pos_off, float* rope_row)
{
    const RopeRow rr = {rope, pos_dev, pos_off, D.hd, D.max_seq, rope_row};
    dim3 grid(ceil_div(D.d, 256), M);
    if (D.wt == WT_BF16)
        hipLaunchKernelGGL(embed_kernel<uint16_t>, grid, dim3(256), 0, s, (const uint16_t*)embed, tok, D.d, D.V, x, rr);
    else if (D.wt == WT_F16)
        hipLaunchKernelGGL(embed_kernel<f16_t>, grid, dim3(256), 0, s, (const f16_t*)embed, tok, D.d, D.V, x, rr);
    else
        hipLaunchKernelGGL(embed_kernel<float>, grid, dim3(256), 0, s, (const float*)embed, tok, D.d, D.V, x, rr);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// single-row weight-streaming GEMV
// ---------------------------------------------------------------------------------------------
// A block has 8 waves.  KS consecutive waves form a group that owns R "logical" weight rows;
// the K dimension is cut into chunks of one 128-bit load per lane (512 bf16 / 256 fp32) and the
// waves of a group take chunks kp, kp+KS, ...  Every wave keeps D chunk-steps of R non-temporal
// loads in flight (weights are read exactly once, they should not displace activations in the
// caches).  The input vector sits in LDS already multiplied by the norm gain; the RMS scale is a
// per-vector scalar and is applied to the finished dot products.
// Logical row order: QKV interleaves the two rows of a rotary pair (i, i + hd/2), gate/up
// interleaves gate row n and up row n, so that one lane holds both operands of the epilogue.
constexpr int GV_WAVES = 8;
constexpr int GV_THREADS = GV_WAVES * 64;

enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_STORE = 3 };

struct GemvP {
    const void* w0; const void* w1; const void* w2;
    const float* in;    // [K]
    const float* part;  // when set (RESID only): the input is the fold of n_splits attention partials of row 0
    int n_splits;       //   laid out [K / hd heads][n_splits][hd + 4] as the attention kernels write them
    const float* gain;  // rmsnorm gain (RESID: none, the input is used as it is)
    float eps;
    int K;
    int n_rows;         // logical rows (QKV: dq + 2 dkv; SWIGLU: 2 f; else N)
    float* y;           // QKV: qbuf; RESID: residual (+=); SWIGLU: act; STORE: logits
    float* tap;
    void* kc; void* vc; int kt;   // cache rows of this layer and their element type (WeightType code)
    const float* rope_row;  // [hd/2][2] (cos, sin) of the row's position
    const int* pos_dev; int pos_off;
    int hd, dq, dkv, max_seq;
    float* vstat;       // STORE only, may be null: per block (max, sum of exp relative to it, arg-max) of the clamped outputs
    float clamp;
};

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

template <typename WT> __device__ __forceinline__ u32x4_t gv_load(const WT* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
}

// LDS position of element i of the staged input vector.  With 8 elements per lane (16-bit weights) a chunk of 512
// elements is stored as two planes of 64 float4: plane 0 holds elements 8 l .. 8 l + 3 of lane l, plane 1 elements
// 8 l + 4 .. 8 l + 7, so that each of a wave's two 128-bit reads covers 1 KB of consecutive LDS (in natural order the
// lanes are 32 bytes apart and every read has two-way bank conflicts: measured 1.6-2 us of a 32 us launch).
template <int VEC> __device__ __forceinline__ int gv_xpos(int i)
{
    if (VEC != 8) return i;
    return (i & ~511) + ((i >> 2) & 1) * 256 + ((i & 511) >> 3) * 4 + (i & 3);
}
constexpr int GV_XB = 256;   // floats between a lane's two float4 (16-bit weights)
constexpr int GV_RES_ROUNDS = 8;   // rounds of a block whose residual values are staged in LDS (later rounds read memory)

// acc += w . x for one 128-bit weight vector; xs points at the lane's activations of this chunk in LDS
template <typename WT> __device__ __forceinline__ float gv_dot(u32x4_t w, const float* xs, float acc);
template <> __device__ __forceinline__ float gv_dot<uint16_t>(u32x4_t w, const float* xs, float acc)
{
    float4 a = *reinterpret_cast<const float4*>(xs), b = *reinterpret_cast<const float4*>(xs + GV_XB);
    acc = fmaf(__uint_as_float(w.x << 16), a.x, acc);
    acc = fmaf(__uint_as_float(w.x & 0xffff0000u), a.y, acc);
    acc = fmaf(__uint_as_float(w.y << 16), a.z, acc);
    acc = fmaf(__uint_as_float(w.y & 0xffff0000u), a.w, acc);
    acc = fmaf(__uint_as_float(w.z << 16), b.x, acc);
    acc = fmaf(__uint_as_float(w.z & 0xffff0000u), b.y, acc);
    acc = fmaf(__uint_as_float(w.w << 16), b.z, acc);
    acc = fmaf(__uint_as_float(w.w & 0xffff0000u), b.w, acc);
    return acc;
}
template <> __device__ __forceinline__ float gv_dot<f16_t>(u32x4_t w, const float* xs, float acc)
{
    const f16x8_t h = __builtin_bit_cast(f16x8_t, w);
    float4 a = *reinterpret_cast<const float4*>(xs), b = *reinterpret_cast<const float4*>(xs + GV_XB);
    acc = fmaf((float)h[0], a.x, acc); acc = fmaf((float)h[1], a.y, acc);
    acc = fmaf((float)h[2], a.z, acc); acc = fmaf((float)h[3], a.w, acc);
    acc = fmaf((float)h[4], b.x, acc); acc = fmaf((float)h[5], b.y, acc);
    acc = fmaf((float)h[6], b.z, acc); acc = fmaf((float)h[7], b.w, acc);
    return acc;
}
template <> __device__ __forceinline__ float gv_dot<float>(u32x4_t w, const float* xs, float acc)
{
    float4 a = *reinterpret_cast<const float4*>(xs);
    acc = fmaf(__uint_as_float(w.x), a.x, acc);
    acc = fmaf(__uint_as_float(w.y), a.y, acc);
    acc = fmaf(__uint_as_float(w.z), a.z, acc);
    acc = fmaf(__uint_as_float(w.w), a.w, acc);
    return acc;
}

template <typename WT, int EPI>
__device__ __forceinline__ const WT* gv_row_ptr(const GemvP& p, int j)
{
    if (EPI == EPI_QKV) {
        if (j < p.dq + p.dkv) {
            const WT* base = (const WT*)p.w0;
            int jj = j;
            if (j >= p.dq) { base = (const WT*)p.w1; jj = j - p.dq; }
            const int head = jj / p.hd, e = jj % p.hd;
            const int i = (e >> 1) + (e & 1) * (p.hd >> 1);
            return base + (size_t)(head * p.hd + i) * p.K;
        }
        return (const WT*)p.w2 + (size_t)(j - p.dq - p.dkv) * p.K;
    } else if (EPI == EPI_SWIGLU) {
        return ((j & 1) ? (const WT*)p.w1 : (const WT*)p.w0) + (size_t)(j >> 1) * p.K;
    } else {
        return (const WT*)p.w0 + (size_t)j * p.K;
    }
}

// running soft-max statistics of the rows a lane has finished: maximum, its lowest row index, sum of exp(v - max)
struct VStat { float m; float z; int arg; };
__device__ __forceinline__ void vstat_add(VStat& a, float v, int idx)
{
    if (v > a.m) { a.z = a.z * __expf(a.m - v) + 1.0f; a.m = v; a.arg = idx; }   // first row: exp(-inf) = 0
    else a.z += __expf(v - a.m);
}
// merge b into a; equal maxima keep the lower index
__device__ __forceinline__ void vstat_merge(VStat& a, const VStat& b)
{
    if (b.m > a.m || (b.m == a.m && b.arg < a.arg)) {
        a.z = (a.m > -INFINITY ? a.z * __expf(a.m - b.m) : 0.f) + b.z;
        a.m = b.m; a.arg = b.arg;
    } else if (b.m > -INFINITY) {
        a.z += b.z * __expf(b.m - a.m);
    }
}

// finished sums s[0..R) of logical rows j0.. ; sc = RMS scale (1 when no norm).  What the epilogue reads besides its
// sums comes out of LDS, staged by the kernel's prologue -- the rotary row of the position (rope_row, QKV) and the
// residual values of the group (res, null = read them from memory) -- so that no memory load sits between the steps
// of the weight pipeline (a load there has to be waited for together with every weight load in flight).
template <typename WT, int EPI, int R>
__device__ __forceinline__ void gv_epilogue(const GemvP& p, int j0, const float (&s)[R], float sc, VStat& vs, int pos,
                                            const float* rope_row, const float* res)
{
    if (EPI == EPI_QKV) {
        const int half = p.hd >> 1;
#pragma unroll
        for (int t = 0; t < R; t += 2) {
            const int j = j0 + t;
            const float a = s[t] * sc, b = s[t + 1] * sc;
            if (j < p.dq + p.dkv) {
                const bool is_q = j < p.dq;
                const int jj = is_q ? j : j - p.dq;
                const int head = jj / p.hd, i = (jj % p.hd) >> 1;
                const float* cs = rope_row + i * 2;
                const float c = cs[0], sn = cs[1];
                const float ra = a * c - b * sn, rb = b * c + a * sn;
                if (is_q) {
                    float* q = p.y + (size_t)head * p.hd + i;
                    q[0] = ra; q[half] = rb;
                } else {
                    const size_t o = ((size_t)head * p.max_seq + pos) * p.hd + i;
                    kv_put(p.kc, o, ra, p.kt);
                    kv_put(p.kc, o + half, rb, p.kt);
                }
            } else {
                const int e = j - p.dq - p.dkv;
                const size_t o = ((size_t)(e / p.hd) * p.max_seq + pos) * p.hd + (e % p.hd);
                kv_put(p.vc, o, a, p.kt);
                kv_put(p.vc, o + 1, b, p.kt);
            }
        }
    } else if (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int t = 0; t < R; t += 2) {
            const float g = s[t] * sc, u = s[t + 1] * sc;
            const float a = g / (1.0f + __expf(-g)) * u;
            p.y[(j0 + t) >> 1] = a;
        }
    } else if (EPI == EPI_RESID) {
#pragma unroll
        for (int t = 0; t < R; t++) {
            const float v = (res ? res[t] : p.y[j0 + t]) + s[t];
            p.y[j0 + t] = v;
            if (p.tap) p.tap[j0 + t] = v;
        }
    } else {
#pragma unroll
        for (int t = 0; t < R; t++) {
            const float v = s[t] * sc;
            p.y[j0 + t] = v;
            if (p.vstat) vstat_add(vs, fminf(fmaxf(v, -p.clamp), p.clamp), j0 + t);   // rows arrive in ascending order
        }
    }
}

// Four elements (i ..) of the input of a projection that folds attention partials: sum_s e^(m_s - m) o_s / sum_s e^(m_s - m) l_s.  All
// partials of an element are requested by independent, unconditional loads (index clamped, weight zeroed past n_splits), so that
// the fold costs one cache round trip, not one per partial.  NF: two, four or eight, the smallest that covers n_splits.
template <int NF>
struct GvFold {
    float mm[NF], ll[NF];
    float4 oo[NF];
    __device__ __forceinline__ void request(const GemvP& p, int i)
    {
        const int hs = p.hd + 4, ns = p.n_splits, d = i % p.hd;
        const float* base = p.part + (size_t)(i / p.hd) * ns * hs;
#pragma unroll
        for (int sp = 0; sp < NF; sp++) {
            const float* ps = base + min(sp, ns - 1) * hs;
            mm[sp] = ps[p.hd];
            ll[sp] = ps[p.hd + 1];
            oo[sp] = *reinterpret_cast<const float4*>(ps + d);
        }
    }
    __device__ __forceinline__ float4 result(int ns) const
    {
        float gm = -INFINITY;
#pragma unroll
        for (int sp = 0; sp < NF; sp++) gm = fmaxf(gm, mm[sp]);   // clamped duplicates do not change the max
        float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
        float den = 0.f;
#pragma unroll
        for (int sp = 0; sp < NF; sp++) {
            const float w = (sp < ns && ll[sp] > 0.f) ? __expf(mm[sp] - gm) : 0.f;
            num.x = fmaf(w, oo[sp].x, num.x); num.y = fmaf(w, oo[sp].y, num.y);
            num.z = fmaf(w, oo[sp].z, num.z); num.w = fmaf(w, oo[sp].w, num.w);
            den = fmaf(w, ll[sp], den);
        }
        return make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
    }
};

// FOLD: 0 = the input is p.in, else the fold of up to FOLD attention partials
template <typename WT, int EPI, int R, int D, int KS, int FOLD = 0>
__global__ __launch_bounds__(GV_THREADS) void gemv_kernel(GemvP p)
{
    extern __shared__ __align__(16) float xs[];
    __shared__ float red[GV_WAVES];
    __shared__ float part[GV_WAVES][R];
    __shared__ float rope_row[EPI == EPI_QKV ? 128 : 1];                                  // (cos, sin) pairs of the position
    __shared__ float res_s[EPI == EPI_RESID ? GV_WAVES * GV_RES_ROUNDS * R : 1];          // [group slot][round][row]
    constexpr int VEC = Elem<WT>::VEC, CH = 64 * VEC, GPB = GV_WAVES / KS;
    const int lane = threadIdx.x & 63;
    // made wave-uniform for the compiler: group numbers and row pointers stay in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int grp = wave / KS, kp = wave % KS;
    const int K = p.K;
    const int n_groups = p.n_rows / R;
    const int nfull = K / CH, tail = K - nfull * CH;   // tail is a multiple of VEC
    // A row is NCH chunks of one load step, the last one partial when tail > 0 (lanes past the row's end are masked).
    // Wave kp owns chunks kp, kp + KS, ..: S steps per group, the same for every wave of the block so that block
    // barriers stay uniform.
    const int NCH = nfull + (tail > 0 ? 1 : 0);
    const int S = (NCH + KS - 1) / KS;
    const int n_gblocks = (n_groups + GPB - 1) / GPB;
    const int n_rounds = (n_gblocks - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int T = n_rounds * S;   // this wave's items (group, step), walked in order
    const int lv_full = lane * VEC;
    const int lv_tail = tail > 0 ? min(lane * VEC, tail - VEC) : 0;   // lanes past a partial chunk re-read its last vector
    const bool lane_in_tail = lane * VEC < tail;

    // Issue side of the software pipeline: D items ahead of the consume side, across groups.  Every issue is
    // UNCONDITIONAL -- a slot past the last group re-reads the last group, a step past the last chunk re-reads the last
    // chunk, and such items are never consumed.  With conditional loads the compiler cannot count what is in flight and
    // waits for everything, the loads just issued included, before every step: one memory latency per step.
    // The waves of a launch start together and their rows lie a multiple of the memory channels' interleave apart:
    // where a wave owns whole rows (KS = 1), group g walks its chunks starting at its (g mod S_kp)-th one and wraps
    // around, so that the waves are spread over the row (and the channels) from the first step on; waves that share a
    // row start at different chunks anyway (measured: the rotation gains 4 % on the 7B LM head, 10 % on the 70B one, and
    // loses 1-3 % where waves share rows; a start at (block / 8) mod S_kp, which is what helps the 16-row kernel, loses
    // up to 15 % here).
    // S_kp = chunks this wave owns.
    const int S_kp = kp < NCH ? (NCH - kp + KS - 1) / KS : 0;
    int ri = 0, ci = 0, rot_i = 0;
    const WT* wi[R];
    auto set_issue_rows = [&]() {
        int g = ((int)blockIdx.x + min(ri, max(n_rounds - 1, 0)) * (int)gridDim.x) * GPB + grp;
        g = min(g, n_groups - 1);
        rot_i = (KS == 1 && S_kp > 0) ? g % S_kp : 0;
#pragma unroll
        for (int r = 0; r < R; r++) wi[r] = gv_row_ptr<WT, EPI>(p, g * R + r);
    };
    set_issue_rows();
    u32x4_t buf[D][R];
    auto issue = [&](int s) {
        int j = ci + rot_i;
        if (j >= S_kp) j -= S_kp;
        const int c = ci < S_kp ? kp + j * KS : NCH - 1;   // (a step past the wave's last chunk re-reads the row's last chunk)
        const size_t off = (size_t)c * CH + (c == nfull ? lv_tail : lv_full);
#pragma unroll
        for (int r = 0; r < R; r++) buf[s][r] = gv_load(wi[r] + off);
        if (++ci == S) { ci = 0; ++ri; set_issue_rows(); }
    };
    // What the block reads besides weights is requested in front of them: loads return in order, and behind the first
    // weights of all blocks (100 KB per CU) the input arrives when these are through, with nothing of the stream in
    // flight until it is staged and the next loads are out.  The first XN four-element pieces per thread (addresses
    // clamped), the rest of a longer input behind: up to 4096 elements of the LM head's and of a folded input, 8192 of a normalised
    // one, 14336 of a plain one, the widths up to 8B and 70B's normalised rows.  A piece past the input's end is requested all the
    // same; with 8192 folded and 28672 plain ones steps of 70B take 0.9 % less (down 71.1 / 69.6 us, folding output projection 25.2 / 24.7),
    // those of 7B, 8B and 13B 0.7 to 1.6 % more (13B down 24.1 / 24.6, folding output projection 13.4 / 14.1).  In the steps of a 7B model, us, input behind / in front: QKV 19.3 / 18.2,
    // output projection with two or three partials 9.0 / 8.0, with seven 11.0 / 10.1, gate/up 28.9 / 28.5, down 17.9 / 16.5; 70B down 74.5 / 72.3.
    constexpr bool GAIN = EPI != EPI_RESID;
    constexpr int XN = FOLD ? 2 : EPI == EPI_STORE ? 2 : EPI == EPI_RESID ? 7 : 4;
    int pos = 0;
    float rope_r = 0.f;
    if (EPI == EPI_QKV) {
        pos = p.pos_dev[0] + p.pos_off;
        rope_r = p.rope_row[min((int)threadIdx.x, p.hd - 1)];   // hd / 2 pairs
    }
    float res_r = 0.f;
    constexpr int NRES = GPB * GV_RES_ROUNDS * R;
    static_assert(NRES <= GV_THREADS, "a residual value per thread");
    if (EPI == EPI_RESID) {
        const int i = min((int)threadIdx.x, NRES - 1), r = i % R, rnd = (i / R) % GV_RES_ROUNDS, gs = i / (R * GV_RES_ROUNDS);
        res_r = p.y[min(((int)blockIdx.x + rnd * (int)gridDim.x) * GPB + gs, n_groups - 1) * R + r];
    }
    float4 xv[XN], xg[XN];
    GvFold<FOLD ? FOLD : 1> xf[FOLD ? XN : 1];
#pragma unroll
    for (int u = 0; u < XN; u++) {
        const int i = min(((int)threadIdx.x + u * GV_THREADS) * 4, K - 4);
        if constexpr (FOLD) xf[u].request(p, i);
        else xv[u] = *reinterpret_cast<const float4*>(p.in + i);
        if (GAIN) xg[u] = *reinterpret_cast<const float4*>(p.gain + i);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < D; s++) issue(s);

    // stage the input vector (times gain); the sum of squares gives the RMS scale
    float ss = 0.f;
    auto stage = [&](int i, float4 v, float4 g) {
        if (GAIN) {
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            v.x *= g.x; v.y *= g.y; v.z *= g.z; v.w *= g.w;
        }
        *reinterpret_cast<float4*>(xs + gv_xpos<VEC>(i)) = v;
    };
    if (EPI == EPI_RESID && (int)threadIdx.x < NRES) res_s[threadIdx.x] = res_r;   // [group of the block][round][row]
    if (EPI == EPI_QKV && (int)threadIdx.x < p.hd) rope_row[threadIdx.x] = rope_r;
#pragma unroll
    for (int u = 0; u < XN; u++) {
        const int i = ((int)threadIdx.x + u * GV_THREADS) * 4;
        if (i < K) {
            if constexpr (FOLD) stage(i, xf[u].result(p.n_splits), make_float4(0.f, 0.f, 0.f, 0.f));
            else stage(i, xv[u], GAIN ? xg[u] : xv[u]);
        }
    }
    for (int i = ((int)threadIdx.x + XN * GV_THREADS) * 4; i < K; i += GV_THREADS * 4) {
        if constexpr (FOLD) {
            GvFold<FOLD ? FOLD : 1> f;
            f.request(p, i);
            stage(i, f.result(p.n_splits), make_float4(0.f, 0.f, 0.f, 0.f));
        } else {
            const float4 v = *reinterpret_cast<const float4*>(p.in + i);
            stage(i, v, GAIN ? *reinterpret_cast<const float4*>(p.gain + i) : v);
        }
    }
    float sc = 1.0f;
    if (GAIN) {
        ss = wave_sum(ss);
        if (lane == 0) red[wave] = ss;
    }
    lds_barrier();   // (the weights in flight are not waited for)
    if (GAIN) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < GV_WAVES; i++) t += red[i];
        sc = 1.0f / sqrtf(t / (float)K + p.eps);
    }

    const float* xp = xs + (size_t)kp * CH + lane * (VEC == 8 ? 4 : VEC);   // the lane's first float4 of chunk kp
    VStat vs = {-INFINITY, 0.f, 0x7fffffff};
    int rc = 0, cc = 0;
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; r++) acc[r] = 0.f;
    auto consume = [&](int s) {
        if (rc < n_rounds) {   // uniform over the block; false only for the padding items behind the last group
            const int g = ((int)blockIdx.x + rc * (int)gridDim.x) * GPB + grp;
            const bool act = g < n_groups;
            int j = cc + ((KS == 1 && S_kp > 0) ? g % S_kp : 0);   // the issue side's chunk order
            if (j >= S_kp) j -= S_kp;
            const int c = kp + j * KS;
            if (act && cc < S_kp && (c < nfull || lane_in_tail)) {
#pragma unroll
                for (int r = 0; r < R; r++) acc[r] = gv_dot<WT>(buf[s][r], xp + (size_t)j * KS * CH, acc[r]);
            }
            if (++cc == S) {  // group finished
#pragma unroll
                for (int r = 0; r < R; r++) acc[r] = wave_sum(acc[r]);
                const float* res = (EPI == EPI_RESID && rc < GV_RES_ROUNDS) ? res_s + (grp * GV_RES_ROUNDS + rc) * R : nullptr;
                if (KS == 1) {
                    if (act && lane == 0) gv_epilogue<WT, EPI, R>(p, g * R, acc, sc, vs, pos, rope_row, res);
                } else {
                    if (lane == 0) {
#pragma unroll
                        for (int r = 0; r < R; r++) part[wave][r] = acc[r];
                    }
                    __syncthreads();
                    if (act && kp == 0 && lane == 0) {
                        float sm[R];
#pragma unroll
                        for (int r = 0; r < R; r++) {
                            float t = 0.f;
#pragma unroll
                            for (int j = 0; j < KS; j++) t += part[grp * KS + j][r];
                            sm[r] = t;
                        }
                        gv_epilogue<WT, EPI, R>(p, g * R, sm, sc, vs, pos, rope_row, res);
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int r = 0; r < R; r++) acc[r] = 0.f;
                cc = 0;
                ++rc;
            }
        }
    };
    // steady state: every step consumes the oldest item and refills its slot; the last D items are consumed without
    // a refill (the item count is padded to a multiple of D: padding items are re-reads that are not consumed)
    const int Tp = (T + D - 1) / D * D;
    for (int t = 0; t + D < Tp; t += D) {
#pragma unroll
        for (int s = 0; s < D; s++) {
            consume(s);
            issue(s);
        }
    }
#pragma unroll
    for (int s = 0; s < D; s++) consume(s);
    if (EPI == EPI_STORE && p.vstat) {   // block partial of the soft-max statistics: lane 0 of every wave holds one
        __shared__ float vred[GV_WAVES * 3];
        if (lane == 0) { vred[wave * 3] = vs.m; vred[wave * 3 + 1] = vs.z; vred[wave * 3 + 2] = __int_as_float(vs.arg); }
        __syncthreads();
        if (threadIdx.x == 0) {
            VStat a = {vred[0], vred[1], __float_as_int(vred[2])};
#pragma unroll
            for (int w = 1; w < GV_WAVES; w++) {
                const VStat b = {vred[w * 3], vred[w * 3 + 1], __float_as_int(vred[w * 3 + 2])};
                vstat_merge(a, b);
            }
            p.vstat[blockIdx.x * 3] = a.m; p.vstat[blockIdx.x * 3 + 1] = a.z; p.vstat[blockIdx.x * 3 + 2] = __int_as_float(a.arg);
        }
    }
}

// End of a single-row step: combines the per-block statistics of the LM-head launch into the greedy token (lowest index
// among equal maxima) and its soft-max probability 1 / sum exp(z - max), and does in the same launch what the next step
// would otherwise need a launch of its own for (about 4 us each in a replayed sequence): the position and the pending token
// of a decode step, or the embedding row that the next draft step starts from.
constexpr int SF_THREADS = 1024;
template <typename WT>
__global__ __launch_bounds__(SF_THREADS) void step_finish_kernel(const float* __restrict__ vstat, int n_blocks, StepOut o, int d, int V, RopeRow rr)
{
    __shared__ VStat sm[SF_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (rr.out && tid < rr.hd) rr.copy(tid);   // of the next step
    // (three reductions over the lanes, an exponential each; merging pairs of records takes six rounds of shuffles and
    // exponentials: 1000 records of a 7B step 5.2 -> 4.3 us, what the shortest launch of a replayed sequence takes)
    auto wave_merge = [](VStat& a) {
        const float m = wave_max_fast(a.m);
        a.z = wave_sum_fast(a.m > -INFINITY ? a.z * __expf(a.m - m) : 0.f);
        a.arg = wave_min_fast(a.m == m ? a.arg : 0x7fffffff);
        a.m = m;
    };
    VStat a = {-INFINITY, 0.f, 0x7fffffff};
    for (int i = tid; i < n_blocks; i += SF_THREADS) {
        const VStat b = {vstat[i * 3], vstat[i * 3 + 1], __float_as_int(vstat[i * 3 + 2])};
        vstat_merge(a, b);
    }
    wave_merge(a);
    if (lane == 0) sm[wave] = a;
    __syncthreads();
    if (wave == 0) {
        a = lane < SF_THREADS / 64 ? sm[lane] : VStat{-INFINITY, 0.f, 0x7fffffff};
        wave_merge(a);
        if (lane == 0) {
            sm[0] = a;
            o.tok_out[0] = a.arg;
            o.tok_host[0] = a.arg;
            o.maxprob_host[0] = 1.0f / a.z;
            bool ok = true;
            if (o.step_ctrl) {   // of a step in one launch: the next launch's tags start behind this one's; a step that gave up commits nothing
                ok = o.step_ctrl[1] == 0;
                o.step_ctrl[0] += o.step_hops;
                if (!ok) o.step_err_host[0] = 1;
            }
            if (o.pos_dev && ok) {
                const int pos = o.pos_dev[0];   // (the next rotary row was copied before the barrier above)
                if (o.tok_log) o.tok_log[pos] = a.arg;
                o.pos_dev[0] = pos + 1; o.tok0[0] = a.arg;
            }
        }
    }
    if (!o.x_next) return;   // uniform
    __syncthreads();
    const WT* row = static_cast<const WT*>(o.embed) + embed_row(sm[0].arg, V) * d;   // (logits that are all NaN leave no arg-max)
    float* x = o.x_next;
    for (int i = tid * 4; i < d; i += SF_THREADS * 4)
        *reinterpret_cast<float4*>(x + i) = make_float4(Elem<WT>::get(row, i), Elem<WT>::get(row, i + 1), Elem<WT>::get(row, i + 2), Elem<WT>::get(row, i + 3));
}

static hipError_t step_finish(const Dims& D, const float* vstat, int blocks, const StepOut& o, hipStream_t s)
{
    const RopeRow rr = {o.rope, o.rope_pos, o.rope_off, D.hd, D.max_seq, o.rope_row};
    if (D.wt == WT_BF16) hipLaunchKernelGGL(step_finish_kernel<uint16_t>, dim3(1), dim3(SF_THREADS), 0, s, vstat, blocks, o, D.d, D.V, rr);
    else if (D.wt == WT_F16) hipLaunchKernelGGL(step_finish_kernel<f16_t>, dim3(1), dim3(SF_THREADS), 0, s, vstat, blocks, o, D.d, D.V, rr);
    else hipLaunchKernelGGL(step_finish_kernel<float>, dim3(1), dim3(SF_THREADS), 0, s, vstat, blocks, o, D.d, D.V, rr);
    return hipGetLastError();
}

// Largest dynamic LDS size a kernel has been enabled for.  A process-wide cache of an idempotent runtime call
// (hipFuncSetAttribute): concurrent contexts may both make the call, never skip it wrongly.
static hipError_t ensure_lds(const void* fn, size_t lds, std::atomic<size_t>& limit)
{
    if (lds <= 64 * 1024 || lds <= limit.load(std::memory_order_acquire)) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    size_t cur = limit.load(std::memory_order_relaxed);
    while (cur < lds && !limit.compare_exchange_weak(cur, lds, std::memory_order_release)) {}
    return hipSuccess;
}

constexpr int gemv_lds_floats(int K, int vec) { return (K + 64 * vec - 1) / (64 * vec) * (64 * vec); }   // whole chunks of one load step

// Rounds of row groups that every block of a launch walks.  Up to four blocks fit a CU (registers: eight waves per SIMD;
// LDS: the staged vector): persistent blocks that are all resident at once leave no second, partial round of blocks.
// Measured: three per CU are best for the layer's GEMVs, four for the LM head.  The variant that folds attention partials
// in its prologue re-reads them per block, so it runs one block per CU.
template <typename WT, int EPI, int R, int KS>
static int gemv_rounds(const GemvP& p, const LaunchOpts* opt)
{
    const size_t lds = (size_t)gemv_lds_floats(p.K, Elem<WT>::VEC) * sizeof(float);
    const int per_cu = (int)std::min<size_t>(EPI == EPI_STORE ? 4 : 3, std::max<size_t>(1, ((size_t)160 << 10) / (lds + 1024)));
    int cap = p.part ? 256 : 256 * per_cu;
    if (opt && opt->gemv_block_cap > 0) cap = opt->gemv_block_cap;
    return std::max(1, ceil_div(ceil_div(p.n_rows / R, GV_WAVES / KS), cap));
}

// blocks_out (may be null) receives the grid size of the launch
template <typename WT, int EPI, int R, int D, int KS, int FOLD>
static hipError_t launch_gemv_fold(const GemvP& p, hipStream_t s, LaunchOpts* opt, int* blocks_out)
{
    const size_t lds = (size_t)gemv_lds_floats(p.K, Elem<WT>::VEC) * sizeof(float);
    static std::atomic<size_t> lds_limit{0};  // per instantiation
    {
        hipError_t e = ensure_lds((const void*)gemv_kernel<WT, EPI, R, D, KS, FOLD>, lds, lds_limit);
        if (e != hipSuccess) return e;
    }
    // equal work per block: with r rounds needed, use just enough blocks for r full rounds (gate/up at 7B:
    // 1376 block-rounds -> 688 blocks x 2 rather than 768 blocks of which 160 would do one round only)
    const int blocks = ceil_div(ceil_div(p.n_rows / R, GV_WAVES / KS), gemv_rounds<WT, EPI, R, KS>(p, opt));
    if (blocks_out) *blocks_out = blocks;
    if (opt && opt->time_start) {
        // timing request for this one launch: the events take the kernel's own begin and end timestamps
        hipExtLaunchKernelGGL((gemv_kernel<WT, EPI, R, D, KS, FOLD>), dim3(blocks), dim3(GV_THREADS), lds, s, opt->time_start,
                              opt->time_stop, 0, p);
        opt->time_start = nullptr;
        opt->time_stop = nullptr;
    } else {
        hipLaunchKernelGGL((gemv_kernel<WT, EPI, R, D, KS, FOLD>), dim3(blocks), dim3(GV_THREADS), lds, s, p);
    }
    return hipGetLastError();
}

template <typename WT, int EPI, int R, int D, int KS>
static hipError_t launch_gemv_cfg(const GemvP& p, hipStream_t s, LaunchOpts* opt, int* blocks_out)
{
    if constexpr (EPI == EPI_RESID) {
        if (p.part) {
            if (p.n_splits <= 2) return launch_gemv_fold<WT, EPI, R, D, KS, 2>(p, s, opt, blocks_out);
            if (p.n_splits <= 4) return launch_gemv_fold<WT, EPI, R, D, KS, 4>(p, s, opt, blocks_out);
            return launch_gemv_fold<WT, EPI, R, D, KS, GV_FOLD_MAX>(p, s, opt, blocks_out);
        }
    }
    return launch_gemv_fold<WT, EPI, R, D, KS, 0>(p, s, opt, blocks_out);
}

// Work split: many rows -> one wave per row pair, deep pipeline; few rows -> split K over the waves
// of a group so that every wave still has a handful of chunks and the chip has thousands of waves.
template <typename WT, int EPI>
static hipError_t launch_gemv_t(const GemvP& p, hipStream_t s, LaunchOpts* opt, int* blocks_out)
{
    const int ch = ceil_div(p.K, 64 * Elem<WT>::VEC);
    if constexpr (EPI == EPI_RESID && sizeof(WT) == 2) {   // tuning hook (kernel_bench sweeps)
        switch (opt && !p.part ? opt->gemv_resid_cfg : 0) {
            case 241: return launch_gemv_fold<WT, EPI, 2, 4, 1, 0>(p, s, opt, blocks_out);
            case 242: return launch_gemv_fold<WT, EPI, 2, 4, 2, 0>(p, s, opt, blocks_out);
            case 244: return launch_gemv_fold<WT, EPI, 2, 4, 4, 0>(p, s, opt, blocks_out);
            case 248: return launch_gemv_fold<WT, EPI, 2, 4, 8, 0>(p, s, opt, blocks_out);
            case 222: return launch_gemv_fold<WT, EPI, 2, 2, 2, 0>(p, s, opt, blocks_out);
            case 224: return launch_gemv_fold<WT, EPI, 2, 2, 4, 0>(p, s, opt, blocks_out);
            case 228: return launch_gemv_fold<WT, EPI, 2, 2, 8, 0>(p, s, opt, blocks_out);
            case 422: return launch_gemv_fold<WT, EPI, 4, 2, 2, 0>(p, s, opt, blocks_out);
            case 424: return launch_gemv_fold<WT, EPI, 4, 2, 4, 0>(p, s, opt, blocks_out);
            case 428: return launch_gemv_fold<WT, EPI, 4, 2, 8, 0>(p, s, opt, blocks_out);
            case 442: return launch_gemv_fold<WT, EPI, 4, 4, 2, 0>(p, s, opt, blocks_out);
            case 444: return launch_gemv_fold<WT, EPI, 4, 4, 4, 0>(p, s, opt, blocks_out);
            default: break;
        }
    }
    if constexpr (EPI != EPI_RESID && sizeof(WT) == 2) {   // tuning hook (kernel_bench sweeps)
        switch (opt ? opt->gemv_cfg : 0) {
            case 281: return launch_gemv_cfg<WT, EPI, 2, 8, 1>(p, s, opt, blocks_out);
            case 441: return launch_gemv_cfg<WT, EPI, 4, 4, 1>(p, s, opt, blocks_out);
            case 421: return launch_gemv_cfg<WT, EPI, 4, 2, 1>(p, s, opt, blocks_out);
            case 221: return launch_gemv_cfg<WT, EPI, 2, 2, 1>(p, s, opt, blocks_out);
            case 242: return launch_gemv_cfg<WT, EPI, 2, 4, 2>(p, s, opt, blocks_out);
            default: break;
        }
    }
    if constexpr (sizeof(WT) == 2) {
        // 16-bit weights: row pairs everywhere (four rows per wave lose 5-20 %); graph replays of one launch per layer, us.
        if constexpr (EPI == EPI_RESID) {
            // Few chunks: two waves per pair.  Folding the attention partials: a wave per pair with four steps in flight, since
            // every block re-reads the partials and there is one block per CU only (7B 9.4 against 10.9 with four waves per
            // pair, both with the input requested behind the weights; at 8192 rows, where a block has two rounds, 27.2 against 28.5 the other
            // way round).  Everything else: four
            // waves per pair; four steps in flight where a wave's share of a pair is longer than that and its items need no
            // padding (7B down projection, 12 items: 16.5 against 16.7 with two; 70B, 112: 71.8
            // against 72.8), else two (Llama-3-8B, 14 items: 22.9 -> 21.4, 13B, 21: 26.7 -> 25.7, 1024-wide, 2: 5.4 -> 5.0; 70B
            // output projection, four steps per pair: 25.3 against 29.4).
            if (ch <= 4) return launch_gemv_cfg<WT, EPI, 2, 2, 2>(p, s, opt, blocks_out);
            if (p.part && p.n_rows < 8192) return launch_gemv_cfg<WT, EPI, 2, 4, 1>(p, s, opt, blocks_out);
            const int steps = ceil_div(ch, 4);
            if (steps > 4 && steps * gemv_rounds<WT, EPI, 2, 4>(p, opt) % 4 == 0) return launch_gemv_cfg<WT, EPI, 2, 4, 4>(p, s, opt, blocks_out);
            return launch_gemv_cfg<WT, EPI, 2, 2, 4>(p, s, opt, blocks_out);
        } else if constexpr (EPI == EPI_QKV) {
            // a wave per pair where there are pairs for every wave slot or hardly any chunks (7B 19.9 -> 19.4, 13B 29.3 -> 28.6,
            // 1024-wide 6.1 -> 5.3), else two (Llama-3-8B, 6144 rows: 11.9 against 13.1)
            if (p.n_rows >= 8192 || ch <= 2) return launch_gemv_cfg<WT, EPI, 2, 2, 1>(p, s, opt, blocks_out);
            return launch_gemv_cfg<WT, EPI, 2, 2, 2>(p, s, opt, blocks_out);
        } else if constexpr (EPI == EPI_SWIGLU) {
            // two waves per pair with four steps in flight where a pair is a multiple of four steps (7B 28.7 against 30.2 with
            // two), else two: the item count is padded to the pipeline's depth (13B, five steps per pair: 48.0 -> 45.9)
            if (ch <= 2) return launch_gemv_cfg<WT, EPI, 2, 2, 1>(p, s, opt, blocks_out);
            if (p.n_rows >= 8192 && ch % 8 == 0) return launch_gemv_cfg<WT, EPI, 2, 4, 2>(p, s, opt, blocks_out);
            return launch_gemv_cfg<WT, EPI, 2, 2, 2>(p, s, opt, blocks_out);
        } else {   // LM head: a wave per pair
            if (p.n_rows >= 8192) return launch_gemv_cfg<WT, EPI, 2, 4, 1>(p, s, opt, blocks_out);
            return launch_gemv_cfg<WT, EPI, 2, 2, 2>(p, s, opt, blocks_out);
        }
    } else {
        if (p.n_rows >= 8192) return launch_gemv_cfg<WT, EPI, 2, 4, 1>(p, s, opt, blocks_out);
        if (ch <= 12) return launch_gemv_cfg<WT, EPI, 2, 2, 2>(p, s, opt, blocks_out);
        if (ch <= 40) return launch_gemv_cfg<WT, EPI, 4, 2, 4>(p, s, opt, blocks_out);
        return launch_gemv_cfg<WT, EPI, 4, 2, 8>(p, s, opt, blocks_out);
    }
}

template <int EPI>
static hipError_t launch_gemv(const Dims& D, const GemvP& p, hipStream_t s, int* blocks_out = nullptr)
{
    if (D.wt == WT_BF16) return launch_gemv_t<uint16_t, EPI>(p, s, D.opt, blocks_out);
    if (D.wt == WT_F16) return launch_gemv_t<f16_t, EPI>(p, s, D.opt, blocks_out);
    return launch_gemv_t<float, EPI>(p, s, D.opt, blocks_out);
}

hipError_t gemv_qkv(const Dims& D, const void* wq, const void* wk, const void* wv, const float* gain, const float* x,
                    const float* rope_row, const int* pos_dev, int pos_off, float* qbuf, void* kc, void* vc, hipStream_t s)
{
    if (!gain || D.hd > 128 || D.hd % 2) return hipErrorInvalidValue;   // the kernel stages one rotary row of hd floats in a 128-float LDS array
    GemvP p = {};
    p.w0 = wq; p.w1 = wk; p.w2 = wv; p.in = x; p.gain = gain; p.eps = D.eps; p.K = D.d;
    p.n_rows = D.dq + 2 * D.dkv;
    p.y = qbuf; p.kc = kc; p.vc = vc; p.kt = D.kt; p.rope_row = rope_row; p.pos_dev = pos_dev; p.pos_off = pos_off;
    p.hd = D.hd; p.dq = D.dq; p.dkv = D.dkv; p.max_seq = D.max_seq;
    return launch_gemv<EPI_QKV>(D, p, s);
}

hipError_t gemv_resid(const Dims& D, const void* w, int N, int K, const float* in, float* x, float* tap, hipStream_t s)
{
    GemvP p = {};
    p.w0 = w; p.in = in; p.gain = nullptr; p.eps = D.eps; p.K = K; p.n_rows = N; p.y = x; p.tap = tap;
    return launch_gemv<EPI_RESID>(D, p, s);
}

hipError_t gemv_resid_attn(const Dims& D, const void* w, const float* part, int n_splits, float* x, float* tap,
                           hipStream_t s)
{
    if (n_splits < 1 || n_splits > GV_FOLD_MAX || D.hd % 4) return hipErrorInvalidValue;
    GemvP p = {};
    p.w0 = w; p.in = nullptr; p.part = part; p.n_splits = n_splits; p.hd = D.hd; p.gain = nullptr; p.eps = D.eps;
    p.K = D.dq; p.n_rows = D.d; p.y = x; p.tap = tap;
    return launch_gemv<EPI_RESID>(D, p, s);
}

hipError_t gemv_swiglu(const Dims& D, const void* wg, const void* wu, const float* gain, const float* x, float* act,
                       hipStream_t s)
{
    if (!gain) return hipErrorInvalidValue;
    GemvP p = {};
    p.w0 = wg; p.w1 = wu; p.in = x; p.gain = gain; p.eps = D.eps; p.K = D.d; p.n_rows = 2 * D.f; p.y = act;
    return launch_gemv<EPI_SWIGLU>(D, p, s);
}

hipError_t gemv_lmhead(const Dims& D, const void* wlm, const float* gain, const float* x, float* logits, hipStream_t s)
{
    if (!gain) return hipErrorInvalidValue;
    GemvP p = {};
    p.w0 = wlm; p.in = x; p.gain = gain; p.eps = D.eps; p.K = D.d; p.n_rows = D.V; p.y = logits;
    return launch_gemv<EPI_STORE>(D, p, s);
}

hipError_t gemv_lmhead_argmax(const Dims& D, const void* wlm, const float* gain, const float* x, float* logits, float clamp,
                              float* vstat, const StepOut& o, hipStream_t s)
{
    if (!gain || !vstat || !o.tok_out || !o.tok_host || !o.maxprob_host || (o.pos_dev && !o.tok0) || (o.x_next && !o.embed)) return hipErrorInvalidValue;
    GemvP p = {};
    p.w0 = wlm; p.in = x; p.gain = gain; p.eps = D.eps; p.K = D.d; p.n_rows = D.V; p.y = logits;
    p.vstat = vstat; p.clamp = clamp;
    int blocks = 0;
    hipError_t e = launch_gemv<EPI_STORE>(D, p, s, &blocks);
    if (e != hipSuccess) return e;
    if (blocks < 1 || blocks > GEMV_MAX_BLOCKS) return hipErrorInvalidValue;
    return step_finish(D, vstat, blocks, o, s);
}

// ---------------------------------------------------------------------------------------------
// multi-row path
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(const float* __restrict__ in, const float* __restrict__ gain,
                                                           int K, float eps, float* __restrict__ out)
{
    __shared__ float red[4];
    const float* x = in + (size_t)blockIdx.x * K;
    float* o = out + (size_t)blockIdx.x * K;
    float ss = 0.f;
    for (int i = threadIdx.x * 4; i < K; i += 1024) {
        float4 v = *reinterpret_cast<const float4*>(x + i);
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    float tot = block_sum<4>(ss, red);
    float sc = 1.0f / sqrtf(tot / (float)K + eps);
    for (int i = threadIdx.x * 4; i < K; i += 1024) {
        float4 v = *reinterpret_cast<const float4*>(x + i);
        float4 g = *reinterpret_cast<const float4*>(gain + i);
        v.x = v.x * sc * g.x; v.y = v.y * sc * g.y; v.z = v.z * sc * g.z; v.w = v.w * sc * g.w;
        *reinterpret_cast<float4*>(o + i) = v;
    }
}

hipError_t rmsnorm_rows(const float* in, const float* gain, int M, int K, float eps, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(rmsnorm_rows_kernel, dim3(M), dim3(256), 0, s, in, gain, K, eps, out);
    return hipGetLastError();
}

struct RowsP {
    const void* w[3];
    int n[3];       // rows of each stacked matrix (multiples of 16)
    int K;
    const float* x; // [M][K]
    float* y; int ldy;
    float* tap; int tap_ld;
    int M;
};

enum { RM_STORE = 0, RM_RESID = 1, RM_SWIGLU = 2 };

__device__ __forceinline__ void rows_epilogue(const RowsP& p, int mode, int r, size_t col, float v, float v2)
{
    if (mode == RM_STORE) {
        p.y[(size_t)r * p.ldy + col] = v;
    } else if (mode == RM_RESID) {
        float* dst = p.y + (size_t)r * p.ldy + col;
        float t = *dst + v;
        *dst = t;
        if (p.tap) p.tap[(size_t)r * p.tap_ld + col] = t;
    } else {
        p.y[(size_t)r * p.ldy + col] = v / (1.0f + __expf(-v)) * v2;
    }
}

// --- bf16 weights: MFMA tiles -------------------------------------------------------------------
// One block owns 16 consecutive output rows (RM_SWIGLU: 16 gate rows and the matching 16 up rows).
// Its 8 waves interleave over the K dimension in steps of 32: the weight tile is the MFMA A
// operand loaded straight from global memory (lane (r, g): row r, 8 consecutive k at 8g), the
// activations are the B operand (lane (c, g): token row c, same 8 k), split on the fly into
// bf16 hi = rne(x) and lo = rne(x - hi), so that hi + lo carries 16 mantissa bits of x.
constexpr int MF_WAVES = 8;
constexpr int MF_THREADS = MF_WAVES * 64;

__device__ __forceinline__ void split_hi_lo(const float (&x)[8], bf16x8_t& hi, bf16x8_t& lo)
{
#pragma unroll
    for (int j = 0; j < 8; j++) {
        __bf16 h = (__bf16)x[j];
        hi[j] = h;
        lo[j] = (__bf16)(x[j] - (float)h);
    }
}

template <int MODE>
__global__ __launch_bounds__(MF_THREADS) void gemm_rows_mfma_kernel(RowsP p)
{
    __shared__ float red[MF_WAVES][2][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int K = p.K;

    // which matrix / row tile does this block own?
    int tile = blockIdx.x;
    const uint16_t* W0; const uint16_t* W1 = nullptr;
    size_t col0;  // first output column of the tile
    if (MODE == RM_SWIGLU) {
        W0 = (const uint16_t*)p.w[0] + (size_t)tile * 16 * K;
        W1 = (const uint16_t*)p.w[1] + (size_t)tile * 16 * K;
        col0 = (size_t)tile * 16;
    } else {
        int t0 = p.n[0] >> 4, t1 = p.n[1] >> 4;
        if (tile < t0) { W0 = (const uint16_t*)p.w[0] + (size_t)tile * 16 * K; col0 = (size_t)tile * 16; }
        else if (tile < t0 + t1) { W0 = (const uint16_t*)p.w[1] + (size_t)(tile - t0) * 16 * K; col0 = (size_t)tile * 16; }
        else { W0 = (const uint16_t*)p.w[2] + (size_t)(tile - t0 - t1) * 16 * K; col0 = (size_t)tile * 16; }
    }
    const uint16_t* a0p = W0 + (size_t)r16 * K + g * 8;
    const uint16_t* a1p = MODE == RM_SWIGLU ? W1 + (size_t)r16 * K + g * 8 : nullptr;
    const bool have_col = r16 < p.M;
    const float* bp = p.x + (size_t)(have_col ? r16 : 0) * K + g * 8;

    f32x4_t acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    const int steps = (K + 31) >> 5;
#pragma unroll 2
    for (int st = wave; st < steps; st += MF_WAVES) {
        const int k0 = st << 5;
        const bool in_k = (k0 + g * 8) < K;  // K is a multiple of 8: a lane's 8 k are all in or all out
        bf16x8_t a0 = {}, a1 = {};
        float xb[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (in_k) {
            a0 = *reinterpret_cast<const bf16x8_t*>(a0p + k0);
            if (MODE == RM_SWIGLU) a1 = *reinterpret_cast<const bf16x8_t*>(a1p + k0);
            if (have_col) {
                float4 t0 = *reinterpret_cast<const float4*>(bp + k0);
                float4 t1 = *reinterpret_cast<const float4*>(bp + k0 + 4);
                xb[0] = t0.x; xb[1] = t0.y; xb[2] = t0.z; xb[3] = t0.w;
                xb[4] = t1.x; xb[5] = t1.y; xb[6] = t1.z; xb[7] = t1.w;
            }
        }
        bf16x8_t bh, bl;
        split_hi_lo(xb, bh, bl);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bh, acc0, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bl, acc0, 0, 0, 0);
        if (MODE == RM_SWIGLU) {
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bh, acc1, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bl, acc1, 0, 0, 0);
        }
    }
    // D layout: lane (c = lane % 16, g = lane / 16) holds rows 4g..4g+3 of column c
#pragma unroll
    for (int j = 0; j < 4; j++) {
        red[wave][0][(g * 4 + j) * 16 + r16] = acc0[j];
        if (MODE == RM_SWIGLU) red[wave][1][(g * 4 + j) * 16 + r16] = acc1[j];
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        int row = threadIdx.x & 15;   // output feature within the tile (fastest: coalesced stores)
        int c = threadIdx.x >> 4;     // token row
        if (c < p.M) {
            float v = 0.f, v2 = 0.f;
#pragma unroll
            for (int w = 0; w < MF_WAVES; w++) {
                v += red[w][0][row * 16 + c];
                if (MODE == RM_SWIGLU) v2 += red[w][1][row * 16 + c];
            }
            rows_epilogue(p, MODE, c, col0 + row, v, v2);
        }
    }
}

// --- fp32 weights, and fp16 shapes outside the MFMA tiling: FMA rows ------------------------------------------------
// One wave owns one pair of output rows (QKV: a rotary pair, or two value rows; SwiGLU: a gate row and its up row) and a
// group of MG token rows, so that even the projections of a 256-wide model are spread over a few hundred waves, and a wave
// has the loads of four steps in flight (what bounds these launches is latency, not bytes).  RMSNorm costs no launch: the
// gain goes into the weights as they are loaded, the sums of squares are taken from the activations that pass by anyway,
// and the row's scale is applied to the finished sums.  Rotary embedding and the cache rows are written by the epilogue.
// Measured on the fp32 model of width 256 with five rows, us per launch: output projection 13.9 -> 4.8, down 13.9 -> 7.7,
// gate/up 8.3 -> 5.4, QKV 7.4 -> 6.1 with norm and rotary embedding; five launches per layer instead of eight.
constexpr int RM_QKV = 3;
struct RowsPlainP {
    const void* w[3];
    int n[3];       // rows of each matrix (multiples of 16)
    int K;
    const float* x; // [M][K]
    const float* gain; float eps;   // RMSNorm of the rows folded in (null: rows as they are)
    float* y; int ldy;
    float* tap; int tap_ld; int tap_only;
    int M;
    const float* rope; const int* pos_dev; int pos_off;   // QKV
    int hd, dq, dkv, max_seq;
    void* kc; void* vc; int kt;
};

template <typename WT, int MODE>
__device__ __forceinline__ void plain_rows(const RowsPlainP& p, int u, const WT*& w0, const WT*& w1)
{
    const size_t K = p.K;
    if (MODE == RM_SWIGLU) { w0 = (const WT*)p.w[0] + u * K; w1 = (const WT*)p.w[1] + u * K; return; }
    if (MODE == RM_QKV) {
        const int j = 2 * u;
        if (j < p.dq + p.dkv) {
            const bool is_q = j < p.dq;
            const int jj = is_q ? j : j - p.dq, head = jj / p.hd, i = (jj % p.hd) >> 1;
            w0 = (const WT*)(is_q ? p.w[0] : p.w[1]) + (size_t)(head * p.hd + i) * K;
            w1 = w0 + (p.hd >> 1) * K;
        } else {
            w0 = (const WT*)p.w[2] + (size_t)(j - p.dq - p.dkv) * K;
            w1 = w0 + K;
        }
        return;
    }
    w0 = (const WT*)p.w[0] + 2 * u * K;   // STORE, RESID: one matrix
    w1 = w0 + K;
}

__device__ __forceinline__ float wave_sum_rows(float v)
{
    v = row16_sum(v);
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// U = load steps of a wave that are in flight together (1 where a row is no longer than that: a quarter of the code, which a
// short launch fetches cold)
template <typename WT, int MODE, int MG, int U>
__global__ __launch_bounds__(256) void rows_plain_kernel(RowsPlainP p)
{
    constexpr int VEC = Elem<WT>::VEC, STEP = 64 * VEC;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int K = p.K, m0 = blockIdx.y * MG, mg = min(MG, p.M - m0);
    const int n_units = MODE == RM_SWIGLU ? p.n[0] : (p.n[0] + p.n[1] + p.n[2]) / 2;
    for (int u = blockIdx.x * 4 + wave; u < n_units; u += gridDim.x * 4) {
        const WT* w0; const WT* w1;
        plain_rows<WT, MODE>(p, u, w0, w1);
        float a0[MG], a1[MG], ss[MG];
#pragma unroll
        for (int m = 0; m < MG; m++) a0[m] = a1[m] = ss[m] = 0.f;
        for (int k0 = 0; k0 < K; k0 += U * STEP) {
            float wa[U][VEC], wb[U][VEC];
#pragma unroll
            for (int t = 0; t < U; t++) {
                const int k = k0 + t * STEP + lane * VEC, kc = min(k, K - VEC);   // lanes past the row re-read its end
                Elem<WT>::load(w0 + kc, wa[t]);
                Elem<WT>::load(w1 + kc, wb[t]);
            }
            if (p.gain) {
#pragma unroll
                for (int t = 0; t < U; t++) {
                    const int kc = min(k0 + t * STEP + lane * VEC, K - VEC);
#pragma unroll
                    for (int j = 0; j < VEC; j++) {
                        const float g = p.gain[kc + j];
                        wa[t][j] *= g; wb[t][j] *= g;
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < MG; m++) {
                if (m >= mg) break;   // uniform
                const float* xr = p.x + (size_t)(m0 + m) * K;
#pragma unroll
                for (int t = 0; t < U; t++) {
                    const int k = k0 + t * STEP + lane * VEC;
                    if (k < K) {
#pragma unroll
                        for (int j = 0; j < VEC; j += 4) {
                            const float4 x = *reinterpret_cast<const float4*>(xr + k + j);
                            a0[m] = fmaf(wa[t][j], x.x, a0[m]); a0[m] = fmaf(wa[t][j + 1], x.y, a0[m]);
                            a0[m] = fmaf(wa[t][j + 2], x.z, a0[m]); a0[m] = fmaf(wa[t][j + 3], x.w, a0[m]);
                            a1[m] = fmaf(wb[t][j], x.x, a1[m]); a1[m] = fmaf(wb[t][j + 1], x.y, a1[m]);
                            a1[m] = fmaf(wb[t][j + 2], x.z, a1[m]); a1[m] = fmaf(wb[t][j + 3], x.w, a1[m]);
                            ss[m] += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
                        }
                    }
                }
            }
        }
        // every lane gets the sums; lane m finishes token row m0 + m
        float a = 0.f, b = 0.f, sq = 0.f;
#pragma unroll
        for (int m = 0; m < MG; m++) {
            if (m >= mg) break;   // uniform
            const float ta = wave_sum_rows(a0[m]), tb = wave_sum_rows(a1[m]), ts = p.gain ? wave_sum_rows(ss[m]) : 0.f;
            if (lane == m) { a = ta; b = tb; sq = ts; }
        }
        if (lane >= mg) continue;
        if (p.gain) {
            const float sc = 1.0f / sqrtf(sq / (float)K + p.eps);
            a *= sc; b *= sc;
        }
        const int r = m0 + lane;
        if (MODE == RM_SWIGLU) {
            p.y[(size_t)r * p.ldy + u] = a / (1.0f + __expf(-a)) * b;
        } else if (MODE == RM_QKV) {
            const int j = 2 * u, pos = p.pos_dev[0] + p.pos_off + r;
            if (j < p.dq + p.dkv) {
                const bool is_q = j < p.dq;
                const int jj = is_q ? j : j - p.dq, head = jj / p.hd, half = p.hd >> 1, i = (jj % p.hd) >> 1;
                const float* cs = p.rope + ((size_t)pos * half + i) * 2;
                const float ra = a * cs[0] - b * cs[1], rb = b * cs[0] + a * cs[1];
                if (is_q) {
                    float* q = p.y + (size_t)r * p.ldy + (size_t)head * p.hd + i;
                    q[0] = ra; q[half] = rb;
                } else {
                    const size_t o = ((size_t)head * p.max_seq + pos) * p.hd + i;
                    kv_put(p.kc, o, ra, p.kt);
                    kv_put(p.kc, o + half, rb, p.kt);
                }
            } else {
                const int e = j - p.dq - p.dkv;
                const size_t o = ((size_t)(e / p.hd) * p.max_seq + pos) * p.hd + (e % p.hd);
                kv_put(p.vc, o, a, p.kt);
                kv_put(p.vc, o + 1, b, p.kt);
            }
        } else {
            float* y = p.y + (size_t)r * p.ldy + 2 * u;
            if (MODE == RM_RESID) {
                a += y[0]; b += y[1];
                if (p.tap && (p.tap_only <= 0 || r == p.tap_only - 1)) {
                    float* tp = p.tap + (size_t)(p.tap_only > 0 ? 0 : r) * p.tap_ld + 2 * u;
                    tp[0] = a; tp[1] = b;
                }
            }
            y[0] = a; y[1] = b;
        }
    }
}

template <typename WT, int MODE>
static hipError_t rows_plain_t(const RowsPlainP& p, hipStream_t s)
{
    const int units = MODE == RM_SWIGLU ? p.n[0] : (p.n[0] + p.n[1] + p.n[2]) / 2;
    const int blocks = std::min(ceil_div(units, 4), 4096);
    // token rows of a wave: four where that covers the launch, else eight (a second group of waves reads the weights again,
    // from the caches)
    const bool one = p.K <= 64 * Elem<WT>::VEC;
    if (p.M <= 4 && one) hipLaunchKernelGGL((rows_plain_kernel<WT, MODE, 4, 1>), dim3(blocks, 1), dim3(256), 0, s, p);
    else if (p.M <= 4) hipLaunchKernelGGL((rows_plain_kernel<WT, MODE, 4, 4>), dim3(blocks, 1), dim3(256), 0, s, p);
    else if (one) hipLaunchKernelGGL((rows_plain_kernel<WT, MODE, 8, 1>), dim3(blocks, ceil_div(p.M, 8)), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((rows_plain_kernel<WT, MODE, 8, 4>), dim3(blocks, ceil_div(p.M, 8)), dim3(256), 0, s, p);
    return hipGetLastError();
}

bool rows_plain_supported(const Dims& D) { return D.wt != WT_BF16; }

hipError_t rows_plain(const Dims& D, const RowsPlain& g, hipStream_t s)
{
    if (!rows_plain_supported(D) || g.M < 1 || g.M > PLAIN_ROWS || g.K % 8) return hipErrorInvalidValue;
    if (g.mode != RM_QKV && g.mode != RM_SWIGLU && (g.n[1] || g.n[2])) return hipErrorInvalidValue;
    if (g.mode == RM_QKV && (g.n[0] != D.dq || g.n[1] != D.dkv || g.n[2] != D.dkv)) return hipErrorInvalidValue;
    RowsPlainP p = {};
    for (int i = 0; i < 3; i++) { p.w[i] = g.w[i]; p.n[i] = g.n[i]; }
    p.K = g.K; p.x = g.x; p.gain = g.gain; p.eps = D.eps; p.y = g.y; p.ldy = g.ldy; p.tap = g.tap; p.tap_ld = g.tap_ld; p.tap_only = g.tap_only; p.M = g.M;
    p.rope = g.rope; p.pos_dev = g.pos_dev; p.pos_off = g.pos_off; p.hd = D.hd; p.dq = D.dq; p.dkv = D.dkv; p.max_seq = D.max_seq;
    p.kc = g.kc; p.vc = g.vc; p.kt = D.kt;
    const bool f16 = D.wt == WT_F16;
    switch (g.mode) {
        case RM_STORE: return f16 ? rows_plain_t<f16_t, RM_STORE>(p, s) : rows_plain_t<float, RM_STORE>(p, s);
        case RM_RESID: return f16 ? rows_plain_t<f16_t, RM_RESID>(p, s) : rows_plain_t<float, RM_RESID>(p, s);
        case RM_SWIGLU: return f16 ? rows_plain_t<f16_t, RM_SWIGLU>(p, s) : rows_plain_t<float, RM_SWIGLU>(p, s);
        case RM_QKV: return f16 ? rows_plain_t<f16_t, RM_QKV>(p, s) : rows_plain_t<float, RM_QKV>(p, s);
    }
    return hipErrorInvalidValue;
}

template <int MODE>
static hipError_t gemm_rows_mode(const Dims& D, const RowsP& p, hipStream_t s)
{
    if (D.wt != WT_BF16) return hipErrorInvalidValue;   // the other types: rows_plain
    int tiles = MODE == RM_SWIGLU ? p.n[0] / 16 : (p.n[0] + p.n[1] + p.n[2]) / 16;
    hipLaunchKernelGGL((gemm_rows_mfma_kernel<MODE>), dim3(tiles), dim3(MF_THREADS), 0, s, p);
    return hipGetLastError();
}

hipError_t gemm_rows(const Dims& D, const RowsGemm& g, hipStream_t s)
{
    RowsP p = {};
    for (int i = 0; i < 3; i++) { p.w[i] = g.w[i]; p.n[i] = g.n[i]; }
    p.K = g.K; p.x = g.x; p.y = g.y; p.ldy = g.ldy; p.tap = g.tap; p.tap_ld = g.tap_ld; p.M = g.M;
    if (g.M < 1 || g.M > 16) return hipErrorInvalidValue;
    switch (g.mode) {
        case RM_STORE: return gemm_rows_mode<RM_STORE>(D, p, s);
        case RM_RESID: return gemm_rows_mode<RM_RESID>(D, p, s);
        case RM_SWIGLU: return gemm_rows_mode<RM_SWIGLU>(D, p, s);
    }
    return hipErrorInvalidValue;
}

// --- bf16 weights, multi-row MFMA GEMM at streaming speed (K a multiple of 64) -----------------------
// The verify / prompt path.  Activations arrive already split into two bf16 arrays hi = rne(x),
// lo = rne(x - hi) (hi + lo carries 16 mantissa bits of x), written once by whoever produced x,
// so the GEMM itself is nothing but loads and MFMAs.  RMSNorm costs no kernel of its own: the
// projection that finishes a residual row block (RESID mode) also writes x * gain of the NEXT norm as
// hi/lo plus, per 16-column tile, the partial sums of x^2; the consumer adds the partials of a row,
// and scales its finished dot products by rsqrt(mean + eps) -- the scale is a per-row scalar and
// commutes with the contraction.
//   * QKV mode orders the 16 rows of a tile as 8 rotary pairs (i, i + hd/2), so the epilogue can
//     rotate q and k and write k, v straight into the cache; SwiGLU mode writes its result
//     directly as the hi/lo pair the down projection consumes.
struct RowsP2 {
    const void* w[3];
    int n[3];  // rows of each stacked matrix (multiples of 16); SWIGLU: n[0] = n[1] = f
    int K;
    const uint16_t* bh; const uint16_t* bl; int ldb;  // activations [M][ldb], bf16 hi and lo
    float* y; int ldy;                                // fp32 output (STORE / RESID / QKV: q)
    uint16_t* oh; uint16_t* ol; int ldo;              // SWIGLU: hi/lo output
    float* tap; int tap_ld;
    int M;
    const float* rope; const int* pos_dev; int pos_off;
    int hd, dq, dkv, max_seq;
    void* kc; void* vc; int kt;                 // cache rows of this layer, element type (WeightType code)
    const float* ssq; int n_ssq; float eps;     // consumer: partial sums of squares [M][n_ssq] of the input rows (or null)
    const float* gain_out; float* ssq_out;      // RESID producer: gain of the next norm -> oh/ol = split(x * gain), ssq_out [M][n/16]
    int ksplit; float* kpart;                   // wide RESID only: K cut into ksplit slices (grid.y), raw sums to kpart [ksplit][M][n]
    int tile0, fin_tile0;                       // large tiles: first weight tile of this launch; first 64-column output tile of its finishing launch
    int tap_only;                               // > 0: only row tap_only - 1 writes its tap (a prompt needs the last row's only)
    float2* vmax; float clamp;                  // 16-row STORE, may be null: per (row, 16-column tile) maximum of the clamped outputs and its lowest column
    int n_tiles;                                // large-tile kernel: weight tiles of the launch
};

// hi = rne(v), lo = rne(v - hi) in the 16-bit storage type (bf16, or fp16 when f16 is set)
__device__ __forceinline__ void split_store(float v, uint16_t* hi, uint16_t* lo, size_t i, bool f16)
{
    const uint16_t h = f32_to_h16_bits(v, f16);
    hi[i] = h;
    lo[i] = f32_to_h16_bits(v - h16_bits_to_f32(h, f16), f16);
}
// 16x16x32 MFMA on two 128-bit operands holding 8 bf16 (or fp16) each
template <bool F16> __device__ __forceinline__ f32x4_t mfma_h16(u32x4_t a, u32x4_t b, f32x4_t c)
{
    if (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// weight row of logical row r16 of tile `tile`
template <int MODE>
__device__ __forceinline__ const uint16_t* m2_row(const RowsP2& p, int tile, int r16, int which /*SWIGLU: 0 gate, 1 up*/)
{
    if (MODE == RM_SWIGLU) return (const uint16_t*)p.w[which] + (size_t)(tile * 16 + r16) * p.K;
    if (MODE == RM_QKV) {
        const int tq = p.dq >> 4, tk = p.dkv >> 4;
        if (tile < tq + tk) {
            const uint16_t* base = (const uint16_t*)p.w[0];
            int tt = tile;
            if (tile >= tq) { base = (const uint16_t*)p.w[1]; tt = tile - tq; }
            const int tph = p.hd >> 4, head = tt / tph, th = tt % tph;
            const int row = head * p.hd + th * 8 + (r16 & 7) + (r16 >> 3) * (p.hd >> 1);
            return base + (size_t)row * p.K;
        }
        return (const uint16_t*)p.w[2] + (size_t)((tile - tq - tk) * 16 + r16) * p.K;
    }
    int row = tile * 16 + r16;
    if (row < p.n[0]) return (const uint16_t*)p.w[0] + (size_t)row * p.K;
    row -= p.n[0];
    if (row < p.n[1]) return (const uint16_t*)p.w[1] + (size_t)row * p.K;
    return (const uint16_t*)p.w[2] + (size_t)(row - p.n[1]) * p.K;
}

// position of activation row 0
template <int MODE> __device__ __forceinline__ int m6_pos0(const RowsP2& p) { return MODE == RM_QKV ? p.pos_dev[0] + p.pos_off : 0; }
// Final step of a tile: sum the KS per-wave partial tiles held in LDS (layout [wave][NT][256], element
// row*16 + column) and apply the mode's epilogue.  Executed by the whole block (it contains barriers in QKV mode).
// rs: per-column (= activation row) RMS scale in LDS, 1 where no norm applies.
// pre: what the epilogue reads from memory besides the sums, loaded by m2_preload while the weights stream (a load there
// costs its whole latency, about 1 us, and for the rotary pair two: the position comes first).
struct M2Pre { float a, b; int pos; };
template <int MODE>
__device__ __forceinline__ M2Pre m2_preload(const RowsP2& p, int t, int pos0)   // pos0: position of row 0 (QKV)
{
    M2Pre r = {0.f, 0.f, 0};
    const int tid = threadIdx.x, rr = tid & 15, c = min((tid >> 4) & 15, p.M - 1);
    if (MODE == RM_QKV) {
        const int tq = p.dq >> 4, tk = p.dkv >> 4;
        r.pos = pos0 + c;
        if (t < tq + tk) {
            const int tt = t < tq ? t : t - tq, th = tt % (p.hd >> 4), half = p.hd >> 1;
            const float* cs = p.rope + ((size_t)r.pos * half + th * 8 + (rr & 7)) * 2;
            r.a = cs[0]; r.b = cs[1];
        }
    } else if (MODE == RM_RESID) {
        const size_t colx = (size_t)t * 16 + rr;
        r.a = p.y[(size_t)c * p.ldy + colx];
        if (p.gain_out) r.b = p.gain_out[colx];
    }
    return r;
}
template <int MODE, bool F16>
__device__ __forceinline__ void m2_epilogue(const RowsP2& p, int t, const float* red, int KS, int ts, float* fin,
                                            const float* rs, const M2Pre& pre)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    const int tid = threadIdx.x;
    const int rr = tid & 15, c = (tid >> 4) & 15;
    float v = 0.f, v2 = 0.f;
    if (tid < 256) {
        for (int j = 0; j < KS; j++) {
            v += red[((ts * KS + j) * NT + 0) * 256 + rr * 16 + c];
            if (MODE == RM_SWIGLU) v2 += red[((ts * KS + j) * NT + 1) * 256 + rr * 16 + c];
        }
        if (MODE != RM_RESID) { v *= rs[c]; v2 *= rs[c]; }
        if (MODE == RM_QKV) fin[rr * 16 + c] = v;
    }
    if (MODE == RM_QKV) __syncthreads();
    if (tid < 256 && c < p.M) {
        if (MODE == RM_QKV) {
            const int tq = p.dq >> 4, tk = p.dkv >> 4;
            const int pos = pre.pos;
            if (t < tq + tk) {
                const bool is_q = t < tq;
                const int tt = is_q ? t : t - tq;
                const int tph = p.hd >> 4, head = tt / tph, th = tt % tph, half = p.hd >> 1;
                const int i = th * 8 + (rr & 7);
                const float av = fin[(rr & 7) * 16 + c], bv = fin[((rr & 7) + 8) * 16 + c];
                const float o = rr < 8 ? av * pre.a - bv * pre.b : bv * pre.a + av * pre.b;
                const int e = rr < 8 ? i : i + half;
                if (is_q) p.y[(size_t)c * p.ldy + (size_t)head * p.hd + e] = o;
                else kv_put(p.kc, ((size_t)head * p.max_seq + pos) * p.hd + e, o, p.kt);
            } else {
                const int e = (t - tq - tk) * 16 + rr;
                kv_put(p.vc, ((size_t)(e / p.hd) * p.max_seq + pos) * p.hd + (e % p.hd), v, p.kt);
            }
        } else {
            const size_t colx = (size_t)t * 16 + rr;
            if (MODE == RM_STORE) {
                p.y[(size_t)c * p.ldy + colx] = v;
                if (p.vmax) {   // the 16 columns of the tile are the 16 lanes of a DPP row, all active together
                    const float z = fminf(fmaxf(v, -p.clamp), p.clamp);
                    const float m = row16_max(z);
                    const unsigned long long eq = __ballot(z == m) >> (threadIdx.x & 48);   // this row's 16 lanes; never empty (z is clamped, no NaN)
                    if (rr == 0) p.vmax[(size_t)c * gridDim.x + t] = make_float2(m, __int_as_float(t * 16 + __ffsll(eq) - 1));
                }
            } else if (MODE == RM_RESID) {
                const float tv = pre.a + v;
                p.y[(size_t)c * p.ldy + colx] = tv;
                if (p.tap) p.tap[(size_t)c * p.tap_ld + colx] = tv;
                if (p.gain_out) {
                    split_store(tv * pre.b, p.oh, p.ol, (size_t)c * p.ldo + colx, F16);
                    // the 16 threads of one column are the 16 lanes of a DPP row, all active together
                    const float sq = row16_sum(tv * tv);
                    if (rr == 0) p.ssq_out[(size_t)c * (p.n[0] >> 4) + t] = sq;
                }
            } else split_store(v / (1.0f + __expf(-v)) * v2, p.oh, p.ol, (size_t)c * p.ldo + colx, F16);
        }
    }
    if (MODE == RM_QKV) __syncthreads();
}

// LDS-staged variant: the block fetches a 16-row x 512-k stripe of the weights the way the single-row
// GEMV does -- every wave two whole rows, 1 KB contiguous per load instruction, which is the access
// shape that streams fastest from HBM -- plus the matching slice of the hi/lo activations, parks both
// in LDS, and the MFMA operands are then read from LDS in fragment order.  Activations never enter
// the in-order global-load queue between weight loads, so the next stripe's loads stay in flight
// during the whole MFMA phase.
constexpr int M3_CK = 512;
constexpr int M3_PITCH = M3_CK * 2 + 16;  // bytes per LDS row (16-byte pad spreads the banks)

// M3_D = stripes in flight per block; F16: fp16 storage, else bf16; NU = activation rows (hi and lo counted) per wave and
// stripe (2 covers up to 8 rows, 3 up to 12, 4 up to 16).  The number of blocks that fit a CU decides how much of the weight
// stream is in flight, and registers decide that number: every row pointer is wave-uniform and lives in scalar registers, so
// that three blocks fit (six waves per SIMD) at all row counts; with per-thread pointers nine rows and more had two.  7B, 9
// rows, fp16: gate/up 42.7 -> 35.0 us, QKV 31.2 -> 23.4, LM head 61 -> 52; 5 rows: QKV 22.5 -> 20.5, gate/up 33.7 -> 32.9.
// 13 to 16 rows: QKV and the residual projections keep 16 bytes per lane in scratch for the third block; two blocks without
// are as fast (verify of 14 / 16 rows, four 7B layers: 0.58 / 0.60 ms either way, 0.67 / 0.68 with per-thread pointers).
template <int MODE, int M3_D, bool F16, int NU>
__global__ __launch_bounds__(512, (M3_D * (MODE == RM_SWIGLU ? 4 + NU : 2 + NU) > 12 ? 4 : 6)) void rows_mfma3_kernel(RowsP2 p)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    extern __shared__ __align__(16) unsigned char sm3[];
    __shared__ float fin[256];
    __shared__ float rs[16];
    unsigned char* As = sm3;                          // [NT][16][PITCH]
    unsigned char* Bh = sm3 + NT * 16 * M3_PITCH;     // [M][PITCH]
    unsigned char* Bl = Bh + p.M * M3_PITCH;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform for the compiler: row pointers in scalar registers
    const int r16 = lane & 15, g = lane >> 4;
    const int tile = blockIdx.x;
    const int K = p.K, M = p.M;
    const int NC = (K + M3_CK - 1) / M3_CK;

    const uint16_t* ap[NT][2];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int j = 0; j < 2; j++) ap[t][j] = m2_row<MODE>(p, tile, 2 * wave + j, t);
    // activation rows of one stripe: hi rows 0 .. M - 1, then the lo rows; wave w takes rows w, w + 8, .. (1 KB each)
    const uint16_t* bsrc[NU];
#pragma unroll
    for (int u = 0; u < NU; u++) {
        const int row = min(wave + u * 8, 2 * M - 1);
        bsrc[u] = row < M ? p.bh + (size_t)row * p.ldb : p.bl + (size_t)(row - M) * p.ldb;
    }
    // Register ring: the loads of the next M3_D stripes are in flight while one stripe is multiplied.  Every load is
    // UNCONDITIONAL: addresses past the end of K (or past the last activation vector) are clamped to valid ones and
    // the values are replaced by zeros when the stripe is stored to LDS.  With loads under conditions the compiler
    // cannot count what is in flight and waits for everything, the stripes just requested included.
    u32x4_t ra[M3_D][NT][2], rb[M3_D][NU];
    const u32x4_t zero4 = {0u, 0u, 0u, 0u};
    auto gload = [&](int slot, int ck) {
        const int k0 = ck * M3_CK;
        const int ka = min(k0 + lane * 8, K - 8);
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int j = 0; j < 2; j++) ra[slot][t][j] = gv_load(ap[t][j] + ka);
#pragma unroll
        for (int u = 0; u < NU; u++) rb[slot][u] = *reinterpret_cast<const u32x4_t*>(bsrc[u] + ka);
    };
    f32x4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int bc = min(r16, M - 1);  // columns >= M read a valid row; their results are never stored
    auto stage = [&](int slot, int ck) {
        const int k0 = ck * M3_CK;
        const bool ok = k0 + lane * 8 < K;
        __syncthreads();  // previous stripe fully consumed
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                *reinterpret_cast<u32x4_t*>(As + (t * 16 + 2 * wave + j) * M3_PITCH + lane * 16) = ok ? ra[slot][t][j] : zero4;
#pragma unroll
        for (int u = 0; u < NU; u++)
            if (wave + u * 8 < 2 * M) *reinterpret_cast<u32x4_t*>(Bh + (wave + u * 8) * M3_PITCH + lane * 16) = ok ? rb[slot][u] : zero4;
        __syncthreads();
    };
    auto multiply = [&](int ck) {
        const int nks = min(M3_CK / 32, (K - ck * M3_CK) / 32);
        for (int s = wave; s < nks; s += 8) {
            const int off = s * 64 + g * 16;
            const u32x4_t bh = *reinterpret_cast<const u32x4_t*>(Bh + bc * M3_PITCH + off);
            const u32x4_t bl = *reinterpret_cast<const u32x4_t*>(Bl + bc * M3_PITCH + off);
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const u32x4_t w = *reinterpret_cast<const u32x4_t*>(As + (t * 16 + r16) * M3_PITCH + off);
                acc[t] = mfma_h16<F16>(w, bh, acc[t]);
                acc[t] = mfma_h16<F16>(w, bl, acc[t]);
            }
        }
    };
    // The blocks of a launch start together and would all ask the memory channels for the same stripe at the same time:
    // block `tile` starts its walk over K at stripe (tile / 8) % NC and wraps around (workgroups go to the eight XCDs
    // round-robin by id, so blocks that follow each other on one XCD start one stripe apart).  Measured against a walk
    // from 0 in every block: 7B QKV 28.0 -> 25.1 us, gate/up 39.4 -> 36.3, down 24.6 -> 22.6; 70B gate/up 170 -> 147,
    // output projection 35 -> 29, LM head 108 -> 90 (a start at tile % NC instead is 20 % SLOWER than a walk from 0 at
    // K = 8192).
    const int rot = (tile / 8) % NC;
    auto sidx = [&](int i) { const int c = min(i, NC - 1) + rot; return c >= NC ? c - NC : c; };
    // RMS scale of every activation row from the producer's per-tile sums of squares (read by the epilogue).  They are requested
    // in front of the weights: loads return in order, and behind the first stripes of all blocks the scales would hold up the
    // first multiplication until these are all there; summed behind the weight stream they cost their latency at the end.
    // Verifications at 7B, 5 rows bf16 / 9 rows fp16, us, before and now: QKV 20.6 -> 20.2 / 23.5 -> 23.0, gate/up 33.2 -> 33.0 /
    // 35.4 -> 34.0, LM head 44.0 -> 42.8 / 52.7 -> 50.0.
    // Every entry, the 1 of a row without a scale included, has a single writer (rows_of_wave): no initial pass by other
    // threads, which would need a barrier of its own before the scales go in.
    constexpr int SQR = NU > 2 ? 2 : 1, SQN = 8;   // rows of a wave that may have a scale (NU = 2: up to 8 rows in all), sums per lane requested here
    const bool scaled = MODE != RM_RESID && p.ssq;
    const int pos0 = m6_pos0<MODE>(p);   // (the rotary pairs are requested once it is there)
    float sq[SQR][SQN];
    if (MODE != RM_RESID) {   // (rows without sums re-read an activation: a condition here would make the compiler wait for the first load)
        const float* src = scaled ? p.ssq : reinterpret_cast<const float*>(p.bh);
        const int n = scaled ? p.n_ssq : 1;
#pragma unroll
        for (int r = 0; r < SQR; r++)
#pragma unroll
            for (int u = 0; u < SQN; u++) sq[r][u] = src[(size_t)min(wave + 8 * r, M - 1) * n + min(lane + u * 64, n - 1)];
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int sl = 0; sl < M3_D; sl++) gload(sl, sidx(sl));
    const M2Pre pre = m2_preload<MODE>(p, tile, pos0);
    rows_of_wave(wave, [&](int c) {
        float v = 1.0f;
        if (scaled && c < M) {
            float t = 0.f;
#pragma unroll
            for (int r = 0; r < SQR; r++)
                if (c == wave + 8 * r) {
#pragma unroll
                    for (int u = 0; u < SQN; u++) t += lane + u * 64 < p.n_ssq ? sq[r][u] : 0.f;
                }
            for (int i = lane + SQN * 64; i < p.n_ssq; i += 64) t += p.ssq[(size_t)c * p.n_ssq + i];
            v = 1.0f / sqrtf(wave_sum(t) / (float)K + p.eps);
        }
        if (lane == 0) rs[c] = v;
    });
    // steady state: every step stores its slot's stripe, refills the slot and multiplies; the stripe count is padded
    // to a multiple of M3_D (a padding request re-reads the last stripe and is never stored); the last M3_D steps
    // request nothing
    const int NCp = (NC + M3_D - 1) / M3_D * M3_D;
    int ck0 = 0;
    for (; ck0 + M3_D < NCp; ck0 += M3_D) {
#pragma unroll
        for (int sl = 0; sl < M3_D; sl++) {
            stage(sl, sidx(ck0 + sl));
            gload(sl, sidx(ck0 + sl + M3_D));
            multiply(sidx(ck0 + sl));
        }
    }
#pragma unroll
    for (int sl = 0; sl < M3_D; sl++) {
        if (ck0 + sl < NC) {   // uniform
            stage(sl, sidx(ck0 + sl));
            multiply(sidx(ck0 + sl));
        }
    }
    __syncthreads();
    float* red = reinterpret_cast<float*>(sm3);  // [8][NT][256] floats fit inside the weight stripe area
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int j = 0; j < 4; j++) red[(wave * NT + t) * 256 + (g * 4 + j) * 16 + r16] = acc[t][j];
    __syncthreads();
    m2_epilogue<MODE, F16>(p, tile, red, 8, 0, fin, rs, pre);
}

template <int MODE, int DEPTH, bool F16, int NU>
static hipError_t launch_mfma3_nu(const RowsP2& p, int n_tiles, hipStream_t s)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    const size_t lds = (size_t)(NT * 16 + 2 * p.M) * M3_PITCH;
    static std::atomic<size_t> lds_limit{0};  // per instantiation
    {
        hipError_t e = ensure_lds((const void*)rows_mfma3_kernel<MODE, DEPTH, F16, NU>, lds, lds_limit);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((rows_mfma3_kernel<MODE, DEPTH, F16, NU>), dim3(n_tiles), dim3(512), lds, s, p);
    return hipGetLastError();
}

template <int MODE, int DEPTH, bool F16>
static hipError_t launch_mfma3(const RowsP2& p, int n_tiles, hipStream_t s)
{
    if (p.M <= 8) return launch_mfma3_nu<MODE, DEPTH, F16, 2>(p, n_tiles, s);
    if (p.M <= 12) return launch_mfma3_nu<MODE, DEPTH, F16, 3>(p, n_tiles, s);
    return launch_mfma3_nu<MODE, DEPTH, F16, 4>(p, n_tiles, s);
}

template <int MODE, bool F16>
static hipError_t rows_fused_mode(const RowsP2& p, hipStream_t s, const LaunchOpts* opt)
{
    const int forced = opt ? opt->rows_depth : 0;
    const int n_tiles = MODE == RM_SWIGLU ? p.n[0] / 16 : (p.n[0] + p.n[1] + p.n[2]) / 16;
    // measured (`KB_ROWS=1 kernel_bench`, and at the 13B / 70B / Llama-3-8B shapes): two stripes in flight are best or
    // equal everywhere (down projection, 5 rows: 17.6 us against 23.2 with one, 19.1 with three) except gate/up, whose ring for
    // two stripes of two matrices is too large for the registers of three blocks per CU from nine rows on, and gains nothing below
    // (in verifications of five rows 32.8 against 33.0 us at 7B, 153.8 against 148.5 at 70B)
    const int depth = forced > 0 ? forced : (MODE == RM_SWIGLU ? 1 : 2);
    switch (depth) {
        case 1: return launch_mfma3<MODE, 1, F16>(p, n_tiles, s);
        case 2: return launch_mfma3<MODE, 2, F16>(p, n_tiles, s);
        default: return launch_mfma3<MODE, 3, F16>(p, n_tiles, s);
    }
}

// --- wide-block variant: up to 64 activation rows per pass (prompt blocks, the 2L confidence rows) -------
// With that many rows a 16-row weight tile would pull eight times more activation bytes out of the cache
// than weight bytes out of HBM.  Here a block owns 64 weight rows (64 of each matrix in SwiGLU mode) and all
// (<= 64) rows.  64 x 128-k stripes of the weights (non-temporal) and of the hi/lo rows go through LDS; a
// stripe has four 32-wide k-steps: wave w takes k-step w & 3 for the weight rows 32 (w >> 2) .. +31 and all
// rows, so every staged byte is read twice only, and the four k-step partials are summed through LDS at the
// end, band by band of 16 rows, where the mode's epilogue is applied.  52 KB of LDS per block (70 KB for
// SwiGLU): two to three blocks share a CU and cover each other's load / stage / multiply phases, which
// measured better than a deeper register ring.  Same modes, same RMSNorm folding and the same rotary-pair
// row order (here 32 pairs per tile) as the 16-row kernel.
constexpr int M6_CK = 128;
constexpr int M6_PITCH = M6_CK * 2 + 16;

// weight row of logical row r64 of tile `tile`
template <int MODE>
__device__ __forceinline__ const uint16_t* m6_row(const RowsP2& p, int tile, int r64, int which /*SWIGLU: 0 gate, 1 up*/)
{
    if (MODE == RM_SWIGLU) return (const uint16_t*)p.w[which] + (size_t)(tile * 64 + r64) * p.K;
    if (MODE == RM_QKV) {
        const int tq = p.dq >> 6, tk = p.dkv >> 6;
        if (tile < tq + tk) {
            const uint16_t* base = (const uint16_t*)p.w[0];
            int tt = tile;
            if (tile >= tq) { base = (const uint16_t*)p.w[1]; tt = tile - tq; }
            const int tph = p.hd >> 6, head = tt / tph, th = tt % tph;
            const int row = head * p.hd + th * 32 + (r64 & 31) + (r64 >> 5) * (p.hd >> 1);
            return base + (size_t)row * p.K;
        }
        return (const uint16_t*)p.w[2] + (size_t)((tile - tq - tk) * 64 + r64) * p.K;
    }
    int row = tile * 64 + r64;
    if (row < p.n[0]) return (const uint16_t*)p.w[0] + (size_t)row * p.K;
    row -= p.n[0];
    if (row < p.n[1]) return (const uint16_t*)p.w[1] + (size_t)row * p.K;
    return (const uint16_t*)p.w[2] + (size_t)(row - p.n[1]) * p.K;
}

// Epilogue of the 64-row tiling, for whole waves: a wave holds the 64 weight rows (= output columns) of tile `tile` for one
// activation row m, nn = lane.  Three parts, because a wave has 8 to 64 rows and what they share must not be done per row:
//   m6_col   where the lane's column goes and what belongs to it (once per wave and tile; the addressing of the cache rows with
//            its divisions took 16 us of a 512-row QKV launch when it was done per row);
//   m6_pre   what a row reads besides its sums (QKV: the rotary pair, RESID: the residual), for several rows at once: a load between
//            the stores of two rows waits for its own latency and for the stores before it;
//   m6_row   the row itself, finished and scaled sums v (and v2 of the second matrix in SwiGLU mode).
// Measured, 7B, 512 rows, in the prompt pass: QKV 135 -> 120 us, residual finishing pass 12.2 -> 11.5; 13B QKV 181 -> 164.
struct M6Col { size_t off; int stride; int kind; float gain; const float* rope; };   // kind: QKV 0 q, 1 k, 2 v
struct M6Pre { float a, b; };
template <int MODE>
__device__ __forceinline__ M6Col m6_col(const RowsP2& p, int tile, int nn, int pos0)
{
    M6Col c = {(size_t)tile * 64 + nn, MODE == RM_SWIGLU ? p.ldo : p.ldy, 0, 0.f, nullptr};
    if (MODE == RM_RESID) {
        if (p.gain_out) c.gain = p.gain_out[c.off];
    } else if (MODE == RM_QKV) {   // rotary pairs are (nn, nn + 32) for nn < 32
        const int tq = p.dq >> 6, tk = p.dkv >> 6, tph = p.hd >> 6, half = p.hd >> 1;   // tph: 1 or 2 tiles per head
        c.kind = tile < tq ? 0 : tile < tq + tk ? 1 : 2;
        const int tt = c.kind == 0 ? tile : c.kind == 1 ? tile - tq : tile - tq - tk, head = tph == 2 ? tt >> 1 : tt, th = tph == 2 ? tt & 1 : 0;
        const int i = th * 32 + (nn & 31), e = c.kind == 2 ? th * 64 + nn : nn < 32 ? i : i + half;
        c.rope = p.rope + ((size_t)pos0 * half + i) * 2;
        if (c.kind == 0) c.off = (size_t)head * p.hd + e;
        else { c.off = ((size_t)head * p.max_seq + pos0) * p.hd + e; c.stride = p.hd; }
    }
    return c;
}
template <int MODE>
__device__ __forceinline__ M6Pre m6_pre(const RowsP2& p, const M6Col& c, int m)
{
    M6Pre r = {0.f, 0.f};
    if (MODE == RM_RESID) {
        r.a = p.y[c.off + (size_t)m * c.stride];
    } else if (MODE == RM_QKV) {
        if (c.kind < 2) {
            const float2 cs = *reinterpret_cast<const float2*>(c.rope + (size_t)m * p.hd);
            r.a = cs.x; r.b = cs.y;
        }
    }
    return r;
}
template <int MODE, bool F16>
__device__ __forceinline__ void m6_row(const RowsP2& p, const M6Col& c, int tile, int m, int nn, float v, float v2, const M6Pre& pre)
{
    const size_t o = c.off + (size_t)m * c.stride;
    if (MODE == RM_STORE) {
        p.y[o] = v;
    } else if (MODE == RM_SWIGLU) {
        split_store(v / (1.0f + __expf(-v)) * v2, p.oh, p.ol, o, F16);
    } else if (MODE == RM_RESID) {
        const float tv = pre.a + v;
        const size_t colx = (size_t)tile * 64 + nn;
        p.y[o] = tv;
        if (p.tap && (p.tap_only <= 0 || m == p.tap_only - 1)) p.tap[(size_t)(p.tap_only > 0 ? 0 : m) * p.tap_ld + colx] = tv;
        if (p.gain_out) {
            split_store(tv * c.gain, p.oh, p.ol, (size_t)m * p.ldo + colx, F16);
            const float sq = wave_sum(tv * tv);   // the wave holds the tile's 64 columns of row m
            if (nn == 0) p.ssq_out[(size_t)m * (p.n[0] >> 6) + tile] = sq;
        }
    } else {
        if (c.kind < 2) {
            const float other = __shfl_xor(v, 32, 64);
            const float av = nn < 32 ? v : other, bv = nn < 32 ? other : v;
            v = nn < 32 ? fmaf(av, pre.a, -(bv * pre.b)) : fmaf(bv, pre.a, av * pre.b);
        }
        if (c.kind == 0) p.y[o] = v;
        else kv_put(c.kind == 1 ? p.kc : p.vc, o, v, p.kt);
    }
}

// RMS scales of activation rows from the producer's sums of squares [M][n_ssq]: a wave takes NR rows, row0 + u * step, and requests the
// sums of all of them together -- in front of its first weights, since loads return in order.  One row after the other, each
// waiting for its own load, 16 rows took a wave of the large-tile kernel 16 us, before anything was multiplied.
template <int NR>
struct RowScales {
    float v[NR];
    __device__ __forceinline__ void load(const float* ssq, int n_ssq, int row0, int step, int M, int i0, int lane)
    {
        const int i = min(i0 + lane, n_ssq - 1);
#pragma unroll
        for (int u = 0; u < NR; u++) v[u] = ssq[(size_t)min(row0 + u * step, M - 1) * n_ssq + i];
    }
    // put(u, scale): called by all lanes, rows past M repeat the last one
    template <typename F>
    __device__ __forceinline__ void finish(const float* ssq, int n_ssq, int row0, int step, int M, int lane, int K, float eps, F&& put)
    {
        float t[NR];
#pragma unroll
        for (int u = 0; u < NR; u++) t[u] = lane < n_ssq ? v[u] : 0.f;
        for (int i0 = 64; i0 < n_ssq; i0 += 64) {
            load(ssq, n_ssq, row0, step, M, i0, lane);
#pragma unroll
            for (int u = 0; u < NR; u++) t[u] += i0 + lane < n_ssq ? v[u] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < NR; u++) put(u, 1.0f / sqrtf(wave_sum(t[u]) / (float)K + eps));
    }
};

template <int MODE, bool F16, int M6_D>  // M6_D = stripes in flight per block
__global__ __launch_bounds__(512) void rows_wide_kernel(RowsP2 p)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    extern __shared__ __align__(16) unsigned char sm6[];
    __shared__ float rs[64];
    unsigned char* As = sm6;                            // [NT * 64][PITCH]
    unsigned char* Bh = sm6 + NT * 64 * M6_PITCH;       // [64][PITCH]
    unsigned char* Bl = Bh + 64 * M6_PITCH;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int tile = blockIdx.x, n0 = tile * 64;
    const int K = p.K, M = p.M;
    // this block's stripes: all of K, or slice blockIdx.y of ksplit (projections with few tiles are cut along K so
    // that every CU has a block; their raw sums go to kpart and rows_finish_resid_kernel adds them up in order)
    const int NCall = K / M6_CK;
    const int S = p.ksplit > 1 ? p.ksplit : 1;
    const int c_begin = (int)((long)NCall * blockIdx.y / S), NC = (int)((long)NCall * (blockIdx.y + 1) / S) - c_begin;
    // weights: wave w loads logical rows 8w .. 8w+7; instruction j covers rows 8w+4j .. 8w+4j+3 (16 lanes = 256 B per row)
    const int arow = 8 * wave + (lane >> 4), acol = (lane & 15) * 8;
    const uint16_t* ap[NT][2];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int j = 0; j < 2; j++) ap[t][j] = m6_row<MODE>(p, tile, arow + 4 * j, t) + acol;
    // activations: 64 rows x 16 vectors per array; thread takes vectors tid and tid + 512 (row clamped to M - 1)
    const uint16_t* bhp[2];
    const uint16_t* blp[2];
    int bdst[2];
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const int v = tid + u * 512, row = v >> 4, kk = (v & 15) * 8;
        const size_t off = (size_t)min(row, M - 1) * p.ldb + kk;
        bhp[u] = p.bh + off; blp[u] = p.bl + off;
        bdst[u] = row * M6_PITCH + kk * 2;
    }
    u32x4_t ra[M6_D][NT][2], rh[M6_D][2], rl[M6_D][2];
    auto gload = [&](int slot, int ck) {
        const int k0 = (c_begin + ck) * M6_CK;
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int j = 0; j < 2; j++) ra[slot][t][j] = gv_load(ap[t][j] + k0);
#pragma unroll
        for (int u = 0; u < 2; u++) {
            rh[slot][u] = *reinterpret_cast<const u32x4_t*>(bhp[u] + k0);
            rl[slot][u] = *reinterpret_cast<const u32x4_t*>(blp[u] + k0);
        }
    };
    auto stage = [&](int slot) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                *reinterpret_cast<u32x4_t*>(As + (t * 64 + arow + 4 * j) * M6_PITCH + acol * 2) = ra[slot][t][j];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            *reinterpret_cast<u32x4_t*>(Bh + bdst[u]) = rh[slot][u];
            *reinterpret_cast<u32x4_t*>(Bl + bdst[u]) = rl[slot][u];
        }
        __syncthreads();
    };
    const int kq = wave & 3, nh = wave >> 2;             // k-step of the stripe, half of the weight rows
    const int MT = (M + 15) >> 4;                        // live 16-row groups of activation rows
    f32x4_t acc[NT][2][4];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 4; j++) acc[t][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&]() {
        const int off = kq * 64 + g * 16;
        u32x4_t a[NT][2];
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int i = 0; i < 2; i++)
                a[t][i] = *reinterpret_cast<const u32x4_t*>(As + (t * 64 + (nh * 2 + i) * 16 + r16) * M6_PITCH + off);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            if (j < MT) {   // uniform
                const u32x4_t h = *reinterpret_cast<const u32x4_t*>(Bh + (j * 16 + r16) * M6_PITCH + off);
                const u32x4_t l = *reinterpret_cast<const u32x4_t*>(Bl + (j * 16 + r16) * M6_PITCH + off);
                // independent accumulators between the two updates of any one of them
#pragma unroll
                for (int t = 0; t < NT; t++)
#pragma unroll
                    for (int i = 0; i < 2; i++) acc[t][i][j] = mfma_h16<F16>(a[t][i], h, acc[t][i][j]);
#pragma unroll
                for (int t = 0; t < NT; t++)
#pragma unroll
                    for (int i = 0; i < 2; i++) acc[t][i][j] = mfma_h16<F16>(a[t][i], l, acc[t][i][j]);
            }
        }
    };
    // RMS scale of every activation row (read by the epilogue); a K-split launch leaves the scaling to its finishing kernel
    const bool scaled = MODE != RM_RESID && p.ssq && S == 1;
    RowScales<8> scales;
    if (scaled) scales.load(p.ssq, p.n_ssq, wave, 8, M, 0, lane);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int sl = 0; sl < M6_D; sl++)
        if (sl < NC) gload(sl, sl);
    if (scaled) scales.finish(p.ssq, p.n_ssq, wave, 8, M, lane, K, p.eps, [&](int u, float v) { if (lane == 0) rs[wave + 8 * u] = v; });
    else if (tid < 64) rs[tid] = 1.0f;
    int ck0 = 0;
    for (; ck0 + 2 * M6_D <= NC; ck0 += M6_D) {   // steady state: every step refills its slot
#pragma unroll
        for (int sl = 0; sl < M6_D; sl++) {
            stage(sl);
            gload(sl, ck0 + sl + M6_D);
            multiply();
        }
    }
    for (; ck0 < NC; ck0 += M6_D) {               // drain
#pragma unroll
        for (int sl = 0; sl < M6_D; sl++) {
            if (ck0 + sl < NC) {
                stage(sl);
                if (ck0 + sl + M6_D < NC) gload(sl, ck0 + sl + M6_D);
                multiply();
            }
        }
    }
    // Sum the four k-step partials of every output, one band of 16 activation rows at a time, through LDS:
    // red[t][wave][i][256], element row * 16 + column of the D layout (lane (c = lane % 16, g) holds weight
    // rows 4g .. 4g+3 of activation row c), then the epilogue: thread -> (weight row nn, activation row c).
    float* red = reinterpret_cast<float*>(sm6);   // NT x 8 x 2 x 256 floats = NT x 16 KB
    const M6Col col = m6_col<MODE>(p, tile, lane, m6_pos0<MODE>(p));
    for (int j = 0; j < MT; j++) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; t++)
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    float v;
                    switch (j) {  // acc is indexed by compile-time constants only
                        case 0: v = acc[t][i][0][e]; break;
                        case 1: v = acc[t][i][1][e]; break;
                        case 2: v = acc[t][i][2][e]; break;
                        default: v = acc[t][i][3][e]; break;
                    }
                    red[((t * 8 + wave) * 2 + i) * 256 + (g * 4 + e) * 16 + r16] = v;
                }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 2; it++) {   // 64 weight rows x 16 activation rows = 1024 outputs, two per thread
            const int o = tid + it * 512;
            const int nn = o & 63, c = o >> 6;      // c (and so m) is uniform over a wave, nn = lane
            const int st = nn >> 4, hh = st >> 1, ii = st & 1;
            float v = 0.f, v2 = 0.f;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                v += red[((hh * 4 + q) * 2 + ii) * 256 + (nn & 15) * 16 + c];
                if (MODE == RM_SWIGLU) v2 += red[(((8 + hh * 4 + q) * 2) + ii) * 256 + (nn & 15) * 16 + c];
            }
            const int m = j * 16 + c;
            if (m >= M) continue;
            if (S > 1) {   // raw sums of this K slice: [slice][matrix][M][n_total]
                const size_t nt = (size_t)gridDim.x * 64;
                p.kpart[(((size_t)blockIdx.y * NT + 0) * M + m) * nt + n0 + nn] = v;
                if (MODE == RM_SWIGLU) p.kpart[(((size_t)blockIdx.y * NT + 1) * M + m) * nt + n0 + nn] = v2;
                continue;
            }
            if (MODE != RM_RESID) { v *= rs[m]; v2 *= rs[m]; }
            m6_row<MODE, F16>(p, col, tile, m, nn, v, v2, m6_pre<MODE>(p, col, m));
        }
    }
}

// Second half of a K-split launch: one wave per (FIN_ROWS rows, 64-column tile) adds the slices in a fixed order,
// applies the RMS scale of each row (summing the producer's partials itself) and runs the mode's epilogue.  The
// loads of the wave's rows are independent and issued together.
constexpr int FIN_ROWS = 4;
template <int MODE, bool F16>
__global__ __launch_bounds__(64) void rows_finish_kernel(RowsP2 p)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    const int tile = blockIdx.x + p.fin_tile0, lane = threadIdx.x;   // kpart covers this launch's tiles only
    const int mbase = blockIdx.y * FIN_ROWS;
    const size_t nt = (size_t)gridDim.x * 64, colx = (size_t)blockIdx.x * 64 + lane;
    const M6Col col = m6_col<MODE>(p, tile, lane, m6_pos0<MODE>(p));
    const bool scaled = MODE != RM_RESID && p.ssq;
    RowScales<FIN_ROWS> scales;
    if (scaled) scales.load(p.ssq, p.n_ssq, mbase, 1, p.M, 0, lane);
    float v[FIN_ROWS], v2[FIN_ROWS], sc[FIN_ROWS];
    M6Pre pre[FIN_ROWS];
#pragma unroll
    for (int r = 0; r < FIN_ROWS; r++) {
        const int m = min(mbase + r, p.M - 1);   // rows past M re-read the last row, never written
        v[r] = v2[r] = 0.f;
        pre[r] = m6_pre<MODE>(p, col, m);
    }
    // two slices of all rows are requested together (slices past the last one re-read it, never added)
    for (int s0 = 0; s0 < p.ksplit; s0 += 2) {
        float a[2][FIN_ROWS], b[2][FIN_ROWS];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int r = 0; r < FIN_ROWS; r++) {
                const int m = min(mbase + r, p.M - 1), sl = min(s0 + u, p.ksplit - 1);
                a[u][r] = p.kpart[(((size_t)sl * NT + 0) * p.M + m) * nt + colx];
                if (MODE == RM_SWIGLU) b[u][r] = p.kpart[(((size_t)sl * NT + 1) * p.M + m) * nt + colx];
            }
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int r = 0; r < FIN_ROWS; r++)
                if (s0 + u < p.ksplit) {   // uniform
                    v[r] += a[u][r];
                    if (MODE == RM_SWIGLU) v2[r] += b[u][r];
                }
    }
    if (scaled) scales.finish(p.ssq, p.n_ssq, mbase, 1, p.M, lane, p.K, p.eps, [&](int u, float x) { sc[u] = x; });
#pragma unroll
    for (int r = 0; r < FIN_ROWS; r++) {
        const int m = mbase + r;
        if (m >= p.M) break;   // uniform
        float a = v[r], b = v2[r];
        if (scaled) { a *= sc[r]; b *= sc[r]; }
        m6_row<MODE, F16>(p, col, tile, m, lane, a, b, pre[r]);
    }
}

// --- large-tile variant: any number of activation rows in one launch (whole prompts, the context window) --------
// With hundreds of rows the work is a real GEMM and the weights should cross the chip once, not once per 64 rows.
// A block owns TN logical weight rows (TN / 2 gate + TN / 2 up rows in SwiGLU mode) x 128 activation rows; the blocks
// that share a weight tile run back to back on one XCD and all but the first find it in that L2.  64-wide K stripes of
// the weights and of the hi / lo rows go through LDS; the waves form a grid of (TN / 4) x 64 sub-tiles (TN = 256, 192:
// eight waves, one block per CU, two staging buffers) or 64 x 64 ones (TN = 128: four waves, two blocks per CU, one
// buffer), 32 (24) MFMAs, hi and lo, per 12 (11) LDS fragment reads.  The finished tile goes back through LDS in two
// halves so that the epilogue sees 64 consecutive columns of a row per wave: the modes, the RMSNorm folding and the order of
// the weight rows (rotary pairs inside every group of 64) are those of the 64-row kernel, whose epilogue it shares.
constexpr int MB_TM = 128, MB_CK = 64;
constexpr int MB_PITCH = MB_CK * 2 + 16;   // bytes per staged row

// weight row of logical row r of tile `tile` (TN logical rows per tile; SwiGLU: TN/2 gate rows, then TN/2 up rows)
template <int MODE, int TN>
__device__ __forceinline__ const uint16_t* mb_row(const RowsP2& p, int tile, int r)
{
    if (MODE == RM_SWIGLU) return (const uint16_t*)p.w[r / (TN / 2)] + (size_t)(tile * (TN / 2) + r % (TN / 2)) * p.K;
    const int row = tile * TN + r;
    return m6_row<MODE>(p, row >> 6, row & 63, 0);
}

// TN = weight rows per tile (see above).  What bounds the 512-thread form is LDS traffic: per stripe the fragment reads
// and staging writes take as many LDS cycles as the MFMAs take matrix cycles, so both have to run all the time.  Hence
// the fragments of a k-step are read while the k-step before it is multiplied (two register sets), the next stripe is
// written to LDS and the one after it requested from memory during the first of a stripe's two k-steps, and the only
// barrier sits between them: behind it the next stripe is staged and nobody reads this one any more.  Scheduling groups
// spread the LDS and memory instructions between the MFMAs.  Measured on random data, 512 rows, K = 4096 (both products
// counted): 256 full tiles 1059 -> 1169 TFLOP/s, 192 tiles 841 -> 941, against reading all fragments at the head of a
// stripe and writing the next one behind its MFMAs; the matrix cores alone reach 1850 here.
template <int MODE, bool F16, int TN>
__global__ __launch_bounds__(TN == 128 ? 256 : 512, 2) void rows_big_kernel(RowsP2 p)
{
    constexpr bool BIG = TN != 128;
    constexpr int NTH = BIG ? 512 : 256, WN = BIG ? 4 : 2;   // threads; waves along the weight rows (x 2 along the activation rows)
    constexpr int WR = TN / WN, WNR = WR / 16;               // weight rows of a wave, in 16-row fragments
    constexpr int RPS = NTH / 8;                // rows covered by one load step of the block
    constexpr int WU = TN / RPS, BU = MB_TM / RPS;   // load steps of the weights / of one activation plane
    constexpr int EP = TN + 4;                  // floats per row of the epilogue tile
    constexpr int BUFB = (TN + 2 * MB_TM) * MB_PITCH;
    static_assert(MODE != RM_SWIGLU || TN % 128 == 0, "a SwiGLU tile holds whole 64-row groups of both matrices");
    extern __shared__ __align__(16) unsigned char smb[];
    __shared__ float rs[MB_TM];
    unsigned char* Ws = smb;                          // [TN][PITCH]
    unsigned char* Bh = smb + TN * MB_PITCH;          // [128][PITCH]
    unsigned char* Bl = Bh + MB_TM * MB_PITCH;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int K = p.K, M = p.M;
    const int NCall = K / MB_CK;
    const int S = p.ksplit > 1 ? p.ksplit : 1;
    // Block id -> (weight tile and K slice, row block).  Workgroups go to the eight XCDs round-robin by id and each
    // XCD has its own L2: ids c, c + 8, c + 16, .. (one XCD, dispatched back to back) take the row blocks of ONE
    // weight tile, so the tile comes out of HBM once per XCD and the other row blocks find it in that L2.
    int tile, slice, m0;
    {
        const int mb = (M + MB_TM - 1) / MB_TM, units = p.n_tiles * S;
        const int L = blockIdx.x, full = units & ~7;
        int unit, y;
        if (L < full * mb) { const int ch = L / (8 * mb), r = L % (8 * mb); unit = ch * 8 + (r & 7); y = r >> 3; }
        else { const int r = L - full * mb, rem = units - full; unit = full + r % rem; y = r / rem; }
        tile = p.tile0 + unit % p.n_tiles; slice = unit / p.n_tiles; m0 = y * MB_TM;
    }
    const int c_begin = (int)((long)NCall * slice / S), NC = (int)((long)NCall * (slice + 1) / S) - c_begin;
    // a stripe is TN + 2 x 128 rows of 8 vectors of 16 bytes; thread takes row tid / 8 + RPS u, vector tid % 8.
    // Addresses are a block-uniform base plus a 32-bit element offset per thread.  A 64-row group of q or k rows is two
    // runs of 32 rows, hd / 2 rows apart (woff_rot); every other load step covers consecutive rows.
    const int kk = (tid & 7) * 8, trow = tid >> 3;
    const uint16_t* wb[WU];   // uniform over the block
    bool rot[WU];             // uniform
    int boff[BU];
    const int woff = trow * K + kk, dst = trow * MB_PITCH + kk * 2;
    const int woff_rot = MODE == RM_QKV && BIG ? ((trow & 31) + (trow >> 5) * (p.hd >> 1)) * K + kk : woff;
#pragma unroll
    for (int u = 0; u < WU; u++) {
        wb[u] = mb_row<MODE, TN>(p, tile, RPS * u);
        rot[u] = MODE == RM_QKV && tile * TN + RPS * u < p.dq + p.dkv;
    }
#pragma unroll
    for (int u = 0; u < BU; u++) boff[u] = min(m0 + trow + RPS * u, M - 1) * p.ldb + kk;   // rows past M read a valid row, never stored
    constexpr int MB_D = BIG ? 1 : 2;   // stripes in flight in registers
    u32x4_t rw[MB_D][WU], rh[MB_D][BU], rl[MB_D][BU];
    auto gload = [&](int slot, int ck) {   // (a stripe past the end re-reads the last one)
        const int k0 = (c_begin + min(ck, NC - 1)) * MB_CK;
#pragma unroll
        for (int u = 0; u < WU; u++)   // cached loads: the other row blocks read the same tile
            rw[slot][u] = *reinterpret_cast<const u32x4_t*>(wb[u] + (rot[u] ? woff_rot : woff) + k0);
#pragma unroll
        for (int u = 0; u < BU; u++) {
            rh[slot][u] = *reinterpret_cast<const u32x4_t*>(p.bh + boff[u] + k0);
            rl[slot][u] = *reinterpret_cast<const u32x4_t*>(p.bl + boff[u] + k0);
        }
    };
    auto put = [&](int slot, int buf) {   // registers of `slot` -> staging buffer `buf`
#pragma unroll
        for (int u = 0; u < WU; u++) *reinterpret_cast<u32x4_t*>(Ws + buf * BUFB + dst + u * RPS * MB_PITCH) = rw[slot][u];
#pragma unroll
        for (int u = 0; u < BU; u++) {
            *reinterpret_cast<u32x4_t*>(Bh + buf * BUFB + dst + u * RPS * MB_PITCH) = rh[slot][u];
            *reinterpret_cast<u32x4_t*>(Bl + buf * BUFB + dst + u * RPS * MB_PITCH) = rl[slot][u];
        }
    };
    const int pos0 = m6_pos0<MODE>(p);   // (requested with the first stripes)
    const int wn = wave % WN, wm = wave / WN;
    f32x4_t acc[WNR][4];
#pragma unroll
    for (int i = 0; i < WNR; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const unsigned char* wfrag = Ws + (wn * WR + r16) * MB_PITCH + g * 16;
    const unsigned char* hfrag = Bh + (wm * 64 + r16) * MB_PITCH + g * 16;
    const unsigned char* lfrag = Bl + (wm * 64 + r16) * MB_PITCH + g * 16;
    // RMS scale of the block's activation rows (a K-split launch leaves the scaling to its finishing kernel)
    constexpr int SR = MB_TM / (NTH / 64);   // rows of a wave
    const bool scaled = MODE != RM_RESID && p.ssq && S == 1;
    RowScales<SR> scales;
    if (scaled) scales.load(p.ssq, p.n_ssq, m0 + wave, NTH / 64, M, 0, lane);
    asm volatile("" ::: "memory");
    auto row_scales = [&]() {
        if (scaled) scales.finish(p.ssq, p.n_ssq, m0 + wave, NTH / 64, M, lane, K, p.eps, [&](int u, float v) { if (lane == 0) rs[wave + NTH / 64 * u] = v; });
        else if (tid < MB_TM) rs[tid] = 1.0f;
    };
    if constexpr (!BIG) {
        // One stripe = 2 k-steps x 4 groups of 16 activation rows.  The weight fragments of both k-steps are read up
        // front; the hi / lo fragments of step t + 1 are requested before the eight MFMAs of step t are issued.  No
        // conditions inside (row groups past M multiply clamped copies of the last row; their results are never stored).
        auto multiply = [&]() {
            constexpr int KS = MB_CK / 32, NSTEP = KS * 4;
            u32x4_t a[KS][WNR], h[2], l[2];
#pragma unroll
            for (int ks = 0; ks < KS; ks++)
#pragma unroll
                for (int i = 0; i < WNR; i++) a[ks][i] = *reinterpret_cast<const u32x4_t*>(wfrag + i * 16 * MB_PITCH + ks * 64);
            h[0] = *reinterpret_cast<const u32x4_t*>(hfrag);
            l[0] = *reinterpret_cast<const u32x4_t*>(lfrag);
#pragma unroll
            for (int t = 0; t < NSTEP; t++) {
                const int ks = t >> 2, j = t & 3;
                if (t + 1 < NSTEP) {
                    const int o = ((t + 1) & 3) * 16 * MB_PITCH + ((t + 1) >> 2) * 64;
                    h[(t + 1) & 1] = *reinterpret_cast<const u32x4_t*>(hfrag + o);
                    l[(t + 1) & 1] = *reinterpret_cast<const u32x4_t*>(lfrag + o);
                }
#pragma unroll
                for (int i = 0; i < WNR; i++) acc[i][j] = mfma_h16<F16>(a[ks][i], h[t & 1], acc[i][j]);
#pragma unroll
                for (int i = 0; i < WNR; i++) acc[i][j] = mfma_h16<F16>(a[ks][i], l[t & 1], acc[i][j]);
            }
        };
        auto stage = [&](int slot) {
            lds_barrier();   // the previous stripe is fully consumed
            put(slot, 0);
            lds_barrier();
        };
        // In front of the weights: a wave has 32 rows here, and their sums beside two stripes in flight are more than its registers
        // hold (36 bytes of scratch per lane in SwiGLU launches, also those cut along K, which scale nothing).  us, behind the first
        // requests / so: 2048 x 5440, 512 rows, uncut 90.0 / 85.3; 1000 rows, the last tiles cut 79.5 / 75.2; 1024 x 2752 26.5 / 25.0.
        row_scales();
#pragma unroll
        for (int sl = 0; sl < MB_D; sl++) gload(sl, sl);
        int ck0 = 0;
        for (; ck0 + 2 * MB_D <= NC; ck0 += MB_D) {   // steady state: every step refills its slot, no conditions
#pragma unroll
            for (int sl = 0; sl < MB_D; sl++) {
                stage(sl);
                gload(sl, ck0 + sl + MB_D);
                multiply();
            }
        }
        for (; ck0 < NC; ck0 += MB_D) {               // drain
#pragma unroll
            for (int sl = 0; sl < MB_D; sl++) {
                if (ck0 + sl < NC) {   // uniform
                    stage(sl);
                    if (ck0 + sl + MB_D < NC) gload(sl, ck0 + sl + MB_D);
                    multiply();
                }
            }
        }
    } else {
        u32x4_t a[2][WNR], h[2][4], l[2][4];   // fragments of two k-steps
        auto frags = [&](int q, int buf, int ks) {
            const int bo = buf * BUFB + ks * 64;
#pragma unroll
            for (int i = 0; i < WNR; i++) a[q][i] = *reinterpret_cast<const u32x4_t*>(wfrag + bo + i * 16 * MB_PITCH);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                h[q][j] = *reinterpret_cast<const u32x4_t*>(hfrag + bo + j * 16 * MB_PITCH);
                l[q][j] = *reinterpret_cast<const u32x4_t*>(lfrag + bo + j * 16 * MB_PITCH);
            }
        };
        auto multiply = [&](int q) {   // row groups past M multiply clamped copies of the last row; never stored
#pragma unroll
            for (int j = 0; j < 4; j++) {
#pragma unroll
                for (int i = 0; i < WNR; i++) acc[i][j] = mfma_h16<F16>(a[q][i], h[q][j], acc[i][j]);
#pragma unroll
                for (int i = 0; i < WNR; i++) acc[i][j] = mfma_h16<F16>(a[q][i], l[q][j], acc[i][j]);
            }
        };
        constexpr int NR = WNR + 8, NM = WNR * 8, NW = WU + 2 * BU;   // fragment reads, MFMAs, staged vectors of a k-step / stripe
        gload(0, 0);
        row_scales();
        put(0, 0);
        gload(0, 1);
        lds_barrier();
        frags(0, 0, 0);
        for (int ck0 = 0; ck0 < NC; ck0 += 2) {
#pragma unroll
            for (int sl = 0; sl < 2; sl++) {
                if (ck0 + sl < NC) {   // uniform
                    // first k-step: its fragments are in registers (set 0).  Meanwhile read those of the second one, write stripe
                    // ck0 + sl + 1 into the other buffer (last read before the barrier one stripe ago) and request the one after it
                    frags(1, sl, 1);
                    put(0, sl ^ 1);
                    gload(0, ck0 + sl + 2);
                    multiply(0);
#pragma unroll
                    for (int z = 0; z < NR; z++) {   // DS read, MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    }
#pragma unroll
                    for (int z = 0; z < NW; z++) {   // DS write, MFMA, memory read
                        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x8, NM - NR - NW, 0);
                    lds_barrier();
                    // second k-step; meanwhile the first fragments of the next stripe (behind the last one: read, never used)
                    frags(0, sl ^ 1, 0);
                    multiply(1);
#pragma unroll
                    for (int z = 0; z < NR; z++) {
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x8, NM - NR, 0);
                }
            }
        }
    }
    // epilogue, 64 activation rows at a time: ep[row][column] through LDS, then a wave takes 64 consecutive columns of a row
    float* ep = reinterpret_cast<float*>(smb);
    constexpr int NG = (MODE == RM_SWIGLU ? TN / 2 : TN) / 64, NWAVE = NTH / 64;   // 64-column groups of the tile's output
    constexpr int EB = 8;   // rows of a wave whose operands are loaded together
    static_assert(64 / NWAVE % EB == 0, "whole batches");
    for (int hf = 0; hf < 2; hf++) {
        if (m0 + hf * 64 >= M) break;   // uniform over the block
        __syncthreads();
        if (wm == hf) {
#pragma unroll
            for (int i = 0; i < WNR; i++)
#pragma unroll
                for (int j = 0; j < 4; j++)
                    *reinterpret_cast<f32x4_t*>(ep + (j * 16 + r16) * EP + wn * WR + i * 16 + 4 * g) = acc[i][j];
        }
        __syncthreads();
        if (S > 1) {   // raw sums of this K slice: [slice][matrix][M][columns of this launch's tiles]
            constexpr int NMAT = MODE == RM_SWIGLU ? 2 : 1;
            const int nt = p.n_tiles * NG * 64, rows = min(64, M - m0 - hf * 64);
            float* kp = p.kpart + ((size_t)slice * NMAT * M + m0 + hf * 64) * nt + (tile - p.tile0) * NG * 64;
            const size_t mat = (size_t)M * nt;
            for (int ml = wave; ml < rows; ml += NWAVE) {
                float* kr = kp + (size_t)ml * nt;
                // a wave takes whole rows of the tile, 16 bytes per lane: 4 bytes with the address worked out per row and 64 columns
                // cost 5 us of a 7B projection, 512 rows (O and down on average 66.4 -> 61.1; 13B 94 -> 86)
                if (lane < NG * 16) {
                    *reinterpret_cast<float4*>(kr + lane * 4) = *reinterpret_cast<const float4*>(ep + ml * EP + lane * 4);
                    if (MODE == RM_SWIGLU) *reinterpret_cast<float4*>(kr + mat + lane * 4) = *reinterpret_cast<const float4*>(ep + ml * EP + TN / 2 + lane * 4);
                }
            }
            continue;
        }
        for (int gr = 0; gr < NG; gr++) {
            const int otile = tile * NG + gr;
            const M6Col col = m6_col<MODE>(p, otile, lane, pos0);
#pragma unroll
            for (int r0 = 0; r0 < 64 / NWAVE; r0 += EB) {
                M6Pre pre[EB];
#pragma unroll
                for (int u = 0; u < EB; u++) pre[u] = m6_pre<MODE>(p, col, min(m0 + hf * 64 + wave + (r0 + u) * NWAVE, M - 1));
#pragma unroll
                for (int u = 0; u < EB; u++) {
                    const int ml = wave + (r0 + u) * NWAVE, m = m0 + hf * 64 + ml;   // uniform over a wave
                    if (m >= M) break;
                    float v = ep[ml * EP + gr * 64 + lane], v2 = MODE == RM_SWIGLU ? ep[ml * EP + TN / 2 + gr * 64 + lane] : 0.f;
                    if (MODE != RM_RESID) { const float sc = rs[hf * 64 + ml]; v *= sc; v2 *= sc; }
                    m6_row<MODE, F16>(p, col, otile, m, lane, v, v2, pre[u]);
                }
            }
        }
    }
}

bool rows_big_supported(const Dims& D)
{
    return D.wt != WT_F32 && D.d % 128 == 0 && D.dq % 128 == 0 && D.dkv % 128 == 0 && D.f % 64 == 0 && D.V % 128 == 0 &&
           (D.hd == 64 || D.hd == 128);
}

bool rows_many_supported(const Dims& D, int N, int K)
{
    return D.wt != WT_F32 && N % 64 == 0 && K % M6_CK == 0 && K >= M6_CK;
}

// every GEMM of a layer and the LM head fit the 64 x 64 x 128 tiling
bool rows_wide_supported(const Dims& D)
{
    return D.wt != WT_F32 && D.d % 128 == 0 && D.dq % 128 == 0 && D.f % 128 == 0 && D.dkv % 64 == 0 && D.V % 64 == 0 &&
           (D.hd == 64 || D.hd == 128);
}

template <int MODE, bool F16, int DEPTH>
static hipError_t launch_wide_d(const RowsP2& p, int n_tiles, hipStream_t s)
{
    constexpr int NT = MODE == RM_SWIGLU ? 2 : 1;
    const size_t lds = (size_t)(NT * 64 + 128) * M6_PITCH;
    static std::atomic<size_t> lds_limit{0};  // per instantiation
    {
        hipError_t e = ensure_lds((const void*)rows_wide_kernel<MODE, F16, DEPTH>, lds, lds_limit);
        if (e != hipSuccess) return e;
    }
    const int S = p.ksplit > 1 ? p.ksplit : 1;
    hipLaunchKernelGGL((rows_wide_kernel<MODE, F16, DEPTH>), dim3(n_tiles, S), dim3(512), lds, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    hipLaunchKernelGGL((rows_finish_kernel<MODE, F16>), dim3(n_tiles, (p.M + FIN_ROWS - 1) / FIN_ROWS), dim3(64), 0, s, p);
    return hipGetLastError();
}

// One stripe in flight per block measured best or equal everywhere: what bounds a block is the 40 GB/s or so
// that a single CU pulls from the cache (a stripe is 48-64 KB of weights and rows), not latency.
template <int MODE, bool F16>
static hipError_t launch_wide(const RowsP2& p, int n_tiles, hipStream_t s, const LaunchOpts* opt)
{
    const int depth = opt && opt->wide_depth > 0 ? opt->wide_depth : 1;
    if (depth >= 4) return launch_wide_d<MODE, F16, 4>(p, n_tiles, s);
    if (depth >= 2) return launch_wide_d<MODE, F16, 2>(p, n_tiles, s);
    return launch_wide_d<MODE, F16, 1>(p, n_tiles, s);
}

static void fill_rows_params(const Dims& D, const RowsFused& f, RowsP2& p)
{
    for (int i = 0; i < 3; i++) { p.w[i] = f.w[i]; p.n[i] = f.n[i]; }
    p.K = f.K; p.bh = f.bh; p.bl = f.bl; p.ldb = f.ldb; p.y = f.y; p.ldy = f.ldy; p.oh = f.oh; p.ol = f.ol; p.ldo = f.ldo;
    p.tap = f.tap; p.tap_ld = f.tap_ld; p.M = f.M; p.rope = f.rope; p.pos_dev = f.pos_dev; p.pos_off = f.pos_off;
    p.hd = D.hd; p.dq = f.mode == RM_QKV ? f.n[0] : D.dq; p.dkv = D.dkv; p.max_seq = D.max_seq; p.kc = f.kc; p.vc = f.vc; p.kt = D.kt;
    p.ssq = f.ssq; p.n_ssq = f.n_ssq; p.eps = D.eps; p.gain_out = f.gain_out; p.ssq_out = f.ssq_out;
    p.tap_only = f.tap_only; p.vmax = f.vmax; p.clamp = f.clamp;
}

hipError_t rows_wide(const Dims& D, const RowsFused& f, hipStream_t s)
{
    if (D.wt == WT_F32 || f.M < 1 || f.M > 64 || f.K % M6_CK || f.K < M6_CK) return hipErrorInvalidValue;
    if (f.n[0] % 64 || f.n[1] % 64 || f.n[2] % 64) return hipErrorInvalidValue;
    if (f.ssq && (f.mode == RM_RESID || f.n_ssq < 1)) return hipErrorInvalidValue;
    if (f.gain_out && (f.mode != RM_RESID || !f.oh || !f.ol || !f.ssq_out)) return hipErrorInvalidValue;
    if (f.mode == RM_QKV && ((f.n[0] && f.n[0] != D.dq) || f.n[1] != D.dkv || f.n[2] != D.dkv || (D.hd != 64 && D.hd != 128)))
        return hipErrorInvalidValue;
    RowsP2 p = {};
    fill_rows_params(D, f, p);
    const int n_tiles = f.mode == RM_SWIGLU ? f.n[0] / 64 : (f.n[0] + f.n[1] + f.n[2]) / 64;
    const bool f16 = D.wt == WT_F16;
    // A block is bound by what one CU pulls from the cache (about 40 GB/s), so a launch with far fewer tiles than
    // CUs (the projections back to d_model) is cut along K until there are about 256 blocks; needs scratch for
    // ksplit x matrices x M x n sums.  With 170 tiles or more (QKV, gate/up at 7B) the cut measured equal or worse.
    p.ksplit = 1; p.kpart = nullptr;
    const int force_ks = D.opt ? D.opt->wide_ksplit : 0;
    if (f.kpart && force_ks != 1 && f.M > 16) {
        const int nmat = f.mode == RM_SWIGLU ? 2 : 1;
        const size_t per_slice = (size_t)nmat * f.M * n_tiles * 64;
        int ks = force_ks > 1 ? force_ks : (n_tiles <= 128 ? 256 / n_tiles : 1);
        const int nc = f.K / M6_CK;
        if (ks > 8) ks = 8;
        if (ks > nc) ks = nc;
        if ((size_t)ks * per_slice > f.kpart_floats) ks = (int)(f.kpart_floats / per_slice);
        if (ks > 1) { p.ksplit = ks; p.kpart = f.kpart; }
    }
    switch (f.mode) {
        case RM_STORE: return f16 ? launch_wide<RM_STORE, true>(p, n_tiles, s, D.opt) : launch_wide<RM_STORE, false>(p, n_tiles, s, D.opt);
        case RM_RESID: return f16 ? launch_wide<RM_RESID, true>(p, n_tiles, s, D.opt) : launch_wide<RM_RESID, false>(p, n_tiles, s, D.opt);
        case RM_SWIGLU: return f16 ? launch_wide<RM_SWIGLU, true>(p, n_tiles, s, D.opt) : launch_wide<RM_SWIGLU, false>(p, n_tiles, s, D.opt);
        case RM_QKV: return f16 ? launch_wide<RM_QKV, true>(p, n_tiles, s, D.opt) : launch_wide<RM_QKV, false>(p, n_tiles, s, D.opt);
        default: return hipErrorInvalidValue;
    }
}

template <int MODE, bool F16, int TN>
static hipError_t launch_big(const RowsP2& p, hipStream_t s)
{
    const size_t lds = (size_t)(TN == 128 ? 1 : 2) * (TN + 2 * MB_TM) * MB_PITCH;
    static_assert((size_t)64 * (TN + 4) * 4 <= (size_t)(TN + 2 * MB_TM) * MB_PITCH, "epilogue tile fits the staging area");
    static std::atomic<size_t> lds_limit{0};  // per instantiation
    {
        hipError_t e = ensure_lds((const void*)rows_big_kernel<MODE, F16, TN>, lds, lds_limit);
        if (e != hipSuccess) return e;
    }
    const int S = p.ksplit > 1 ? p.ksplit : 1;
    hipLaunchKernelGGL((rows_big_kernel<MODE, F16, TN>), dim3(p.n_tiles * ((p.M + MB_TM - 1) / MB_TM) * S), dim3(TN == 128 ? 256 : 512), lds, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    hipLaunchKernelGGL((rows_finish_kernel<MODE, F16>), dim3(p.n_tiles * (MODE == RM_SWIGLU ? TN / 128 : TN / 64), (p.M + FIN_ROWS - 1) / FIN_ROWS), dim3(64), 0, s, p);
    return hipGetLastError();
}

template <int MODE, bool F16>
static hipError_t launch_big_tn(const RowsP2& p, int tn, hipStream_t s)
{
    if constexpr (MODE == RM_QKV)
        if (tn == 192) return launch_big<MODE, F16, 192>(p, s);
    return tn == 256 ? launch_big<MODE, F16, 256>(p, s) : launch_big<MODE, F16, 128>(p, s);
}

hipError_t rows_big(const Dims& D, const RowsFused& f, hipStream_t s)
{
    if (D.wt == WT_F32 || f.M < 1 || f.K % MB_CK || f.K < MB_CK) return hipErrorInvalidValue;
    if (f.mode == RM_SWIGLU ? (f.n[0] % 64 || f.n[1] != f.n[0]) : (f.n[0] % 128 || f.n[1] % 128 || f.n[2] % 128))
        return hipErrorInvalidValue;
    if (f.ssq && (f.mode == RM_RESID || f.n_ssq < 1)) return hipErrorInvalidValue;
    if (f.gain_out && (f.mode != RM_RESID || !f.oh || !f.ol || !f.ssq_out)) return hipErrorInvalidValue;
    if (f.mode == RM_QKV && ((f.n[0] && f.n[0] != D.dq) || f.n[1] != D.dkv || f.n[2] != D.dkv || (D.hd != 64 && D.hd != 128)))
        return hipErrorInvalidValue;
    RowsP2 p = {};
    fill_rows_params(D, f, p);
    const int m_blocks = (f.M + MB_TM - 1) / MB_TM;
    const int n_total = f.mode == RM_SWIGLU ? 2 * f.n[0] : f.n[0] + f.n[1] + f.n[2];   // logical weight rows
    // 256-row tiles (one 512-thread block per CU, staging double-buffered in LDS: measured 20-30 % faster per MFMA, and
    // a launch fills the CUs with the same granularity as two 128-row blocks per CU would) wherever every stacked
    // matrix is a whole number of them; else 128-row tiles
    const int force_tn = D.opt ? D.opt->wide_depth : 0;   // tuning hook: 128, 192 (QKV) or 256
    const bool fits256 = n_total % 256 == 0;   // (tiles are made of 64-row groups, which never straddle two matrices)
    int tn = f.mode == RM_QKV ? qkv_tile_rows(n_total, m_blocks) : fits256 ? 256 : 128;
    if (force_tn == 128 || (force_tn == 192 && f.mode == RM_QKV && n_total % 192 == 0) || (force_tn == 256 && fits256)) tn = force_tn;
    const int n_tiles = n_total / tn;
    p.n_tiles = n_tiles;
    const bool f16 = D.wt == WT_F16;
    // A residual projection or a QKV launch that leaves resident slots empty (two per CU for the small tile, one for the
    // large) is cut along K: its raw sums go to kpart, rows_finish_kernel adds the slices in a fixed order and runs the epilogue.
    p.ksplit = 1; p.kpart = nullptr;
    const int force_ks = D.opt ? D.opt->wide_ksplit : 0;
    const int slots = tn != 128 ? 256 : 512, nc = f.K / MB_CK;
    if (f.kpart && (f.mode == RM_RESID || f.mode == RM_QKV) && force_ks != 1) {
        const size_t per_slice = (size_t)f.M * n_tiles * tn;
        int ks = force_ks > 1 ? force_ks : k_slices(n_tiles * m_blocks, slots, nc, 4.0 * (double)per_slice, f.mode == RM_QKV ? 4 : 8);
        if (ks > nc) ks = nc;
        if ((size_t)ks * per_slice > f.kpart_floats) ks = (int)(f.kpart_floats / per_slice);
        if (ks > 1) { p.ksplit = ks; p.kpart = f.kpart; }
    }
    // Gate / up with a last round that would leave most CUs idle (7B, 512 rows: 344 blocks for 256 slots): the tiles
    // of the whole rounds run as they are, the rest (all of them when there is no whole round) are cut along K, and the
    // finishing kernel adds the slices and applies SwiGLU (there 1 + 1/2 block times instead of 2).
    if (f.kpart && f.mode == RM_SWIGLU && force_ks != 1) {
        const int units = n_tiles * m_blocks;
        const int whole_tiles = units / slots * slots / m_blocks, tail_tiles = n_tiles - whole_tiles;
        const int tail_units = tail_tiles * m_blocks;
        if (tail_tiles > 0) {
            const size_t per_slice = (size_t)2 * f.M * tail_tiles * (tn / 2);
            int ks = force_ks > 1 ? force_ks : k_slices(tail_units, slots, nc, 4.0 * (double)per_slice, 4);
            if (ks > nc) ks = nc;
            if ((size_t)ks * per_slice > f.kpart_floats) ks = (int)(f.kpart_floats / per_slice);
            if (ks > 1) {
                if (whole_tiles > 0) {
                    RowsP2 a = p;
                    a.n_tiles = whole_tiles;
                    const hipError_t e = f16 ? launch_big_tn<RM_SWIGLU, true>(a, tn, s) : launch_big_tn<RM_SWIGLU, false>(a, tn, s);
                    if (e != hipSuccess) return e;
                }
                p.tile0 = whole_tiles; p.n_tiles = tail_tiles; p.fin_tile0 = whole_tiles * (tn / 128);
                p.ksplit = ks; p.kpart = f.kpart;
            }
        }
    }
    switch (f.mode) {
        case RM_STORE: return f16 ? launch_big_tn<RM_STORE, true>(p, tn, s) : launch_big_tn<RM_STORE, false>(p, tn, s);
        case RM_RESID: return f16 ? launch_big_tn<RM_RESID, true>(p, tn, s) : launch_big_tn<RM_RESID, false>(p, tn, s);
        case RM_SWIGLU: return f16 ? launch_big_tn<RM_SWIGLU, true>(p, tn, s) : launch_big_tn<RM_SWIGLU, false>(p, tn, s);
        case RM_QKV: return f16 ? launch_big_tn<RM_QKV, true>(p, tn, s) : launch_big_tn<RM_QKV, false>(p, tn, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t rows_many(const Dims& D, const void* w, int N, int K, const uint16_t* bh, const uint16_t* bl, int ldb, int M,
                     float* y, int ldy, hipStream_t s)
{
    if (!rows_many_supported(D, N, K)) return hipErrorInvalidValue;
    RowsFused f = {};
    f.w[0] = w; f.n[0] = N; f.K = K; f.bh = bh; f.bl = bl; f.ldb = ldb; f.y = y; f.ldy = ldy; f.M = M; f.mode = RM_STORE;
    return rows_wide(D, f, s);
}

bool rows_fused_supported(const Dims& D)
{
    return D.wt != WT_F32 && D.d % 64 == 0 && D.dq % 64 == 0 && D.f % 64 == 0;
}

hipError_t rows_fused(const Dims& D, const RowsFused& f, hipStream_t s)
{
    if (!rows_fused_supported(D) || f.M < 1 || f.M > 16 || f.K % 64) return hipErrorInvalidValue;
    RowsP2 p = {};
    fill_rows_params(D, f, p);
    if (f.ssq && (f.mode == RM_RESID || f.n_ssq < 1)) return hipErrorInvalidValue;
    if (f.gain_out && (f.mode != RM_RESID || !f.oh || !f.ol || !f.ssq_out)) return hipErrorInvalidValue;
    switch (f.mode) {
        case RM_STORE: return D.wt == WT_F16 ? rows_fused_mode<RM_STORE, true>(p, s, D.opt) : rows_fused_mode<RM_STORE, false>(p, s, D.opt);
        case RM_RESID: return D.wt == WT_F16 ? rows_fused_mode<RM_RESID, true>(p, s, D.opt) : rows_fused_mode<RM_RESID, false>(p, s, D.opt);
        case RM_SWIGLU: return D.wt == WT_F16 ? rows_fused_mode<RM_SWIGLU, true>(p, s, D.opt) : rows_fused_mode<RM_SWIGLU, false>(p, s, D.opt);
        case RM_QKV: return D.wt == WT_F16 ? rows_fused_mode<RM_QKV, true>(p, s, D.opt) : rows_fused_mode<RM_QKV, false>(p, s, D.opt);
    }
    return hipErrorInvalidValue;
}

// hi/lo bf16 split of M rows of length K, optionally RMS-normalised first (gain != nullptr)
__global__ __launch_bounds__(256) void rows_prep_kernel(const float* __restrict__ in, int ldx, const float* __restrict__ gain,
                                                        int K, float eps, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                                        bool f16)
{
    __shared__ float red[4];
    const float* x = in + (size_t)blockIdx.x * ldx;
    float sc = 1.0f;
    if (gain) {
        float ss = 0.f;
        for (int i = threadIdx.x * 4; i < K; i += 1024) {
            const float4 v = *reinterpret_cast<const float4*>(x + i);
            ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        }
        sc = 1.0f / sqrtf(block_sum<4>(ss, red) / (float)K + eps);
    }
    for (int i = threadIdx.x * 4; i < K; i += 1024) {
        float4 v = *reinterpret_cast<const float4*>(x + i);
        if (gain) {
            const float4 g = *reinterpret_cast<const float4*>(gain + i);
            v.x = v.x * sc * g.x; v.y = v.y * sc * g.y; v.z = v.z * sc * g.z; v.w = v.w * sc * g.w;
        }
        const size_t o = (size_t)blockIdx.x * K + i;
        split_store(v.x, hi, lo, o, f16); split_store(v.y, hi, lo, o + 1, f16);
        split_store(v.z, hi, lo, o + 2, f16); split_store(v.w, hi, lo, o + 3, f16);
    }
}

hipError_t rows_prep(const Dims& D, const float* in, int ldx, const float* gain, int M, int K, float eps, uint16_t* hi,
                     uint16_t* lo, hipStream_t s)
{
    hipLaunchKernelGGL(rows_prep_kernel, dim3(M), dim3(256), 0, s, in, ldx, gain, K, eps, hi, lo, D.wt == WT_F16);
    return hipGetLastError();
}

// Entry of the fused path: the embedding rows of M tokens as fp32 rows x and as what a RESID projection leaves behind for
// its consumer, hi/lo = split(x * gain) without the norm scale and the sums of squares of every GROUP (16 or 64)
// consecutive elements.  A thread owns four elements, a block 1024 of one row.  (As two launches, a gather and a split in
// which one thread walked a whole group: 9.7 + 12 us for 512 rows of 4096, 4.5 + 3.6 us for five.)
template <typename WT, int GROUP>
__global__ __launch_bounds__(256) void embed_split_kernel(const WT* __restrict__ E, Tokens tok, int d, int V,
                                                          const float* __restrict__ gain, float* __restrict__ x,
                                                          uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                                                          float* __restrict__ ssq)
{
    constexpr bool F16 = IsF16<WT>::value;
    const int r = blockIdx.y, i = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= d) return;   // whole DPP rows: d is a multiple of 64
    const uint2 w = *reinterpret_cast<const uint2*>(E + embed_row(token_of(tok, r), V) * d + i);
    const float4 g = *reinterpret_cast<const float4*>(gain + i);
    const float4 v = make_float4(h16_bits_to_f32(w.x & 0xffff, F16), h16_bits_to_f32(w.x >> 16, F16),
                                 h16_bits_to_f32(w.y & 0xffff, F16), h16_bits_to_f32(w.y >> 16, F16));
    const size_t o = (size_t)r * d + i;
    *reinterpret_cast<float4*>(x + o) = v;
    const float y[4] = {v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w};
    unsigned h[4], l[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        h[j] = f32_to_h16_bits(y[j], F16);
        l[j] = f32_to_h16_bits(y[j] - h16_bits_to_f32(h[j], F16), F16);
    }
    *reinterpret_cast<uint2*>(hi + o) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    *reinterpret_cast<uint2*>(lo + o) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
    float sq = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    if (GROUP == 64) sq = row16_sum(sq);                       // 16 lanes of four elements
    else sq = dpp_add<0x4E>(dpp_add<0xB1>(sq));                // the four lanes of a quad
    if ((i & (GROUP - 1)) == 0) ssq[(size_t)r * (d / GROUP) + i / GROUP] = sq;
}

hipError_t embed_split(const Dims& D, const void* embed, Tokens tok, int M, const float* gain, float* x, uint16_t* hi,
                       uint16_t* lo, float* ssq, int group, hipStream_t s)
{
    if ((group != 16 && group != 64) || D.d % 64 || D.wt == WT_F32 || !gain || M < 1) return hipErrorInvalidValue;
    const dim3 grid(ceil_div(D.d, 1024), M);
    auto go = [&](auto kernel, auto e) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, e, tok, D.d, D.V, gain, x, hi, lo, ssq);
        return hipGetLastError();
    };
    if (D.wt == WT_F16) return group == 16 ? go(embed_split_kernel<f16_t, 16>, (const f16_t*)embed) : go(embed_split_kernel<f16_t, 64>, (const f16_t*)embed);
    return group == 16 ? go(embed_split_kernel<uint16_t, 16>, (const uint16_t*)embed) : go(embed_split_kernel<uint16_t, 64>, (const uint16_t*)embed);
}

// rotary + cache write for the multi-row path: one thread per (row, head slot, pair index)
template <typename KT>
__global__ void rope_kv_rows_kernel(float* __restrict__ qkv, const float* __restrict__ rope, const int* pos_dev,
                                    int pos_off, int M, int H, int Hkv, int hd, int max_seq, KT* __restrict__ kc,
                                    KT* __restrict__ vc)
{
    const int half = hd >> 1;
    const int dq = H * hd, dkv = Hkv * hd, ld = dq + 2 * dkv;
    const int per_row = (H + Hkv) * half + dkv;  // q pairs, k pairs, v elements
    int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= M * per_row) return;
    int r = idx / per_row, e = idx % per_row;
    int pos = pos_dev[0] + pos_off + r;
    float* row = qkv + (size_t)r * ld;
    if (e < (H + Hkv) * half) {
        int hs = e / half, i = e % half;  // head slot over q heads then k heads
        const float* cs = rope + ((size_t)pos * half + i) * 2;
        float c = cs[0], s = cs[1];
        if (hs < H) {
            float* v = row + (size_t)hs * hd;
            float a = v[i], b = v[i + half];
            v[i] = a * c - b * s;
            v[i + half] = b * c + a * s;
        } else {
            int kvh = hs - H;
            const float* v = row + dq + (size_t)kvh * hd;
            float a = v[i], b = v[i + half];
            size_t o = ((size_t)kvh * max_seq + pos) * hd;
            Elem<KT>::put(kc, o + i, a * c - b * s);
            Elem<KT>::put(kc, o + i + half, b * c + a * s);
        }
    } else {
        int j = e - (H + Hkv) * half;  // element of v
        int kvh = j / hd, i = j % hd;
        Elem<KT>::put(vc, ((size_t)kvh * max_seq + pos) * hd + i, row[dq + dkv + j]);
    }
}

hipError_t rope_kv_rows(const Dims& D, float* qkv, const float* rope, const int* pos_dev, int pos_off, int M, void* kc,
                        void* vc, hipStream_t s)
{
    int per_row = (D.H + D.Hkv) * (D.hd / 2) + D.dkv;
    int blocks = ceil_div(M * per_row, 256);
    if (D.kt == WT_BF16)
        hipLaunchKernelGGL(rope_kv_rows_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s, qkv, rope, pos_dev, pos_off, M,
                           D.H, D.Hkv, D.hd, D.max_seq, (uint16_t*)kc, (uint16_t*)vc);
    else if (D.kt == WT_F16)
        hipLaunchKernelGGL(rope_kv_rows_kernel<f16_t>, dim3(blocks), dim3(256), 0, s, qkv, rope, pos_dev, pos_off, M,
                           D.H, D.Hkv, D.hd, D.max_seq, (f16_t*)kc, (f16_t*)vc);
    else
        hipLaunchKernelGGL(rope_kv_rows_kernel<float>, dim3(blocks), dim3(256), 0, s, qkv, rope, pos_dev, pos_off, M, D.H,
                           D.Hkv, D.hd, D.max_seq, (float*)kc, (float*)vc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// attention over the cache: split over the sequence, K/V tiles staged through LDS
// ---------------------------------------------------------------------------------------------
constexpr int AT_THREADS = 256;
constexpr int AT_QPASS = 16;   // query vectors handled per pass over the staged chunk

// P.V for up to NQ query vectors at once: acc[qi] += e[qi][j] * V[j][d] over this thread's positions
template <typename KT, int NQ>
__device__ __forceinline__ void attn_pv(const KT* vtile, int rowb, const float* sc, int d, int grp, int ng, int n,
                                        float (&acc)[AT_QPASS])
{
    for (int j = grp; j < n; j += ng) {
        const float v = Elem<KT>::get(reinterpret_cast<const KT*>(reinterpret_cast<const unsigned char*>(vtile) + (size_t)j * rowb), d);
#pragma unroll
        for (int qi = 0; qi < NQ; qi++) acc[qi] = fmaf(sc[qi * AT_CHUNK + j], v, acc[qi]);
    }
}

// One block = one KV head x one chunk of positions x ALL query vectors that read this head (the G
// query heads of the group times the M rows), so K and V are fetched once however many rows verify.
// All global loads of the chunk are issued up front, land in LDS (rows padded by 16 bytes to spread
// banks), and the three phases -- scores, softmax statistics, P.V -- then run out of LDS only.
// partial layout per (row, head, split): [hd] unnormalised output, then m (max score), l (sum of exp), 2 pad
// (stride hd + 4 floats keeps every partial 16-byte aligned)
template <typename KT, int HD>
__global__ __launch_bounds__(AT_THREADS) void attn_kernel(const float* __restrict__ q, int ldq,
                                                          const KT* __restrict__ kc, const KT* __restrict__ vc,
                                                          const int* pos_dev, int pos_off, int M, int H, int Hkv,
                                                          int max_seq, int n_splits, float* __restrict__ part,
                                                          float* __restrict__ outp, int dq,
                                                          uint16_t* __restrict__ out_hi, uint16_t* __restrict__ out_lo,
                                                          bool out_f16)
{
    constexpr int ROWB = HD * (int)sizeof(KT) + 16;
    constexpr int EPV = 16 / (int)sizeof(KT);  // elements per 16-byte vector
    constexpr int VPR = HD / EPV;              // vectors per cache row
    constexpr int NG = AT_THREADS / HD;        // position groups in the P.V phase
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* ktile = smem;
    unsigned char* vtile = smem + AT_CHUNK * ROWB;
    float* qs = reinterpret_cast<float*>(smem + 2 * AT_CHUNK * ROWB);  // [AT_QPASS][HD], pre-scaled
    float* sc = qs + AT_QPASS * HD;                                    // [AT_QPASS][AT_CHUNK]
    float* ml = sc + AT_QPASS * AT_CHUNK;                              // [AT_QPASS][2]
    float* fold = ml + AT_QPASS * 2;                                   // [NG][AT_QPASS][HD]

    const int split = blockIdx.x, kvh = blockIdx.y;
    const int G = H / Hkv, Q = G * M;
    const int p0 = pos_dev[0] + pos_off;
    const int total = p0 + M;                                  // positions the last row sees
    const int j0 = split * AT_CHUNK;
    const int n = min(AT_CHUNK, total - j0);                   // may be <= 0
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    if (n > 0) {  // stage K and V of the chunk: every load is issued before the first is used
        const KT* kbase = kc + ((size_t)kvh * max_seq + j0) * HD;
        const KT* vbase = vc + ((size_t)kvh * max_seq + j0) * HD;
        constexpr int NV = (AT_CHUNK * VPR + AT_THREADS - 1) / AT_THREADS;
        uint4 kr[NV], vr[NV];
        const int vmax = n * VPR - 1;
#pragma unroll
        for (int t = 0; t < NV; t++) {  // clamped, not predicated: the loads stay in registers and in flight together
            const int v = min(tid + t * AT_THREADS, vmax);
            kr[t] = *reinterpret_cast<const uint4*>(kbase + (size_t)(v / VPR) * HD + (v % VPR) * EPV);
            vr[t] = *reinterpret_cast<const uint4*>(vbase + (size_t)(v / VPR) * HD + (v % VPR) * EPV);
        }
#pragma unroll
        for (int t = 0; t < NV; t++) {
            const int v = tid + t * AT_THREADS;
            if (v <= vmax) {
                *reinterpret_cast<uint4*>(ktile + (v / VPR) * ROWB + (v % VPR) * 16) = kr[t];
                *reinterpret_cast<uint4*>(vtile + (v / VPR) * ROWB + (v % VPR) * 16) = vr[t];
            }
        }
    }
    const float scale = 1.0f / sqrtf((float)HD);
    for (int q0 = blockIdx.z * AT_QPASS; q0 < Q; q0 += gridDim.z * AT_QPASS) {   // uniform over the block
        const int nq = min(AT_QPASS, Q - q0);
        __syncthreads();                         // staged tiles visible / previous pass done with qs, sc
        for (int e = tid; e < nq * HD; e += AT_THREADS) {
            const int qi = q0 + e / HD, r = qi / G, g = qi % G;
            qs[e] = q[(size_t)r * ldq + (size_t)(kvh * G + g) * HD + (e % HD)] * scale;
        }
        __syncthreads();
        if (n > 0) {
            // phase A: scores. 2 lanes per position, each holding half a key row in registers
            constexpr int DPT = HD / 2;
            for (int jb = 0; jb < n; jb += AT_THREADS / 2) {
                const int j = jb + (tid >> 1), half = tid & 1;
                float kf[DPT];
                if (j < n) {
                    const KT* krow = reinterpret_cast<const KT*>(ktile + j * ROWB) + half * DPT;
#pragma unroll
                    for (int i = 0; i < DPT; i += EPV) {
                        float t8[EPV];
                        Elem<KT>::load(krow + i, t8);
#pragma unroll
                        for (int u = 0; u < EPV; u++) kf[i + u] = t8[u];
                    }
                }
                for (int qi = 0; qi < nq; qi++) {
                    float dot = 0.f;
                    if (j < n) {
                        const float* qv = qs + qi * HD + half * DPT;
#pragma unroll
                        for (int i = 0; i < DPT; i += 4) {
                            const float4 t4 = *reinterpret_cast<const float4*>(qv + i);
                            dot = fmaf(kf[i], t4.x, dot); dot = fmaf(kf[i + 1], t4.y, dot);
                            dot = fmaf(kf[i + 2], t4.z, dot); dot = fmaf(kf[i + 3], t4.w, dot);
                        }
                    }
                    dot += __shfl_xor(dot, 1, 64);
                    if (j < n && half == 0) sc[qi * AT_CHUNK + j] = dot;
                }
            }
        }
        __syncthreads();
        // phase B: per query vector (one wave each): causal mask, max, exp, sum
        for (int qi = wave; qi < nq; qi += AT_THREADS / 64) {
            const int r = (q0 + qi) / G;
            const int vis = min(n, p0 + r + 1 - j0);   // positions of this chunk the row may see
            float mx = -INFINITY;
            for (int j = lane; j < vis; j += 64) mx = fmaxf(mx, sc[qi * AT_CHUNK + j]);
            mx = wave_max(mx);
            float ls = 0.f;
            for (int j = lane; j < n; j += 64) {
                const float e = j < vis ? __expf(sc[qi * AT_CHUNK + j] - mx) : 0.f;
                sc[qi * AT_CHUNK + j] = e;
                ls += e;
            }
            ls = wave_sum(ls);
            if (lane == 0) { ml[qi * 2] = mx; ml[qi * 2 + 1] = ls; }
        }
        __syncthreads();
        // phase C: o[qi][d] = sum_j e[qi][j] V[j][d]; thread = (position group, d), all nq accumulators in registers
        const int d = tid % HD, grp = tid / HD;
        float acc[AT_QPASS];
#pragma unroll
        for (int qi = 0; qi < AT_QPASS; qi++) acc[qi] = 0.f;
        const KT* vcol = reinterpret_cast<const KT*>(vtile);
        if (nq == 1) attn_pv<KT, 1>(vcol, ROWB, sc, d, grp, NG, n, acc);
        else if (nq <= 4) attn_pv<KT, 4>(vcol, ROWB, sc, d, grp, NG, n, acc);
        else if (nq <= 8) attn_pv<KT, 8>(vcol, ROWB, sc, d, grp, NG, n, acc);
        else attn_pv<KT, AT_QPASS>(vcol, ROWB, sc, d, grp, NG, n, acc);
        // fold the NG position groups and write this split's result
#pragma unroll
        for (int qi = 0; qi < AT_QPASS; qi++)
            if (qi < nq) fold[(grp * AT_QPASS + qi) * HD + d] = acc[qi];
        __syncthreads();
        for (int e = tid; e < nq * HD; e += AT_THREADS) {
            const int qi = e / HD, dd = e % HD;
            float o = 0.f;
#pragma unroll
            for (int gg = 0; gg < NG; gg++) o += fold[(gg * AT_QPASS + qi) * HD + dd];
            const int qg = q0 + qi, r = qg / G, head = kvh * G + qg % G;
            const float mx = ml[qi * 2], ls = ml[qi * 2 + 1];
            if (n_splits == 1) {
                const size_t oo = (size_t)r * dq + (size_t)head * HD + dd;
                if (out_hi) split_store(o / ls, out_hi, out_lo, oo, out_f16);
                else outp[oo] = o / ls;
            } else {
                float* mine = part + (((size_t)r * H + head) * n_splits + split) * (HD + 4);
                mine[dd] = o;
                if (dd == 0) { mine[HD] = n > 0 ? mx : -INFINITY; mine[HD + 1] = ls; }
            }
        }
    }
}

// MFMA form of the kernel above for 16-bit caches: one block per KV head, chunk of positions and group of 16
// query vectors; same staging of K, same softmax statistics and the same partial layout, but the two
// contractions run on the matrix cores.  Scores: A = 16 query vectors (fp32 -> hi + lo in the cache's 16-bit
// type), B = K rows read from LDS in fragment order.  P.V: A = the 16 x 96 exponentials (hi + lo), B = V, which
// is therefore staged transposed ([dim][position]) so that a fragment is one 128-bit LDS read.
constexpr int AM_VPITCH = AT_CHUNK * 2 + 16;   // bytes per row of the transposed V tile
// One block fits a CU (120 KB of LDS for an fp32 cache), and what it does with a wave per SIMD is a chain of latencies.  Hence
// eight waves instead of four, conversions two at a time, and the position by the scalar path instead of behind all of K and V:
// 7B, 5 rows behind 550 positions of an fp32 cache 9.5 -> 8.8 us; 70B, 1 and 5 rows behind 300 7.9 -> 6.8.
constexpr int AM_WAVES = 8, AM_THREADS = AM_WAVES * 64;

// hi = rne(x), lo = rne(x - hi) of two fp32 values, packed with the first one in the low half: one conversion instruction takes both
template <bool F16>
__device__ __forceinline__ void pair_hi_lo(float a, float b, unsigned& hi, unsigned& lo)
{
    if (F16) {
        const f16_t ha = (f16_t)a, hb = (f16_t)b;
        hi = __builtin_bit_cast(uint16_t, ha) | ((unsigned)__builtin_bit_cast(uint16_t, hb) << 16);
        lo = __builtin_bit_cast(uint16_t, (f16_t)(a - (float)ha)) | ((unsigned)__builtin_bit_cast(uint16_t, (f16_t)(b - (float)hb)) << 16);
    } else {
        hi = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
        lo = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_t{a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u)}, bf16x2_t));
    }
}
// 8 fp32 values -> two packed fragments hi, lo
template <bool F16>
__device__ __forceinline__ void pack_hi_lo(const float (&v)[8], u32x4_t& hi, u32x4_t& lo)
{
    unsigned h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; i++) pair_hi_lo<F16>(v[2 * i], v[2 * i + 1], h[i], l[i]);
    hi = u32x4_t{h[0], h[1], h[2], h[3]};
    lo = u32x4_t{l[0], l[1], l[2], l[3]};
}
// the same for 8 consecutive values in LDS
template <bool F16>
__device__ __forceinline__ void split8(const float* x, u32x4_t& hi, u32x4_t& lo)
{
    // two 128-bit reads (x is 32-byte aligned), not eight dependent scalar ones
    const float4 a = *reinterpret_cast<const float4*>(x), b = *reinterpret_cast<const float4*>(x + 4);
    const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    pack_hi_lo<F16>(v, hi, lo);
}

// Four cache vectors (the same EPV dims of four consecutive positions) into a V^T tile: dim e of them as 8 bytes at
// dst + e * pitch; fp32 elements as hi = rne(x) there and lo = rne(x - hi) `plane` bytes further on.
template <typename KT>
__device__ __forceinline__ void store_v4(const u32x4_t (&v)[4], unsigned char* dst, int pitch, int plane)
{
    unsigned w[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++) { w[i][0] = v[i].x; w[i][1] = v[i].y; w[i][2] = v[i].z; w[i][3] = v[i].w; }
#pragma unroll
    for (int e = 0; e < 16 / (int)sizeof(KT); e++) {
        if constexpr (sizeof(KT) == 4) {
            uint2 h, l;
            pair_hi_lo<false>(__uint_as_float(w[0][e]), __uint_as_float(w[1][e]), h.x, l.x);
            pair_hi_lo<false>(__uint_as_float(w[2][e]), __uint_as_float(w[3][e]), h.y, l.y);
            *reinterpret_cast<uint2*>(dst + e * pitch) = h;
            *reinterpret_cast<uint2*>(dst + plane + e * pitch) = l;
        } else {
            unsigned h[4];
#pragma unroll
            for (int i = 0; i < 4; i++) h[i] = (w[i][e >> 1] >> ((e & 1) * 16)) & 0xffffu;
            *reinterpret_cast<uint2*>(dst + e * pitch) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        }
    }
}

// Elements dd .. dd + 3 of the output of (row, head) rh, folded from partials part[rh][n_splits][HD + 4] (unnormalised output, maximum,
// sum), eight of them requested together.  DEV: they come from blocks of the same launch and are loaded at device scope (each XCD
// has its own L2); the partials of all n_rows are less than 2 GiB then.
struct AttnAcc { float4 num; float m, den; };   // output relative to maximum m
__device__ __forceinline__ void attn_acc_add(AttnAcc& a, const AttnAcc& b)
{
    const float m = fmaxf(a.m, b.m), ca = a.m > -INFINITY ? __expf(a.m - m) : 0.f, cb = b.m > -INFINITY ? __expf(b.m - m) : 0.f;
    a.num = make_float4(a.num.x * ca + b.num.x * cb, a.num.y * ca + b.num.y * cb, a.num.z * ca + b.num.z * cb, a.num.w * ca + b.num.w * cb);
    a.den = a.den * ca + b.den * cb;
    a.m = m;
}
__device__ __forceinline__ float4 attn_acc_out(const AttnAcc& a) { return make_float4(a.num.x / a.den, a.num.y / a.den, a.num.z / a.den, a.num.w / a.den); }
template <int HD, bool DEV>
__device__ __forceinline__ AttnAcc attn_fold(const float* part, int n_rows, int rh, int n_splits, int first, int end, int dd)   // ranges first .. end - 1
{
    constexpr int ROW = HD + 4;
    const float* p = part + (size_t)rh * n_splits * ROW;
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(part), 0, DEV ? n_rows * n_splits * ROW * 4 : 0, 0x00020000);
    AttnAcc a = {make_float4(0.f, 0.f, 0.f, 0.f), -INFINITY, 0.f};
    for (int s0 = first; s0 < end; s0 += 8) {
        u32x4_t o[8], ml[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {   // (past the last one it is read again and weighs nothing)
            const int sl = min(s0 + u, end - 1);
            if (DEV) {
                const int b = (rh * n_splits + sl) * ROW * 4;
                ml[u] = __builtin_amdgcn_raw_buffer_load_b128(r, b + HD * 4, 0, 16 /* sc1: device scope */);
                o[u] = __builtin_amdgcn_raw_buffer_load_b128(r, b + dd * 4, 0, 16);
            } else {
                ml[u] = *reinterpret_cast<const u32x4_t*>(p + sl * ROW + HD);
                o[u] = *reinterpret_cast<const u32x4_t*>(p + sl * ROW + dd);
            }
        }
        AttnAcc b = {make_float4(0.f, 0.f, 0.f, 0.f), -INFINITY, 0.f};
#pragma unroll
        for (int u = 0; u < 8; u++) b.m = fmaxf(b.m, __uint_as_float(ml[u].x));
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const float l = __uint_as_float(ml[u].y), w = s0 + u < end && l > 0.f ? __expf(__uint_as_float(ml[u].x) - b.m) : 0.f;
            b.num.x = fmaf(w, __uint_as_float(o[u].x), b.num.x); b.num.y = fmaf(w, __uint_as_float(o[u].y), b.num.y);
            b.num.z = fmaf(w, __uint_as_float(o[u].z), b.num.z); b.num.w = fmaf(w, __uint_as_float(o[u].w), b.num.w);
            b.den = fmaf(w, l, b.den);
        }
        attn_acc_add(a, b);
    }
    return a;
}
__device__ __forceinline__ void attn_put4(float4 o, size_t i, float* out, uint16_t* out_hi, uint16_t* out_lo, bool f16)
{
    if (!out_hi) { *reinterpret_cast<float4*>(out + i) = o; return; }
    uint2 h, l;
    if (f16) { pair_hi_lo<true>(o.x, o.y, h.x, l.x); pair_hi_lo<true>(o.z, o.w, h.y, l.y); }
    else { pair_hi_lo<false>(o.x, o.y, h.x, l.x); pair_hi_lo<false>(o.z, o.w, h.y, l.y); }
    *reinterpret_cast<uint2*>(out_hi + i) = h;
    *reinterpret_cast<uint2*>(out_lo + i) = l;
}
// The block of a (KV head, group of queries) = (blockIdx.y, blockIdx.z) that arrives last folds the partials of all ranges; nobody
// waits.  A block counts itself in when its stores, made at device scope, are acknowledged; the last one sets the counter back to
// zero for the next launch.  Called by the whole block.  Attention and the launch that folded, before / attention now: 7B, 5 rows behind
// 550 positions 8.8 + 5.4 / 10.8 us, 9 rows behind 100 of an fp16 cache 5.9 + 4.7 / 8.7.  (Fences in place of device-scope
// accesses write whole L2s back and cost more than the launch.)
__device__ __forceinline__ bool attn_last(unsigned* arrive)
{
    __shared__ int last;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned* c = arrive + blockIdx.y * gridDim.z + blockIdx.z;
        last = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (last) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return last;
}

// The fold for query vectors q0 .. q0 + nq - 1 (vector qg: row qg / G, head kvh G + qg % G), by the last block.  Threads that the outputs
// leave over share the ranges, eight and more each, and meet in LDS.
template <int HD, int NT>
__device__ __forceinline__ void attn_fold_block(const float* part, int M, int H, int G, int kvh, int q0, int nq, int n_splits, float* outp, uint16_t* out_hi,
                                                uint16_t* out_lo, bool out_f16)
{
    __shared__ AttnAcc acc[NT];
    const int items = nq * (HD / 4), tid = threadIdx.x;
    int shares = 1;
    while (shares * 2 * items <= NT && shares * 16 <= n_splits + 8) shares *= 2;
    const int per = (n_splits + shares - 1) / shares;
    auto row = [&](int f) { const int qg = q0 + f / (HD / 4); return qg / G * H + kvh * G + qg % G; };
    if (shares == 1) {
        for (int f = tid; f < items; f += NT) {
            const int rh = row(f), dd = f % (HD / 4) * 4;
            attn_put4(attn_acc_out(attn_fold<HD, true>(part, M * H, rh, n_splits, 0, n_splits, dd)), (size_t)rh * HD + dd, outp, out_hi, out_lo, out_f16);
        }
        return;
    }
    const int f = tid % items, sh = tid / items, rh = row(f), dd = f % (HD / 4) * 4;
    if (sh < shares) acc[tid] = attn_fold<HD, true>(part, M * H, rh, n_splits, min(sh * per, n_splits), min(sh * per + per, n_splits), dd);
    __syncthreads();
    if (sh == 0) {
        AttnAcc a = acc[f];
        for (int u = 1; u < shares; u++) attn_acc_add(a, acc[u * items + f]);
        attn_put4(attn_acc_out(a), (size_t)rh * HD + dd, outp, out_hi, out_lo, out_f16);
    }
}

// fp32 caches take the same kernel: while a chunk is staged every K / V element is split into two bf16 planes
// (hi = rne(x), lo = rne(x - hi), 16 mantissa bits together), and each contraction becomes three MFMAs
// (hi.hi + lo.hi + hi.lo; the lo.lo term is below the 16 bits the planes carry).
template <typename KT, int HD>
__global__ __launch_bounds__(AM_THREADS) void attn_mfma_kernel(const float* __restrict__ q, int ldq,
                                                               const KT* __restrict__ kc, const KT* __restrict__ vc,
                                                               const int* __restrict__ pos_dev, int pos_off, int M, int H, int Hkv,
                                                               int max_seq, int n_splits, float* __restrict__ part,
                                                               float* __restrict__ outp, int dq,
                                                               uint16_t* __restrict__ out_hi, uint16_t* __restrict__ out_lo,
                                                               bool out_f16, unsigned* arrive)
{
    constexpr bool F32 = sizeof(KT) == 4;
    constexpr bool F16 = IsF16<KT>::value;     // operand type of the MFMAs: fp16 for fp16 caches, else bf16
    constexpr int NP = F32 ? 2 : 1;            // planes per staged tile
    constexpr int ROWB = HD * 2 + 16;
    constexpr int EPV = 16 / (int)sizeof(KT);  // cache elements per 16-byte vector
    constexpr int VPR = HD / EPV;              // 16-byte vectors per cache row
    constexpr int KSTEPS = HD / 32;            // MFMA k-steps of a score
    constexpr int PT = AT_CHUNK / 16;          // position tiles of the chunk (6)
    constexpr int PS = AT_CHUNK / 32;          // k-steps of P.V (3)
    constexpr int DT = HD / 16;                // output dim tiles (8 or 4)
    constexpr int KPLANE = AT_CHUNK * ROWB, VPLANE = HD * AM_VPITCH;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* ktile = smem;                                       // [NP][AT_CHUNK][ROWB]
    unsigned char* vT = smem + NP * KPLANE;                            // [NP][HD][AM_VPITCH]
    float* qs = reinterpret_cast<float*>(vT + NP * VPLANE);            // [16][HD], pre-scaled
    float* sc = qs + AT_QPASS * HD;                                    // [16][AT_CHUNK]
    float* ml = sc + AT_QPASS * AT_CHUNK;                              // [16][2]

    const int split = blockIdx.x, kvh = blockIdx.y;
    const int G = H / Hkv, Q = G * M;
    const int j0 = split * AT_CHUNK;   // chunks of fixed length: where they lie does not depend on the position
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    // the block's group of 16 query vectors (blockIdx.z)
    const int q0 = blockIdx.z * AT_QPASS;
    const int nq = min(AT_QPASS, Q - q0);
    constexpr int QPT = AT_QPASS * HD / AM_THREADS;   // query elements per thread
    float qreg[QPT];
    constexpr int NV = (AT_CHUNK * VPR + AM_THREADS - 1) / AM_THREADS;
    constexpr int VU = AT_CHUNK / 4 * VPR, NVU = (VU + AM_THREADS - 1) / AM_THREADS;   // V units of 4 positions x EPV dims; per thread
    u32x4_t kr[NV], vr[NVU][4];
    // Query vectors, K and V are all requested before the position is known (one memory latency less on the way through the
    // kernel): cache rows past it may hold anything and are replaced by zeros when they are stored to LDS.
    // K: consecutive lanes take consecutive vectors of a row.  V: a thread takes the vectors of four consecutive positions, so
    // that the transpose stores 8 bytes at a time; four lanes share a row's 64 bytes.  (2-byte stores with a lane per position:
    // 11.4 us against 9.5, 7B, 5 rows behind 540 positions of an fp32 cache.)
    auto v_unit = [](int u, int& pg, int& dg) { const int w = u >> 2; pg = w % (AT_CHUNK / 4); dg = w / (AT_CHUNK / 4) * 4 + (u & 3); };
    {
        const KT* kbase = kc + (size_t)kvh * max_seq * HD;
        const KT* vbase = vc + (size_t)kvh * max_seq * HD;
#pragma unroll
        for (int t = 0; t < NV; t++) {
            const int v = min(tid + t * AM_THREADS, AT_CHUNK * VPR - 1);
            kr[t] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)min(j0 + v / VPR, max_seq - 1) * HD + (v % VPR) * EPV);
        }
        asm volatile("" ::: "memory");   // (the divisions of the queries' addresses behind the requests for K)
#pragma unroll
        for (int t = 0; t < QPT; t++) {
            const int e = tid + t * AM_THREADS, qg = q0 + min(e / HD, nq - 1);
            qreg[t] = q[(size_t)(qg / G) * ldq + (size_t)(kvh * G + qg % G) * HD + (e % HD)];
        }
#pragma unroll
        for (int t = 0; t < NVU; t++) {
            int pg, dg;
            v_unit(min(tid + t * AM_THREADS, VU - 1), pg, dg);
#pragma unroll
            for (int i = 0; i < 4; i++)
                vr[t][i] = *reinterpret_cast<const u32x4_t*>(vbase + (size_t)min(j0 + pg * 4 + i, max_seq - 1) * HD + dg * EPV);
        }
    }
    const int p0 = pos_dev[0] + pos_off;
    const int total = p0 + M;
    const int n = min(AT_CHUNK, total - j0);                   // may be <= 0
    const auto prsrc = __builtin_amdgcn_make_buffer_rsrc(part, 0, arrive ? M * H * n_splits * (HD + 4) * 4 : 0, 0x00020000);
    auto put_partial = [&](float* to, float4 v) {
        if (arrive) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), prsrc, (int)(to - part) * 4, 0, 16 /* sc1: device scope */);
        else *reinterpret_cast<float4*>(to) = v;
    };
    auto fold = [&]() {
        if (arrive && attn_last(arrive)) attn_fold_block<HD, AM_THREADS>(part, M, H, G, kvh, q0, nq, n_splits, outp, out_hi, out_lo, out_f16);
    };
    // A chunk that lies wholly behind the causal horizon of the block's LAST query row contributes nothing (in a
    // prompt pass that is half of all blocks): leave empty partials and go.  Uniform over the block.
    if (n_splits > 1 && (n <= 0 || j0 > p0 + (q0 + nq - 1) / G)) {
        for (int f = tid; f < nq * (HD / 4); f += AM_THREADS) {
            const int qi = f / (HD / 4), dd = (f % (HD / 4)) * 4;
            const int qg = q0 + qi, r = qg / G, head = kvh * G + qg % G;
            float* mine = part + (((size_t)r * H + head) * n_splits + split) * (HD + 4);
            put_partial(mine + dd, make_float4(0.f, 0.f, 0.f, 0.f));
            if (dd == 0) put_partial(mine + HD, make_float4(-INFINITY, 0.f, 0.f, 0.f));
        }
        fold();
        return;
    }
    if (n > 0) {  // stage K (row-major) and V (transposed)
        const int vmax = n * VPR - 1;
        const u32x4_t zero = {0u, 0u, 0u, 0u};   // positions past the chunk: zero keys and values
#pragma unroll
        for (int t = 0; t < NV; t++) {
            const int v = tid + t * AM_THREADS;
            if (v < AT_CHUNK * VPR) {
                const int pos = v / VPR, d0 = (v % VPR) * EPV;
                const u32x4_t kk = v <= vmax ? kr[t] : zero;
                if constexpr (F32) {
                    uint2 h, l;
                    pair_hi_lo<false>(__uint_as_float(kk.x), __uint_as_float(kk.y), h.x, l.x);
                    pair_hi_lo<false>(__uint_as_float(kk.z), __uint_as_float(kk.w), h.y, l.y);
                    *reinterpret_cast<uint2*>(ktile + pos * ROWB + d0 * 2) = h;
                    *reinterpret_cast<uint2*>(ktile + KPLANE + pos * ROWB + d0 * 2) = l;
                } else {
                    *reinterpret_cast<u32x4_t*>(ktile + pos * ROWB + d0 * 2) = kk;
                }
            }
        }
#pragma unroll
        for (int t = 0; t < NVU; t++) {
            const int u = tid + t * AM_THREADS;
            if (VU % AM_THREADS == 0 || u < VU) {
                int pg, dg;
                v_unit(u, pg, dg);
                const u32x4_t w4[4] = {pg * 4 < n ? vr[t][0] : zero, pg * 4 + 1 < n ? vr[t][1] : zero, pg * 4 + 2 < n ? vr[t][2] : zero,
                                       pg * 4 + 3 < n ? vr[t][3] : zero};
                store_v4<KT>(w4, vT + dg * EPV * AM_VPITCH + pg * 8, AM_VPITCH, VPLANE);
            }
        }
    }
    const float scale = 1.0f / sqrtf((float)HD);
    {   // one group of 16 query vectors per block: the groups of a head run side by side on different CUs instead of
        // one after the other, each re-staging the chunk out of the cache
#pragma unroll
        for (int t = 0; t < QPT; t++) {   // rows past nq: zero queries (their results are never stored)
            const int e = tid + t * AM_THREADS;
            qs[e] = e / HD < nq ? qreg[t] * scale : 0.f;
        }
        __syncthreads();   // K, V^T and the query vectors are staged
        if (n > 0) {
            // phase A: scores.  Wave w takes position tile w (w + 8, ..); D: lane (c = position, g) holds queries 4g .. 4g+3
            u32x4_t qh[KSTEPS], ql[KSTEPS];
#pragma unroll
            for (int st = 0; st < KSTEPS; st++) split8<F16>(qs + r16 * HD + st * 32 + g * 8, qh[st], ql[st]);
            for (int pt = wave; pt < PT; pt += AM_WAVES) {
                f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < KSTEPS; st++) {
                    const unsigned char* kp = ktile + (pt * 16 + r16) * ROWB + (st * 32 + g * 8) * 2;
                    const u32x4_t kf = *reinterpret_cast<const u32x4_t*>(kp);
                    acc = mfma_h16<F16>(qh[st], kf, acc);
                    acc = mfma_h16<F16>(ql[st], kf, acc);
                    if constexpr (F32) acc = mfma_h16<F16>(qh[st], *reinterpret_cast<const u32x4_t*>(kp + KPLANE), acc);
                }
#pragma unroll
                for (int jx = 0; jx < 4; jx++) sc[(g * 4 + jx) * AT_CHUNK + pt * 16 + r16] = acc[jx];
            }
        }
        __syncthreads();
        // phase B: causal mask, max, exp, sum.  Wave w < 4 owns queries 4w .. 4w+3, one per 16-lane row, so the two
        // reductions are DPP row operations; entries past the visible range (and rows past nq) become 0
        if (wave < 4) {
            const int qi = wave * 4 + g;
            int vis = 0;
            if (qi < nq) vis = min(n, p0 + (q0 + qi) / G + 1 - j0);   // positions of this chunk the row may see
            float sv[AT_CHUNK / 16];
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < AT_CHUNK / 16; t++) {
                const int j = r16 + 16 * t;
                sv[t] = sc[qi * AT_CHUNK + j];
                if (j < vis) mx = fmaxf(mx, sv[t]);
            }
            mx = row16_max(mx);
            float ls = 0.f;
#pragma unroll
            for (int t = 0; t < AT_CHUNK / 16; t++) {
                const int j = r16 + 16 * t;
                const float e = j < vis ? __expf(sv[t] - mx) : 0.f;
                sc[qi * AT_CHUNK + j] = e;
                ls += e;
            }
            ls = row16_sum(ls);
            if (r16 == 0) { ml[qi * 2] = mx; ml[qi * 2 + 1] = ls; }
        }
        __syncthreads();
        // phase C: O = P.V.  Wave w takes output dim tile w; A: lane (r = query, g) holds P[r][32 s + 8g ..],
        // B: lane (c = dim, g) holds V^T[dim][32 s + 8g ..]; D: lane (c = dim, g) holds queries 4g .. 4g+3
        u32x4_t ph[PS], pl[PS];
#pragma unroll
        for (int st = 0; st < PS; st++) split8<F16>(sc + r16 * AT_CHUNK + st * 32 + g * 8, ph[st], pl[st]);
#pragma unroll
        for (int dt = wave; dt < DT; dt += AM_WAVES) {
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
            if (n > 0) {
#pragma unroll
                for (int st = 0; st < PS; st++) {
                    const unsigned char* vp = vT + (dt * 16 + r16) * AM_VPITCH + (st * 32 + g * 8) * 2;
                    const u32x4_t vf = *reinterpret_cast<const u32x4_t*>(vp);
                    acc = mfma_h16<F16>(ph[st], vf, acc);
                    acc = mfma_h16<F16>(pl[st], vf, acc);
                    if constexpr (F32) acc = mfma_h16<F16>(ph[st], *reinterpret_cast<const u32x4_t*>(vp + VPLANE), acc);
                }
            }
            // the tile goes back through LDS (the query buffer is free by now) so that the block can write whole
            // rows: scattered 4-byte stores straight from the D layout kept every block waiting on the write path
#pragma unroll
            for (int jx = 0; jx < 4; jx++) qs[(g * 4 + jx) * HD + dt * 16 + r16] = acc[jx];
        }
        __syncthreads();
        for (int f = tid; f < nq * (HD / 4); f += AM_THREADS) {
            const int qi = f / (HD / 4), dd = (f % (HD / 4)) * 4;
            const float4 o = *reinterpret_cast<const float4*>(qs + qi * HD + dd);
            const int qg = q0 + qi, r = qg / G, head = kvh * G + qg % G;
            const float mx = ml[qi * 2], ls = ml[qi * 2 + 1];
            if (n_splits == 1) {
                const size_t oo = (size_t)r * dq + (size_t)head * HD + dd;
                const float inv = 1.0f / ls;
                if (out_hi) {
                    split_store(o.x * inv, out_hi, out_lo, oo, out_f16); split_store(o.y * inv, out_hi, out_lo, oo + 1, out_f16);
                    split_store(o.z * inv, out_hi, out_lo, oo + 2, out_f16); split_store(o.w * inv, out_hi, out_lo, oo + 3, out_f16);
                } else {
                    *reinterpret_cast<float4*>(outp + oo) = make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
                }
            } else {
                float* mine = part + (((size_t)r * H + head) * n_splits + split) * (HD + 4);
                put_partial(mine + dd, o);
                if (dd == 0) put_partial(mine + HD, make_float4(n > 0 ? mx : -INFINITY, n > 0 ? ls : 0.f, 0.f, 0.f));
            }
        }
    }
    if (n_splits > 1) fold();
}

// ---- prompt passes: one block per KV head and 64 query vectors walks the whole causal range -----------------
// Eight waves share the staged K / V^T chunks (64 positions at a time, the same 16-bit planes as above): wave w takes the
// 16 query vectors 16 (w & 3) .. against half w >> 2 of every chunk, so that a SIMD has two waves to switch between although a
// prompt of 512 rows gives a CU one block only.  A wave keeps its HD x 16 output tile and the running maximum / sum of every
// query vector in registers and rescales them chunk by chunk (online soft-max); the two halves are merged at the end.
// Nothing is written but the finished output, and a chunk is staged once per 64 query vectors instead of once per 16.
// Both products are taken transposed, S^T = K Q^T and O^T = V^T P^T: a lane (c, g) then owns query c in the scores (positions
// 4g .. 4g+3 of every 16), in the exponentials as the B operand of the second product, and in the output tile (dims
// 4g .. 4g+3), so the exponentials never leave their registers and the statistics are two shuffles.  The B operand wants
// eight positions of a 32-wide k-step per lane and the lane has four of either 16-wide half: a contraction does not care
// about the order of its terms, so V^T is staged in that order (slot 8g + 4h + x of a k-step = position 16h + 4g + x).
// V is loaded four positions at a time per thread, so that the transpose writes 8 bytes where it wrote 2.  The next chunk is
// requested before the present one is multiplied; blocks with the longest causal range start first.  What is left is LDS
// traffic and the conversion of fp32 caches.  512 rows, fp32 cache: 7B 49.6 -> 32 us per layer, 13B (second pass of 1000) 127 -> 52 on average.
constexpr int AP_Q = 64;                 // query vectors per block
constexpr int AP_C = 64;                 // cache positions per step
constexpr int AP_THREADS = 512;
constexpr int AP_VPITCH = AP_C * 2 + 32; // bytes per row of the transposed V tile (conflict-free 8-byte writes and 16-byte reads)

template <typename KT, int HD>
static constexpr size_t attn_prompt_lds_bytes()
{
    return (sizeof(KT) == 4 ? 4 : 2) * ((size_t)AP_C * (HD * 2 + 16) + (size_t)HD * AP_VPITCH);   // two buffers
}

template <typename KT, int HD>
__global__ __launch_bounds__(AP_THREADS, 2) void attn_prompt_kernel(const float* __restrict__ q, int ldq,
                                                                 const KT* __restrict__ kc, const KT* __restrict__ vc,
                                                                 const int* __restrict__ pos_dev, int pos_off, int M, int H, int Hkv,
                                                                 int max_seq, float* __restrict__ outp, int dq,
                                                                 uint16_t* __restrict__ out_hi, uint16_t* __restrict__ out_lo,
                                                                 bool out_f16)
{
    constexpr bool F32 = sizeof(KT) == 4;
    constexpr bool F16 = IsF16<KT>::value;
    constexpr int NP = F32 ? 2 : 1;
    constexpr int ROWB = HD * 2 + 16;
    constexpr int EPV = 16 / (int)sizeof(KT);
    constexpr int VPR = HD / EPV;
    constexpr int KSTEPS = HD / 32;
    constexpr int PT = AP_C / 32;              // position tiles of a wave's half of a chunk (2, one k-step of P.V)
    constexpr int DT = HD / 16;                // output dim tiles per wave (8 or 4)
    constexpr int KPLANE = AP_C * ROWB, VPLANE = HD * AP_VPITCH;
    constexpr int NK = AP_C * VPR / AP_THREADS;                                // K vectors per thread
    constexpr int VU = AP_C / 4 * VPR, NVU = (VU + AP_THREADS - 1) / AP_THREADS;  // V units of 4 positions x EPV dims; per thread
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int BUF = NP * (KPLANE + VPLANE);   // a buffer: K planes [NP][AP_C][ROWB], V^T planes [NP][HD][AP_VPITCH]

    const int G = H / Hkv, Q = G * M;
    // Block id -> (KV head, query block), longest causal range first.  Workgroups go to the eight XCDs round-robin by id: with
    // a multiple of eight heads every head stays on one XCD, whose L2 then fetches its K and V once for all query blocks.
    int kvh, qb;
    {
        const int id = blockIdx.x, nqb = (int)gridDim.x / Hkv;
        if (Hkv % 8 == 0) { const int hpx = Hkv >> 3, i = id >> 3; kvh = (id & 7) * hpx + i % hpx; qb = i / hpx; }
        else { kvh = id % Hkv; qb = id / Hkv; }
        qb = nqb - 1 - qb;
    }
    const int p0 = pos_dev[0] + pos_off;
    const int total = p0 + M;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const int wq = wave & 3, half = wave >> 2;             // query group, half of every chunk
    const int q0 = qb * AP_Q;
    const int nq = min(AP_Q, Q - q0);
    const int last_vis = p0 + (q0 + nq - 1) / G;          // last position any query vector of the block may see
    const float scale = 1.0f / sqrtf((float)HD);

    // K / V of the chunk at j0 into registers; positions past the end re-read the last one (zeroed when stored to LDS)
    u32x4_t kr[NK], vr[NVU][4];
    const KT* kbase = kc + (size_t)kvh * max_seq * HD;
    const KT* vbase = vc + (size_t)kvh * max_seq * HD;
    auto load = [&](int j0) {
#pragma unroll
        for (int t = 0; t < NK; t++) {
            const int v = tid + t * AP_THREADS;
            kr[t] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)min(j0 + v / VPR, total - 1) * HD + (v % VPR) * EPV);
        }
#pragma unroll
        for (int t = 0; t < NVU; t++) {
            const int u = min(tid + t * AP_THREADS, VU - 1);   // 16 lanes = the 16 position groups of one dim group
#pragma unroll
            for (int i = 0; i < 4; i++)
                vr[t][i] = *reinterpret_cast<const u32x4_t*>(vbase + (size_t)min(j0 + (u & 15) * 4 + i, total - 1) * HD + (u >> 4) * EPV);
        }
    };
    auto stage = [&](unsigned char* ktile, int n) {   // registers -> a buffer; n = positions of the chunk that exist
        unsigned char* vT = ktile + NP * KPLANE;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < NK; t++) {
            const int v = tid + t * AP_THREADS, pos = v / VPR, d0 = (v % VPR) * EPV;
            const u32x4_t kk = pos < n ? kr[t] : zero;
            if constexpr (F32) {
                uint2 h, l;
                pair_hi_lo<false>(__uint_as_float(kk.x), __uint_as_float(kk.y), h.x, l.x);
                pair_hi_lo<false>(__uint_as_float(kk.z), __uint_as_float(kk.w), h.y, l.y);
                *reinterpret_cast<uint2*>(ktile + pos * ROWB + d0 * 2) = h;
                *reinterpret_cast<uint2*>(ktile + KPLANE + pos * ROWB + d0 * 2) = l;
            } else {
                *reinterpret_cast<u32x4_t*>(ktile + pos * ROWB + d0 * 2) = kk;
            }
        }
#pragma unroll
        for (int t = 0; t < NVU; t++) {
            const int u = tid + t * AP_THREADS;
            if (VU % AP_THREADS && u >= VU) break;
            const int pg = u & 15, d0 = (u >> 4) * EPV;
            const int slot = (pg >> 3) * 32 + (pg & 3) * 8 + ((pg >> 2) & 1) * 4;   // of positions 4 pg .. 4 pg + 3
            const u32x4_t w4[4] = {pg * 4 < n ? vr[t][0] : zero, pg * 4 + 1 < n ? vr[t][1] : zero, pg * 4 + 2 < n ? vr[t][2] : zero,
                                   pg * 4 + 3 < n ? vr[t][3] : zero};
            store_v4<KT>(w4, vT + d0 * AP_VPITCH + slot * 2, AP_VPITCH, VPLANE);
        }
    };
    load(0);

    // the wave's 16 query vectors as hi / lo fragments (B operand: lane (r16 = query, g) holds dims 32 st + 8 g ..)
    const int myq = wq * 16 + r16;                           // the lane's query vector within the block
    const int qv = q0 + min(myq, nq - 1);                      // vectors past nq read a valid one; never stored
    u32x4_t qh[KSTEPS], ql[KSTEPS];
    {
        const float* qp = q + (size_t)(qv / G) * ldq + (size_t)(kvh * G + qv % G) * HD;
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) {
            const float4 a = *reinterpret_cast<const float4*>(qp + st * 32 + g * 8), b = *reinterpret_cast<const float4*>(qp + st * 32 + g * 8 + 4);
            const float x[8] = {a.x * scale, a.y * scale, a.z * scale, a.w * scale, b.x * scale, b.y * scale, b.z * scale, b.w * scale};
            pack_hi_lo<F16>(x, qh[st], ql[st]);
        }
    }
    const int horizon = myq < nq ? p0 + qv / G : -1;           // last position the lane's query may see; -1 = padding
    const int wave_vis = wq * 16 < nq ? p0 + (q0 + min(wq * 16 + 15, nq - 1)) / G : -1;   // the same over the wave
    float mrun = -INFINITY, lrun = 0.f;                        // lrun: the lane's own positions only, folded at the end
    f32x4_t oacc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; dt++) oacc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Chunk c is multiplied out of buffer c % 2 while chunk c + 1 goes from registers into the other one.  The first half's
    // waves store first and multiply then, the second half's the other way round: of the two waves of a SIMD one converts and
    // stores while the other one multiplies.  One barrier per chunk: behind it this chunk is staged and the last one consumed.
    stage(smem, min(AP_C, total));
    if (AP_C <= last_vis) load(AP_C);
    auto stage_next = [&](int j0) {
        if (j0 + AP_C <= last_vis) {
            stage(smem + ((j0 / AP_C + 1) & 1) * BUF, min(AP_C, total - j0 - AP_C));
            if (j0 + 2 * AP_C <= last_vis) load(j0 + 2 * AP_C);
        }
    };
    auto multiply = [&](int j0) {
        const unsigned char* ktile = smem + (j0 / AP_C & 1) * BUF;
        const unsigned char* vT = ktile + NP * KPLANE;
        // scores of the half's 32 positions for the lane's query, masked; running maximum
        float sv[PT][4];
        float mnew = mrun;
#pragma unroll
        for (int pt = 0; pt < PT; pt++) {
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < KSTEPS; st++) {
                const unsigned char* kp = ktile + (half * 32 + pt * 16 + r16) * ROWB + (st * 32 + g * 8) * 2;
                const u32x4_t kf = *reinterpret_cast<const u32x4_t*>(kp);
                acc = mfma_h16<F16>(kf, qh[st], acc);
                acc = mfma_h16<F16>(kf, ql[st], acc);
                if constexpr (F32) acc = mfma_h16<F16>(*reinterpret_cast<const u32x4_t*>(kp + KPLANE), qh[st], acc);
            }
#pragma unroll
            for (int jx = 0; jx < 4; jx++) {
                sv[pt][jx] = j0 + half * 32 + pt * 16 + g * 4 + jx <= horizon ? acc[jx] : -INFINITY;
                mnew = fmaxf(mnew, sv[pt][jx]);
            }
        }
        mnew = fmaxf(mnew, __shfl_xor(mnew, 16, 64));
        mnew = fmaxf(mnew, __shfl_xor(mnew, 32, 64));
        const float alpha = mrun > -INFINITY ? __expf(mrun - mnew) : 0.f;
        mrun = mnew;
        lrun *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
#pragma unroll
            for (int jx = 0; jx < 4; jx++) oacc[dt][jx] *= alpha;
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const float v = sv[i >> 2][i & 3];
            e[i] = v > -INFINITY ? __expf(v - mnew) : 0.f;
            lrun += e[i];
        }
        u32x4_t ph, pl;
        pack_hi_lo<F16>(e, ph, pl);
#pragma unroll
        for (int dt = 0; dt < DT; dt++) {
            const unsigned char* vp = vT + (dt * 16 + r16) * AP_VPITCH + (half * 32 + g * 8) * 2;
            const u32x4_t vf = *reinterpret_cast<const u32x4_t*>(vp);
            oacc[dt] = mfma_h16<F16>(vf, ph, oacc[dt]);
            oacc[dt] = mfma_h16<F16>(vf, pl, oacc[dt]);
            if constexpr (F32) oacc[dt] = mfma_h16<F16>(*reinterpret_cast<const u32x4_t*>(vp + VPLANE), ph, oacc[dt]);
        }
    };
    for (int j0 = 0; j0 <= last_vis; j0 += AP_C) {
        lds_barrier();
        if (half == 0) stage_next(j0);
        if (j0 + half * 32 <= wave_vis) multiply(j0);          // uniform over the wave
        if (half == 1) stage_next(j0);
    }
    lrun += __shfl_xor(lrun, 16, 64);
    lrun += __shfl_xor(lrun, 32, 64);
    // the second half's waves hand their tile and statistics over through LDS
    float4* mo = reinterpret_cast<float4*>(smem) + wq * DT * 64 + lane;                      // [4][DT][64]
    float2* ms = reinterpret_cast<float2*>(smem + 4 * DT * 64 * 16) + wq * 16 + r16;          // [4][16]
    static_assert((size_t)4 * DT * 64 * 16 + 4 * 16 * 8 <= attn_prompt_lds_bytes<KT, HD>(), "the merge fits the staging area");
    lds_barrier();                                             // the last chunk is fully consumed
    if (half == 1) {
#pragma unroll
        for (int dt = 0; dt < DT; dt++) mo[dt * 64] = make_float4(oacc[dt][0], oacc[dt][1], oacc[dt][2], oacc[dt][3]);
        if (g == 0) *ms = make_float2(mrun, lrun);
    }
    lds_barrier();
    if (half == 1 || myq >= nq) return;
    {
        const float2 s1 = *ms;
        const float m = fmaxf(mrun, s1.x);                     // position 0 is visible to every query: finite
        const float w0 = mrun > -INFINITY ? __expf(mrun - m) : 0.f, w1 = s1.x > -INFINITY ? __expf(s1.x - m) : 0.f;
        lrun = lrun * w0 + s1.y * w1;
#pragma unroll
        for (int dt = 0; dt < DT; dt++) {
            const float4 o1 = mo[dt * 64];
            oacc[dt][0] = oacc[dt][0] * w0 + o1.x * w1; oacc[dt][1] = oacc[dt][1] * w0 + o1.y * w1;
            oacc[dt][2] = oacc[dt][2] * w0 + o1.z * w1; oacc[dt][3] = oacc[dt][3] * w0 + o1.w * w1;
        }
    }
    const size_t oo = (size_t)(qv / G) * dq + (size_t)(kvh * G + qv % G) * HD + g * 4;
#pragma unroll
    for (int dt = 0; dt < DT; dt++) {
        const float o[4] = {oacc[dt][0] / lrun, oacc[dt][1] / lrun, oacc[dt][2] / lrun, oacc[dt][3] / lrun};
        if (out_hi) {
            unsigned h[4], l[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                h[i] = f32_to_h16_bits(o[i], out_f16);
                l[i] = f32_to_h16_bits(o[i] - h16_bits_to_f32(h[i], out_f16), out_f16);
            }
            *reinterpret_cast<uint2*>(out_hi + oo + dt * 16) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            *reinterpret_cast<uint2*>(out_lo + oo + dt * 16) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
        } else {
            *reinterpret_cast<float4*>(outp + oo + dt * 16) = make_float4(o[0], o[1], o[2], o[3]);
        }
    }
}

template <typename KT, int HD>
static size_t attn_mfma_lds_bytes()
{
    const size_t planes = sizeof(KT) == 4 ? 2 : 1;
    return planes * ((size_t)AT_CHUNK * (HD * 2 + 16) + (size_t)HD * AM_VPITCH) + (size_t)AT_QPASS * HD * 4 +
           (size_t)AT_QPASS * AT_CHUNK * 4 + (size_t)AT_QPASS * 2 * 4;
}

template <typename KT, int HD>
static size_t attn_lds_bytes()
{
    return (size_t)2 * AT_CHUNK * (HD * sizeof(KT) + 16) + (size_t)AT_QPASS * HD * 4 + (size_t)AT_QPASS * AT_CHUNK * 4 +
           (size_t)AT_QPASS * 2 * 4 + (size_t)AT_THREADS * AT_QPASS * 4;
}

// Folds the split partials of one (row, head) into the attention output, where the attention launch does not do so itself.
template <int HD>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part, int n_rows, int n_splits, float* __restrict__ out,
                                                           uint16_t* __restrict__ out_hi, uint16_t* __restrict__ out_lo, bool f16)
{
    const int i = blockIdx.x * 256 + threadIdx.x, rh = i / (HD / 4), dd = i % (HD / 4) * 4;   // rh: (row, head)
    if (rh >= n_rows) return;
    attn_put4(attn_acc_out(attn_fold<HD, false>(part, n_rows, rh, n_splits, 0, n_splits, dd)), (size_t)rh * HD + dd, out, out_hi, out_lo, f16);
}

// ---- register-resident variant for few query vectors (decoding, short verification blocks) ----------
// One block = one KV head x one range of positions x up to NQ query vectors.  No LDS staging: a lane
// owns 16 bytes of a cache row (LPP lanes per position, PPL = 64 / LPP positions per wave-wide load)
// and every wave keeps NL such K loads and NL V loads in flight, consecutive waves reading
// consecutive 1 KB pieces.  Scores are reduced over the LPP lanes of a position by shuffles, each wave
// runs an online softmax over its positions, and the NW waves are folded through LDS at the end.  With
// one range per head the block writes the finished output and no second kernel is needed.
template <typename KT> __device__ __forceinline__ void aw_unpack(u32x4_t w, float (&o)[16 / sizeof(KT)]);
template <> __device__ __forceinline__ void aw_unpack<uint16_t>(u32x4_t w, float (&o)[8])
{
    o[0] = __uint_as_float(w.x << 16); o[1] = __uint_as_float(w.x & 0xffff0000u);
    o[2] = __uint_as_float(w.y << 16); o[3] = __uint_as_float(w.y & 0xffff0000u);
    o[4] = __uint_as_float(w.z << 16); o[5] = __uint_as_float(w.z & 0xffff0000u);
    o[6] = __uint_as_float(w.w << 16); o[7] = __uint_as_float(w.w & 0xffff0000u);
}
template <> __device__ __forceinline__ void aw_unpack<f16_t>(u32x4_t w, float (&o)[8])
{
    const f16x8_t h = __builtin_bit_cast(f16x8_t, w);
#pragma unroll
    for (int i = 0; i < 8; i++) o[i] = (float)h[i];
}
template <> __device__ __forceinline__ void aw_unpack<float>(u32x4_t w, float (&o)[4])
{
    o[0] = __uint_as_float(w.x); o[1] = __uint_as_float(w.y); o[2] = __uint_as_float(w.z); o[3] = __uint_as_float(w.w);
}
// sum over the LPP lanes of one position (every lane of the segment gets it).  Segments of 8 and 16
// lanes lie inside one DPP row: rotations by 8, 4, 2, 1 (or a half-row mirror and two quad swaps) add all
// of them without going through the LDS crossbar.
template <int LPP> __device__ __forceinline__ float aw_seg_sum(float v)
{
    if (LPP == 16 || LPP == 32) {
        v = dpp_add<0x128>(v);  // row_ror:8
        v = dpp_add<0x124>(v);  // row_ror:4
        v = dpp_add<0x122>(v);  // row_ror:2
        v = dpp_add<0x121>(v);  // row_ror:1
        if (LPP == 32) v += __shfl_xor(v, 16, 64);
    } else if (LPP == 8) {
        v = dpp_add<0x141>(v);  // row_half_mirror: lane i <- lane 7 - i of its half row
        v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
        v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    } else {
#pragma unroll
        for (int o = LPP / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    }
    return v;
}
// sum / max across the segments of a wave, for values already uniform inside each segment
template <int LPP> __device__ __forceinline__ float aw_xseg_sum(float v)
{
#pragma unroll
    for (int o = 32; o >= LPP; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <int LPP> __device__ __forceinline__ float aw_xseg_max(float v)
{
#pragma unroll
    for (int o = 32; o >= LPP; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

template <typename KT, int HD, int NQ, int NW, int NL>
__global__ __launch_bounds__(NW * 64) void attn_wide_kernel(const float* __restrict__ q, int ldq,
                                                            const KT* __restrict__ kc, const KT* __restrict__ vc,
                                                            const int* pos_dev, int pos_off, int M, int H, int Hkv,
                                                            int max_seq, int n_splits, int chunk, float* __restrict__ part,
                                                            float* __restrict__ outp, int dq,
                                                            uint16_t* __restrict__ out_hi, uint16_t* __restrict__ out_lo,
                                                            bool out_f16, unsigned* arrive)
{
    constexpr int EPV = 16 / (int)sizeof(KT), LPP = HD / EPV, PPL = 64 / LPP, NT = NW * 64;
    constexpr int PASS = NL * NW * PPL;  // positions one pass of the block covers
    __shared__ __align__(16) float qs[NQ * HD];     // query vectors, pre-scaled
    __shared__ float wacc[NW * NQ * HD];            // per-wave unnormalised outputs
    __shared__ float wml[NW * NQ * 2];              // per-wave (max, sum)
    const int split = blockIdx.x, kvh = blockIdx.y, q0 = blockIdx.z * NQ;
    const int G = H / Hkv, Q = G * M, nq = min(NQ, Q - q0);
    const int j0 = split * chunk;    // ranges of fixed length: where they lie does not depend on the position
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seg = lane / LPP, sl = (lane % LPP) * EPV;
    const int jlast = min(j0 + chunk, max_seq) - 1;   // last cache row of the range (may lie past the position)
    const KT* kbase = kc + (size_t)kvh * max_seq * HD + sl;
    const KT* vbase = vc + (size_t)kvh * max_seq * HD + sl;

    u32x4_t kr[NL], vr[NL];
    // addresses are clamped to the last row of the range, never predicated: all loads of a pass stay in flight together.  The
    // first pass is requested before the position is known (one memory latency less on the way through the kernel):
    // rows past it may hold anything, their scores are masked and their values replaced by zeros.
    auto issue_k = [&](int pass) {
#pragma unroll
        for (int t = 0; t < NL; t++) {
            const int j = min(j0 + ((pass * NL + t) * NW + wave) * PPL + seg, jlast);
            kr[t] = *reinterpret_cast<const u32x4_t*>(kbase + (size_t)j * HD);
        }
    };
    auto issue_v = [&](int pass) {
#pragma unroll
        for (int t = 0; t < NL; t++) {
            const int j = min(j0 + ((pass * NL + t) * NW + wave) * PPL + seg, jlast);
            vr[t] = *reinterpret_cast<const u32x4_t*>(vbase + (size_t)j * HD);
        }
    };
    issue_k(0);
    issue_v(0);
    const int p0 = pos_dev[0] + pos_off, total = p0 + M;
    const int n = min(chunk, total - j0);  // may be <= 0
    const int n_pass = n > 0 ? (n + PASS - 1) / PASS : 0;

    const float scale = 1.0f / sqrtf((float)HD);
    for (int e = tid; e < NQ * HD; e += NT) {
        const int qi = e / HD;
        float v = 0.f;
        if (qi < nq) {
            const int qg = q0 + qi;
            v = q[(size_t)(qg / G) * ldq + (size_t)(kvh * G + qg % G) * HD + (e % HD)] * scale;
        }
        qs[e] = v;
    }
    int vis[NQ];  // first position a query may NOT see
#pragma unroll
    for (int qi = 0; qi < NQ; qi++) vis[qi] = qi < nq ? min(p0 + (q0 + qi) / G + 1, j0 + n) : j0;
    __syncthreads();

    float m[NQ], l[NQ], acc[NQ][EPV];
#pragma unroll
    for (int qi = 0; qi < NQ; qi++) {
        m[qi] = -INFINITY; l[qi] = 0.f;
#pragma unroll
        for (int u = 0; u < EPV; u++) acc[qi][u] = 0.f;
    }
    for (int pass = 0; pass < n_pass; pass++) {
        float sc[NQ][NL];
#pragma unroll
        for (int t = 0; t < NL; t++) {
            float kf[EPV];
            aw_unpack<KT>(kr[t], kf);
            const int j = j0 + ((pass * NL + t) * NW + wave) * PPL + seg;
#pragma unroll
            for (int qi = 0; qi < NQ; qi++) {
                const float* qv = qs + qi * HD + sl;
                float dot = 0.f;
#pragma unroll
                for (int u = 0; u < EPV; u += 4) {
                    const float4 t4 = *reinterpret_cast<const float4*>(qv + u);
                    dot = fmaf(kf[u], t4.x, dot); dot = fmaf(kf[u + 1], t4.y, dot);
                    dot = fmaf(kf[u + 2], t4.z, dot); dot = fmaf(kf[u + 3], t4.w, dot);
                }
                dot = aw_seg_sum<LPP>(dot);
                sc[qi][t] = j < vis[qi] ? dot : -INFINITY;
            }
        }
        if (pass + 1 < n_pass) issue_k(pass + 1);
#pragma unroll
        for (int qi = 0; qi < NQ; qi++) {
            float mx = sc[qi][0];
#pragma unroll
            for (int t = 1; t < NL; t++) mx = fmaxf(mx, sc[qi][t]);
            mx = aw_xseg_max<LPP>(mx);
            const float mn = fmaxf(m[qi], mx);          // uniform over the wave
            const bool live = mn > -INFINITY;
            const float c = live ? __expf(m[qi] - mn) : 1.0f;   // exp(-inf) = 0 on the first live pass
            l[qi] *= c;
#pragma unroll
            for (int u = 0; u < EPV; u++) acc[qi][u] *= c;
            m[qi] = mn;
#pragma unroll
            for (int t = 0; t < NL; t++) {
                const float e = live ? __expf(sc[qi][t] - mn) : 0.f;  // masked scores give 0
                sc[qi][t] = e;
                l[qi] += e;
            }
        }
#pragma unroll
        for (int t = 0; t < NL; t++) {
            float vf[EPV];
            const bool live = ((pass * NL + t) * NW + wave) * PPL + seg < n;
            aw_unpack<KT>(live ? vr[t] : u32x4_t{0u, 0u, 0u, 0u}, vf);
#pragma unroll
            for (int qi = 0; qi < NQ; qi++)
#pragma unroll
                for (int u = 0; u < EPV; u++) acc[qi][u] = fmaf(sc[qi][t], vf[u], acc[qi][u]);
        }
        if (pass + 1 < n_pass) issue_v(pass + 1);
    }
    // fold the position segments of the wave, then the waves of the block
#pragma unroll
    for (int qi = 0; qi < NQ; qi++) {
        l[qi] = aw_xseg_sum<LPP>(l[qi]);
#pragma unroll
        for (int u = 0; u < EPV; u++) acc[qi][u] = aw_xseg_sum<LPP>(acc[qi][u]);
        if (seg == 0) {
#pragma unroll
            for (int u = 0; u < EPV; u++) wacc[(wave * NQ + qi) * HD + sl + u] = acc[qi][u];
        }
        if (lane == 0) { wml[(wave * NQ + qi) * 2] = m[qi]; wml[(wave * NQ + qi) * 2 + 1] = l[qi]; }
    }
    __syncthreads();
    const auto prsrc = __builtin_amdgcn_make_buffer_rsrc(part, 0, arrive ? M * H * n_splits * (HD + 4) * 4 : 0, 0x00020000);
    for (int e = tid; e < nq * HD; e += NT) {
        const int qi = e / HD, d = e % HD;
        float gm = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; w++) gm = fmaxf(gm, wml[(w * NQ + qi) * 2]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const float mw = wml[(w * NQ + qi) * 2];
            if (mw > -INFINITY) {
                const float c = __expf(mw - gm);
                num = fmaf(c, wacc[(w * NQ + qi) * HD + d], num);
                den = fmaf(c, wml[(w * NQ + qi) * 2 + 1], den);
            }
        }
        const int qg = q0 + qi, r = qg / G, head = kvh * G + qg % G;
        if (n_splits == 1) {
            const size_t oo = (size_t)r * dq + (size_t)head * HD + d;
            if (out_hi) split_store(num / den, out_hi, out_lo, oo, out_f16);
            else outp[oo] = num / den;
        } else {
            float* mine = part + (((size_t)r * H + head) * n_splits + split) * (HD + 4);
            if (arrive) {   // at device scope: see the fold below
                const int o = (int)(mine - part) * 4;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(num), prsrc, o + d * 4, 0, 16);
                if (d < 2) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d == 0 ? gm : den), prsrc, o + (HD + d) * 4, 0, 16);
            } else {
                mine[d] = num;
                if (d == 0) { mine[HD] = gm; mine[HD + 1] = den; }
            }
        }
    }
    if (arrive && n_splits > 1 && attn_last(arrive)) attn_fold_block<HD, NT>(part, M, H, G, kvh, q0, nq, n_splits, outp, out_hi, out_lo, out_f16);
}

// folds: the launch can fold its partials itself
static AttnPlan attn_plan(const Dims& D, int ctx, int M, bool folds = false)
{
    const AttnShape a = {D.H / D.Hkv, D.Hkv, D.hd, D.kt == WT_F32, D.wt == WT_F32};
    const int splits = D.opt ? D.opt->attn_splits : 0, kernel = D.opt ? D.opt->attn_kernel : 0;
    return folds && M == 1 && D.H <= ATTN_COUNTERS ? attn_plan_many(a, ctx, splits, kernel) : attn_plan(a, ctx, M, splits, kernel);
}

long attention_splits(const Dims& D, int ctx, int M)
{
    const AttnPlan pl = attn_plan(D, ctx, M);
    if (!pl.wide) return pl.n_splits;
    const AttnPlan many = attn_plan(D, ctx, M, true);
    return -((long)pl.n_splits + 64 * (long)pl.chunk + ((long)many.n_splits + 128 * (long)many.chunk) * (1l << 32));  // distinct values for distinct launch shapes
}

int attention_ranges(const Dims& D, int ctx, int M) { return attn_plan(D, ctx, M).n_splits; }

size_t attention_scratch_floats(const Dims& D, int max_rows)
{
    size_t splits = (size_t)ceil_div(D.max_seq, AT_CHUNK);
    if (splits < 64) splits = 64;  // room for the tuning hook
    return (size_t)max_rows * D.H * splits * (D.hd + 4);
}

template <typename KT, int HD, int NQ, int NW, int NL>
static void launch_attn_wide(const Dims& D, const float* q, int ldq, const void* kc, const void* vc, const int* pos_dev,
                             int pos_off, int n_splits, int chunk, int zq, int M, float* part, float* out, uint16_t* out_hi,
                             uint16_t* out_lo, unsigned* arrive, hipStream_t s)
{
    hipLaunchKernelGGL((attn_wide_kernel<KT, HD, NQ, NW, NL>), dim3(n_splits, D.Hkv, zq), dim3(NW * 64), 0, s, q, ldq,
                       (const KT*)kc, (const KT*)vc, pos_dev, pos_off, M, D.H, D.Hkv, D.max_seq, n_splits, chunk, part, out, D.dq,
                       out_hi, out_lo, D.wt == WT_F16, arrive);
}

// LDS-staged kernel: MFMA form for 16-bit caches, plain form for fp32 caches
template <typename KT, int HD>
static void launch_attn_staged(const Dims& D, const float* q, int ldq, const void* kc, const void* vc, const int* pos_dev,
                               int pos_off, int n_splits, int M, float* part, float* out, uint16_t* out_hi, uint16_t* out_lo,
                               unsigned* arrive, hipStream_t s)
{
    {
        // MFMA form: 16-bit caches always; fp32 caches when the model's weights are 16-bit (its hi/lo planes carry 16
        // mantissa bits, the precision the multi-row path of such a model works at anyway; an fp32 model keeps fp32)
        if (!(D.opt && D.opt->attn_kernel == 3) && (sizeof(KT) == 2 || D.wt != WT_F32)) {
            const size_t lds = attn_mfma_lds_bytes<KT, HD>();
            static std::atomic<size_t> lds_limit{0};  // per instantiation
            if (ensure_lds((const void*)attn_mfma_kernel<KT, HD>, lds, lds_limit) != hipSuccess)
                return;   // the launch below then fails and reports
            const int Q = (D.H / D.Hkv) * M;
            hipLaunchKernelGGL((attn_mfma_kernel<KT, HD>), dim3(n_splits, D.Hkv, ceil_div(Q, AT_QPASS)), dim3(AM_THREADS), lds, s, q, ldq,
                               (const KT*)kc, (const KT*)vc, pos_dev, pos_off, M, D.H, D.Hkv, D.max_seq, n_splits, part, out, D.dq,
                               out_hi, out_lo, D.wt == WT_F16, arrive);
            return;
        }
    }
    const size_t lds = attn_lds_bytes<KT, HD>();
    static std::atomic<size_t> lds_limit{0};  // per instantiation
    if (ensure_lds((const void*)attn_kernel<KT, HD>, lds, lds_limit) != hipSuccess) return;
    // groups of 16 query vectors side by side, each staging the chunk for itself (one after the other in a block they took 12 us each)
    hipLaunchKernelGGL((attn_kernel<KT, HD>), dim3(n_splits, D.Hkv, ceil_div((D.H / D.Hkv) * M, AT_QPASS)), dim3(AT_THREADS), lds, s, q, ldq, (const KT*)kc,
                       (const KT*)vc, pos_dev, pos_off, M, D.H, D.Hkv, D.max_seq, n_splits, part, out, D.dq, out_hi, out_lo,
                       D.wt == WT_F16);
}

template <typename KT, int HD>
static hipError_t attention_t(const Dims& D, const float* q, int ldq, const void* kc, const void* vc, const int* pos_dev,
                              int pos_off, AttnPlan pl, int ctx, int M, float* part, float* out, uint16_t* out_hi,
                              uint16_t* out_lo, unsigned* arrive, hipStream_t s)
{
    const int n_splits = pl.n_splits;
    // the matrix-core and the register-resident kernel fold their partials themselves unless another launch does, a counter per group of blocks
    const bool mfma = !pl.wide && !(D.opt && D.opt->attn_kernel == 3) && (sizeof(KT) == 2 || D.wt != WT_F32);
    if (!(mfma || pl.wide) || n_splits == 1 || pl.defer_fold || D.H * M > ATTN_COUNTERS ||
        (size_t)M * D.H * n_splits * (HD + 4) * 4 >= (size_t)1 << 31)
        arrive = nullptr;
    if (n_splits < 1 || (n_splits > 64 && n_splits > ceil_div(D.max_seq, AT_CHUNK))) return hipErrorInvalidValue;
    // prompt passes (more than 16 rows) of models with 16-bit weights: one kernel over the whole causal range, where
    // it has blocks for a quarter of the CUs at least or the range is short (a block walks the range chunk by chunk:
    // 64 rows behind 640 cached positions take 62 us in 32 blocks, 40 us through the split kernel and its fold)
    if (M > 16 && !pl.wide && (sizeof(KT) == 2 || D.wt != WT_F32) && !(D.opt && D.opt->attn_kernel) &&
        (ceil_div((D.H / D.Hkv) * M, AP_Q) * D.Hkv >= 64 || ctx <= 4 * AP_C)) {
        constexpr size_t lds = attn_prompt_lds_bytes<KT, HD>();
        static std::atomic<size_t> lds_limit{0};  // per instantiation
        hipError_t e = ensure_lds((const void*)attn_prompt_kernel<KT, HD>, lds, lds_limit);
        if (e != hipSuccess) return e;
        const int Q = (D.H / D.Hkv) * M;
        hipLaunchKernelGGL((attn_prompt_kernel<KT, HD>), dim3(ceil_div(Q, AP_Q) * D.Hkv), dim3(AP_THREADS), lds, s, q, ldq, (const KT*)kc,
                           (const KT*)vc, pos_dev, pos_off, M, D.H, D.Hkv, D.max_seq, out, D.dq, out_hi, out_lo, D.wt == WT_F16);
        return hipGetLastError();
    }
    if (pl.wide) {
        int Q = (D.H / D.Hkv) * M, zq = 1;
        if (Q > AW_MAXQ_TOTAL) {  // one block per row (its group of heads, or half of a group of 8) and range
            const int G = D.H / D.Hkv;
            Q = G > 4 ? 4 : G;
            zq = M * (G / Q);
        }
        const int span = pl.chunk * (HD / (16 / (int)sizeof(KT)));  // lanes' worth of 16-byte vectors per range
        if (Q == 1 && span <= 8 * 64 * 4) launch_attn_wide<KT, HD, 1, 8, 4>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
        else if (Q == 1 && span <= 16 * 64 * 4) launch_attn_wide<KT, HD, 1, 16, 4>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
        else if (Q == 1) launch_attn_wide<KT, HD, 1, 8, 16>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
        else if (Q == 2) launch_attn_wide<KT, HD, 2, 16, 4>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
        else if (span <= 8 * 64 * 4) launch_attn_wide<KT, HD, 4, 8, 4>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
        else launch_attn_wide<KT, HD, 4, 8, 8>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, pl.chunk, zq, M, part, out, out_hi, out_lo, arrive, s);
    } else {
        launch_attn_staged<KT, HD>(D, q, ldq, kc, vc, pos_dev, pos_off, n_splits, M, part, out, out_hi, out_lo, arrive, s);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_splits == 1 || pl.defer_fold || arrive) return e;
    hipLaunchKernelGGL((attn_combine_kernel<HD>), dim3(ceil_div(M * D.H * (HD / 4), 256)), dim3(256), 0, s, part, M * D.H, n_splits, out, out_hi,
                       out_lo, D.wt == WT_F16);
    return hipGetLastError();
}

hipError_t attention(const Dims& D, const float* q, int ldq, const void* kc, const void* vc, const int* pos_dev,
                     int pos_off, int pos_host_hint, int M, float* part, float* out, uint16_t* out_hi, uint16_t* out_lo,
                     hipStream_t s, int* deferred_splits, unsigned* arrive)
{
    int ctx = pos_host_hint + pos_off + M;  // positions the last row sees
    if (ctx < 1 || ctx > D.max_seq || M < 1) return hipErrorInvalidValue;
    AttnPlan pl = attn_plan(D, ctx, M, arrive != nullptr);
    if (deferred_splits) {  // single row: the consumer (gemv_resid_attn) folds the partials itself
        if (M != 1) return hipErrorInvalidValue;
        pl.defer_fold = pl.n_splits > 1 && pl.n_splits <= GV_FOLD_MAX;
        *deferred_splits = pl.defer_fold ? pl.n_splits : 0;
    }
    if (D.kt == WT_BF16) {
        if (D.hd == 128) return attention_t<uint16_t, 128>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
        if (D.hd == 64) return attention_t<uint16_t, 64>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
    } else if (D.kt == WT_F16) {
        if (D.hd == 128) return attention_t<f16_t, 128>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
        if (D.hd == 64) return attention_t<f16_t, 64>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
    } else {
        if (D.hd == 128) return attention_t<float, 128>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
        if (D.hd == 64) return attention_t<float, 64>(D, q, ldq, kc, vc, pos_dev, pos_off, pl, ctx, M, part, out, out_hi, out_lo, arrive, s);
    }
    return hipErrorInvalidValue;
}

// ---- whole single-row steps of narrow models in one launch ---------------------------------------------------------------
// A layer of a 1024-wide model is 26 MB: its five launches cost their fixed time, not their bytes.  Here the blocks of ONE
// launch, one per CU and all resident, walk the layers.  What bounds it is the hand-over of a stage's output vector to all
// blocks, five per layer, and the arithmetic of the few waves that own rows in between.  Hence:
//  * the vectors travel as 64-bit words (value, tag): a reader polls the data itself until every word carries the tag of the
//    hand-over it waits for, so there is no counter, no second round trip, and nothing has to be reset;
//  * a reader first waits ST_FIRST_POLL: polls that arrive while the words are being written take the line away from the
//    writers again and again.  With the pause a hand-over is 0.8 to 0.9 us, without 2 to 2.6 (step below: 443 -> 351 us);
//  * a block's outputs leave in one store where several waves own them;
//  * the weights do not wait for anything: a wave holds its rows of all of a layer's stages in registers and requests those
//    of the next layer when it no longer needs the present ones and has the input of the stage it is in (loads return in order:
//    requested before a poll they delay it: 351 -> 333 us);
//  * a wave owns whole rows, so that no sum crosses waves; K and V of the cached positions are requested before the query is there.
// Measured, 24 layers of 1024 (FFN 2816), 300 positions, 32000-row LM head: 620 us with a launch per matrix, 333 so.
// Every wait is bounded (wait_ticks of the 100 MHz clock): when blocks are not all resident -- another stream or process holds
// CUs for that long -- the launch drains, the error flag tells the host, and the step is run again by the launches per matrix.
// Tags are 32 bits of a running number and could only be mistaken after 2^32 hand-overs without a write to the word.
constexpr int ST_THREADS = ST_WAVES * 64;
constexpr int ST_FIRST_POLL = 18;         // x 64 clocks (10: 344 us, 13: 340, 16: 333 to 335, 19: 333, 22: 334)

struct StepP {
    const StepWeights* layers; int L;
    uint64_t mask[2];           // bit l: layer l is executed
    const void* lm_head; const float* final_norm;
    const float* x; const float* rope_row; const int* pos_dev; int pos_off;
    char* kv; size_t kv_layer;  // cache, bytes of K (or V) of one layer
    float* logits; float* vstat; float clamp;
    unsigned long long* mail; StepMail off;
    int d, dq, dkv, f, V, H, Hkv, max_seq; float eps;
    int n_splits, chunk;
    long wait_ticks;
};

__device__ __forceinline__ void mail_put(unsigned long long* p, float v, unsigned tag)
{
    __hip_atomic_store(p, ((unsigned long long)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until the word pairs at pair[0..N) below n_pairs all carry `tag` (those at n_pairs and above count as there); v
// receives their values.  Called by whole waves.  A word is written by one 8-byte store, so the halves of a 16-byte load are
// each whole.
template <int N>
__device__ __forceinline__ void mail_take(const int (&pair)[N], float2 (&v)[N], unsigned long long* base, int n_pairs, unsigned tag, unsigned* ctrl,
                                          bool& alive, long wait_ticks, bool pause = true)
{
    const auto r = __builtin_amdgcn_make_buffer_rsrc(base, 0, n_pairs * 16, 0x00020000);
    u32x4_t w[N];
    int spins = 0;
    long t0 = 0;
    if (pause) __builtin_amdgcn_s_sleep(ST_FIRST_POLL);
    while (true) {
        bool ok = true;
        asm volatile("" ::: "memory");   // the words change under the loop
#pragma unroll
        for (int u = 0; u < N; u++) w[u] = __builtin_amdgcn_raw_buffer_load_b128(r, pair[u] * 16, 0, 16 /* sc1: device scope */);
#pragma unroll
        for (int u = 0; u < N; u++) ok = ok && ((w[u].y == tag && w[u].w == tag) || pair[u] >= n_pairs);
        if (__all(ok) || !alive) break;
        if ((++spins & 63) == 0) {
            const long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (__hip_atomic_load(ctrl + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) alive = false;
            else if (now - t0 > wait_ticks) {
                __hip_atomic_store(ctrl + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                alive = false;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < N; u++) v[u] = make_float2(__uint_as_float(w[u].x), __uint_as_float(w[u].z));
}
// next set bit of a 128-bit mask (low, high word) at l or above, -1 if there is none
__device__ __forceinline__ int next_layer(uint64_t lo, uint64_t hi, int l)
{
    if (l < 64) {
        const unsigned long long b = lo >> l << l;
        if (b) return __ffsll(b) - 1;
        l = 64;
    }
    const unsigned long long b = l < 128 ? hi >> (l - 64) << (l - 64) : 0;
    return b ? 63 + __ffsll(b) : -1;
}
// the same over the segments of LPP lanes of a wave, for values that are uniform inside each segment or belong to its lanes
template <int LPP> __device__ __forceinline__ float seg_sum_fast(float v)
{
    if (LPP == 8) v = dpp_add<0x128>(v);    // the other half of the row
    if (LPP <= 16) return rows_swap_sum(v);
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int LPP> __device__ __forceinline__ float seg_max_fast(float v)
{
    if (LPP == 8) v = dpp_max<0x128>(v);
    if (LPP <= 16) return rows_swap_max(v);
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <typename WT, typename KT, int HD, bool LACK = false>
__global__ __launch_bounds__(ST_THREADS) void step_kernel(StepP p)
{
    constexpr int VEC = Elem<WT>::VEC, CH = 64 * VEC, CD = ST_CD, CF = ST_CF, XF = CF * CH;
    constexpr int EPV = 16 / (int)sizeof(KT), LPP = HD / EPV, PPL = 64 / LPP, NL = 4, PASS = NL * ST_WAVES * PPL;
    constexpr int NX = (CD * CH + 2 * ST_THREADS - 1) / (2 * ST_THREADS), NF = (XF + 2 * ST_THREADS - 1) / (2 * ST_THREADS);   // pairs of elements of a d- or dq-, of an f-vector per thread
    extern __shared__ __align__(16) float st_sm[];
    float* xs = st_sm;                                                   // [2][XF] input vector of a stage, alternating
    const unsigned long long* tab = reinterpret_cast<const unsigned long long*>(st_sm + 2 * XF);   // weight pointers [L][9]
    __shared__ float red[2][ST_WAVES];
    __shared__ float rope[HD];
    __shared__ __align__(16) float qs[3 * HD];                           // query (scaled), new key and value of the head
    __shared__ float outs[2 * ST_WAVES];                                 // outputs of the block's rows, handed over by one store
    __shared__ float wacc[ST_WAVES * HD], wml[ST_WAVES * 2];
    // What depends on the lane is worked out anew in every stage (fresh): kept over the layers it would not fit beside the
    // weights and go to scratch memory.
    int tid = threadIdx.x, lane = tid & 63;
    auto fresh = [&]() { asm volatile("" : "+v"(tid)); lane = tid & 63; };
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x, NB = gridDim.x;
    if (LACK && b + 1 == NB) return;   // (a test's launch: the others wait in vain.  As a run-time switch it cost a step 0.8 %)
    const int d = p.d, dq = p.dq, dkv = p.dkv, f = p.f;
    unsigned* ctrl = reinterpret_cast<unsigned*>(p.mail);
    unsigned long long* const mx = p.mail + p.off.x;
    unsigned long long* const mqkv = p.mail + p.off.qkv;
    unsigned long long* const mpart = p.mail + p.off.part;
    unsigned long long* const mact = p.mail + p.off.act;

    {
        unsigned long long* t = reinterpret_cast<unsigned long long*>(st_sm + 2 * XF);
        const unsigned long long* src = reinterpret_cast<const unsigned long long*>(p.layers);
        for (int i = tid; i < p.L * 9; i += ST_THREADS) t[i] = src[i];
        if (tid < HD) rope[tid] = p.rope_row[tid];
    }
    unsigned tag = ctrl[0];
    bool alive = ctrl[1] == 0;                  // an earlier launch of the sequence has given up: drain
    const int p0 = p.pos_dev[0] + p.pos_off;
    // what this block and wave own: rows of the residual stream, pairs of q / k / v rows, gate / up pairs, pairs of LM-head rows
    const int xr0 = step_begin(d, b, NB) + wave;
    const bool has_x = xr0 < step_begin(d, b + 1, NB);
    const int nqp = (dq + 2 * dkv) / 2;
    const int qp = step_begin(nqp, b, NB) + wave;
    const bool has_q = qp < step_begin(nqp, b + 1, NB);
    const int gp0 = step_begin(f, b, NB) + wave, gp_end = step_begin(f, b + 1, NB);
    const int lp_end = step_begin(p.V / 2, b + 1, NB), lp0 = step_begin(p.V / 2, b, NB) + wave;
    // rows of the q / k / v pair: the two rows of a rotary pair, or consecutive rows of v
    auto qkv_rows = [&](int pair, int& m, int& r0, int& r1) {
        const int j = 2 * pair;
        if (j < dq + dkv) {
            m = j < dq ? 0 : 1;
            const int jj = m ? j - dq : j, head = jj / HD, i = (jj % HD) >> 1;
            r0 = head * HD + i; r1 = r0 + HD / 2;
        } else {
            m = 2; r0 = j - dq - dkv; r1 = r0 + 1;
        }
    };
    int qm, qr0, qr1;
    qkv_rows(qp, qm, qr0, qr1);
    float xr = has_x ? p.x[xr0] : 0.f;          // residual value of this wave's row
    __syncthreads();

    auto ptr = [&](int l, int which) -> const char* {   // uniform: scalar registers
        const unsigned long long v = tab[l * 9 + which];
        return reinterpret_cast<const char*>(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                                             (unsigned)__builtin_amdgcn_readfirstlane((int)v));
    };
    enum { P_AN = 0, P_Q, P_K, P_V, P_O, P_MN, P_G, P_U, P_D };
    // Weights of the next executed layer.  Loads are unconditional, through a buffer descriptor that is empty where there is
    // nothing to load (such lanes get zeros and cost no memory request): behind a branch the compiler merges old and new
    // registers by copies, which wait for the loads just issued (1 to 3 us per stage).
    u32x4_t bq[2][CD], bo[CD], bg[ST_GU][2][CD], bd[CF];
    auto row_load = [&](u32x4_t* w, int C, const char* m, size_t row, int K, bool ok) {
        auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(m) + row * K * sizeof(WT), 0, ok ? K * (int)sizeof(WT) : 0, 0x00020000);
#pragma unroll
        for (int c = 0; c < CF; c++)
            if (c < C) w[c] = __builtin_amdgcn_raw_buffer_load_b128(r, (c * CH + lane * VEC) * (int)sizeof(WT), 0, 2 /* nt */);
    };
    auto lm_load = [&](u32x4_t (*w)[CD], int pair) {
        row_load(w[0], CD, static_cast<const char*>(p.lm_head), (size_t)pair * 2, d, pair < lp_end);
        row_load(w[1], CD, static_cast<const char*>(p.lm_head), (size_t)pair * 2 + 1, d, pair < lp_end);
    };
    float2 gq[NX], gg[NX];                      // norm gains of this thread's elements: next attention sub-block (or LM head), next MLP
    auto xe = [&](int u) { return min(2 * (u * ST_THREADS + tid), d - 2); };
    auto gain = [&](float2 (&o)[NX], const char* g) {
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(g), 0, d * 4, 0x00020000);
#pragma unroll
        for (int u = 0; u < NX; u++) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(r, (u * ST_THREADS + tid) * 8, 0, 0);
            o[u] = make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
        }
    };
    auto load_qkv = [&](int l) {                // of layer l, or, l < 0, the first pair of LM-head rows
        const int t = max(l, 0);
        const char* m = l < 0 ? static_cast<const char*>(p.lm_head) : ptr(t, P_Q + qm);
        const bool ok = l < 0 ? lp0 < lp_end : has_q;
        row_load(bq[0], CD, m, l < 0 ? (size_t)lp0 * 2 : (size_t)qr0, d, ok);
        row_load(bq[1], CD, m, l < 0 ? (size_t)lp0 * 2 + 1 : (size_t)qr1, d, ok);
        gain(gq, l < 0 ? reinterpret_cast<const char*>(p.final_norm) : ptr(t, P_AN));
    };
    auto load_o = [&](int l) { row_load(bo, CD, ptr(max(l, 0), P_O), xr0, dq, l >= 0 && has_x); };
    auto load_gu = [&](int l) {                 // or the next pairs of LM-head rows
        const int t = max(l, 0);
        const char* lh = static_cast<const char*>(p.lm_head);
        const char* wg = l < 0 ? lh : ptr(t, P_G);
        const char* wu = l < 0 ? lh : ptr(t, P_U);
#pragma unroll
        for (int u = 0; u < ST_GU; u++) {
            const int pair = lp0 + (u + 1) * ST_WAVES, gp = gp0 + u * ST_WAVES;
            const bool ok = l < 0 ? pair < lp_end : gp < gp_end;
            row_load(bg[u][0], CD, wg, l < 0 ? (size_t)pair * 2 : (size_t)gp, d, ok);
            row_load(bg[u][1], CD, wu, l < 0 ? (size_t)pair * 2 + 1 : (size_t)gp, d, ok);
        }
        gain(gg, ptr(t, P_MN));
    };
    auto load_d = [&](int l) { row_load(bd, CF, ptr(max(l, 0), P_D), xr0, f, l >= 0 && has_x); };

    auto mail_wait = [&](const auto& pair, auto& v, unsigned long long* base, int n_pairs) {
        mail_take(pair, v, base, n_pairs, tag, ctrl, alive, p.wait_ticks);
    };

    int buf = 0, xpar = 0;
    bool first = true;                          // the residual stream is still the embedding row in memory
    // residual stream into LDS, times the gain; returns the RMS scale
    auto take_x = [&](const float2 (&gain)[NX]) -> float {
        fresh();
        float2 v[NX];
        if (first) {
#pragma unroll
            for (int u = 0; u < NX; u++) v[u] = *reinterpret_cast<const float2*>(p.x + xe(u));
        } else {
            int pr[NX];
#pragma unroll
            for (int u = 0; u < NX; u++) pr[u] = u * ST_THREADS + tid;
            mail_wait(pr, v, mx + (size_t)xpar * d, d / 2);
        }
        buf ^= 1;
        float ss = 0.f;
#pragma unroll
        for (int u = 0; u < NX; u++) {
            const int i = 2 * (u * ST_THREADS + tid);
            if (i < d) {
                *reinterpret_cast<float2*>(xs + buf * XF + gv_xpos<VEC>(i)) = make_float2(v[u].x * gain[u].x, v[u].y * gain[u].y);
                ss += v[u].x * v[u].x + v[u].y * v[u].y;
            }
        }
        ss = wave_sum_fast(ss);
        if (lane == 0) red[buf][wave] = ss;
        lds_barrier();
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < ST_WAVES; i++) t += red[buf][i];
        return 1.0f / sqrtf(t / (float)d + p.eps);
    };
    auto dot = [&](const u32x4_t* w, int C, int K) -> float {
        const float* x = xs + buf * XF + lane * (VEC == 8 ? 4 : VEC);
        float a = 0.f;
#pragma unroll
        for (int c = 0; c < CF; c++)
            if (c < C && c * CH + lane * VEC < K) a = gv_dot<WT>(w[c], x + c * CH, a);
        return wave_sum_fast(a);
    };
    // the block's share of the residual stream to everybody
    auto give_x = [&]() {
        tag++; xpar ^= 1; first = false;
        if (lane == 0) outs[wave] = xr;
        lds_barrier();
        const int x0 = step_begin(d, b, NB), i = tid;
        if (i < step_begin(d, b + 1, NB) - x0) mail_put(mx + (size_t)xpar * d + x0 + i, outs[i], tag);
    };

    int ln = next_layer(p.mask[0], p.mask[1], 0);
    load_qkv(ln); load_o(ln); load_gu(ln); load_d(ln);
    while (ln >= 0) {
        const int l = ln;
        ln = next_layer(p.mask[0], p.mask[1], l + 1);
        KT* kc = reinterpret_cast<KT*>(p.kv + (size_t)(2 * l) * p.kv_layer);
        KT* vc = reinterpret_cast<KT*>(p.kv + (size_t)(2 * l + 1) * p.kv_layer);
        // ---- q, k, v ----
        {
            const float sc = take_x(gq);
            tag++;
            if (has_q) {
                const float a = dot(bq[0], CD, d) * sc, c = dot(bq[1], CD, d) * sc;
                float o0 = a, o1 = c;
                if (qm < 2) {
                    const int i = qr0 % HD;
                    const float cs = rope[2 * i], sn = rope[2 * i + 1];
                    o0 = a * cs - c * sn; o1 = c * cs + a * sn;
                }
                if (lane < 2) {
                    float o = lane == 0 ? o0 : o1;
                    if (qm > 0) {
                        const int r = lane == 0 ? qr0 : qr1;
                        KT* row = (qm == 1 ? kc : vc) + ((size_t)(r / HD) * p.max_seq + p0) * HD;
                        Elem<KT>::put(row, r % HD, o);
                        if (sizeof(KT) == 2) { KT t; Elem<KT>::put(&t, 0, o); o = Elem<KT>::get(&t, 0); }   // attention sees what the cache holds
                    }
                    outs[lane * ST_WAVES + wave] = o;
                }
            }
            lds_barrier();
            if (wave == 0 && lane < 2 * ST_WAVES) {   // lane: pair lane % ST_WAVES of the block, its row lane / ST_WAVES
                const int pr = step_begin(nqp, b, NB) + lane % ST_WAVES;
                int m, r0, r1;
                qkv_rows(pr, m, r0, r1);
                if (pr < step_begin(nqp, b + 1, NB))
                    mail_put(mqkv + (m == 0 ? 0 : m == 1 ? dq : dq + dkv) + (lane < ST_WAVES ? r0 : r1), outs[lane], tag);
            }
        }
        // ---- attention: one block per query head and range of positions ----
        if (b < p.H * p.n_splits) {
            fresh();
            const int head = b / p.n_splits, split = b % p.n_splits, kvh = head / (p.H / p.Hkv);
            const int j0 = split * p.chunk, jlast = min(j0 + p.chunk, p.max_seq) - 1;
            const int n = min(p.chunk, p0 + 1 - j0);   // may be <= 0
            const int n_pass = n > 0 ? (n + PASS - 1) / PASS : 0;
            const bool has_cur = n > 0 && j0 + n == p0 + 1;
            const int seg = lane / LPP, sl = (lane % LPP) * EPV;
            const KT* kb = kc + (size_t)kvh * p.max_seq * HD + sl;
            const KT* vb = vc + (size_t)kvh * p.max_seq * HD + sl;
            u32x4_t kr[NL], vr[NL];
            auto issue = [&](int pass) {
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = min(j0 + ((pass * NL + t) * ST_WAVES + wave) * PPL + seg, jlast);
                    kr[t] = *reinterpret_cast<const u32x4_t*>(kb + (size_t)j * HD);
                    vr[t] = *reinterpret_cast<const u32x4_t*>(vb + (size_t)j * HD);
                }
            };
            issue(0);
            if (wave < 3 && (wave == 0 || has_cur)) {   // wave 0: the query, waves 1 and 2: the position's key and value
                const int pr[1] = {(wave == 0 ? head * HD : dq + (wave - 1) * dkv + kvh * HD) / 2 + min(lane, HD / 2 - 1)};
                const float sc = wave == 0 ? 1.0f / sqrtf((float)HD) : 1.0f;
                float2 v[1];
                mail_wait(pr, v, mqkv, (dq + 2 * dkv) / 2);
                if (lane < HD / 2) *reinterpret_cast<float2*>(qs + wave * HD + 2 * lane) = make_float2(v[0].x * sc, v[0].y * sc);
            }
            lds_barrier();
            float m = -INFINITY, lsum = 0.f, acc[EPV];
#pragma unroll
            for (int u = 0; u < EPV; u++) acc[u] = 0.f;
            for (int pass = 0; pass < n_pass; pass++) {
                if (pass) issue(pass);
                float s[NL];
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = j0 + ((pass * NL + t) * ST_WAVES + wave) * PPL + seg;
                    float kf[EPV];
                    aw_unpack<KT>(kr[t], kf);
                    if (has_cur && j == p0) {
#pragma unroll
                        for (int u = 0; u < EPV; u++) kf[u] = qs[HD + sl + u];
                    }
                    float a = 0.f;
#pragma unroll
                    for (int u = 0; u < EPV; u++) a = fmaf(kf[u], qs[sl + u], a);
                    a = aw_seg_sum<LPP>(a);
                    s[t] = j <= p0 && j < j0 + n ? a : -INFINITY;
                }
                float mt = s[0];
#pragma unroll
                for (int t = 1; t < NL; t++) mt = fmaxf(mt, s[t]);
                mt = seg_max_fast<LPP>(mt);
                const float mn = fmaxf(m, mt);
                const bool live = mn > -INFINITY;
                const float c = live ? __expf(m - mn) : 1.0f;
                lsum *= c;
#pragma unroll
                for (int u = 0; u < EPV; u++) acc[u] *= c;
                m = mn;
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = j0 + ((pass * NL + t) * ST_WAVES + wave) * PPL + seg;
                    const float e = live ? __expf(s[t] - mn) : 0.f;
                    lsum += e;
                    float vf[EPV];
                    aw_unpack<KT>(j < j0 + n ? vr[t] : u32x4_t{0u, 0u, 0u, 0u}, vf);   // rows past the position may hold anything
                    if (has_cur && j == p0) {
#pragma unroll
                        for (int u = 0; u < EPV; u++) vf[u] = qs[2 * HD + sl + u];
                    }
#pragma unroll
                    for (int u = 0; u < EPV; u++) acc[u] = fmaf(e, vf[u], acc[u]);
                }
            }
            lsum = seg_sum_fast<LPP>(lsum);
#pragma unroll
            for (int u = 0; u < EPV; u++) {
                acc[u] = seg_sum_fast<LPP>(acc[u]);
                if (seg == 0) wacc[wave * HD + sl + u] = acc[u];
            }
            if (lane == 0) { wml[wave * 2] = m; wml[wave * 2 + 1] = lsum; }
            lds_barrier();
            if (tid < HD) {
                float gm = -INFINITY, num = 0.f, den = 0.f;
#pragma unroll
                for (int w = 0; w < ST_WAVES; w++) gm = fmaxf(gm, wml[w * 2]);
#pragma unroll
                for (int w = 0; w < ST_WAVES; w++) {
                    const float mw = wml[w * 2], c = mw > -INFINITY ? __expf(mw - gm) : 0.f;
                    num = fmaf(c, wacc[w * HD + tid], num);
                    den = fmaf(c, wml[w * 2 + 1], den);
                }
                unsigned long long* o = mpart + (size_t)b * (HD + 2);
                mail_put(o + tid, num, tag + 1);
                if (tid < 2) mail_put(o + HD + tid, tid == 0 ? gm : den, tag + 1);
            }
        }
        // ---- output projection: its input is the fold of the heads' partials ----
        {
            fresh();
            tag++;
            const int ns = p.n_splits, np = p.H * ns * (HD / 2 + 1);
            float gm[NX], den[NX];
            float2 num[NX];
#pragma unroll
            for (int x = 0; x < NX; x++) { gm[x] = -INFINITY; den[x] = 0.f; num[x] = make_float2(0.f, 0.f); }
            for (int s0 = 0; s0 < ns; s0 += 4) {
                int pr[8 * NX];
                float2 v[8 * NX];   // per split: two elements of the output, (maximum, sum)
#pragma unroll
                for (int x = 0; x < NX; x++) {
                    const int e = 2 * (x * ST_THREADS + tid);
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        const int r = e < dq && s0 + u < ns ? ((e / HD) * ns + s0 + u) * (HD / 2 + 1) : np;   // np: nothing to wait for
                        pr[8 * x + 2 * u] = r + (e % HD) / 2; pr[8 * x + 2 * u + 1] = r + HD / 2;
                    }
                }
                mail_wait(pr, v, mpart, np);
#pragma unroll
                for (int x = 0; x < NX; x++) {
                    const float2* w = v + 8 * x;
                    float mn = gm[x];
#pragma unroll
                    for (int u = 0; u < 4; u++) mn = s0 + u < ns ? fmaxf(mn, w[2 * u + 1].x) : mn;
                    const float c = gm[x] > -INFINITY ? __expf(gm[x] - mn) : 0.f;
                    num[x].x *= c; num[x].y *= c; den[x] *= c;
                    gm[x] = mn;
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        const float q = s0 + u < ns && w[2 * u + 1].y > 0.f ? __expf(w[2 * u + 1].x - mn) : 0.f;
                        num[x].x = fmaf(q, w[2 * u].x, num[x].x); num[x].y = fmaf(q, w[2 * u].y, num[x].y);
                        den[x] = fmaf(q, w[2 * u + 1].y, den[x]);
                    }
                }
            }
            load_qkv(ln);
            buf ^= 1;
#pragma unroll
            for (int x = 0; x < NX; x++) {
                const int i = 2 * (x * ST_THREADS + tid);
                if (i < dq) *reinterpret_cast<float2*>(xs + buf * XF + gv_xpos<VEC>(i)) = make_float2(num[x].x / den[x], num[x].y / den[x]);
            }
            lds_barrier();
            if (has_x) xr += dot(bo, CD, dq);
            give_x();
            fresh();
            load_o(ln);
        }
        // ---- gate and up ----
        {
            const float sc = take_x(gg);
            tag++;
#pragma unroll
            for (int u = 0; u < ST_GU; u++) {
                const int gp = gp0 + u * ST_WAVES;
                if (gp < gp_end) {
                    const float a = dot(bg[u][0], CD, d) * sc, c = dot(bg[u][1], CD, d) * sc;
                    if (lane == 0) outs[u * ST_WAVES + wave] = a / (1.0f + __expf(-a)) * c;
                }
            }
            lds_barrier();
            if (wave == 0 && lane < gp_end - gp0) mail_put(mact + gp0 + lane, outs[lane], tag);
        }
        // ---- down projection ----
        {
            fresh();
            int pr[NF];
            float2 v[NF];
#pragma unroll
            for (int u = 0; u < NF; u++) pr[u] = u * ST_THREADS + tid;
            mail_wait(pr, v, mact, f / 2);
            load_gu(ln);
            buf ^= 1;
#pragma unroll
            for (int u = 0; u < NF; u++) {
                const int i = 2 * (u * ST_THREADS + tid);
                if (i < f) *reinterpret_cast<float2*>(xs + buf * XF + gv_xpos<VEC>(i)) = v[u];
            }
            lds_barrier();
            if (has_x) xr += dot(bd, CF, f);
            give_x();
            fresh();
            load_d(ln);
        }
    }
    // ---- LM head: the first three row pairs of every wave are in registers, a used one is replaced by the third next ----
    const float sc = take_x(gq);
    VStat vs = {-INFINITY, 0.f, 0x7fffffff};
    auto lm_rows = [&](const u32x4_t (*w)[CD], int pair) {
        const float a = dot(w[0], CD, d) * sc, c = dot(w[1], CD, d) * sc;
        if (lane == 0) *reinterpret_cast<float2*>(p.logits + (size_t)pair * 2) = make_float2(a, c);
        vstat_add(vs, fminf(fmaxf(a, -p.clamp), p.clamp), pair * 2);
        vstat_add(vs, fminf(fmaxf(c, -p.clamp), p.clamp), pair * 2 + 1);
    };
    constexpr int LR = (1 + ST_GU) * ST_WAVES;   // pairs that the block's registers hold
    for (int i = lp0; i < lp_end; i += LR) {
        lm_rows(bq, i);
        lm_load(bq, i + LR);
#pragma unroll
        for (int u = 0; u < ST_GU; u++) {
            const int j = i + (u + 1) * ST_WAVES;
            if (j < lp_end) lm_rows(bg[u], j);
            lm_load(bg[u], j + LR);
        }
    }
    __shared__ VStat vred[ST_WAVES];
    if (lane == 0) vred[wave] = vs;
    lds_barrier();
    if (tid == 0) {
        VStat a = vred[0];
#pragma unroll
        for (int w = 1; w < ST_WAVES; w++) vstat_merge(a, vred[w]);
        p.vstat[b * 3] = a.m; p.vstat[b * 3 + 1] = a.z; p.vstat[b * 3 + 2] = __int_as_float(a.arg);
    }
}

// ---- whole verifications of narrow models in one launch -------------------------------------------------------------------
// The step above for the k + 1 rows of a verification, and for the same reason: the six launches of a layer of 26 MB take 35 us
// (5 rows, the gaps between them not counted), most of it their fixed time.  Same blocks, same owners, same hand-overs; what is different:
//  * every word exists once per row, so a hand-over moves R times the bytes (5 rows of 2816 activations: 28 MB over all blocks);
//  * a wave multiplies its weights with all rows: a vector of activations is read from LDS once for all the weight rows a wave
//    owns in a stage, and R (3, 5 or 9: the smallest that holds the rows) is part of the kernel so that these reads are
//    independent; rows past M are zeros that nobody hands over;
//  * attention is one block per head and row over all positions, without partials: a fold would be another hand-over, of more
//    bytes.  The position's own K and V and those of the rows before it come by hand-over, the earlier ones from the cache.
//    They are requested behind the block's own q, k and v: in front of its products they delay the words it hands over
//    (8 layers: 179 -> 185 us);
//  * a lane finishes one row's sum (wave_sums): reduced one by one, the sums of a stage and what is done with them took longer
//    than the products.
// fp32 arithmetic throughout.  Measured, 5 rows, embedding and arg-max launches not counted: 8 layers of 1024 (FFN 2816, 32000-row
// LM head) at 200 to 260 positions: 300 us with a launch per matrix, 207 with every sum reduced by itself, 179, now 175;
// 4 layers of 256 in fp32: 112, 84, 67, 64.  A layer of the former spends 1.8 us waiting for the residual rows, twice, 1 for q, k, v,
// 2 for attention's output and 4 for the activations (112 KB per block: what a CU pulls in 2 us), and 8 on arithmetic.
struct RowsStepP {
    const StepWeights* layers; int L, M;
    const void* lm_head; const float* final_norm;
    const float* x; const float* rope; const int* pos_dev;
    char* kv; size_t kv_layer;  // cache, bytes of K (or V) of one layer
    float* logits; float* taps; size_t tap_ld; float2* vmax; float clamp;
    unsigned* ctrl; unsigned long long* mail; RowsMail off;
    int d, dq, dkv, f, V, H, Hkv, max_seq; float eps;
    long wait_ticks;
};

// o[j][r] = this lane's part of weight row j (C vectors) . row r in LDS
template <typename WT, int J, int C, int R>
__device__ __forceinline__ void rows_dots(const u32x4_t (&w)[J][C], const float* xs, int lane, int K, float (&o)[J][R])
{
    constexpr int VEC = Elem<WT>::VEC, CH = 64 * VEC, XF = ST_CF * CH;
#pragma unroll
    for (int j = 0; j < J; j++)
#pragma unroll
        for (int r = 0; r < R; r++) o[j][r] = 0.f;
#pragma unroll
    for (int c = 0; c < C; c++) {
        if (c * CH + lane * VEC < K) {
            float wf[J][VEC];
#pragma unroll
            for (int j = 0; j < J; j++) aw_unpack<WT>(w[j][c], wf[j]);
#pragma unroll
            for (int r = 0; r < R; r++) {
                const float* x = xs + r * XF + c * CH + lane * 4;
                float xv[8];
                *reinterpret_cast<float4*>(xv) = *reinterpret_cast<const float4*>(x);
                if (VEC == 8) *reinterpret_cast<float4*>(xv + 4) = *reinterpret_cast<const float4*>(x + GV_XB);
#pragma unroll
                for (int j = 0; j < J; j++)
#pragma unroll
                    for (int e = 0; e < VEC; e++) o[j][r] = fmaf(wf[j][e], xv[e], o[j][r]);
            }
        }
    }
}

// Sums of N values over the wave; sum v is returned in the lane whose wave_slot is v.  Four values share a register after two
// exchanges, so that the adds inside the rows of 16 lanes are done once for all four: 11 instructions instead of 40.
__device__ __forceinline__ int wave_slot(int lane) { return 4 * (lane & 15) + (lane >> 4); }
template <int N>
__device__ __forceinline__ float wave_sums(const float (&v)[N], int lane)
{
    static_assert(N <= 64, "one lane per sum");
    float out = 0.f;
#pragma unroll
    for (int q = 0; q < (N + 3) / 4; q++) {
        auto at = [&](int i) { return i < N ? __float_as_uint(v[i < N ? i : 0]) : 0u; };
        auto a = __builtin_amdgcn_permlane32_swap(at(4 * q), at(4 * q + 2), false, false);         // halves: 4q, 4q + 2
        auto b = __builtin_amdgcn_permlane32_swap(at(4 * q + 1), at(4 * q + 3), false, false);     // 4q + 1, 4q + 3
        const float x = __uint_as_float(a[0]) + __uint_as_float(a[1]), y = __uint_as_float(b[0]) + __uint_as_float(b[1]);
        auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);   // rows: 4q .. 4q + 3
        const float z = row16_sum(__uint_as_float(c[0]) + __uint_as_float(c[1]));
        out = q == 0 || (lane & 15) == q ? z : out;
    }
    return out;
}

template <typename WT, typename KT, int HD, int R, bool LACK = false>
__global__ __launch_bounds__(ST_THREADS) void rows_step_kernel(RowsStepP p)
{
    constexpr int VEC = Elem<WT>::VEC, CH = 64 * VEC, CD = ST_CD, CF = ST_CF, XF = CF * CH;
    constexpr int EPV = 16 / (int)sizeof(KT), LPP = HD / EPV, PPL = 64 / LPP, NL = 4, PASS = NL * ST_WAVES * PPL;
    constexpr int NX = (CD * CH + 2 * ST_THREADS - 1) / (2 * ST_THREADS), NF = (XF + 2 * ST_THREADS - 1) / (2 * ST_THREADS);   // pairs of elements of a d- or dq-, of an f-vector per thread
    constexpr int NQ = ((2 * R + 1) * HD / 2 + ST_THREADS - 1) / ST_THREADS;
    extern __shared__ __align__(16) float st_sm[];
    float* xs = st_sm;                                                   // [R][XF] input rows of a stage
    const unsigned long long* tab = reinterpret_cast<const unsigned long long*>(st_sm + R * XF);   // weight pointers [L][9]
    __shared__ float red[R * ST_WAVES];
    __shared__ float rope[R * HD];
    __shared__ __align__(16) float qs[(2 * R + 1) * HD];                 // query (scaled), new keys, new values of the head
    __shared__ float outs[2 * ST_WAVES * R];                             // outputs of the block, [unit][row]
    __shared__ float wacc[ST_WAVES * HD], wml[ST_WAVES * 2];
    static_assert(ST_GU <= 2 && 2 * ST_WAVES * R <= ST_THREADS, "one thread per output");
    int tid = threadIdx.x, lane = tid & 63;
    auto fresh = [&]() { asm volatile("" : "+v"(tid)); lane = tid & 63; };   // as above
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x, NB = gridDim.x;
    if (LACK && b + 1 == NB) return;
    const int d = p.d, dq = p.dq, dkv = p.dkv, f = p.f, M = p.M, nqkv = dq + 2 * dkv;
    unsigned* ctrl = p.ctrl;
    unsigned long long* const mx = p.mail + p.off.x;
    unsigned long long* const mqkv = p.mail + p.off.qkv;
    unsigned long long* const matt = p.mail + p.off.att;
    unsigned long long* const mact = p.mail + p.off.act;

    const int p0 = p.pos_dev[0];
    {
        unsigned long long* t = reinterpret_cast<unsigned long long*>(st_sm + R * XF);
        const unsigned long long* src = reinterpret_cast<const unsigned long long*>(p.layers);
        for (int i = tid; i < p.L * 9; i += ST_THREADS) t[i] = src[i];
        for (int i = tid; i < M * HD; i += ST_THREADS) rope[i] = p.rope[(size_t)p0 * HD + i];
    }
    unsigned tag = ctrl[0];
    bool alive = ctrl[1] == 0;
    // what this block and wave own, as above
    const int xb0 = step_begin(d, b, NB), xb1 = step_begin(d, b + 1, NB), xr0 = xb0 + wave;
    const bool has_x = xr0 < xb1;
    const int nqp = nqkv / 2;
    const int qp = step_begin(nqp, b, NB) + wave;
    const bool has_q = qp < step_begin(nqp, b + 1, NB);
    const int gb0 = step_begin(f, b, NB), gp0 = gb0 + wave, gp_end = step_begin(f, b + 1, NB);
    const int lp_end = step_begin(p.V / 2, b + 1, NB), lp0 = step_begin(p.V / 2, b, NB) + wave;
    auto qkv_rows = [&](int pair, int& m, int& r0, int& r1) {
        const int j = 2 * pair;
        if (j < dq + dkv) {
            m = j < dq ? 0 : 1;
            const int jj = m ? j - dq : j, head = jj / HD, i = (jj % HD) >> 1;
            r0 = head * HD + i; r1 = r0 + HD / 2;
        } else {
            m = 2; r0 = j - dq - dkv; r1 = r0 + 1;
        }
    };
    int qm, qr0, qr1;
    qkv_rows(qp, qm, qr0, qr1);
    float xr = has_x && wave_slot(lane) < M ? p.x[(size_t)wave_slot(lane) * d + xr0] : 0.f;   // of this wave's row: lane of slot r, residual row r
    __syncthreads();

    auto ptr = [&](int l, int which) -> const char* {   // uniform: scalar registers
        const unsigned long long v = tab[l * 9 + which];
        return reinterpret_cast<const char*>(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                                             (unsigned)__builtin_amdgcn_readfirstlane((int)v));
    };
    enum { P_AN = 0, P_Q, P_K, P_V, P_O, P_MN, P_G, P_U, P_D };
    // weights of the next layer: loads are unconditional, as above
    u32x4_t bq[2][CD], bo[1][CD], bg[2 * ST_GU][CD], bd[1][CF];   // bg: gate, up, gate, up
    auto row_load = [&](u32x4_t* w, int C, const char* m, size_t row, int K, bool ok) {
        auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(m) + row * K * sizeof(WT), 0, ok ? K * (int)sizeof(WT) : 0, 0x00020000);
#pragma unroll
        for (int c = 0; c < CF; c++)
            if (c < C) w[c] = __builtin_amdgcn_raw_buffer_load_b128(r, (c * CH + lane * VEC) * (int)sizeof(WT), 0, 2 /* nt */);
    };
    float2 gq[NX], gg[NX];                      // norm gains of this thread's elements
    auto gain = [&](float2 (&o)[NX], const char* g) {
        const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(g), 0, d * 4, 0x00020000);
#pragma unroll
        for (int u = 0; u < NX; u++) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(r, (u * ST_THREADS + tid) * 8, 0, 0);
            o[u] = make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
        }
    };
    const char* const lh = static_cast<const char*>(p.lm_head);
    auto load_qkv = [&](int l) {                // of layer l, or, l == L, the first pair of LM-head rows
        const bool lm = l >= p.L;
        const char* m = lm ? lh : ptr(l, P_Q + qm);
        const bool ok = lm ? lp0 < lp_end : has_q;
        row_load(bq[0], CD, m, lm ? (size_t)lp0 * 2 : (size_t)qr0, d, ok);
        row_load(bq[1], CD, m, lm ? (size_t)lp0 * 2 + 1 : (size_t)qr1, d, ok);
        gain(gq, lm ? reinterpret_cast<const char*>(p.final_norm) : ptr(l, P_AN));
    };
    auto load_o = [&](int l) { row_load(bo[0], CD, ptr(min(l, p.L - 1), P_O), xr0, dq, l < p.L && has_x); };
    auto load_gu = [&](int l) {                 // or the next pairs of LM-head rows
        const bool lm = l >= p.L;
        const int t = min(l, p.L - 1);
        const char* wg = lm ? lh : ptr(t, P_G);
        const char* wu = lm ? lh : ptr(t, P_U);
#pragma unroll
        for (int u = 0; u < ST_GU; u++) {
            const int pair = lp0 + (u + 1) * ST_WAVES, gp = gp0 + u * ST_WAVES;
            const bool ok = lm ? pair < lp_end : gp < gp_end;
            row_load(bg[2 * u], CD, wg, lm ? (size_t)pair * 2 : (size_t)gp, d, ok);
            row_load(bg[2 * u + 1], CD, wu, lm ? (size_t)pair * 2 + 1 : (size_t)gp, d, ok);
        }
        gain(gg, ptr(t, P_MN));
    };
    auto load_d = [&](int l) { row_load(bd[0], CF, ptr(min(l, p.L - 1), P_D), xr0, f, l < p.L && has_x); };

    int xpar = 0;
    bool first = true;                          // the residual rows are still the embedding rows in memory
    // pair u of this thread of a row of n elements into LDS
    auto put_row = [&](int r, int u, float2 v, int n) {
        const int i = 2 * (u * ST_THREADS + tid);
        if (i < n) *reinterpret_cast<float2*>(xs + r * XF + gv_xpos<VEC>(i)) = v;
    };
    // residual rows into LDS, times the gain, and their sums of squares
    auto take_x = [&](const float2 (&gain)[NX]) {
        fresh();
        float2 v[R * NX];
        if (first) {
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < NX; u++) {
                    const int i = 2 * (u * ST_THREADS + tid);
                    v[r * NX + u] = r < M && i < d ? *reinterpret_cast<const float2*>(p.x + (size_t)r * d + i) : make_float2(0.f, 0.f);
                }
        } else {
            const int np = M * (d / 2);
            int pr[R * NX];
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < NX; u++) {
                    const int i = u * ST_THREADS + tid;
                    pr[r * NX + u] = r < M && 2 * i < d ? r * (d / 2) + i : np;
                }
            mail_take(pr, v, mx + (size_t)xpar * RS_ROWS * d, np, tag, ctrl, alive, p.wait_ticks);
        }
        float ss[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            ss[r] = 0.f;
#pragma unroll
            for (int u = 0; u < NX; u++) {
                const float2 x = v[r * NX + u];
                put_row(r, u, make_float2(x.x * gain[u].x, x.y * gain[u].y), d);
                ss[r] += x.x * x.x + x.y * x.y;
            }
        }
        const float sum = wave_sums(ss, lane);
        if (wave_slot(lane) < R) red[wave_slot(lane) * ST_WAVES + wave] = sum;
        lds_barrier();
    };
    auto scale = [&](int r) -> float {          // RMS scale of residual row r, behind take_x
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < ST_WAVES; i++) t += red[r * ST_WAVES + i];
        return 1.0f / sqrtf(t / (float)d + p.eps);
    };
    // the block's share of the residual rows to everybody, and into the taps
    auto give_x = [&](int l, int which) {
        tag++; xpar ^= 1; first = false;
        if (wave_slot(lane) < R) outs[wave * R + wave_slot(lane)] = xr;
        lds_barrier();
        const int i = tid / R, r = tid % R;
        if (i < xb1 - xb0 && r < M) {
            const float v = outs[tid];
            mail_put(mx + ((size_t)xpar * RS_ROWS + r) * d + xb0 + i, v, tag);
            p.taps[r * p.tap_ld + (size_t)(2 * l + which) * d + xb0 + i] = v;
        }
    };

    load_qkv(0); load_o(0); load_gu(0); load_d(0);
    for (int l = 0; l < p.L; l++) {
        KT* kc = reinterpret_cast<KT*>(p.kv + (size_t)(2 * l) * p.kv_layer);
        KT* vc = reinterpret_cast<KT*>(p.kv + (size_t)(2 * l + 1) * p.kv_layer);
        // ---- q, k, v ----
        {
            take_x(gq);
            tag++;
            float o[2][R];
            rows_dots<WT>(bq, xs, lane, d, o);
            const int slot = wave_slot(lane), sr = min(slot, R - 1), hi = qr0 % HD;
            const float sc = scale(sr), a = wave_sums(o[0], lane) * sc, c = wave_sums(o[1], lane) * sc;
            float o0 = a, o1 = c;
            if (qm < 2) {
                const float cs = rope[sr * HD + 2 * hi], sn = rope[sr * HD + 2 * hi + 1];   // (rows past M: nobody takes the result)
                o0 = a * cs - c * sn; o1 = c * cs + a * sn;
            }
            if (slot < R) { outs[wave * R + slot] = o0; outs[(ST_WAVES + wave) * R + slot] = o1; }
            lds_barrier();
            const int unit = tid / R, r = tid % R, pr = step_begin(nqp, b, NB) + unit % ST_WAVES;
            if (unit < 2 * ST_WAVES && r < M && pr < step_begin(nqp, b + 1, NB)) {
                int m, r0, r1;
                qkv_rows(pr, m, r0, r1);
                const int row = unit < ST_WAVES ? r0 : r1;
                float v = outs[tid];
                if (m > 0) {
                    KT* c = (m == 1 ? kc : vc) + ((size_t)(row / HD) * p.max_seq + p0 + r) * HD;
                    Elem<KT>::put(c, row % HD, v);
                    if (sizeof(KT) == 2) { KT t; Elem<KT>::put(&t, 0, v); v = Elem<KT>::get(&t, 0); }   // attention sees what the cache holds
                }
                mail_put(mqkv + (size_t)r * nqkv + (m == 0 ? 0 : m == 1 ? dq : dq + dkv) + row, v, tag);
            }
        }
        // ---- attention: one block per query head and row; the blocks of a head run on as few XCDs as the head count allows ----
        if (b < p.H * M) {
            fresh();
            const int head = b % p.H, row = b / p.H, kvh = head / (p.H / p.Hkv);
            const int n = p0 + row + 1, jlast = max(p0 - 1, 0);   // positions the row sees; the last one that is in the cache
            const int n_pass = (n + PASS - 1) / PASS;
            const int seg = lane / LPP, sl = (lane % LPP) * EPV;
            const KT* kb = kc + (size_t)kvh * p.max_seq * HD + sl;
            const KT* vb = vc + (size_t)kvh * p.max_seq * HD + sl;
            u32x4_t kr[2][NL], vr[2][NL];   // two passes: their loads are in flight together (one of twice the length: tiny contexts pay for all of it)
            auto issue = [&](u32x4_t (&kr)[NL], u32x4_t (&vr)[NL], int pass) {
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = min(((pass * NL + t) * ST_WAVES + wave) * PPL + seg, jlast);
                    kr[t] = *reinterpret_cast<const u32x4_t*>(kb + (size_t)j * HD);
                    vr[t] = *reinterpret_cast<const u32x4_t*>(vb + (size_t)j * HD);
                }
            };
            issue(kr[0], vr[0], 0);
            if (n_pass > 1) issue(kr[1], vr[1], 1);
            {   // the query, then the keys and the values of rows 0 .. row
                const int units = 2 * row + 3, np = M * nqkv / 2;
                const float qsc = 1.0f / sqrtf((float)HD);
                int pr[NQ];
                float2 v[NQ];
#pragma unroll
                for (int u = 0; u < NQ; u++) {
                    const int i = u * ST_THREADS + tid, unit = i / (HD / 2), e = i % (HD / 2);
                    const int rr = unit == 0 ? row : unit <= row + 1 ? unit - 1 : unit - row - 2;
                    const int at = unit == 0 ? head * HD : unit <= row + 1 ? dq + kvh * HD : dq + dkv + kvh * HD;
                    pr[u] = unit < units ? (rr * nqkv + at) / 2 + e : np;
                }
                mail_take(pr, v, mqkv, np, tag, ctrl, alive, p.wait_ticks);
#pragma unroll
                for (int u = 0; u < NQ; u++) {
                    const int i = u * ST_THREADS + tid, unit = i / (HD / 2);
                    const float s = unit == 0 ? qsc : 1.0f;
                    if (unit < units) *reinterpret_cast<float2*>(qs + 2 * i) = make_float2(v[u].x * s, v[u].y * s);
                }
            }
            lds_barrier();
            float m = -INFINITY, lsum = 0.f, acc[EPV];
#pragma unroll
            for (int u = 0; u < EPV; u++) acc[u] = 0.f;
            auto attend = [&](const u32x4_t (&kr)[NL], const u32x4_t (&vr)[NL], int pass) {
                float s[NL];
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = ((pass * NL + t) * ST_WAVES + wave) * PPL + seg;
                    float kf[EPV];
                    aw_unpack<KT>(kr[t], kf);
                    if (j >= p0 && j < n) {
#pragma unroll
                        for (int u = 0; u < EPV; u++) kf[u] = qs[(1 + j - p0) * HD + sl + u];
                    }
                    float a = 0.f;
#pragma unroll
                    for (int u = 0; u < EPV; u++) a = fmaf(kf[u], qs[sl + u], a);
                    a = aw_seg_sum<LPP>(a);
                    s[t] = j < n ? a : -INFINITY;
                }
                float mt = s[0];
#pragma unroll
                for (int t = 1; t < NL; t++) mt = fmaxf(mt, s[t]);
                mt = seg_max_fast<LPP>(mt);
                const float mn = fmaxf(m, mt);
                const bool live = mn > -INFINITY;
                const float c = live ? __expf(m - mn) : 1.0f;
                lsum *= c;
#pragma unroll
                for (int u = 0; u < EPV; u++) acc[u] *= c;
                m = mn;
#pragma unroll
                for (int t = 0; t < NL; t++) {
                    const int j = ((pass * NL + t) * ST_WAVES + wave) * PPL + seg;
                    const float e = live ? __expf(s[t] - mn) : 0.f;
                    lsum += e;
                    float vf[EPV];
                    aw_unpack<KT>(j < p0 ? vr[t] : u32x4_t{0u, 0u, 0u, 0u}, vf);   // rows from the position on may hold anything
                    if (j >= p0 && j < n) {
#pragma unroll
                        for (int u = 0; u < EPV; u++) vf[u] = qs[(2 + row + j - p0) * HD + sl + u];
                    }
#pragma unroll
                    for (int u = 0; u < EPV; u++) acc[u] = fmaf(e, vf[u], acc[u]);
                }
            };
            for (int pass = 0; pass < n_pass; pass += 2) {
                attend(kr[0], vr[0], pass);
                if (pass + 2 < n_pass) issue(kr[0], vr[0], pass + 2);
                if (pass + 1 >= n_pass) break;
                attend(kr[1], vr[1], pass + 1);
                if (pass + 3 < n_pass) issue(kr[1], vr[1], pass + 3);
            }
            lsum = seg_sum_fast<LPP>(lsum);
#pragma unroll
            for (int u = 0; u < EPV; u++) {
                acc[u] = seg_sum_fast<LPP>(acc[u]);
                if (seg == 0) wacc[wave * HD + sl + u] = acc[u];
            }
            if (lane == 0) { wml[wave * 2] = m; wml[wave * 2 + 1] = lsum; }
            lds_barrier();
            if (tid < HD) {
                float gm = -INFINITY, num = 0.f, den = 0.f;
#pragma unroll
                for (int w = 0; w < ST_WAVES; w++) gm = fmaxf(gm, wml[w * 2]);
#pragma unroll
                for (int w = 0; w < ST_WAVES; w++) {
                    const float mw = wml[w * 2], c = mw > -INFINITY ? __expf(mw - gm) : 0.f;
                    num = fmaf(c, wacc[w * HD + tid], num);
                    den = fmaf(c, wml[w * 2 + 1], den);
                }
                mail_put(matt + (size_t)row * dq + head * HD + tid, num / den, tag + 1);
            }
        }
        // ---- output projection ----
        {
            fresh();
            tag++;
            const int np = M * (dq / 2);
            int pr[R * NX];
            float2 v[R * NX];
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < NX; u++) {
                    const int i = u * ST_THREADS + tid;
                    pr[r * NX + u] = r < M && 2 * i < dq ? r * (dq / 2) + i : np;
                }
            mail_take(pr, v, matt, np, tag, ctrl, alive, p.wait_ticks);
            load_qkv(l + 1);
#pragma unroll
            for (int r = 0; r < R; r++)
#pragma unroll
                for (int u = 0; u < NX; u++) put_row(r, u, v[r * NX + u], dq);
            lds_barrier();
            float o[1][R];
            rows_dots<WT>(bo, xs, lane, dq, o);
            xr += wave_sums(o[0], lane);
            give_x(l, 0);
            fresh();
            load_o(l + 1);
        }
        // ---- gate and up ----
        {
            take_x(gg);
            tag++;
            float o[2 * ST_GU][R], og[ST_GU * R], ou[ST_GU * R];
            rows_dots<WT>(bg, xs, lane, d, o);
#pragma unroll
            for (int u = 0; u < ST_GU; u++)
#pragma unroll
                for (int r = 0; r < R; r++) { og[u * R + r] = o[2 * u][r]; ou[u * R + r] = o[2 * u + 1][r]; }
            const int slot = wave_slot(lane);
            const float sc = scale(slot % R), a = wave_sums(og, lane) * sc, c = wave_sums(ou, lane) * sc;
            if (slot < ST_GU * R) outs[(slot / R * ST_WAVES + wave) * R + slot % R] = a / (1.0f + __expf(-a)) * c;
            lds_barrier();
            const int unit = tid / R, r = tid % R;
            if (unit < gp_end - gb0 && r < M) mail_put(mact + (size_t)r * f + gb0 + unit, outs[tid], tag);
        }
        // ---- down projection ----
        {
            fresh();
            constexpr int RG = R > 5 ? (R + 1) / 2 : R;   // rows per wait: what the registers hold
            const int np = M * (f / 2);
#pragma unroll
            for (int r0 = 0; r0 < R; r0 += RG) {
                int pr[RG * NF];
                float2 v[RG * NF];
#pragma unroll
                for (int r = 0; r < RG; r++)
#pragma unroll
                    for (int u = 0; u < NF; u++) {
                        const int i = u * ST_THREADS + tid;
                        pr[r * NF + u] = r0 + r < M && 2 * i < f ? (r0 + r) * (f / 2) + i : np;
                    }
                mail_take(pr, v, mact, np, tag, ctrl, alive, p.wait_ticks, r0 == 0);
#pragma unroll
                for (int r = 0; r < RG; r++)
#pragma unroll
                    for (int u = 0; u < NF; u++)
                        if (r0 + r < R) put_row(r0 + r, u, v[r * NF + u], f);
            }
            load_gu(l + 1);
            lds_barrier();
            float o[1][R];
            rows_dots<WT>(bd, xs, lane, f, o);
            xr += wave_sums(o[0], lane);
            give_x(l, 1);
            fresh();
            load_d(l + 1);
        }
    }
    // ---- LM head: the first three row pairs of every wave are in registers, a used one is replaced by the third next ----
    take_x(gq);
    const int slot = wave_slot(lane);           // row of the logits that this lane finishes
    const float sc = scale(min(slot, R - 1));
    float best = -INFINITY;
    int arg = 0x7fffffff;
    auto lm_rows = [&](const u32x4_t (&w)[2][CD], int pair) {
        float o[2][R];
        rows_dots<WT>(w, xs, lane, d, o);
        const float a = wave_sums(o[0], lane) * sc, c = wave_sums(o[1], lane) * sc;
        if (slot < M) *reinterpret_cast<float2*>(p.logits + (size_t)slot * p.V + (size_t)pair * 2) = make_float2(a, c);
        const float ca = fminf(fmaxf(a, -p.clamp), p.clamp), cc = fminf(fmaxf(c, -p.clamp), p.clamp);
        if (ca > best) { best = ca; arg = pair * 2; }         // ascending columns: the first of equal maxima stays
        if (cc > best) { best = cc; arg = pair * 2 + 1; }
    };
    auto lm_load = [&](u32x4_t* w0, u32x4_t* w1, int pair) {
        row_load(w0, CD, lh, (size_t)pair * 2, d, pair < lp_end);
        row_load(w1, CD, lh, (size_t)pair * 2 + 1, d, pair < lp_end);
    };
    constexpr int LR = (1 + ST_GU) * ST_WAVES;   // pairs that the block's registers hold
    for (int i = lp0; i < lp_end; i += LR) {
        lm_rows(bq, i);
        lm_load(bq[0], bq[1], i + LR);
#pragma unroll
        for (int u = 0; u < ST_GU; u++) {
            const int j = i + (u + 1) * ST_WAVES;
            u32x4_t w[2][CD];
#pragma unroll
            for (int c = 0; c < CD; c++) { w[0][c] = bg[2 * u][c]; w[1][c] = bg[2 * u + 1][c]; }
            if (j < lp_end) lm_rows(w, j);
            lm_load(bg[2 * u], bg[2 * u + 1], j + LR);
        }
    }
    __shared__ float2 vred[ST_WAVES * R];
    if (slot < R) vred[wave * R + slot] = make_float2(best, __int_as_float(arg));
    lds_barrier();
    if (tid < M) {
        float2 a = vred[tid];
        for (int w = 1; w < ST_WAVES; w++) {
            const float2 e = vred[w * R + tid];
            if (e.x > a.x || (e.x == a.x && __float_as_int(e.y) < __float_as_int(a.y))) a = e;
        }
        p.vmax[(size_t)tid * NB + b] = a;
    }
}

static StepShape step_shape(const Dims& D) { return {D.d, D.dq, D.dkv, D.f, D.V, D.hd, D.H, D.Hkv, D.wt, D.kt, D.L}; }

size_t step_scratch_bytes(const Dims& D)
{
    const StepShape s = step_shape(D);
    return step_blocks(s, ST_BLOCKS) ? step_table_offset(D) + (size_t)D.L * sizeof(StepWeights) : 0;
}

// control words and words of the single-row step, words of the verification, weight table
size_t step_table_offset(const Dims& D)
{
    const StepShape s = step_shape(D);
    return (step_mail(s).total + rows_mail(s).total) * 8;
}

// Kernels whose last block leaves at once exist for one type and head size, which is enough to test what the others do then.
static bool step_can_lack(const Dims& D) { return D.wt == WT_F32 && D.hd == 64; }

template <typename WT, typename KT>
static const void* step_fn(const Dims& D)
{
    return D.hd == 64 ? (const void*)step_kernel<WT, KT, 64> : (const void*)step_kernel<WT, KT, 128>;
}
static const void* step_fn(const Dims& D, bool lack)
{
    if (lack && step_can_lack(D)) return (const void*)step_kernel<float, float, 64, true>;
    if (D.wt == WT_F32) return step_fn<float, float>(D);
    if (D.wt == WT_BF16) return D.kt == WT_F32 ? step_fn<uint16_t, float>(D) : step_fn<uint16_t, uint16_t>(D);
    return D.kt == WT_F32 ? step_fn<f16_t, float>(D) : step_fn<f16_t, f16_t>(D);
}
static size_t step_lds_bytes(const Dims& D)
{
    return (size_t)2 * ST_CF * 64 * (D.wt == WT_F32 ? 4 : 8) * sizeof(float) + (size_t)D.L * sizeof(StepWeights);
}

// The verification kernel that computes R rows, enabled for its LDS.
template <typename WT, typename KT, int HD, bool LACK = false>
static hipError_t rows_step_fn(const Dims& D, int R, const void** fn, size_t* lds)
{
    constexpr size_t XF = (size_t)ST_CF * 64 * Elem<WT>::VEC;
    static std::atomic<size_t> lds_limit[3];   // per instantiation
    *fn = R == 3 ? (const void*)rows_step_kernel<WT, KT, HD, 3, LACK> : R == 5 ? (const void*)rows_step_kernel<WT, KT, HD, 5, LACK>
                                                                               : (const void*)rows_step_kernel<WT, KT, HD, RS_ROWS, LACK>;
    *lds = R * XF * sizeof(float) + (size_t)D.L * sizeof(StepWeights);
    return ensure_lds(*fn, *lds, lds_limit[R == 3 ? 0 : R == 5 ? 1 : 2]);
}
template <typename WT, typename KT>
static hipError_t rows_step_fn(const Dims& D, int R, const void** fn, size_t* lds)
{
    return D.hd == 64 ? rows_step_fn<WT, KT, 64>(D, R, fn, lds) : rows_step_fn<WT, KT, 128>(D, R, fn, lds);
}
static hipError_t rows_step_fn(const Dims& D, int R, bool lack, const void** fn, size_t* lds)
{
    if (lack && step_can_lack(D)) return rows_step_fn<float, float, 64, true>(D, R, fn, lds);
    if (D.wt == WT_F32) return rows_step_fn<float, float>(D, R, fn, lds);
    if (D.wt == WT_BF16) return D.kt == WT_F32 ? rows_step_fn<uint16_t, float>(D, R, fn, lds) : rows_step_fn<uint16_t, uint16_t>(D, R, fn, lds);
    return D.kt == WT_F32 ? rows_step_fn<f16_t, float>(D, R, fn, lds) : rows_step_fn<f16_t, f16_t>(D, R, fn, lds);
}

hipError_t step_device_blocks(const Dims& D, int device, int* blocks_out, int* max_rows_out)
{
    *blocks_out = *max_rows_out = 0;
    if (!step_scratch_bytes(D)) return hipSuccess;
    int cus = 0, per_cu = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    const size_t lds = step_lds_bytes(D);   // below 64 KB
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, step_fn(D, false), ST_THREADS, lds);
    if (e != hipSuccess) return e;
    if (per_cu >= 1) *blocks_out = step_blocks(step_shape(D), cus);
    // the verification kernels ask for more registers and four to five times the LDS: up to the widest that fits
    for (int R : {3, 5, RS_ROWS}) {
        const void* fn;
        size_t rows_lds;
        if (*blocks_out == 0 || rows_step_fn(D, R, false, &fn, &rows_lds) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, ST_THREADS, rows_lds) != hipSuccess || per_cu < 1) {
            (void)hipGetLastError();   // a kernel that does not fit is no error of this call
            break;
        }
        *max_rows_out = R;
    }
    return hipSuccess;
}

bool step_plan_fits(const Dims& D, int ctx, int blocks)
{
    const AttnPlan pl = attn_plan(D, ctx, 1);
    return pl.wide && pl.n_splits <= AW_MAX_RANGES && D.H * pl.n_splits <= blocks;
}

hipError_t step_fused(const Dims& D, const StepLaunch& a, const StepOut& o, hipStream_t s)
{
    const int ctx = a.plan_ctx;
    if (a.blocks < 1 || !step_plan_fits(D, ctx, a.blocks) || a.blocks != step_blocks(step_shape(D), a.blocks) || ctx < 1 || ctx > D.max_seq)
        return hipErrorInvalidValue;
    if (!o.tok_out || !o.tok_host || !o.maxprob_host || (o.pos_dev && !o.tok0) || (o.x_next && !o.embed) || !o.step_ctrl) return hipErrorInvalidValue;
    const AttnPlan pl = attn_plan(D, ctx, 1);
    StepP p = {};
    p.off = step_mail(step_shape(D));
    p.mail = static_cast<unsigned long long*>(a.scratch);
    p.layers = reinterpret_cast<const StepWeights*>(static_cast<char*>(a.scratch) + step_table_offset(D)); p.L = D.L;
    StepOut out = o;
    out.step_hops = 0;
    for (int l = 0; l < D.L; l++) {
        if (a.sub && a.sub[2 * l] != a.sub[2 * l + 1]) return hipErrorInvalidValue;
        if (!(a.sub && a.sub[2 * l])) { p.mask[l >> 6] |= 1ull << (l & 63); out.step_hops += 5; }
    }
    p.lm_head = a.lm_head; p.final_norm = a.final_norm; p.x = a.x; p.rope_row = a.rope_row; p.pos_dev = a.pos_dev; p.pos_off = a.pos_off;
    p.kv = static_cast<char*>(a.kv); p.kv_layer = a.kv_layer;
    p.logits = a.logits; p.vstat = a.vstat; p.clamp = a.clamp;
    p.d = D.d; p.dq = D.dq; p.dkv = D.dkv; p.f = D.f; p.V = D.V; p.H = D.H; p.Hkv = D.Hkv; p.max_seq = D.max_seq; p.eps = D.eps;
    p.n_splits = pl.n_splits; p.chunk = pl.chunk;
    p.wait_ticks = a.wait_ticks;
    void* args[] = {&p};
    const void* fn = step_fn(D, a.wait_ticks < 0 && out.step_hops > 0);   // (without a layer nobody waits for anybody)
    hipError_t e = hipLaunchKernel(fn, dim3(a.blocks), dim3(ST_THREADS), args, step_lds_bytes(D), s);
    if (e != hipSuccess) return e;
    return step_finish(D, a.vstat, a.blocks, out, s);
}

bool rows_step_fits(const Dims& D, int M, int ctx, int blocks, int max_rows)
{
    return ctx <= D.max_seq && rows_step_fits(step_shape(D), M, ctx, blocks, max_rows);
}

hipError_t rows_step_fused(const Dims& D, const RowsStepLaunch& a, hipStream_t s)
{
    if (!rows_step_fits(D, a.M, a.ctx, a.blocks, RS_ROWS) || a.blocks != step_blocks(step_shape(D), a.blocks) || !a.tok_out || !a.tok_host || !a.err_host ||
        !a.taps || !a.vmax) return hipErrorInvalidValue;
    RowsStepP p = {};
    p.ctrl = static_cast<unsigned*>(a.scratch);
    p.mail = static_cast<unsigned long long*>(a.scratch) + step_mail(step_shape(D)).total;
    p.off = rows_mail(step_shape(D));
    p.layers = reinterpret_cast<const StepWeights*>(static_cast<char*>(a.scratch) + step_table_offset(D)); p.L = D.L; p.M = a.M;
    p.lm_head = a.lm_head; p.final_norm = a.final_norm; p.x = a.x; p.rope = a.rope; p.pos_dev = a.pos_dev;
    p.kv = static_cast<char*>(a.kv); p.kv_layer = a.kv_layer;
    p.logits = a.logits; p.taps = a.taps; p.tap_ld = (size_t)D.L * 2 * D.d; p.vmax = a.vmax; p.clamp = a.clamp;
    p.d = D.d; p.dq = D.dq; p.dkv = D.dkv; p.f = D.f; p.V = D.V; p.H = D.H; p.Hkv = D.Hkv; p.max_seq = D.max_seq; p.eps = D.eps;
    p.wait_ticks = a.wait_ticks;
    const void* fn;
    size_t lds;
    hipError_t e = rows_step_fn(D, rows_step_rows(a.M), a.wait_ticks < 0, &fn, &lds);
    if (e != hipSuccess) return e;
    void* args[] = {&p};
    e = hipLaunchKernel(fn, dim3(a.blocks), dim3(ST_THREADS), args, lds, s);
    if (e != hipSuccess) return e;
    return argmax_tiles(a.vmax, a.M, a.blocks, a.tok_out, a.tok_host, s, p.ctrl, 5 * D.L, a.err_host);
}

// ---------------------------------------------------------------------------------------------
// vocabulary reduction: arg-max, softmax max-probability, entropy confidence (Eq. 1-4)
// ---------------------------------------------------------------------------------------------
constexpr int VR_THREADS = 1024;

// maximum of a wave and its lowest index
__device__ __forceinline__ void argmax_wave(float& m, int& mi)
{
    const float wm = wave_max_fast(m);
    mi = wave_min_fast(m == wm ? mi : 0x7fffffff);
    m = wm;
}

__global__ __launch_bounds__(VR_THREADS) void vocab_reduce_kernel(const float* __restrict__ logits, int V, float clamp,
                                                                  float eps, int32_t* tok_out, int32_t* tok_host,
                                                                  int32_t* argmax_out, float* maxprob_out, float* conf_out)
{
    __shared__ float rv[16];
    __shared__ int ri[16];
    __shared__ double rd[16];
    const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* z = logits + (size_t)r * V;
    // pass 1: max and its lowest index
    float m = -INFINITY;
    int mi = 0x7fffffff;
    for (int i = tid; i < V; i += VR_THREADS) {
        float v = fminf(fmaxf(z[i], -clamp), clamp);
        if (v > m) { m = v; mi = i; }  // ascending i per thread: first occurrence kept
    }
    argmax_wave(m, mi);
    if (lane == 0) { rv[wave] = m; ri[wave] = mi; }
    __syncthreads();
    m = rv[0]; mi = ri[0];
#pragma unroll
    for (int w = 1; w < 16; w++) {
        float om = rv[w]; int oi = ri[w];
        if (om > m || (om == m && oi < mi)) { m = om; mi = oi; }
    }
    // pass 2: Z = sum exp(z - m)
    // (both sums in 64 bits: a rounding error of Z or H moves every confidence of the row)
    double zs = 0.0;
    for (int i = tid; i < V; i += VR_THREADS) zs += expf(fminf(fmaxf(z[i], -clamp), clamp) - m);
    const double Z = block_sum<16>(zs, rd);
    if (tid == 0) {
        if (tok_out) { tok_out[r] = mi; tok_host[r] = mi; }
        if (argmax_out) argmax_out[r] = mi;
        if (maxprob_out) maxprob_out[r] = (float)(1.0 / Z);
    }
    if (conf_out) {
        // pass 3: H = -sum p log(p + eps)
        double hs = 0.0;
        const double invZ = 1.0 / Z;
        for (int i = tid; i < V; i += VR_THREADS) {
            const double pr = expf(fminf(fmaxf(z[i], -clamp), clamp) - m) * invZ;
            hs -= pr * logf((float)pr + eps);
        }
        const double Hs = block_sum<16>(hs, rd);
        if (tid == 0) conf_out[r] = (float)(1.0 - Hs / log((double)V));
    }
}

// Greedy token of every row of a 16-row LM-head launch from the per-tile maxima its epilogue left behind: one block per
// row, lowest column among equal maxima.  (Reading the logits back instead is one block walking 128-513 KB: 18.5 us at
// 32 000 columns, 65 us at 128 256.)
__global__ __launch_bounds__(VR_THREADS) void argmax_tiles_kernel(const float2* __restrict__ vmax, int n_tiles,
                                                                  int32_t* __restrict__ tok_out, int32_t* __restrict__ tok_host,
                                                                  unsigned* step_ctrl, unsigned step_hops, int32_t* step_err_host)
{
    if (step_ctrl && blockIdx.x == 0 && threadIdx.x == 0) {   // end of a verification in one launch, as in step_finish_kernel
        step_ctrl[0] += step_hops;
        if (step_ctrl[1]) step_err_host[0] = 1;
    }
    __shared__ float rv[16];
    __shared__ int ri[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float2* v = vmax + (size_t)blockIdx.x * n_tiles;
    float m = -INFINITY;
    int mi = 0x7fffffff;
    for (int i = tid; i < n_tiles; i += VR_THREADS) {
        const float2 e = v[i];
        if (e.x > m) { m = e.x; mi = __float_as_int(e.y); }   // ascending tiles per thread: first occurrence kept
    }
    argmax_wave(m, mi);
    if (lane == 0) { rv[wave] = m; ri[wave] = mi; }
    __syncthreads();
    if (wave == 0) {
        m = lane < 16 ? rv[lane] : -INFINITY;
        mi = lane < 16 ? ri[lane] : 0x7fffffff;
        argmax_wave(m, mi);
        if (lane == 0) { tok_out[blockIdx.x] = mi; tok_host[blockIdx.x] = mi; }
    }
}
hipError_t argmax_tiles(const float2* vmax, int M, int n_tiles, int32_t* tok_out, int32_t* tok_host, hipStream_t s, unsigned* step_ctrl,
                        unsigned step_hops, int32_t* step_err_host)
{
    if (M < 1 || n_tiles < 1 || !tok_host) return hipErrorInvalidValue;
    hipLaunchKernelGGL(argmax_tiles_kernel, dim3(M), dim3(VR_THREADS), 0, s, vmax, n_tiles, tok_out, tok_host, step_ctrl, step_hops, step_err_host);
    return hipGetLastError();
}

// Confidence rows, cut along the vocabulary: `ns` blocks per row leave (max, sum of exp relative to it, arg-max) of their
// slice, a second launch merges a row's records (every block for itself, in slice order) and adds up its slice of the
// entropy, a third adds the slices.  One block per row walks 32 000 logits three times in 27 us while most CUs idle (16
// or 64 rows); the three short launches take 22 us together for 64 rows of 32 000 logits, 19 us for 16.
constexpr int VS_THREADS = 256;
struct VRec { double z, h; float m; int arg; };   // sums in 64 bits, as above

__device__ __forceinline__ void vs_slice(int V, int ns, int sl, int& b, int& e)
{
    b = (int)((long)V * sl / ns);
    e = (int)((long)V * (sl + 1) / ns);
}
__global__ __launch_bounds__(VS_THREADS) void vocab_part_kernel(const float* __restrict__ logits, int V, int ns, float clamp,
                                                                VRec* __restrict__ rec)
{
    __shared__ float rv[VS_THREADS / 64];
    __shared__ int ri[VS_THREADS / 64];
    __shared__ double rd[VS_THREADS / 64];
    const int sl = blockIdx.x, r = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* z = logits + (size_t)r * V;
    int b, e;
    vs_slice(V, ns, sl, b, e);
    float m = -INFINITY;
    int mi = 0x7fffffff;
    for (int i = b + tid; i < e; i += VS_THREADS) {
        const float v = fminf(fmaxf(z[i], -clamp), clamp);
        if (v > m) { m = v; mi = i; }
    }
    argmax_wave(m, mi);
    if (lane == 0) { rv[wave] = m; ri[wave] = mi; }
    __syncthreads();
    m = rv[0]; mi = ri[0];
#pragma unroll
    for (int w = 1; w < VS_THREADS / 64; w++)
        if (rv[w] > m || (rv[w] == m && ri[w] < mi)) { m = rv[w]; mi = ri[w]; }
    double zs = 0.0;
    if (m > -INFINITY)   // (infinite clamp: a slice of -inf only has no terms; exp(-inf - -inf) would be NaN.  Uniform.)
        for (int i = b + tid; i < e; i += VS_THREADS) zs += expf(fminf(fmaxf(z[i], -clamp), clamp) - m);
    const double Z = block_sum<VS_THREADS / 64>(zs, rd);
    if (tid == 0) rec[(size_t)r * ns + sl] = VRec{Z, 0.0, m, mi};
}
// merged maximum, its lowest index and sum of exp of the ns records of a row
__device__ __forceinline__ void vs_merge(const VRec* rec, int ns, float& m, double& Z, int& mi)
{
    m = -INFINITY; mi = 0x7fffffff;
    for (int i = 0; i < ns; i++)
        if (rec[i].m > m) { m = rec[i].m; mi = rec[i].arg; }   // ascending slices: first occurrence kept
    Z = 0.0;
    for (int i = 0; i < ns; i++) Z += rec[i].z * expf(rec[i].m - m);
}
__global__ __launch_bounds__(VS_THREADS) void vocab_entropy_kernel(const float* __restrict__ logits, int V, int ns, float clamp,
                                                                   float eps, VRec* __restrict__ rec)
{
    __shared__ double rd[VS_THREADS / 64];
    const int sl = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
    const float* z = logits + (size_t)r * V;
    VRec* row = rec + (size_t)r * ns;
    int b, e, mi;
    float m;
    double Z;
    vs_slice(V, ns, sl, b, e);
    vs_merge(row, ns, m, Z, mi);
    const double invZ = 1.0 / Z;
    double hs = 0.0;
    for (int i = b + tid; i < e; i += VS_THREADS) {
        const double pr = expf(fminf(fmaxf(z[i], -clamp), clamp) - m) * invZ;
        hs -= pr * logf((float)pr + eps);
    }
    const double H = block_sum<VS_THREADS / 64>(hs, rd);
    if (tid == 0) row[sl].h = H;   // (the other blocks of the row read m, z and arg only)
}
__global__ __launch_bounds__(64) void vocab_sum_kernel(const VRec* __restrict__ rec, int V, int ns, int32_t* argmax_out,
                                                       float* maxprob_out, float* conf_out)
{
    const int r = blockIdx.x, lane = threadIdx.x;   // one wave per row, a lane per slice
    const VRec v = rec[(size_t)r * ns + min(lane, ns - 1)];
    const bool own = lane < ns;
    float m = own ? v.m : -INFINITY;
    int mi = own ? v.arg : 0x7fffffff;
    argmax_wave(m, mi);
    double Z = own ? v.z * expf(v.m - m) : 0.0, H = own ? v.h : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { Z += __shfl_xor(Z, o, 64); H += __shfl_xor(H, o, 64); }
    if (lane == 0) {
        if (argmax_out) argmax_out[r] = mi;
        if (maxprob_out) maxprob_out[r] = (float)(1.0 / Z);
        conf_out[r] = (float)(1.0 - H / log((double)V));
    }
}

// Slices per row: 16, or what leaves at least 1024 logits to each and the scratch holds -- whatever the row count, so that
// batches of different size give the same bits.  More than 256 rows fill the chip by themselves and a short vocabulary
// is one quick block: those keep the one-block-per-row kernel.
hipError_t vocab_confidence(const float* logits, int M, int V, float clamp, float eps, int32_t* argmax_out, float* maxprob_out,
                            float* conf_out, void* scratch, size_t scratch_bytes, hipStream_t s)
{
    if (M < 1 || V < 1 || !conf_out) return hipErrorInvalidValue;
    const int ns = (int)std::min<size_t>(std::min(V / 1024, 16), scratch ? scratch_bytes / ((size_t)M * sizeof(VRec)) : 0);
    if (M > 256 || ns < 4) return vocab_reduce(logits, M, V, clamp, eps, nullptr, nullptr, argmax_out, maxprob_out, conf_out, s);
    VRec* rec = static_cast<VRec*>(scratch);
    hipLaunchKernelGGL(vocab_part_kernel, dim3(ns, M), dim3(VS_THREADS), 0, s, logits, V, ns, clamp, rec);
    hipLaunchKernelGGL(vocab_entropy_kernel, dim3(ns, M), dim3(VS_THREADS), 0, s, logits, V, ns, clamp, eps, rec);
    hipLaunchKernelGGL(vocab_sum_kernel, dim3(M), dim3(64), 0, s, rec, V, ns, argmax_out, maxprob_out, conf_out);
    return hipGetLastError();
}

// means[t] = mean over p < n_pos of v[p * n_taps + t], summed in position order (one thread per tap row)
__global__ void window_mean_kernel(const float* __restrict__ v, int n_pos, int n_taps, float* __restrict__ means)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_taps) return;
    float s = 0.f;
    for (int p = 0; p < n_pos; p++) s += v[(size_t)p * n_taps + t];
    means[t] = s / (float)n_pos;
}
hipError_t window_mean(const float* v, int n_pos, int n_taps, float* means, hipStream_t s)
{
    if (n_pos < 1 || n_taps < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(window_mean_kernel, dim3(ceil_div(n_taps, 64)), dim3(64), 0, s, v, n_pos, n_taps, means);
    return hipGetLastError();
}

hipError_t vocab_reduce(const float* logits, int M, int V, float clamp, float eps, int32_t* tok_out, int32_t* tok_host,
                        int32_t* argmax_out, float* maxprob_out, float* conf_out, hipStream_t s)
{
    hipLaunchKernelGGL(vocab_reduce_kernel, dim3(M), dim3(VR_THREADS), 0, s, logits, V, clamp, eps, tok_out, tok_host,
                       argmax_out, maxprob_out, conf_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// static scratch (for the entry point that allocates nothing)
// ---------------------------------------------------------------------------------------------
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)12 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

size_t static_scratch_bytes() { return STATIC_SCRATCH_BYTES; }

// `scratch` names the array only in device code; in host code the name is a stand-in, not an address.  The device
// address is asked of the runtime once per device, with that device current, and kept.
hipError_t static_scratch_for_device(int device, void** ptr_out)
{
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static void* ptr[MAX_DEV] = {};
    if (!ptr_out || device < 0 || device >= MAX_DEV) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[device] = p;
    }
    *ptr_out = ptr[device];
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// state kernels
// ---------------------------------------------------------------------------------------------
__global__ void set_state_kernel(int32_t* tok0, int32_t token, int* pos_dev, int pos)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) { tok0[0] = token; pos_dev[0] = pos; }
}
hipError_t set_state(int32_t* tok0, int32_t token, int* pos_dev, int pos, hipStream_t s)
{
    hipLaunchKernelGGL(set_state_kernel, dim3(1), dim3(64), 0, s, tok0, token, pos_dev, pos);
    return hipGetLastError();
}

__global__ void advance_state_kernel(int* pos_dev, int delta, int32_t* tok0, const int32_t* src)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        pos_dev[0] += delta;
        if (src) tok0[0] = src[0];
    }
}
hipError_t advance_state(int* pos_dev, int delta, int32_t* tok0, const int32_t* src, hipStream_t s)
{
    hipLaunchKernelGGL(advance_state_kernel, dim3(1), dim3(64), 0, s, pos_dev, delta, tok0, src);
    return hipGetLastError();
}

template <typename KT>
__global__ void kv_poison_kernel(KT* kv, int planes, int max_seq, int hd, const int* pos_dev)
{
    // kv: [planes][max_seq][hd] where planes = L * 2 * Hkv
    const int from = pos_dev[0];
    size_t per_plane = (size_t)(max_seq - from) * hd;
    size_t total = per_plane * planes;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        size_t pl = i / per_plane, o = i % per_plane;
        Elem<KT>::put(kv, (pl * max_seq + from) * hd + o, __int_as_float(0x7fc00000));
    }
}
hipError_t kv_poison(const Dims& D, void* kv_all, const int* pos_dev, hipStream_t s)
{
    int planes = D.L * 2 * D.Hkv;
    if (D.kt == WT_BF16)
        hipLaunchKernelGGL(kv_poison_kernel<uint16_t>, dim3(1024), dim3(256), 0, s, (uint16_t*)kv_all, planes, D.max_seq,
                           D.hd, pos_dev);
    else if (D.kt == WT_F16)
        hipLaunchKernelGGL(kv_poison_kernel<f16_t>, dim3(1024), dim3(256), 0, s, (f16_t*)kv_all, planes, D.max_seq, D.hd,
                           pos_dev);
    else
        hipLaunchKernelGGL(kv_poison_kernel<float>, dim3(1024), dim3(256), 0, s, (float*)kv_all, planes, D.max_seq, D.hd,
                           pos_dev);
    return hipGetLastError();
}

__global__ void copy_f32_kernel(const float* __restrict__ src, float* __restrict__ dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}
hipError_t copy_f32(const float* src, float* dst, size_t n, hipStream_t s)
{
    int blocks = (int)((n + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(copy_f32_kernel, dim3(blocks), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

// Read-only streaming probe: every lane keeps eight non-temporal 128-bit loads in flight (the access shape of the
// weight-streaming kernels, minus their arithmetic); a wave reads 1 KB contiguous per load instruction.
__global__ __launch_bounds__(256) void read_probe_kernel(const u32x4_t* __restrict__ src, size_t n_vec, float* sink)
{
    uint32_t acc = 0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 7 * stride < n_vec; i += 8 * stride) {
        u32x4_t v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
        for (int u = 0; u < 8; u++) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < n_vec; i += stride) {
        const u32x4_t a = __builtin_nontemporal_load(src + i);
        acc ^= a.x ^ a.y ^ a.z ^ a.w;
    }
    if (acc == 0x9e3779b9u) sink[0] = 1.0f;  // practically never true; keeps the loads alive
}
hipError_t read_probe(const void* dev, size_t bytes, float* sink_dev, hipStream_t s)
{
    hipLaunchKernelGGL(read_probe_kernel, dim3(256 * 8), dim3(256), 0, s, (const u32x4_t*)dev, bytes / 16, sink_dev);
    return hipGetLastError();
}

}  // namespace ssdk
