// Building blocks of the chunked fp64 kernels (fp32 inputs): fp64 MFMA tiles, DPP
// sums, the per-token inputs of a walk lane and the group transfers of the precision
// walk.  Shared by the sequential chunk kernels (chunk64.hip) and the chunk-parallel
// ones (chunk64_par.hip).
#pragma once
#include "kla_buf.hpp"
#include "kla_device.hpp"

namespace kla {

constexpr int kC64 = 32;    // tokens per chunk

typedef double d4 __attribute__((ext_vector_type(4)));

// D += A B over four columns of A (v_mfma_f64_16x16x4_f64): lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; D[i][j] is component i / 4 of lane
// j + 16 (i % 4).
__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ d4 zero_d4() { return d4{0.0, 0.0, 0.0, 0.0}; }

// acc += sum_{k < K} A(i, k) B(k, j) for the 16x16 tile whose A rows start at pa and
// B columns at pb (LDS), A(i, k) = pa[i AI + k AK], B(k, j) = pb[k BK + j BJ].  The
// triangular products run over the whole chunk: the tile above the diagonal of the
// masked matrices is stored as zeros.
template <int K, int AI, int AK, int BK, int BJ>
__device__ __forceinline__ d4 tile_mm(d4 acc, const double* pa, const double* pb, int lane) {
    const int li = lane & 15, lk = lane >> 4;
    double av[K / 4], bv[K / 4];
#pragma unroll
    for (int s = 0; s < K / 4; ++s) {
        av[s] = pa[li * AI + (4 * s + lk) * AK];
        bv[s] = pb[(4 * s + lk) * BK + li * BJ];
    }
#pragma unroll
    for (int s = 0; s < K / 4; ++s) acc = mfma64(av[s], bv[s], acc);
    return acc;
}

// Sum over the DK lanes of one walk group (DK = 32: a half wave, DK = 16: a DPP row),
// valid in the group's last lane (n = DK - 1).
template <int DK>
__device__ __forceinline__ double slot_sum(double x) {
    if constexpr (DK == 32) {
        return half_sum(x);
    } else {
        x += dpp<0xB1, 0xf>(x);    // quad_perm [1,0,3,2]
        x += dpp<0x4E, 0xf>(x);    // quad_perm [2,3,0,1]
        x += dpp<0x141, 0xf>(x);   // row_half_mirror
        x += dpp<0x140, 0xf>(x);   // row_mirror
        return x;
    }
}

// row of component r of a D tile, relative to the tile (its column is lane % 16)
__device__ __forceinline__ int drow(int r, int lane) { return 4 * r + (lane >> 4); }

__device__ __forceinline__ float bld32(rsrc_t r, uint32_t voff) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0));
}

// Stores through a buffer: a lane whose offset lies past the end stores nothing.
__device__ __forceinline__ void bst32(rsrc_t r, uint32_t voff, float x) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, voff, 0, 0);
}

typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

__device__ __forceinline__ void bst64(rsrc_t r, uint32_t voff, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, voff, 0, 0);
}

// N (2 or 4) consecutive floats through a buffer in one load (offset aligned to 4 N bytes)
template <int N>
__device__ __forceinline__ void bldN(rsrc_t r, uint32_t voff, float* out) {
    if constexpr (N == 4) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = __uint_as_float(v[i]);
    } else {
        static_assert(N == 2, "2 or 4 floats");
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0);
        out[0] = __uint_as_float(v[0]);
        out[1] = __uint_as_float(v[1]);
    }
}

// N (2 or 4) consecutive floats from LDS (aligned to 4 N bytes) stored through a buffer in one store
template <int N>
__device__ __forceinline__ void bstN_lds(rsrc_t r, uint32_t voff, const float* src) {
    if constexpr (N == 4) {
        const float4 v = *reinterpret_cast<const float4*>(src);
        __builtin_amdgcn_raw_buffer_store_b128(
            u32x4{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)}, r, voff, 0, 0);
    } else {
        static_assert(N == 2, "2 or 4 floats");
        const float2 v = *reinterpret_cast<const float2*>(src);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(v.x), __float_as_uint(v.y)}, r, voff, 0, 0);
    }
}

// Buffers over one chunk's rows of the per-token tensors of head h: [t][H][DK] rows
// (abar, pbar, k, q) and [t][H] (r), each ending at the chunk's last valid token, so
// that tokens past the sequence end read as zero.
struct ChunkBufs {
    rsrc_t a, p, k, q, r;
    __device__ ChunkBufs(const float* ga, const float* gp, const float* gk, const float* gq, const float* gr,
                         size_t tok0, int H, int h, int DK, int nt) {
        const size_t e0 = (tok0 * H + h) * DK;
        const uint32_t bytes = (uint32_t)((nt - 1) * H * DK + DK) * 4;
        a = make_rsrc(ga ? ga + e0 : gk, ga ? bytes : 0u);
        p = make_rsrc(gp ? gp + e0 : gk, gp ? bytes : 0u);
        k = make_rsrc(gk + e0, bytes);
        q = make_rsrc(gq + e0, bytes);
        r = make_rsrc(gr + tok0 * H + h, (uint32_t)((nt - 1) * H + 1) * 4);
    }
};

// Per-token inputs of a walk lane, slot n, tokens t0 .. t0 + TPG - 1 of a chunk
// (t0 = gq TPG), as loaded (fp32).  Tokens past the sequence end (j >= nv) read as
// zeros, and abar as 1: the identity step.
template <int DK, int TPG, bool TI>
struct WalkIn {
    float a[TPG], p[TPG], k[TPG], q[TPG], r[TPG];
    int nv;
    double ca, cp;   // time-invariant gates (TI)
    __device__ void load(const ChunkBufs& cb, int H, int n, int t0, int nt) {
        nv = min(max(nt - t0, 0), TPG);
#pragma unroll
        for (int j = 0; j < TPG; ++j) {
            const uint32_t vo = (uint32_t)((t0 + j) * H * DK + n) * 4;
            if constexpr (!TI) {
                a[j] = bld32(cb.a, vo);
                p[j] = bld32(cb.p, vo);
            }
            k[j] = bld32(cb.k, vo);
            q[j] = bld32(cb.q, vo);
            r[j] = bld32(cb.r, (uint32_t)((t0 + j) * H) * 4);
        }
    }
    __device__ double A(int j) const { return j < nv ? (TI ? ca : (double)a[j]) : 1.0; }
    __device__ double P(int j) const { return TI ? (j < nv ? cp : 0.0) : (double)p[j]; }
    __device__ double K(int j) const { return (double)k[j]; }
    __device__ double Q(int j) const { return (double)q[j]; }
    __device__ double R(int j) const { return (double)r[j]; }
};

// The 2x2 transfer of a lane's tokens (the images of (1, 0) and (0, 1) under the
// homogeneous precision map) and the product of abar, into qs[gq][5][DK].
template <int DK, int TPG, bool TI>
__device__ __forceinline__ void group_transfer(const WalkIn<DK, TPG, TI>& in, double* qs, int gq, int n) {
    double m00 = 1.0, m10 = 0.0, m01 = 0.0, m11 = 1.0, aq = 1.0;
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const double av = in.A(j), kv = in.K(j);
        const double a2 = av * av, phi = kv * kv * in.R(j);
        const double z0 = fma(in.P(j), m00, a2 * m10), z1 = fma(in.P(j), m01, a2 * m11);
        m00 = fma(phi, z0, m00);
        m01 = fma(phi, z1, m01);
        m10 = z0;
        m11 = z1;
        aq *= av;
    }
    qs[(gq * 5 + 0) * DK + n] = m00;
    qs[(gq * 5 + 1) * DK + n] = m10;
    qs[(gq * 5 + 2) * DK + n] = m01;
    qs[(gq * 5 + 3) * DK + n] = m11;
    qs[(gq * 5 + 4) * DK + n] = aq;
}

// (x, z, A) before the lane's first token: the transfers of the earlier groups
// applied to the chunk start (lam, 1, 1).
template <int DK, int G>
__device__ __forceinline__ void chain_start(const double* qs, int gq, int n, double lam, double& x, double& z,
                                            double& A) {
    x = lam;
    z = 1.0;
    A = 1.0;
#pragma unroll
    for (int g2 = 0; g2 < G - 1; ++g2) {   // every lane the same steps, applied while g2 < gq
        const double m00 = qs[(g2 * 5 + 0) * DK + n], m10 = qs[(g2 * 5 + 1) * DK + n];
        const double m01 = qs[(g2 * 5 + 2) * DK + n], m11 = qs[(g2 * 5 + 3) * DK + n];
        const double aq = qs[(g2 * 5 + 4) * DK + n];
        const bool use = g2 < gq;
        const double xn = fma(m00, x, m01 * z), zn = fma(m10, x, m11 * z);
        x = use ? xn : x;
        z = use ? zn : z;
        A = use ? A * aq : A;
    }
}

}  // namespace kla
