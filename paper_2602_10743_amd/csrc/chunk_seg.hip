// Segment-parallel forward for few sequences.
//
// With B H small, one workgroup per (b, h, value tile) leaves most of the chip idle for
// the whole sequence.  The sequence is cut into ns segments of lc chunks (the last one as
// long as is left) and both recursions are carried across segment boundaries by their
// composition laws (Corollaries 1 and 2):
//   1. per piece of a segment and key slot, the product of Theorem 1's 2x2 matrices over
//      the piece's tokens (seg_prec_kernel), with prod abar, then the product over each
//      segment's pieces (seg_compose_kernel);
//   2. an exclusive scan over the segments gives the precision at every segment start and
//      the segment's gate product P_s = prod_t F_t (seg_lam_scan_kernel);
//   3. the chunked forward over every segment but the last at once, from those precisions
//      and a zero state, without readout, gives the state each segment adds on its own, U_s;
//   4. an exclusive scan of H_{s+1} = diag(P_s) H_s + U_s gives the state at every segment
//      start (seg_state_scan_kernel);
//   5. the chunked forward over every segment from the exact start belief writes y (and
//      yvar, the saved context and, from the last segment, the final belief).
#include "kla_device.hpp"
#include "kla_internal.hpp"

namespace kla {
namespace {

constexpr int kCS = 32;   // tokens per chunk

struct Cut {
    int ns, lc;      // segments, chunks per segment (all but the last full)
    int pl, pps;     // chunks per piece, pieces per segment
};

// Per (b, h, piece): lanes = key slots.  The images of (1, 0) and (0, 1) under the piece's
// matrices, with prod abar, rescaled together every 16 tokens by the largest entry (the
// matrix is projective and P = A / z is unchanged by a common scale).
template <int DK, bool TI>
__global__ __launch_bounds__(DK) void seg_prec_kernel(Shape s, Cut cut, FwdArgs g, float* __restrict__ mseg) {
    const uint16_t *a = static_cast<const uint16_t*>(g.a), *p = static_cast<const uint16_t*>(g.p);
    const uint16_t *k = static_cast<const uint16_t*>(g.k), *r = static_cast<const uint16_t*>(g.r);
    const int np = (cut.ns - 1) * cut.pps, pc = blockIdx.x % np, bh = blockIdx.x / np;
    const int seg = pc / cut.pps, pi = pc % cut.pps;
    const int H = s.H, b = bh / H, h = bh % H, n = threadIdx.x;
    const int c0 = seg * cut.lc + pi * cut.pl, c1 = min(c0 + cut.pl, (seg + 1) * cut.lc);
    float ca = 0.f, cp = 0.f;
    if constexpr (TI) ou_gates(g.ou_a[h * DK + n], g.ou_p[h * DK + n], g.ou_d[h * DK + n], ca, cp);
    float x0 = 1.f, z0 = 0.f, x1 = 0.f, z1 = 1.f, A = 1.f;
    for (int t0 = c0 * kCS; t0 < c1 * kCS; t0 += 16) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const size_t tok = ((size_t)b * s.T + t0 + j) * H + h;
            const float av = TI ? ca : ld(a, tok * DK + n), pv = TI ? cp : ld(p, tok * DK + n);
            const float kv = ld(k, tok * DK + n);
            const float phi = kv * kv * ld(r, tok);
            const float a2 = av * av;
            const float zn0 = fmaf(pv, x0, a2 * z0), zn1 = fmaf(pv, x1, a2 * z1);
            x0 = fmaf(phi, zn0, x0);
            x1 = fmaf(phi, zn1, x1);
            z0 = zn0;
            z1 = zn1;
            A *= av;
        }
        const float m = fmaxf(fmaxf(fabsf(x0), fabsf(z0)), fmaxf(fabsf(x1), fabsf(z1)));
        const float sc = 1.f / m;
        x0 *= sc;
        z0 *= sc;
        x1 *= sc;
        z1 *= sc;
        A *= sc;
    }
    float* o = mseg + ((size_t)bh * np + pc) * 5 * DK;
    o[0 * DK + n] = x0;
    o[1 * DK + n] = z0;
    o[2 * DK + n] = x1;
    o[3 * DK + n] = z1;
    o[4 * DK + n] = A;
}

// Per (b, h, segment, key slot): the product of the segment's piece matrices (later pieces
// on the left) with their abar products, rescaled by the largest entry after each piece;
// written over the segment's first piece.
__global__ __launch_bounds__(64) void seg_compose_kernel(int nseg, int DK, int pps, float* __restrict__ mseg) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nseg * DK) return;
    const int n = i % DK, seg = i / DK;   // seg over all sequences
    float* m0 = mseg + (size_t)seg * pps * 5 * DK + n;
    constexpr int U = 4;   // pieces loaded before their products
    float x0 = 1.f, z0 = 0.f, x1 = 0.f, z1 = 1.f, A = 1.f;
    for (int u0 = 0; u0 < pps; u0 += U) {
        float m[U][5];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 5; ++e) m[u][e] = m0[((size_t)min(u0 + u, pps - 1) * 5 + e) * DK];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u0 + u < pps) {
                const float nx0 = fmaf(m[u][0], x0, m[u][2] * z0), nz0 = fmaf(m[u][1], x0, m[u][3] * z0);
                const float nx1 = fmaf(m[u][0], x1, m[u][2] * z1), nz1 = fmaf(m[u][1], x1, m[u][3] * z1);
                A *= m[u][4];
                const float sc = 1.f / fmaxf(fmaxf(fabsf(nx0), fabsf(nz0)), fmaxf(fabsf(nx1), fabsf(nz1)));
                x0 = nx0 * sc;
                z0 = nz0 * sc;
                x1 = nx1 * sc;
                z1 = nz1 * sc;
                A *= sc;
            }
    }
    m0[0 * DK] = x0;
    m0[1 * DK] = z0;
    m0[2 * DK] = x1;
    m0[3 * DK] = z1;
    m0[4 * DK] = A;
}

// Per (b, h, key slot): lam at every segment start [bh ns + seg][DK] and the gate product of
// every segment but the last.
__global__ __launch_bounds__(64) void seg_lam_scan_kernel(int nbh, int DK, Cut cut, const float* __restrict__ mseg,
                                                          const float* __restrict__ lam0,
                                                          float* __restrict__ lam_start, float* __restrict__ pseg) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbh * DK) return;
    const int n = i % DK, bh = i / DK;
    float lam = lam0 ? lam0[i] : 1.f;
    const float* m = mseg + (size_t)bh * (cut.ns - 1) * cut.pps * 5 * DK + n;
    constexpr int U = 4;
    for (int s0 = 0; s0 < cut.ns; s0 += U) {
        float c[U][5];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 5; ++e)   // the composed segments
                c[u][e] = m[((size_t)min(s0 + u, cut.ns - 2) * cut.pps * 5 + e) * DK];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int sg = s0 + u;
            if (sg < cut.ns) {
                const size_t v = (size_t)bh * cut.ns + sg;
                lam_start[v * DK + n] = lam;
                const float x = fmaf(c[u][0], lam, c[u][2]), z = fmaf(c[u][1], lam, c[u][3]);
                if (sg < cut.ns - 1) pseg[v * DK + n] = c[u][4] / z;
                lam = x / z;
            }
        }
    }
}

// Per element (b, h, n, d): H at every segment start, in place of the states U that the
// segments before it add (h[bh ns + s] holds U_s on entry, H_s on return).
__global__ __launch_bounds__(256) void seg_state_scan_kernel(int nbh, int DK, int DV, int ns,
                                                             const float* __restrict__ pseg,
                                                             const float* __restrict__ eta0, float* __restrict__ h) {
    const size_t per = (size_t)DK * DV, i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)nbh * per) return;
    const size_t e = i % per, bh = i / per;
    const int n = (int)(e / DV);
    float st = eta0 ? eta0[i] : 0.f;
    constexpr int U = 8;
    float* o = h + bh * ns * per + e;
    const float* pn = pseg + bh * ns * DK + n;
    for (int s0 = 0; s0 < ns; s0 += U) {
        float u[U], p[U];
#pragma unroll
        for (int m = 0; m < U; ++m) {
            const int sg = min(s0 + m, ns - 2);
            u[m] = o[(size_t)sg * per];
            p[m] = pn[(size_t)sg * DK];
        }
#pragma unroll
        for (int m = 0; m < U; ++m)
            if (s0 + m < ns) {
                o[(size_t)(s0 + m) * per] = st;
                st = fmaf(p[m], st, u[m]);
            }
    }
}

// The cut of a shape.  One workgroup fills a CU, so segments are added until every CU has
// one (as many workgroups as fit 256, one per head and segment where dv = 128 runs wide).
// The costs (us per chunk round, and of the four kernels around the passes and their launches) are
// those with which the rule chose best over 1 to 128 heads, 300 to 8192 tokens and eight pairs of
// widths, each timed whole and in both cuts, with and without a saved context: at most 5% (12% at a
// few) from the best, but for some of one to four heads with 128 value channels, whose hundreds of
// segments cost more in the scans than the rule knows.  With one set of rounds for all widths, those
// of few workgroups, 100 heads of 64 x 64 over 2048 tokens took two segments, 148 us against 135, and
// 128 of 128 x 128 over 4096 with a saved context 589 against 446.
// Against the whole walk: 3001 tokens of 16 heads 238 -> 75 us, with OU gates and a saved context
// (B2 T2048 H16) 167 -> 85 us; 65536 tokens, 8 segments of two 64-channel tiles -> 16 wide ones,
// 1460 -> 1067 us (kernel times).
Cut cut_of(const Shape& s) {
    const int nct = (s.T + kCS - 1) / kCS, bh = s.B * s.H;
    Cut c{1, nct, 1, 1};
    if (!chunked_supported(s) || nct < 4) return c;
    const int ntile = s.dv == 128 ? 2 : 1;
    struct Us {
        double walk, exact, wide, state, fixed;   // whole walk, exact pass (wide), state-only pass
    };
    const bool two = ntile == 2;
    const Us us = s.dk == 128  ? (two ? Us{2.6, 2.25, 4.6, 1.35, 22.0} : Us{2.3, 2.25, 0.0, 1.85, 16.0})
                  : s.dk == 64 ? (two ? Us{1.95, 1.6, 3.3, 1.2, 17.0} : Us{1.7, 1.6, 0.0, 1.65, 15.0})
                               : (two ? Us{1.85, 1.45, 0.0, 1.35, 17.0} : Us{1.46, 1.6, 0.0, 1.35, 13.0});
    auto rounds = [](int wg) { return (wg + 255) / 256; };
    double best = nct * us.walk;
    for (int wg : {256 / (bh * ntile), 256 / bh}) {
        if (wg < 2) continue;
        const int lc = (nct + wg - 1) / wg, ns = (nct + lc - 1) / lc;
        if (ns < 2) continue;
        const double exact = chunked_wide(s, ns) ? us.wide * rounds(bh * ns) : us.exact * rounds(bh * ns * ntile);
        const double cost = lc * (us.state + exact) + us.fixed;
        if (cost < best) {
            best = cost;
            c.ns = ns;
            c.lc = lc;
        }
    }
    if (c.ns > 1) {   // pieces: enough of them to fill the chip with walks of at most 8 chunks
        const long chunks = (long)bh * (c.ns - 1) * c.lc;
        c.pl = (int)(chunks / 2048 < 1 ? 1 : chunks / 2048 > 8 ? 8 : chunks / 2048);
        c.pps = (c.lc + c.pl - 1) / c.pl;
    }
    return c;
}

}  // namespace

int forward_segments(const Shape& s) { return cut_of(s).ns; }

size_t forward_segmented_workspace(const Shape& s) {
    const Cut c = cut_of(s);
    if (c.ns < 2) return 0;
    const size_t nbh = (size_t)s.B * s.H, nl = nbh * c.ns * s.dk;
    // mseg (5 per piece and slot), lam_start and pseg, the states
    return (5 * nbh * (c.ns - 1) * c.pps * s.dk + 2 * nl + nl * s.dv) * sizeof(float) + 4 * 256;
}

hipError_t launch_forward_segmented(const Shape& s, const FwdArgs& a, void* saved, void* ws, hipStream_t st) {
    const Cut cut = cut_of(s);
    const int nbh = s.B * s.H, nseg = nbh * (cut.ns - 1);
    const size_t nl = (size_t)nbh * cut.ns * s.dk;
    auto carve = [&](size_t count) {
        float* p = static_cast<float*>(ws);
        ws = static_cast<char*>(ws) + (count * sizeof(float) + 255) / 256 * 256;
        return p;
    };
    float* mseg = carve(5 * (size_t)nseg * cut.pps * s.dk);
    float* lam_start = carve(nl);
    float* pseg = carve(nl);
    float* h = carve(nl * s.dv);
    const dim3 pgrid((unsigned)(nseg * cut.pps));
#define KLA_SEG_PREC(DK_)                                                                                     \
    if (s.dk == DK_) {                                                                                        \
        if (a.ou_a)                                                                                           \
            hipLaunchKernelGGL((seg_prec_kernel<DK_, true>), pgrid, dim3(DK_), 0, st, s, cut, a, mseg);       \
        else                                                                                                  \
            hipLaunchKernelGGL((seg_prec_kernel<DK_, false>), pgrid, dim3(DK_), 0, st, s, cut, a, mseg);      \
    }
    KLA_SEG_PREC(32) KLA_SEG_PREC(64) KLA_SEG_PREC(128)
#undef KLA_SEG_PREC
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (cut.pps > 1)
        hipLaunchKernelGGL(seg_compose_kernel, dim3((unsigned)((nseg * s.dk + 63) / 64)), dim3(64), 0, st, nseg, s.dk,
                           cut.pps, mseg);
    hipLaunchKernelGGL(seg_lam_scan_kernel, dim3((unsigned)((nbh * s.dk + 63) / 64)), dim3(64), 0, st, nbh, s.dk, cut,
                       mseg, a.lam0, lam_start, pseg);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    FwdArgs zero = a;   // the state each segment adds from a zero start (no readout)
    zero.lam0 = lam_start;
    zero.eta0 = nullptr;
    zero.y = nullptr;
    zero.yvar = nullptr;
    zero.lamT = nullptr;
    zero.etaT = h;
    if ((e = launch_forward_chunked_seg(s, cut.ns, cut.lc, cut.ns - 1, zero, nullptr, st)) != hipSuccess) return e;
    const size_t nel = (size_t)nbh * s.dk * s.dv;
    hipLaunchKernelGGL(seg_state_scan_kernel, dim3((unsigned)((nel + 255) / 256)), dim3(256), 0, st, nbh, s.dk, s.dv,
                       cut.ns, pseg, a.eta0, h);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    FwdArgs full = a;   // the exact pass, from every segment's start belief
    full.lam0 = lam_start;
    full.eta0 = h;
    return launch_forward_chunked_seg(s, cut.ns, cut.lc, cut.ns, full, saved, st);
}

}  // namespace kla
