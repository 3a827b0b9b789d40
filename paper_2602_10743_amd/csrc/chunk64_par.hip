// Chunk-parallel fp64 kernels for fp32 inputs.
//
// The chunk form of chunk64.hip (same recursions, same adjoint; see its header for the
// notation), cut the other way: there one workgroup walks a sequence chunk by chunk with
// the state in registers, here every (b, h, 32-token chunk) is a workgroup of its own and
// only the three short recursions that join the chunks run along the sequence, each as a
// small scan kernel over values the chunk kernels left in memory:
//   forward   lam at the chunk starts, from the chunks' 2x2 maps (Theorem 1)
//             H_{c+1} = P_c H_c + U_c,              U_c = diag(P_c) Kn^T V
//   backward  G_{c-1} = P_c G_c + E_c,              E_c = Qp^T dY
//             (c, S)  <-  (A c + B S + C, S + D),   the chunk's composed adjoint steps
// so the length of the dependent chain is one multiply-add per 32 tokens instead of a
// whole chunk round, and a batch-1 sequence fills the chip.
//
// Which is the better one is decided in c64p_supported.
//
// Range: a chunk's walk needs prod abar, prod (abar^2 + pbar lam) and their products with
// lam inside fp64's range over 32 tokens.  At widths of 64 and 128, which the
// token-recurrent kernels take without such a limit, every walk tests it, and a chunk
// that leaves it sets a flag on the device; the token-recurrent kernels are launched
// behind this path, return at once while the flag is clear, and otherwise overwrite
// every output and the saved context with theirs.  A q or v that is not finite sets the flag
// too: the products with the zeros above the diagonal of the chunk's masked matrices would carry
// it to earlier tokens (v into y; q, in the backward, into the gradients of later ones).
//
// Saved context: that of chunk64.hip (lam at every chunk start [BH][nchunk][dk], the
// states at every chunk start and after the last token [BH][nchunk+1][dk][dv]), followed
// at widths of 64 and 128 by the flag; the region is at least recurrent_saved_bytes long.
#include "kla_chunk64.hpp"
#include "kla_internal.hpp"

namespace kla {
namespace {

constexpr int C = kC64;

// Sequences bh0 .. bh0 + nb - 1 and chunks c0 .. c0 + nc - 1 of them: what one pass of
// the kernels covers.  Per-chunk work buffers are indexed [local bh][local chunk].
struct Win {
    int bh0, nb, c0, nc;
};

// The states of a window: those of local sequence i start at base + i * seq, slot j
// (chunk start c0 + j) dk dv doubles further each.
struct States {
    double* base;
    size_t seq;
};

// Threads of a workgroup: a lane walks C DK / NT tokens, 8 at dk >= 64.  The contraction
// kernels are slower on twice the threads at dk = 64 (more group maps to chain: par_adj_kernel
// 50 against 45 us at 960 chunks), par_grad_kernel, which keeps five values per token, is
// faster (24.6 against 27.1 us): GRAD.
template <int DK, bool GRAD = false>
struct Par {
    static constexpr int NT = DK == 128 || (GRAD && DK == 64) ? 512 : 256;
    static constexpr int W = NT / 64, G = NT / DK, TPG = C / G;
    static constexpr int PQ = DK + 1;
};

struct Ins {
    const float *q, *k, *a, *p, *r;
    const float *oa, *op, *od;   // OU parameters, or none
};

struct Tok {   // a window's workgroup: its (b, h), chunk and token rows
    int bh, b, h, c, i, j, nt;   // i: local bh, j: local chunk
    size_t tok0;
    __device__ Tok(const Shape& s, const Win& w) {
        j = blockIdx.x % w.nc;
        i = blockIdx.x / w.nc;
        bh = w.bh0 + i;
        b = bh / s.H;
        h = bh % s.H;
        c = w.c0 + j;
        nt = min(C, s.T - c * C);
        tok0 = (size_t)b * s.T + (size_t)c * C;
    }
};

template <int DK, int TPG, bool TI>
__device__ __forceinline__ void load_lane(WalkIn<DK, TPG, TI>& in, const Ins& g, const Shape& s,
                                          const Tok& t, int n, int gq) {
    if constexpr (TI) ou_gates(g.oa[t.h * DK + n], g.op[t.h * DK + n], g.od[t.h * DK + n], in.ca, in.cp);
    in.load(ChunkBufs(TI ? nullptr : g.a, TI ? nullptr : g.p, g.k, g.q, g.r, t.tok0, s.H, t.h, DK, t.nt), s.H, n,
            gq * TPG, t.nt);
}

// Range test of a walk: at widths up to 32 the sum of Qp Kn (finite exactly while every
// one is, as in chunk64.hip); at wider ones every factor well inside fp64's normal range.
template <bool WIDE>
struct Range {
    double sum = 0.0;
    bool bad = false;
    __device__ void token(double qp, double kn, double z, double A, double R) {
        if constexpr (WIDE)   // z, 1 / (x A) and P = A / z
            bad = bad || !(z >= 1.0e-270 && z <= 1.0e270 && R <= 1.0e290 && A >= 1.0e-290 * z && A <= 1.0e290 * z);
        else
            sum = fma(qp, kn, sum);
    }
    __device__ void end(double x, double A) {
        if constexpr (WIDE) bad = bad || !(A >= 1.0e-270 && x <= 1.0e270);
    }
    __device__ void report(int* flag) const {
        if (flag && (WIDE ? bad : !(fabs(sum) <= 1.0e300))) *flag = 1;
    }
};

// four values of a tile, whose sum is finite exactly while they are
__device__ __forceinline__ bool all_finite(const d4& x) { return fabs((x[0] + x[1]) + (x[2] + x[3])) <= 1.0e300; }

// Per token of a lane, what its walk leaves for the adjoint walk.
template <int TPG>
struct Kept {
    double lam_p[TPG], P[TPG], il[TPG], rho[TPG], irho[TPG];
};

// ---------------------------------------------------------------- forward, precision
// The chunk's 2x2 map of (x, z) (images of (1, 0) and (0, 1), scaled by the largest entry
// after each group: the map is projective).
template <int DK, bool TI>
__global__ __launch_bounds__(Par<DK>::NT) void par_map_kernel(Shape s, Win w, Ins g, double* __restrict__ map) {
    using P = Par<DK>;
    __shared__ double qs[P::G * 5 * DK];
    const Tok t(s, w);
    const int n = threadIdx.x % DK, gq = threadIdx.x / DK;
    WalkIn<DK, P::TPG, TI> in;
    load_lane(in, g, s, t, n, gq);
    group_transfer(in, qs, gq, n);
    __syncthreads();
    if (gq) return;
    double x0 = qs[0 * DK + n], z0 = qs[1 * DK + n], x1 = qs[2 * DK + n], z1 = qs[3 * DK + n];
#pragma unroll
    for (int g2 = 1; g2 < P::G; ++g2) {
        const double* m = qs + g2 * 5 * DK;
        const double m00 = m[0 * DK + n], m10 = m[1 * DK + n], m01 = m[2 * DK + n], m11 = m[3 * DK + n];
        const double nx0 = fma(m00, x0, m01 * z0), nz0 = fma(m10, x0, m11 * z0);
        const double nx1 = fma(m00, x1, m01 * z1), nz1 = fma(m10, x1, m11 * z1);
        const double sc = rcpa(fmax(fmax(nx0, nz0), fmax(nx1, nz1)));
        x0 = nx0 * sc;
        z0 = nz0 * sc;
        x1 = nx1 * sc;
        z1 = nz1 * sc;
    }
    double* o = map + ((size_t)t.i * w.nc + t.j) * 4 * DK + n;
    o[0 * DK] = x0;
    o[1 * DK] = z0;
    o[2 * DK] = x1;
    o[3 * DK] = z1;
}

// lam at the window's chunk starts, lam[(i lseq + j) dk + n]; carry[bh dk + n]: lam at the
// window's start (after the first window) and, on return, after its last chunk.
__global__ __launch_bounds__(64) void par_lam_kernel(Win w, int dk, const double* __restrict__ map,
                                                     const float* __restrict__ lam0, double* __restrict__ carry,
                                                     double* __restrict__ lam, size_t lseq, float* __restrict__ lamT,
                                                     int* __restrict__ flag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (flag && i == 0) *flag = 0;   // cleared before the first kernel that may set it
    if (i >= w.nb * dk) return;
    const int n = i % dk, il = i / dk;
    const size_t e = (size_t)w.bh0 * dk + i;
    double x = w.c0 ? carry[i] : lam0 ? (double)lam0[e] : 1.0;
    const double* m = map + (size_t)il * w.nc * 4 * dk + n;
    double* o = lam + (size_t)il * lseq + n;
    constexpr int U = 8;   // the maps of U chunks are loaded while those of the U before are applied
    double b[U][4], nx[U][4];
    auto load = [&](double (&d)[U][4], int j0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) d[u][r] = m[((size_t)min(j0 + u, w.nc - 1) * 4 + r) * dk];
    };
    load(nx, 0);
    for (int j0 = 0; j0 < w.nc; j0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) b[u][r] = nx[u][r];
        load(nx, j0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u < w.nc) {
                o[(size_t)(j0 + u) * dk] = x;
                x = fma(b[u][0], x, b[u][2]) * rcpa(fma(b[u][1], x, b[u][3]));
            }
    }
    carry[i] = x;
    if (lamT) lamT[e] = (float)x;
}

// ---------------------------------------------------------------- chunk contributions to the states
// ADJ = false: U = diag(P_C) Kn^T V into slot j + 1; ADJ = true: E = Qp^T dY into slot j.
// Also the chunk's gate product P_C.  fp64 MFMA bound: dk dv / 256 tiles of 8 products of
// 64 cycles over the CU's four matrix cores, 1 us at 64 x 64; the 16-channel columns of the
// value rows go straight from memory into the B operands.
template <int DK, int DV, bool TI, bool ADJ>
__global__ __launch_bounds__(Par<DK>::NT) void par_state_kernel(Shape s, Win w, Ins g, const float* __restrict__ val,
                                                                const double* __restrict__ lam, size_t lseq,
                                                                States st, double* __restrict__ pc, int* flag) {
    using P = Par<DK>;
    constexpr int PQ = P::PQ, TPG = P::TPG, G = P::G, W = P::W, NTN = DK / 16, NTD = DV / 16;
    __shared__ double sM[C * PQ], qs[G * 5 * DK], sPC[DK];
    const Tok t(s, w);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = tid % DK, gq = tid / DK, H = s.H;
    WalkIn<DK, TPG, TI> in;
    load_lane(in, g, s, t, n, gq);
    group_transfer(in, qs, gq, n);
    const double lam0 = lam[(size_t)t.i * lseq + (size_t)t.j * DK + n];
    __syncthreads();
    double x, z, A;
    chain_start<DK, G>(qs, gq, n, lam0, x, z, A);
    constexpr bool WIDE = DK > 32 || DV > 32;
    Range<WIDE> range;
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const double av = in.A(j), kv = in.K(j);
        const double kr = kv * in.R(j);
        const double zn = fma(in.P(j), x, av * av * z);
        const double xn = fma(kr * kv, zn, x);
        const double An = A * av;
        const double R = rcpa(xn * An);
        const double qp = in.Q(j) * An * (An * R), kn = kr * zn * (xn * R);
        range.token(qp, kn, zn, An, R);
        sM[(gq * TPG + j) * PQ + n] = ADJ ? qp : kn;
        x = xn;
        z = zn;
        A = An;
    }
    range.end(x, A);
    range.report(flag);
    if (gq == G - 1) {
        const double d = A * rcpa(z);
        sPC[n] = d;
        pc[((size_t)t.i * w.nc + t.j) * DK + n] = d;
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4, tn = wave % NTN;
    constexpr int WD = W / NTN > 0 ? W / NTN : 1;   // waves per 16 key slots
    const rsrc_t rv = make_rsrc(val + (t.tok0 * H + t.h) * DV, (uint32_t)((t.nt - 1) * H * DV + DV) * 4);
    double* out = st.base + (size_t)t.i * st.seq + (size_t)(ADJ ? t.j : t.j + 1) * DK * DV;
    bool finite = true;
    double av[C / 4];
#pragma unroll
    for (int k4 = 0; k4 < C / 4; ++k4) av[k4] = sM[(4 * k4 + lk) * PQ + 16 * tn + li];
    for (int td = wave / NTN; td < NTD; td += WD) {
        float bv[C / 4];
#pragma unroll
        for (int k4 = 0; k4 < C / 4; ++k4) bv[k4] = bld32(rv, (uint32_t)((4 * k4 + lk) * H * DV + 16 * td + li) * 4);
        d4 acc = zero_d4();
#pragma unroll
        for (int k4 = 0; k4 < C / 4; ++k4) acc = mfma64(av[k4], (double)bv[k4], acc);
        if constexpr (WIDE && !ADJ) finite = finite && all_finite(acc);   // a v that is not shows in every slot
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * tn + drow(r, lane);
            out[(size_t)row * DV + 16 * td + li] = ADJ ? acc[r] : acc[r] * sPC[row];
        }
    }
    if (flag && !finite) *flag = 1;
}

// Scan of the states along the window's chunks, one thread per element.
// REV = false: slots 1 .. nc hold U and become the states, slot 0 the state at the window's
// start: eta0 (first window) or carry.  REV = true: slots nc - 1 .. 0 hold E and become the
// adjoints of the chunks' last states, starting from detaT (last window) or carry.  carry
// receives the value that leaves the window; fin (etaT / deta0), where given, its rounding.
template <bool REV>
__global__ __launch_bounds__(256) void par_scan_kernel(Win w, int dk, int dv, const double* __restrict__ pc, States st,
                                                       bool first, const float* __restrict__ init,
                                                       double* __restrict__ carry, float* __restrict__ fin) {
    const size_t per = (size_t)dk * dv, i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= w.nb * per) return;
    const size_t il = i / per, e = i % per;
    const size_t ge = (size_t)w.bh0 * per + i;
    double x = first ? (init ? (double)init[ge] : 0.0) : carry[i];
    double* o = st.base + il * st.seq + e;
    const double* pcn = pc + il * w.nc * dk + e / dv;
    constexpr int U = 8;   // chunks loaded before their steps
    if (!REV) o[0] = x;
    for (int j0 = 0; j0 < w.nc; j0 += U) {
        double u[U], p[U];
#pragma unroll
        for (int m = 0; m < U; ++m) {
            const int j = min(j0 + m, w.nc - 1), jj = REV ? w.nc - 1 - j : j;
            u[m] = o[(size_t)(REV ? jj : jj + 1) * per];
            p[m] = pcn[(size_t)jj * dk];
        }
#pragma unroll
        for (int m = 0; m < U; ++m)
            if (j0 + m < w.nc) {
                const int jj = REV ? w.nc - 1 - (j0 + m) : j0 + m;
                if (REV) {
                    o[(size_t)jj * per] = x;
                    x = fma(p[m], x, u[m]);
                } else {
                    x = fma(p[m], x, u[m]);
                    o[(size_t)(jj + 1) * per] = x;
                }
            }
    }
    carry[i] = x;
    if (fin) fin[ge] = (float)x;
}

// ---------------------------------------------------------------- forward, readout
// y = M(Qp Kn^T) V + Qp H_c, yvar.  The chunk-start state and V go straight from memory
// into the B operands.
template <int DK, int DV, bool TI>
__global__ __launch_bounds__(Par<DK>::NT) void par_out_kernel(Shape s, Win w, Ins g, const float* __restrict__ val,
                                                              const double* __restrict__ lam, size_t lseq, States st,
                                                              float* __restrict__ y, float* __restrict__ yvar,
                                                              int* flag) {
    using P = Par<DK>;
    constexpr int PQ = P::PQ, TPG = P::TPG, G = P::G, W = P::W, NTD = DV / 16, PS = C + 1, NT = P::NT;
    __shared__ double sQp[C * PQ], sKn[C * PQ], sS[C * PS];
    __shared__ double qs[G * 5 * DK > C * PQ ? G * 5 * DK : C * PQ];   // group transfers, then q^2 / lam
    const Tok t(s, w);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = tid % DK, gq = tid / DK, H = s.H;
    WalkIn<DK, TPG, TI> in;
    load_lane(in, g, s, t, n, gq);
    group_transfer(in, qs, gq, n);
    const double lam0 = lam[(size_t)t.i * lseq + (size_t)t.j * DK + n];
    __syncthreads();
    double x, z, A, wv[TPG];
    chain_start<DK, G>(qs, gq, n, lam0, x, z, A);
    float q0 = 0.f;   // zero exactly while every q is finite
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const double av = in.A(j), kv = in.K(j), qv = in.Q(j);
        q0 = fmaf(in.q[j], 0.f, q0);
        const double kr = kv * in.R(j);
        const double zn = fma(in.P(j), x, av * av * z);
        const double xn = fma(kr * kv, zn, x);
        const double An = A * av;
        const double R = rcpa(xn * An);
        const double AR = An * R;   // 1 / x_t
        sQp[(gq * TPG + j) * PQ + n] = qv * An * AR;
        sKn[(gq * TPG + j) * PQ + n] = kr * zn * (xn * R);
        wv[j] = qv * qv * zn * AR;
        x = xn;
        z = zn;
        A = An;
    }
    __syncthreads();
    // S = M(Qp Kn^T): tiles (0, 0), (1, 0), (1, 1)
    for (int st3 = wave; st3 < 3; st3 += W) {
        const int si = st3 == 0 ? 0 : 1, sj = st3 == 2 ? 1 : 0;
        const d4 acc = tile_mm<DK, PQ, 1, 1, PQ>(zero_d4(), sQp + 16 * si * PQ, sKn + 16 * sj * PQ, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = drow(r, lane), j = lane & 15;
            sS[(16 * si + i) * PS + 16 * sj + j] = (si == sj && j > i) ? 0.0 : acc[r];
        }
    }
    if (yvar)
#pragma unroll
        for (int j = 0; j < TPG; ++j) qs[(gq * TPG + j) * PQ + n] = wv[j];
    __syncthreads();
    if (yvar) {   // NT / C lanes per token
        constexpr int L = NT / C;
        const int tt = tid / L, l = tid % L;
        double acc = 0.0;
        for (int m = l; m < DK; m += L) acc += qs[tt * PQ + m];
#pragma unroll
        for (int o = L / 2; o; o /= 2) acc += __shfl_xor(acc, o, 64);
        if (l == 0 && tt < t.nt) yvar[(t.tok0 + tt) * H + t.h] = (float)acc;
    }
    const int li = lane & 15, lk = lane >> 4;
    const uint32_t vbytes = (uint32_t)((t.nt - 1) * H * DV + DV) * 4;
    const rsrc_t rv = make_rsrc(val + (t.tok0 * H + t.h) * DV, vbytes);
    const rsrc_t ry = make_rsrc(y + (t.tok0 * H + t.h) * DV, vbytes);
    const double* H0 = st.base + (size_t)t.i * st.seq + (size_t)t.j * DK * DV;
    constexpr int NI = NTD >= W ? 2 : 1, NJ = NTD * 2 / NI;   // a wave's row tiles per job, jobs
#pragma unroll 1
    for (int job = wave; job < NJ; job += W) {
        const int td = job % NTD, i0 = NI == 2 ? 0 : job / NTD;
        d4 acc[NI];
        double hv[DK / 4];
        float bv[C / 4];
#pragma unroll
        for (int k4 = 0; k4 < DK / 4; ++k4) hv[k4] = H0[(size_t)(4 * k4 + lk) * DV + 16 * td + li];
#pragma unroll
        for (int k4 = 0; k4 < C / 4; ++k4) bv[k4] = bld32(rv, (uint32_t)((4 * k4 + lk) * H * DV + 16 * td + li) * 4);
#pragma unroll
        for (int m = 0; m < NI; ++m) {
            const int ti = i0 + m;
            acc[m] = zero_d4();
#pragma unroll
            for (int k4 = 0; k4 < DK / 4; ++k4) acc[m] = mfma64(sQp[(16 * ti + li) * PQ + 4 * k4 + lk], hv[k4], acc[m]);
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) acc[m] = mfma64(sS[(16 * ti + li) * PS + 4 * k4 + lk], (double)bv[k4], acc[m]);
            if (ti == 1)
#pragma unroll
                for (int k4 = 4; k4 < 8; ++k4)
                    acc[m] = mfma64(sS[(16 * ti + li) * PS + 4 * k4 + lk], (double)bv[k4], acc[m]);
#pragma unroll
            for (int r = 0; r < 4; ++r)   // rows past the chunk's last token fall outside the buffer
                bst32(ry, (uint32_t)((16 * ti + drow(r, lane)) * H * DV + 16 * td + li) * 4, (float)acc[m][r]);
        }
    }
    if constexpr (DK > 32 || DV > 32)   // at the end: before the walk the branch costs registers, and waves
        if (flag && !(q0 == 0.f)) *flag = 1;
}

// ---------------------------------------------------------------- backward, contractions and adjoint summary
// The lane's walk with everything the adjoint needs kept (see chunk64.hip).
template <int DK, int TPG, bool TI>
__device__ __forceinline__ void walk_kept(const WalkIn<DK, TPG, TI>& in, double x, double z, double A, Kept<TPG>& kp) {
    double izp = rcpa(z);
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const double av = in.A(j), kv = in.K(j);
        const double kr = kv * in.R(j);
        const double zn = fma(in.P(j), x, av * av * z);
        const double xn = fma(kr * kv, zn, x);
        const double An = A * av;
        const double R = rcpa(xn * An), iz = rcpa(zn);
        const double AR = An * R;   // 1 / x_t
        kp.lam_p[j] = x * izp;
        kp.P[j] = An * iz;
        kp.il[j] = zn * AR;
        kp.rho[j] = z * iz;
        kp.irho[j] = zn * izp;   // 1 / rho_t = z_t / z_{t-1}
        izp = iz;
        x = xn;
        z = zn;
        A = An;
    }
}

// Adjoint pass 1 over the lane's tokens in reverse, composed into
// c_out = Am c_in + Bm S_in + Cm, S_out = S_in + Dm, into qs[gq][4][DK].
template <int DK, int TPG, bool TI>
__device__ __forceinline__ void adjoint_summary(const WalkIn<DK, TPG, TI>& in, const Kept<TPG>& kp,
                                                const double (&dqt)[TPG], const double (&dkh)[TPG],
                                                const float (&gv)[TPG], double* qs, int gq, int n) {
    double Am = 1.0, Bm = 0.0, Cm = 0.0, Dm = 0.0;
#pragma unroll
    for (int j = TPG - 1; j >= 0; --j) {
        const double qv = in.Q(j), av = in.A(j), qi = qv * kp.il[j];
        const double u = qi * dqt[j] - in.K(j) * in.R(j) * dkh[j];
        const double w = qi * fma(qv, (double)gv[j], dqt[j]) * kp.il[j];
        const double al = av * av * kp.rho[j] * kp.rho[j], be = in.P(j) * kp.rho[j];
        Cm = al * Cm - be * Dm - (al * w + be * u);
        Bm = al * Bm - be;
        Am = al * Am;
        Dm = Dm + u;
    }
    qs[(gq * 4 + 0) * DK + n] = Am;
    qs[(gq * 4 + 1) * DK + n] = Bm;
    qs[(gq * 4 + 2) * DK + n] = Cm;
    qs[(gq * 4 + 3) * DK + n] = Dm;
}

template <int TPG>
__device__ __forceinline__ void load_gv(float (&gv)[TPG], const float* dyvar, const Shape& s, const Tok& t, int gq) {
    const rsrc_t rg = make_rsrc(dyvar + t.tok0 * s.H + t.h, dyvar ? (uint32_t)((t.nt - 1) * s.H + 1) * 4 : 0u);
#pragma unroll
    for (int j = 0; j < TPG; ++j) gv[j] = bld32(rg, (uint32_t)((gq * TPG + j) * s.H) * 4);
}

// One chunk: S = M(Qp Kn^T), B = M(dY V^T), then
//   dV = S^T dY + Kn Gs,  X = dY H_c^T + B Kn,  Y = V Gs^T + B^T Qp    (Gs = diag(P_C) G_c)
// and the chunk's composed adjoint step coef [4][dk].  dqt = P X and dkh = Y / P go to
// xy [2][C][dk] for par_grad_kernel.  X and Y stay in the accumulators until every wave is
// done with Qp and Kn and then take their place in LDS.  The state operands of X and Y run
// along a row of H_c / G_c per lane (lane group g takes channels g dv / 4 ..; the
// contraction index may be permuted), so each lane reads whole cache lines; 624 products of
// 64 cycles over four matrix cores at 64 x 64, 4.2 us.
template <int DK, int DV, bool TI>
__global__ __launch_bounds__(Par<DK>::NT) void par_adj_kernel(Shape s, Win w, Ins g, const float* __restrict__ val,
                                                              const float* __restrict__ dy,
                                                              const float* __restrict__ dyvar,
                                                              const double* __restrict__ lam, size_t lseq, States sh,
                                                              States sg, float* __restrict__ dv,
                                                              double* __restrict__ xy, double* __restrict__ coef,
                                                              int* flag) {
    using P = Par<DK>;
    constexpr int PQ = P::PQ, TPG = P::TPG, G = P::G, W = P::W, NT = P::NT, PS = C + 1, PD = DV + 1;
    constexpr int NTN = DK / 16, NTD = DV / 16;
    __shared__ double sQp[C * PQ], sKn[C * PQ], sPC[DK];
    // the group transfers, then S and B, then the adjoint summaries of the groups
    __shared__ double sU[G * 5 * DK > 2 * C * PS ? G * 5 * DK : 2 * C * PS];
    double *qs = sU, *sS = sU, *sB = sU + C * PS;
    __shared__ float sV[C * PD], sD[C * PD];
    const Tok t(s, w);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = tid % DK, gq = tid / DK, H = s.H;
    WalkIn<DK, TPG, TI> in;
    load_lane(in, g, s, t, n, gq);
    float gv[TPG];
    load_gv(gv, dyvar, s, t, gq);
    const uint32_t vbytes = (uint32_t)((t.nt - 1) * H * DV + DV) * 4;
    const size_t v0 = (t.tok0 * H + t.h) * DV;
    {
        const rsrc_t rv = make_rsrc(val + v0, vbytes), rd = make_rsrc(dy + v0, vbytes);
#pragma unroll
        for (int m = 0; m < C * DV / NT; ++m) {
            const int e = tid + NT * m, tt = e / DV, d = e % DV;
            sV[tt * PD + d] = bld32(rv, (uint32_t)(tt * H * DV + d) * 4);
            sD[tt * PD + d] = bld32(rd, (uint32_t)(tt * H * DV + d) * 4);
        }
    }
    group_transfer(in, qs, gq, n);
    const double lam0 = lam[(size_t)t.i * lseq + (size_t)t.j * DK + n];
    __syncthreads();
    double x0, z0, A0;
    chain_start<DK, G>(qs, gq, n, lam0, x0, z0, A0);
    Range<(DK > 32 || DV > 32)> range;
    {
        double x = x0, z = z0, A = A0;
#pragma unroll
        for (int j = 0; j < TPG; ++j) {
            const double av = in.A(j), kv = in.K(j);
            const double kr = kv * in.R(j);
            const double zn = fma(in.P(j), x, av * av * z);
            const double xn = fma(kr * kv, zn, x);
            const double An = A * av;
            const double R = rcpa(xn * An);
            const double qp = in.Q(j) * An * (An * R), kn = kr * zn * (xn * R);
            range.token(qp, kn, zn, An, R);
            sQp[(gq * TPG + j) * PQ + n] = qp;
            sKn[(gq * TPG + j) * PQ + n] = kn;
            x = xn;
            z = zn;
            A = An;
        }
        if (gq == G - 1) sPC[n] = A * rcpa(z);
    }
    if (DK <= 32 && DV <= 32) range.report(flag);
    __syncthreads();
    // ---- S and B, tiles (0, 0), (1, 0), (1, 1) of each
    for (int job = wave; job < 6; job += W) {
        const int st3 = job % 3, si = st3 == 0 ? 0 : 1, sj = st3 == 2 ? 1 : 0;
        const int li = lane & 15, lk = lane >> 4;
        d4 acc = zero_d4();
        double* dst = job < 3 ? sS : sB;
        if (job < 3) {
            acc = tile_mm<DK, PQ, 1, 1, PQ>(acc, sQp + 16 * si * PQ, sKn + 16 * sj * PQ, lane);
        } else {
#pragma unroll
            for (int k4 = 0; k4 < DV / 4; ++k4)
                acc = mfma64((double)sD[(16 * si + li) * PD + 4 * k4 + lk], (double)sV[(16 * sj + li) * PD + 4 * k4 + lk],
                             acc);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = drow(r, lane), j = lane & 15;
            dst[(16 * si + i) * PS + 16 * sj + j] = (si == sj && j > i) ? 0.0 : acc[r];
        }
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    const double* H0 = sh.base + (size_t)t.i * sh.seq + (size_t)t.j * DK * DV;
    const double* G0 = sg.base + (size_t)t.i * sg.seq + (size_t)t.j * DK * DV;
    // ---- dV, 16 tokens x 16 channels at a time
    {
        const rsrc_t rdv = make_rsrc(dv + v0, vbytes);
        double sum = 0.0;   // of all outputs: finite exactly while they are
        constexpr int NI = NTD >= W ? 2 : 1, NJ = NTD * 2 / NI;
#pragma unroll 1
        for (int job = wave; job < NJ; job += W) {
            const int td = job % NTD, i0 = NI == 2 ? 0 : job / NTD;
            double gvv[DK / 4];
#pragma unroll
            for (int k4 = 0; k4 < DK / 4; ++k4)
                gvv[k4] = G0[(size_t)(4 * k4 + lk) * DV + 16 * td + li] * sPC[4 * k4 + lk];
#pragma unroll
            for (int m = 0; m < NI; ++m) {
                const int tj = i0 + m;
                d4 acc = zero_d4();
#pragma unroll
                for (int k4 = 0; k4 < DK / 4; ++k4)
                    acc = mfma64(sKn[(16 * tj + li) * PQ + 4 * k4 + lk], gvv[k4], acc);
                for (int k4 = 4 * tj; k4 < 8; ++k4)   // tokens i >= 16 tj
                    acc = mfma64(sS[(4 * k4 + lk) * PS + 16 * tj + li], (double)sD[(4 * k4 + lk) * PD + 16 * td + li], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    bst32(rdv, (uint32_t)((16 * tj + drow(r, lane)) * H * DV + 16 * td + li) * 4, (float)acc[r]);
                sum += (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
        }
        // a dY that is not finite has met the zeros of S: the wave's tiles again without them, so that
        // it stays out of the tokens after its own
        if (__any(!(fabs(sum) <= 1.0e300)))
#pragma unroll 1
            for (int e = 0; e < (NJ - wave + W - 1) / W * NI * 4; ++e) {
                const int job = wave + e / (NI * 4) * W, tj = NI == 2 ? e / 4 % 2 : job / NTD;
                const int j = 16 * tj + drow(e % 4, lane), d = 16 * (job % NTD) + li;
                double x = 0.0;
#pragma unroll 1   // here and below: unrolled, the registers of this rare path cost the kernel a wave per SIMD
                for (int m = 0; m < DK; ++m) x = fma(sKn[j * PQ + m], G0[(size_t)m * DV + d] * sPC[m], x);
#pragma unroll 1
                for (int i = j; i < C; ++i) x = fma(sS[i * PS + j], (double)sD[i * PD + d], x);
                bst32(rdv, (uint32_t)(j * H * DV + d) * 4, (float)x);
            }
    }
    // ---- X, Y: wave's key-slot tile nn and token tiles tq0 .. tq0 + NX - 1
    constexpr int NX = 2 * NTN >= 2 * W ? 2 : 1;
    static_assert(NTN <= W, "one key-slot tile per wave");
    const int nn = wave % NTN, tq0 = NX == 2 ? 0 : wave / NTN;
    const bool own = tq0 < 2;
    d4 xa[NX], ya[NX];
#pragma unroll
    for (int m = 0; m < NX; ++m) xa[m] = ya[m] = zero_d4();
    if (own) {
        const double* hr = H0 + (size_t)(16 * nn + li) * DV + lk * (DV / 4);
        const double* gr = G0 + (size_t)(16 * nn + li) * DV + lk * (DV / 4);
        constexpr int B8 = DV / 4 < 8 ? DV / 4 : 8;   // state values per lane and batch
#pragma unroll 1
        for (int b8 = 0; b8 < DV / 4; b8 += B8) {
            double hv[B8], gg[B8];
#pragma unroll
            for (int e = 0; e < B8; e += 2) {
                const double2 h2 = *reinterpret_cast<const double2*>(hr + b8 + e);
                const double2 g2 = *reinterpret_cast<const double2*>(gr + b8 + e);
                hv[e] = h2.x;
                hv[e + 1] = h2.y;
                gg[e] = g2.x;
                gg[e + 1] = g2.y;
            }
#pragma unroll
            for (int m = 0; m < NX; ++m) {
                const int row = 16 * (tq0 + m) + li;
#pragma unroll
                for (int e = 0; e < B8; ++e) {
                    const int d = lk * (DV / 4) + b8 + e;
                    xa[m] = mfma64((double)sD[row * PD + d], hv[e], xa[m]);
                    ya[m] = mfma64((double)sV[row * PD + d], gg[e], ya[m]);
                }
            }
        }
        const double pcn = sPC[16 * nn + li];
#pragma unroll
        for (int m = 0; m < NX; ++m) {
            const int tq = tq0 + m;
#pragma unroll
            for (int r = 0; r < 4; ++r) ya[m][r] *= pcn;
            for (int k4 = 0; k4 < 4 + 4 * tq; ++k4)   // tokens j < 16 (tq + 1)
                xa[m] = mfma64(sB[(16 * tq + li) * PS + 4 * k4 + lk], sKn[(4 * k4 + lk) * PQ + 16 * nn + li], xa[m]);
            for (int k4 = 4 * tq; k4 < 8; ++k4)   // tokens t >= 16 tq
                ya[m] = mfma64(sB[(4 * k4 + lk) * PS + 16 * tq + li], sQp[(4 * k4 + lk) * PQ + 16 * nn + li], ya[m]);
        }
    }
    __syncthreads();   // Qp, Kn read
    if (own)
#pragma unroll
        for (int m = 0; m < NX; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = (16 * (tq0 + m) + drow(r, lane)) * PQ + 16 * nn + li;
                sQp[o] = xa[m][r];
                sKn[o] = ya[m][r];
            }
    __syncthreads();
    // ---- the chunk's composed adjoint step
    Kept<TPG> kp;
    walk_kept(in, x0, z0, A0, kp);
    double dqt[TPG], dkh[TPG];
    double* o = xy + ((size_t)t.i * w.nc + t.j) * 2 * C * DK;
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const int tt = gq * TPG + j;
        dqt[j] = kp.P[j] * sQp[tt * PQ + n];
        dkh[j] = sKn[tt * PQ + n] * rcpa(kp.P[j]);
        o[tt * DK + n] = dqt[j];
        o[(C + tt) * DK + n] = dkh[j];
    }
    adjoint_summary(in, kp, dqt, dkh, gv, qs, gq, n);   // S and B were read before a barrier
    __syncthreads();
    if (gq == 0) {
        double Am = 1.0, Bm = 0.0, Cm = 0.0, Dm = 0.0;
#pragma unroll
        for (int g2 = G - 1; g2 >= 0; --g2) {
            const double A2 = qs[(g2 * 4 + 0) * DK + n], B2 = qs[(g2 * 4 + 1) * DK + n];
            const double C2 = qs[(g2 * 4 + 2) * DK + n], D2 = qs[(g2 * 4 + 3) * DK + n];
            Cm = fma(A2, Cm, fma(B2, Dm, C2));
            Bm = fma(A2, Bm, B2);
            Am *= A2;
            Dm += D2;
        }
        double* cf = coef + ((size_t)t.i * w.nc + t.j) * 4 * DK + n;
        cf[0 * DK] = Am;
        cf[1 * DK] = Bm;
        cf[2 * DK] = Cm;
        cf[3 * DK] = Dm;
    }
}

// (c, S) at the end of every chunk of the window, into the chunk's rows 0 and 1 of coef;
// carry [nb][2][dk].  The last window starts from dlamT and sum_d detaT H_T (hT: the final
// states, one per hseq doubles).
__global__ __launch_bounds__(64) void par_carry_kernel(Win w, int dk, int dv, bool last, double* __restrict__ coef,
                                                       double* __restrict__ carry, const float* __restrict__ dlamT,
                                                       const float* __restrict__ detaT, const double* __restrict__ hT,
                                                       size_t hseq, float* __restrict__ dlam0) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= w.nb * dk) return;
    const int n = i % dk, il = i / dk;
    const size_t e = (size_t)w.bh0 * dk + i;
    double* cr = carry + (size_t)il * 2 * dk + n;
    double c = 0.0, S = 0.0;
    if (!last) {
        c = cr[0];
        S = cr[dk];
    } else {
        if (dlamT) c = (double)dlamT[e];
        if (detaT) {
            const double* h = hT + (size_t)il * hseq + (size_t)n * dv;
            const float* d = detaT + e * dv;
#pragma unroll 8
            for (int m = 0; m < dv; ++m) S = fma((double)d[m], h[m], S);
        }
    }
    double* cf = coef + (size_t)il * w.nc * 4 * dk + n;
    constexpr int U = 8;   // the steps of U chunks are loaded while those of the U after are applied
    double b[U][4], nx[U][4];
    auto load = [&](double (&d)[U][4], int j0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) d[u][r] = cf[((size_t)max(j0 - u, 0) * 4 + r) * dk];
    };
    load(nx, w.nc - 1);
    for (int j0 = w.nc - 1; j0 >= 0; j0 -= U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) b[u][r] = nx[u][r];
        load(nx, j0 - U);   // rows of other chunks than those written below
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 - u >= 0) {
                double* o = cf + (size_t)(j0 - u) * 4 * dk;
                o[0] = c;
                o[dk] = S;
                c = fma(b[u][0], c, fma(b[u][1], S, b[u][2]));
                S += b[u][3];
            }
    }
    cr[0] = c;
    cr[dk] = S;
    if (dlam0) dlam0[e] = (float)c;
}

// The gradients of a chunk's tokens from dqt, dkh and (c, S) at its end: the walk, the
// groups' summaries chained from the chunk end, and adjoint pass 2.
template <int DK, bool TI>
__global__ __launch_bounds__((Par<DK, true>::NT)) void par_grad_kernel(Shape s, Win w, Ins g,
                                                               const float* __restrict__ dyvar,
                                                               const double* __restrict__ lam, size_t lseq,
                                                               const double* __restrict__ xy,
                                                               const double* __restrict__ coef, float* __restrict__ dq,
                                                               float* __restrict__ dk, float* __restrict__ da,
                                                               float* __restrict__ dp, float* __restrict__ dr,
                                                               double* __restrict__ oupart) {
    using P = Par<DK, true>;
    constexpr int PQ = P::PQ, TPG = P::TPG, G = P::G, NT = P::NT;
    __shared__ double qs[G * 5 * DK], qa[G * 4 * DK], sR[C * PQ];
    const Tok t(s, w);
    const int tid = threadIdx.x, n = tid % DK, gq = tid / DK, H = s.H;
    WalkIn<DK, TPG, TI> in;
    load_lane(in, g, s, t, n, gq);
    float gv[TPG];
    load_gv(gv, dyvar, s, t, gq);
    double dqt[TPG], dkh[TPG];
    const double* o = xy + ((size_t)t.i * w.nc + t.j) * 2 * C * DK;
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        dqt[j] = o[(gq * TPG + j) * DK + n];
        dkh[j] = o[(C + gq * TPG + j) * DK + n];
    }
    const double* cf = coef + ((size_t)t.i * w.nc + t.j) * 4 * DK + n;
    double cc = cf[0], SS = cf[DK];
    const double lam0 = lam[(size_t)t.i * lseq + (size_t)t.j * DK + n];
    group_transfer(in, qs, gq, n);
    __syncthreads();
    double x, z, A;
    chain_start<DK, G>(qs, gq, n, lam0, x, z, A);
    Kept<TPG> kp;
    walk_kept(in, x, z, A, kp);
    adjoint_summary(in, kp, dqt, dkh, gv, qa, gq, n);
    __syncthreads();
#pragma unroll
    for (int g2 = G - 1; g2 >= 1; --g2) {   // through the later groups
        const double A2 = qa[(g2 * 4 + 0) * DK + n], B2 = qa[(g2 * 4 + 1) * DK + n];
        const double C2 = qa[(g2 * 4 + 2) * DK + n], D2 = qa[(g2 * 4 + 3) * DK + n];
        const bool use = g2 > gq;
        const double cn = fma(A2, cc, fma(B2, SS, C2));
        cc = use ? cn : cc;
        SS = use ? SS + D2 : SS;
    }
    const size_t k0 = (t.tok0 * H + t.h) * DK;
    const uint32_t kbytes = (uint32_t)((t.nt - 1) * H * DK + DK) * 4;
    const rsrc_t rq = make_rsrc(dq + k0, kbytes), rk = make_rsrc(dk + k0, kbytes);
    const rsrc_t ra = make_rsrc(TI ? dq : da + k0, TI ? 0u : kbytes), rp = make_rsrc(TI ? dq : dp + k0, TI ? 0u : kbytes);
    double sum_da = 0.0, sum_dp = 0.0;
#pragma unroll
    for (int j = TPG - 1; j >= 0; --j) {
        const int tt = gq * TPG + j;
        const double qv = in.Q(j), kv = in.K(j), rv = in.R(j), av = in.A(j), qi = qv * kp.il[j];
        const double r2 = kp.rho[j] * kp.rho[j];
        SS += qi * dqt[j] - kv * rv * dkh[j];
        const double gl = cc - qi * fma(qv, (double)gv[j], dqt[j]) * kp.il[j];
        const double drho = fma(gl, kp.lam_p[j], SS * kp.irho[j]);
        const double dav = fma(-2.0 * av * r2, drho, SS * rcpa(av));
        const double dpv = -kp.lam_p[j] * r2 * drho;
        sR[tt * PQ + n] = fma(kv * kv, gl, kv * dkh[j]);
        cc = fma(av * av * r2, gl, -(in.P(j) * kp.rho[j]) * SS);
        const uint32_t vo = (uint32_t)(tt * H * DK + n) * 4;   // tokens past the end fall outside
        bst32(rq, vo, (float)(fma(2.0 * qv, (double)gv[j], dqt[j]) * kp.il[j]));
        bst32(rk, vo, (float)fma(2.0 * kv * rv, gl, rv * dkh[j]));
        if constexpr (TI) {
            if (tt < t.nt) {
                sum_da += dav;
                sum_dp += dpv;
            }
        } else {
            bst32(ra, vo, (float)dav);
            bst32(rp, vo, (float)dpv);
        }
    }
    if constexpr (TI) {
        qs[gq * DK + n] = sum_da;   // the transfers were read before a barrier
        qs[(G + gq) * DK + n] = sum_dp;
    }
    __syncthreads();
    {   // dr: the sum over the slots, NT / C lanes per token
        constexpr int L = NT / C;
        const int tt = tid / L, l = tid % L;
        double acc = 0.0;
        for (int m = l; m < DK; m += L) acc += sR[tt * PQ + m];
#pragma unroll
        for (int of = L / 2; of; of /= 2) acc += __shfl_xor(acc, of, 64);
        if (l == 0 && tt < t.nt) dr[(t.tok0 + tt) * H + t.h] = (float)acc;
    }
    if constexpr (TI)
        if (gq < 2) {   // the chunk's sums of the gate gradients [2][dk]
            double acc = 0.0;
#pragma unroll
            for (int g2 = 0; g2 < G; ++g2) acc += qs[(gq * G + g2) * DK + n];
            oupart[(((size_t)t.i * w.nc + t.j) * 2 + gq) * DK + n] = acc;
        }
}

// OU parts [2][BH][dk] += the window's chunk sums, later chunks first.
__global__ __launch_bounds__(64) void par_ou_kernel(Win w, int dk, int nbh, bool last, const double* __restrict__ sums,
                                                    double* __restrict__ part) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= w.nb * 2 * dk) return;
    const int n = i % dk, q = i / dk % 2, il = i / (2 * dk);
    double* o = part + ((size_t)q * nbh + w.bh0 + il) * dk + n;
    double acc = last ? 0.0 : *o;
#pragma unroll 8
    for (int j = w.nc - 1; j >= 0; --j) acc += sums[(((size_t)il * w.nc + j) * 2 + q) * dk + n];
    *o = acc;
}

// ---------------------------------------------------------------- host side
// Work memory of a pass is bounded: sequences are taken a batch at a time and, when one
// sequence alone is over the bound, its chunks a window at a time.
constexpr size_t kMaxWork = 192u << 20, kMinWork = 56u << 20;

size_t up(size_t x) { return (x + 255) / 256 * 256; }

struct Plan {
    int nb, nc;      // sequences per batch, chunks per window
    size_t bytes;    // work memory
};

// per (sequence, chunk) and per sequence bytes of the work buffers
template <typename PerChunk, typename PerSeq>
Plan plan(int BH, int NC, PerChunk chunk, PerSeq seq, size_t limit) {
    Plan p{BH, NC, 0};
    auto need = [&](int nb, int nc) { return (size_t)nb * (seq(nc) + (size_t)nc * chunk) + 16 * 256; };
    if (need(BH, NC) > limit) {
        const size_t one = need(1, NC);
        if (one <= limit) {
            const int most = (int)((limit - 16 * 256) / (one - 16 * 256));
            const int batches = (BH + most - 1) / most;
            p.nb = (BH + batches - 1) / batches;   // equal batches
        } else {
            p.nb = 1;
            const size_t fixed = seq(0) + 16 * 256 + (seq(1) - seq(0));
            const int most = (int)((limit - fixed) / (chunk + (seq(2) - seq(1))));
            const int wins = (NC + most - 1) / most;
            p.nc = (NC + wins - 1) / wins;
        }
    }
    p.bytes = need(p.nb, p.nc);
    return p;
}

int chunks_of(const Shape& s) { return (s.T + C - 1) / C; }
bool wide(const Shape& s) { return s.dk > 32 || s.dv > 32; }

Plan fwd_plan(const Shape& s, bool save, size_t limit) {
    const size_t d = sizeof(double), st = (size_t)s.dk * s.dv * d;
    const size_t chunk = (5 + (save ? 0 : 1)) * s.dk * d + (save ? 0 : st);   // map, P_C, lam; states
    auto seq = [&](int) { return s.dk * d + st + (save ? 0 : st); };          // lam and state carries, one more slot
    return plan(s.B * s.H, chunks_of(s), chunk, seq, limit);
}

Plan bwd_plan(const Shape& s, size_t limit) {
    const size_t d = sizeof(double), st = (size_t)s.dk * s.dv * d;
    const size_t chunk = st + (2 * (size_t)C + 4 + 1 + 2) * s.dk * d;   // adjoint state; dqt, dkh; coef, P_C, OU sums
    auto seq = [&](int) { return st + 2 * s.dk * d; };
    return plan(s.B * s.H, chunks_of(s), chunk, seq, limit);
}

struct Carver {
    char* p;
    double* operator()(size_t n) {
        double* r = reinterpret_cast<double*>(p);
        p += up(n * sizeof(double));
        return r;
    }
};

dim3 blocks(size_t n, int per) { return dim3((unsigned)((n + per - 1) / per)); }

struct SavedP {
    double *lam, *H;
    int* flag;
};
SavedP saved_par(const Shape& s, const void* saved) {
    char* p = static_cast<char*>(const_cast<void*>(saved));
    SavedP r{nullptr, nullptr, nullptr};
    if (!p) return r;
    r.lam = reinterpret_cast<double*>(p);
    r.H = r.lam + (size_t)s.B * s.H * chunks_of(s) * s.dk;
    if (wide(s)) r.flag = reinterpret_cast<int*>(p + c64p_saved_bytes(s) - 256);
    return r;
}

template <int DK, int DV, bool TI>
hipError_t fwd_par(const Shape& s, const FwdArgs& a, void* saved, void* ws, int* flag, hipStream_t st) {
    const int NC = chunks_of(s), BH = s.B * s.H;
    const bool save = saved != nullptr;
    const Plan pl = fwd_plan(s, save, kMaxWork);
    const SavedP sv = saved_par(s, saved);
    const Ins in{static_cast<const float*>(a.q), static_cast<const float*>(a.k), static_cast<const float*>(a.a),
                 static_cast<const float*>(a.p), static_cast<const float*>(a.r), a.ou_a, a.ou_p, a.ou_d};
    const float* v = static_cast<const float*>(a.v);
    Carver carve{static_cast<char*>(ws)};
    constexpr size_t ST = (size_t)DK * DV;
    double* map = carve((size_t)pl.nb * pl.nc * 4 * DK);
    double* pc = carve((size_t)pl.nb * pl.nc * DK);
    double* clam = carve((size_t)pl.nb * DK);
    double* cst = carve((size_t)pl.nb * ST);
    double* wlam = save ? nullptr : carve((size_t)pl.nb * pl.nc * DK);
    double* wst = save ? nullptr : carve((size_t)pl.nb * (pl.nc + 1) * ST);
    constexpr int NT = Par<DK>::NT;
    for (int bh0 = 0; bh0 < BH; bh0 += pl.nb)
        for (int c0 = 0; c0 < NC; c0 += pl.nc) {
            const Win w{bh0, min(pl.nb, BH - bh0), c0, min(pl.nc, NC - c0)};
            const bool last = c0 + w.nc == NC;
            double* lam = save ? sv.lam + ((size_t)bh0 * NC + c0) * DK : wlam;
            const size_t lseq = (size_t)(save ? NC : w.nc) * DK;
            const States sts{save ? sv.H + ((size_t)bh0 * (NC + 1) + c0) * ST : wst, (save ? NC + 1 : w.nc + 1) * ST};
            const dim3 grid((unsigned)(w.nb * w.nc));
            hipLaunchKernelGGL((par_map_kernel<DK, TI>), grid, dim3(NT), 0, st, s, w, in, map);
            hipLaunchKernelGGL(par_lam_kernel, blocks((size_t)w.nb * DK, 64), dim3(64), 0, st, w, DK, map, a.lam0, clam,
                               lam, lseq, last ? a.lamT : nullptr, wide(s) && bh0 == 0 && c0 == 0 ? flag : nullptr);
            hipLaunchKernelGGL((par_state_kernel<DK, DV, TI, false>), grid, dim3(NT), 0, st, s, w, in, v, lam, lseq, sts,
                               pc, flag);
            hipLaunchKernelGGL(par_scan_kernel<false>, blocks(w.nb * ST, 256), dim3(256), 0, st, w, DK, DV, pc, sts,
                               c0 == 0, a.eta0, cst, last ? a.etaT : nullptr);
            hipLaunchKernelGGL((par_out_kernel<DK, DV, TI>), grid, dim3(NT), 0, st, s, w, in, v, lam, lseq, sts,
                               static_cast<float*>(a.y), a.yvar, flag);
        }
    return hipGetLastError();
}

template <int DK, int DV, bool TI>
hipError_t bwd_par(const Shape& s, const BwdArgs& a, const void* saved, void* ws, size_t limit, int* flag,
                   hipStream_t st) {
    const int NC = chunks_of(s), BH = s.B * s.H;
    const Plan pl = bwd_plan(s, limit);
    const SavedP sv = saved_par(s, saved);
    const Ins in{static_cast<const float*>(a.q), static_cast<const float*>(a.k), static_cast<const float*>(a.a),
                 static_cast<const float*>(a.p), static_cast<const float*>(a.r), a.ou_a, a.ou_p, a.ou_d};
    const float *v = static_cast<const float*>(a.v), *dy = static_cast<const float*>(a.dy);
    Carver carve{static_cast<char*>(ws)};
    constexpr size_t ST = (size_t)DK * DV;
    double* wg = carve((size_t)pl.nb * pl.nc * ST);
    double* xy = carve((size_t)pl.nb * pl.nc * 2 * C * DK);
    double* coef = carve((size_t)pl.nb * pl.nc * 4 * DK);
    double* pc = carve((size_t)pl.nb * pl.nc * DK);
    double* ous = carve((size_t)pl.nb * pl.nc * 2 * DK);
    double* cst = carve((size_t)pl.nb * ST);
    double* ccs = carve((size_t)pl.nb * 2 * DK);
    constexpr int NT = Par<DK>::NT;
    for (int bh0 = 0; bh0 < BH; bh0 += pl.nb)
        for (int c1 = NC; c1 > 0; c1 -= pl.nc) {
            const int c0 = c1 > pl.nc ? c1 - pl.nc : 0;
            const Win w{bh0, min(pl.nb, BH - bh0), c0, c1 - c0};
            const bool last = c1 == NC, first = c0 == 0;
            const double* lam = sv.lam + ((size_t)bh0 * NC + c0) * DK;
            const size_t lseq = (size_t)NC * DK;
            const States sh{sv.H + ((size_t)bh0 * (NC + 1) + c0) * ST, (size_t)(NC + 1) * ST};
            const States sg{wg, (size_t)w.nc * ST};
            const dim3 grid((unsigned)(w.nb * w.nc));
            hipLaunchKernelGGL((par_state_kernel<DK, DV, TI, true>), grid, dim3(NT), 0, st, s, w, in, dy, lam, lseq, sg,
                               pc, nullptr);
            hipLaunchKernelGGL(par_scan_kernel<true>, blocks(w.nb * ST, 256), dim3(256), 0, st, w, DK, DV, pc, sg, last,
                               a.detaT, cst, first ? a.deta0 : nullptr);
            hipLaunchKernelGGL((par_adj_kernel<DK, DV, TI>), grid, dim3(NT), 0, st, s, w, in, v, dy, a.dyvar, lam, lseq,
                               sh, sg, static_cast<float*>(a.dv), xy, coef, flag);
            hipLaunchKernelGGL(par_carry_kernel, blocks((size_t)w.nb * DK, 64), dim3(64), 0, st, w, DK, DV, last, coef,
                               ccs, a.dlamT, a.detaT, sh.base + (size_t)w.nc * ST, sh.seq, first ? a.dlam0 : nullptr);
            hipLaunchKernelGGL((par_grad_kernel<DK, TI>), grid, dim3((Par<DK, true>::NT)), 0, st, s, w, in, a.dyvar, lam,
                               lseq, xy, coef, static_cast<float*>(a.dq), static_cast<float*>(a.dk), static_cast<float*>(a.da),
                               static_cast<float*>(a.dp), static_cast<float*>(a.dr), ous);
            if (TI)
                hipLaunchKernelGGL(par_ou_kernel, blocks((size_t)w.nb * 2 * DK, 64), dim3(64), 0, st, w, DK, BH, last,
                                   ous, static_cast<double*>(a.ou_part));
        }
    return hipGetLastError();
}

}  // namespace

// Against the kernels it replaces, forward + backward on one MI355X (a forward alone is slower
// here only with 128 value channels: 16 x 128 over 65 to 128 tokens 22 against 15 to 19 us,
// 64 x 128 over 65 tokens 26 against 22):
//   widths of 64 and 128 (token-recurrent, about 1.3 us per token at any batch up to the
//   chip's width): always from the third chunk on (2825 -> 240 us at B1 T2048 H15 64 x 64);
//   up to 64 tokens the recurrent walk is as fast as the launches here;
//   widths up to 32 (chunk64.hip, one workgroup per sequence): there 10 + 8.3 us per chunk
//   while the sequences fit one per CU, here 43 us + 0.034 (dk = 16) or 0.055 us (dk = 32)
//   per chunk of every sequence.  Measured crossings at dk = dv = 32: 64 sequences between
//   5 and 8 chunks (80 -> 63 us at 8), 128 between 8 and 16 (151 -> 143 us at 16), at 256
//   never (163 against 255 us at 16).
bool c64p_supported(const Shape& s) {
    if (s.bf16 || s.T <= 2 * C) return false;
    // a chunk's rows lie within 32 bits of byte offsets
    if ((size_t)s.H * (s.dk > s.dv ? s.dk : s.dv) * C * sizeof(float) > (size_t)1 << 32) return false;
    if (wide(s)) return true;
    return chunks_of(s) * (8.3 - (s.dk == 16 ? 0.034 : 0.055) * s.B * s.H) > 33.0;
}

bool c64p_wide(const Shape& s) { return wide(s); }

size_t c64p_saved_bytes(const Shape& s) {
    const size_t nc = chunks_of(s);
    const size_t par = (size_t)s.B * s.H * s.dk * (nc + (nc + 1) * (size_t)s.dv) * sizeof(double);
    if (!wide(s)) return par;
    const size_t rec = recurrent_saved_bytes(s);
    return up(par > rec ? par : rec) + 256;   // the range flag in the last 256 bytes
}

size_t c64p_fwd_workspace(const Shape& s, bool save) { return fwd_plan(s, save, kMaxWork).bytes; }

size_t c64p_bwd_workspace(const Shape& s, bool least) {
    const size_t a = bwd_plan(s, least ? kMinWork : kMaxWork).bytes;
    const size_t b = wide(s) ? backward_recurrent_workspace(s) : 0;   // should the range flag be set
    return a > b ? a : b;
}

const int* c64p_flag(const Shape& s, const void* saved) { return saved_par(s, saved).flag; }

#define KLA_C64P_ROW(F, TI, DK_, ...)                                  \
    if (s.dk == DK_ && s.dv == 16) return F<DK_, 16, TI>(__VA_ARGS__); \
    if (s.dk == DK_ && s.dv == 32) return F<DK_, 32, TI>(__VA_ARGS__); \
    if (s.dk == DK_ && s.dv == 64) return F<DK_, 64, TI>(__VA_ARGS__); \
    if (s.dk == DK_ && s.dv == 128) return F<DK_, 128, TI>(__VA_ARGS__);
#define KLA_C64P_CASES(F, ...)                                                                           \
    if (a.ou_a) {                                                                                        \
        KLA_C64P_ROW(F, true, 16, __VA_ARGS__) KLA_C64P_ROW(F, true, 32, __VA_ARGS__)                    \
        KLA_C64P_ROW(F, true, 64, __VA_ARGS__) KLA_C64P_ROW(F, true, 128, __VA_ARGS__)                   \
    } else {                                                                                             \
        KLA_C64P_ROW(F, false, 16, __VA_ARGS__) KLA_C64P_ROW(F, false, 32, __VA_ARGS__)                  \
        KLA_C64P_ROW(F, false, 64, __VA_ARGS__) KLA_C64P_ROW(F, false, 128, __VA_ARGS__)                 \
    }

hipError_t launch_forward_c64p(const Shape& s, const FwdArgs& a, void* saved, void* ws, int* flag, hipStream_t st) {
    if (saved && wide(s)) flag = saved_par(s, saved).flag;
    KLA_C64P_CASES(fwd_par, s, a, saved, ws, flag, st)
    return hipErrorInvalidValue;
}

hipError_t launch_backward_c64p(const Shape& s, const BwdArgs& a, const void* saved, void* ws, bool least, int* flag,
                                hipStream_t st) {
    KLA_C64P_CASES(bwd_par, s, a, saved, ws, least ? kMinWork : kMaxWork, flag, st)
    return hipErrorInvalidValue;
}

}  // namespace kla
