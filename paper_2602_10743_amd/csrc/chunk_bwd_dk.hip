// Chunked backward, key side: dq, dk, dabar, dpbar, dr and dlam0.
//
// Notation per chunk of kC = 32 tokens (local t), with P_t, Qp, Kn from the
// precision walk (kla_chunk.hpp) redone from the saved walk state:
//   H_t  = P_t (H0 + sum_{j<=t} Kn_j v_j^T)          (state rows, H0 = saved chunk-start state)
//   G    = adjoint of the chunk's last state from later tokens (detaT for the
//          last chunk), Gs = diag(P_C) G
//   B    = dY V^T                                    (kC x kC)
// then, with M() keeping j <= t,
//   X    = dY H0^T + M(B) Kn     dqt = P X   (gradient of qt = q / lam_t)
//   Y    = M(B)^T Qp + V Gs^T    dkh = Y / P (gradient of kh = r k)
//   G'   = Qp^T dY + Gs                          (carried into the previous chunk)
// The adjoint of log F_t is the reverse running sum S_t of qt dqt - kh dkh (plus
// the final-state term sum_d detaT H_T).  Over a whole chunk the attention parts of
// X and Y cancel exactly: the chunk's total of qt dqt - kh dkh is
// sum_t Qp_t (dY H0^T)_t - sum_j Kn_j (V Gs^T)_j, and S is carried from chunk to
// chunk by that total (per token, only within the chunk, by the running sum);
// summed token by token, the rounding of the large attention terms would add up
// over the sequence.  The adjoint c of lam follows
//   g_t = c_t - q_t dqt_t / lam_t^2,    c_T = dlamT,
//   c_{t-1} = abar_t^2 rho_t^2 g_t - pbar_t rho_t S_t,
// from which the input gradients follow by the chain rule through rho, lam, F
// (Theorem 1's update, differentiated by hand):
//   dq = dqt / lam,  dk = r dkh + 2 k r g,  dr = sum_n (k dkh + k^2 g),
//   drho = g lam_{t-1} + S / rho,  dabar = S / abar - 2 abar rho^2 drho,
//   dpbar = -lam_{t-1} rho^2 drho,  dlam0 = c after the first token.
// An upstream gradient gv_t of the readout variance yvar_t = sum_n q^2 / lam_t
// adds 2 q gv / lam to dq and -q^2 gv / lam^2 to g_t (YG instantiations; the
// others leave out its load and arithmetic).
//
// One workgroup per (batch, head, 64 key slots); a pair of waves owns 16 key
// slots n0 + 16 p .. + 15, and the pairs share only the dY / V tiles.  Wave e of
// a pair takes the tokens 16 e .. 16 e + 15 of each chunk in the walks:
//   walk   lanes = (slot nl = lane % 16, group g = lane / 16 of 4 tokens): each
//          lane forms its group's transfer -- the 2x2 map of (x, z) of
//          Theorem 1 over 4 tokens, with prod abar --, the four groups of each
//          half (the wave's four 16-lane rows) are chained by lane swaps from
//          the saved state at the start of the half (lam_0, or lam_16 and
//          P_16), and each lane walks its 4 tokens from the group start,
//          writing Qp and Kn (slot-major, split bf16) and keeping lam_t, P_t and
//          the reciprocals the adjoint walk needs;
//   MFMA   split by operand instead: wave 0 forms B^T and X^T (with the chunk's
//          saved start state H0 in registers), wave 1 forms B and Y^T and
//          carries G^T[dv, 16] in registers;
//   adjoint per lane: its group's tokens in reverse, once to summarise the
//          group as an affine map of the incoming (c, S), then -- the groups
//          chained through LDS -- once more for the gradients.
// The chunks are walked last to first, four LDS barriers per chunk separating
// the phases.  The next chunk's inputs go straight into LDS, requested during
// the first pass of a round's adjoint walk; the chunk's saved state rows come
// into wave 0's registers at the start of its round.
//
// What bounds it is issue: two waves per SIMD walk dependent fp32 chains between barriers,
// with LDS instructions the largest share.  The per-pair tiles are slot-major (nt_off) so that a lane
// writes its four tokens with one 8-byte store and reads them with one transposing read, the
// group summaries are one vector per slot, and the sum over slots for dr is taken in registers:
// 746 -> 418 LDS instructions in the 128 x 128 kernel.  Reads whose bytes came by direct loads
// are written out in asm with their own wait, since for the builtin the compiler also waits for
// every request in flight.  8 sequences of 2048, 16 heads of 128 x 128: 447 -> 427 us; the
// split kernel at 2 sequences: 95 -> 89 us (with OU gates 85).
//
// TI (gates from OU parameters, the same for every token of a key slot): abar
// and pbar are formed once per lane and not loaded; dabar and dpbar are not
// stored per token but summed over the lane's tokens, one part per (batch row,
// wave of the pair), for the parameter gradients.
#include <algorithm>
#include <type_traits>

#include "kla_chunk.hpp"
#include "kla_internal.hpp"

namespace kla {
namespace {

template <int DK, int DV>
struct DkCfg {
    static constexpr int NP = DK / 16 < 4 ? DK / 16 : 4;   // wave pairs, 16 key slots each
    static constexpr int NW = 2 * NP;                       // waves
    static constexpr int NTN = 16 * NP;                     // key slots per workgroup
    static constexpr int NNT = DK / NTN;                    // workgroups per (b, h)
    static constexpr int NTHR = 64 * NW;
    static constexpr int KSD = DV / 32;                     // 32-deep steps over the value channels
    static constexpr int NRD = DV / 16;                     // 16-row tiles over the value channels
    static constexpr int CPR = DV / 8;                      // 16-byte chunks per dY / V row
    static constexpr int TPV = 512 / DV;                    // rows per 1 KiB load of a dY / V tile
    static constexpr int NVL = kC / TPV;                    // 1 KiB loads per dY / V tile
    static constexpr int TQ = 16 * kC * 2;                  // bytes of a per-pair slot-major bf16 tile (nt_off)
    static constexpr int LX = 20;                           // row stride of per-pair [t][16] fp32 tiles
    static constexpr int NG = 8;                            // token groups per chunk (4 tokens each)
    // shared: dY and V tiles [2 buffers][2][kC][DV] (16-byte chunks swizzled by row)
    static constexpr int TILE = kC * DV * 2;
    static constexpr int PAIR0 = 2 * 2 * TILE;
    // per pair (offsets from the pair's base)
    static constexpr int STG = 0;                                   // [2][4][kC][16] bf16: abar, pbar, k, q
    static constexpr int RW = STG + 2 * 4 * kC * 16 * 2;            // [2][64] r words
    static constexpr int LW = RW + 2 * 64 * 4;                      // [2][64] walk state: lam_0, lam_16, P_16 [3][16]
    static constexpr int GV = LW + 2 * 64 * 4;                      // [2][64] yvar gradient (fp32)
    static constexpr int QH = GV + 2 * 64 * 4;                      // Qp, Kn split bf16 (slot, t)
    static constexpr int QL = QH + TQ, KH = QL + TQ, KL = KH + TQ;
    static constexpr int XT = KL + TQ, YT = XT + kC * LX * 4;   // X, Y fp32 [kC][LX]
    static constexpr int QS = YT + kC * LX * 4;                     // adjoint group summaries [NG][16][4] fp32
    static constexpr int PC = QS + NG * 4 * 16 * 4;                 // chunk decay P_C [16] fp32
    static constexpr int WT = PC + 16 * 4;                          // chunk totals of the state parts [2][16]
    static constexpr int PAIR = (WT + 2 * 16 * 4 + 15) / 16 * 16;
    static constexpr int BYTES = PAIR0 + NP * PAIR;   // dynamic part
    // The gradient tiles dq, dk, dabar, dpbar (slot, t) bf16 of each pair live in a
    // separate static array: they are read back while the next chunk's direct-to-LDS
    // loads are in flight, and as a distinct object they are seen not to alias those
    // loads' destinations.
    static constexpr int STATIC = NP * 4 * kC * 16 * 2;
    static_assert(DK >= 32 && DK % 16 == 0 && DV >= 32 && DV % 32 == 0, "backward tile sizes");
    static_assert(NVL >= 1 && TPV * CPR == 64, "value tile loads");
    static_assert(4 + 2 * ((NVL + NW - 1) / NW) <= 8, "requests spread over 4 tokens, two each");
    static_assert(3 + 2 * ((NVL + NW - 1) / NW) <= 8, "requests spread over 4 tokens, two each");
    static_assert(BYTES + STATIC <= 160 * 1024, "LDS budget of one workgroup");
};

// Element (row t, column d) of a swizzled [kC][DV] bf16 tile: the 16-byte chunk
// d / 8 of row t sits at chunk (d / 8) ^ (t % CPR), so that 16 consecutive rows
// read at one column fall into distinct banks.
template <int DV>
__device__ __forceinline__ const uint16_t* swz(const uint16_t* tile, int t, int d) {
    constexpr int CPR = DV / 8;
    return tile + t * DV + ((((d >> 3) ^ (t % CPR)) << 3) | (d & 7));
}

template <int DV>
__device__ __forceinline__ bf16x8 lds8_swz(const uint16_t* tile, int t, int d0) {
    return lds8(swz<DV>(tile, t, d0));
}

template <int DV>
__device__ __forceinline__ bf16x8 lds4x2_swz(const uint16_t* tile, int t, int d0, int d1) {
    return lds4x2(swz<DV>(tile, t, d0), swz<DV>(tile, t, d1));
}

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4_t;

// byte address of an LDS object, as the DS instructions take it
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// Two operands of lds_tr8 (four transposing reads at the given byte addresses) with their wait
// written out: as a builtin such a read waits, besides, for every direct load into LDS in flight.
__device__ __forceinline__ void tr8x2(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, bf16x8& x, bf16x8& y) {
    uint64_t p, q, r, t;
    asm volatile(
        "ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %5\n\t"
        "ds_read_b64_tr_b16 %2, %6\n\tds_read_b64_tr_b16 %3, %7\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(p), "=&v"(q), "=&v"(r), "=&v"(t) : "v"(a0), "v"(a1), "v"(b0), "v"(b1) : "memory");
    typedef __attribute__((__vector_size__(2 * sizeof(uint64_t)))) uint64_t u64x2_t;
    x = __builtin_bit_cast(bf16x8, u64x2_t{p, q});
    y = __builtin_bit_cast(bf16x8, u64x2_t{r, t});
}

// 8-byte LDS write through a scalar type (a vector struct's store is taken to alias the direct
// loads in flight, and waits for them)
__device__ __forceinline__ void st_b64(uint16_t* p, uint32_t lo, uint32_t hi) {
    *reinterpret_cast<uint64_t*>(p) = (uint64_t)lo | ((uint64_t)hi << 32);
}

// sum over each 16-lane row, held by every lane of the row
__device__ __forceinline__ float row_sum16f(float x) {
    x += dpp<0xB1, 0xf>(x);    // quad_perm [1,0,3,2]
    x += dpp<0x4E, 0xf>(x);    // quad_perm [2,3,0,1]
    x += dpp<0x141, 0xf>(x);   // row_half_mirror
    x += dpp<0x140, 0xf>(x);   // row_mirror
    return x;
}

__device__ __forceinline__ void buf_st128(uint4 v, rsrc_t r, uint32_t voff) {
    typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.x, v.y, v.z, v.w}, r, voff, 0, 0);
}

__device__ __forceinline__ void buf_st32(float v, rsrc_t r, uint32_t voff) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, 0, 0);
}

// SPLIT (segments of few sequences, which run side by side): the precision adjoint c that a
// segment starts from is not known yet, so phase 5 is left to bwd_grad_kernel: dqt and dkh go
// to xy [B H][window's chunk][2][kC][dk] and the chunk's composed adjoint step, with the exact
// change of S, to coef [B H][window's chunk][4][dk].  gend [B H][run]: the adjoints of the last
// states of the segments run.
template <int DK, int DV, bool TI, bool YG, bool SPLIT>
__global__ __launch_bounds__((DkCfg<DK, DV>::NTHR)) void bwd_dk_kernel(Shape s, Seg sg, BwdArgs g,
                                                                       const float* __restrict__ saved_lam,
                                                                       const float* __restrict__ saved_H,
                                                                       float* __restrict__ dr_part,
                                                                       const float* __restrict__ gend,
                                                                       float* __restrict__ xy,
                                                                       float* __restrict__ coef) {
    using Cfg = DkCfg<DK, DV>;
    constexpr int NP = Cfg::NP, NW = Cfg::NW, KSD = Cfg::KSD, NRD = Cfg::NRD, LX = Cfg::LX;
    constexpr int NG = Cfg::NG;
    // stores per round: dq, dk(, dabar, dpbar) and dr; SPLIT: dqt, dkh of 4 tokens, two of coef
    constexpr int NST = SPLIT ? 10 : TI ? 3 : 5;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) uint16_t s_out[NP * 4 * kC * 16];

    const uint16_t* a = static_cast<const uint16_t*>(g.a);
    const uint16_t* p = static_cast<const uint16_t*>(g.p);
    const uint16_t* k = static_cast<const uint16_t*>(g.k);
    const uint16_t* q = static_cast<const uint16_t*>(g.q);
    const uint16_t* r = static_cast<const uint16_t*>(g.r);
    const uint16_t* vv = static_cast<const uint16_t*>(g.v);
    const uint16_t* dy = static_cast<const uint16_t*>(g.dy);

    int vi, ntile;
    xcd_tile_map(blockIdx.x, s.B * s.H * sg.run, Cfg::NNT, vi, ntile);
    const int bh = vi / sg.run, seg = sg.first + vi % sg.run;
    const int b = bh / s.H, h = bh % s.H;
    const int c0 = seg * sg.lc, nct = (s.T + kC - 1) / kC;   // this segment's first chunk, the sequence's chunks
    const int H = s.H, T = min(s.T - c0 * kC, sg.lc * kC);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int pr = wave % NP, e = wave / NP;     // pair, half of the chunk (a pair shares a SIMD)
    const int l16 = lane & 15, g4 = lane >> 4;   // MFMA lane coordinates
    const int nl = l16, gg = 4 * e + g4;         // walk lanes: slot, token group (tokens 4 gg .. 4 gg + 3)
    const int n0w = ntile * Cfg::NTN + 16 * pr;  // the pair's first key slot
    const int nchunk = (T + kC - 1) / kC;
    const size_t seq0 = (size_t)b * s.T + (size_t)c0 * kC;
    const size_t row_c0 = (size_t)bh * nct + c0;       // the first chunk's row of the saved walk states
    // and of the window's work arrays
    const size_t win_c0 = (size_t)bh * min(sg.run * sg.lc, nct - sg.first * sg.lc) + (c0 - sg.first * sg.lc);
    const size_t slot_c0 = (size_t)bh * (nct + 1) + c0;   // and its slot of the saved states
    const size_t nbt = (size_t)s.B * s.T * H;
    unsigned char* wb = smem + Cfg::PAIR0 + pr * Cfg::PAIR;
    const uint32_t tok_k = (uint32_t)H * DK * 2;   // bytes between tokens of a [.., H, DK] tensor
    const uint32_t tok_v = (uint32_t)H * DV * 2;

    // ---- carries of the reverse recursions (every lane of both waves holds its slot's values)
    float cT = !SPLIT && g.dlamT ? g.dlamT[(size_t)bh * DK + n0w + nl] : 0.f;
    float ST = 0.f;
    if (!SPLIT && g.detaT) {   // final-state term sum_d detaT H_T, split over the four lane groups
        const float* HT = saved_H + ((slot_c0 + nchunk) * DK + n0w + nl) * DV;
        const float* dT = g.detaT + ((size_t)bh * DK + n0w + nl) * DV;
        for (int d = g4 * (DV / 4); d < (g4 + 1) * (DV / 4); ++d) ST += dT[d] * HT[d];
    }
    ST += __shfl_xor(ST, 16, 64);
    ST += __shfl_xor(ST, 32, 64);
    // range check of the walk: Qp Kn (= q r k / lam) summed over the lane's tokens stays
    // finite exactly while every Qp and Kn is
    float chk = 0.f;
    // time-invariant gates of the slot and the lane's sums of their gradients
    float ca = 0.f, cp = 0.f, sum_da = 0.f, sum_dp = 0.f;
    if constexpr (TI) {
        const int o = h * DK + n0w + nl;
        ou_gates(g.ou_a[o], g.ou_p[o], g.ou_d[o], ca, cp);
    }

    // G^T[d, n] for d = 16 rd + 4 g4 + rr, n = n0w + l16 (carried by wave 1 of the pair)
    const float* gsrc = SPLIT ? gend + (size_t)vi * DK * DV : g.detaT ? g.detaT + (size_t)bh * DK * DV : nullptr;
    f32x4 GT[NRD];
#pragma unroll
    for (int rd = 0; rd < NRD; ++rd)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
            GT[rd][rr] = (e == 1 && gsrc) ? gsrc[(size_t)(n0w + l16) * DV + 16 * rd + 4 * g4 + rr] : 0.f;

    // ---- requests of chunk cn into buffer bb (chunks outside the sequence: empty, writing
    // zeros), one load per part so that they can be spread over a round:
    //   wave 0: 0..3  abar, pbar, k, q of the pair's slots (1 KiB each, lane -> (t = lane / 2, 8 slots));
    //                 TI: 0, 1  k, q
    //   wave 1: 0..2  r (lanes >= nt read as 0), the chunk-start lam of the 16 slots and (YG)
    //                 the yvar gradient
    //   then this wave's share of the dY and V tiles (loads i = wave, wave + NW, ...), swizzled
    const int nin = e == 0 ? (TI ? 2 : 4) : (YG ? 3 : 2);
    const int nvw = wave < Cfg::NVL ? (Cfg::NVL - wave + NW - 1) / NW : 0;
    const int nparts = nin + 2 * nvw;
    auto issue_part = [&](int cn, int bb, int part) {
        const bool in = cn >= 0 && cn < nchunk;
        const int t0 = in ? cn * kC : 0, nt = in ? min(kC, T - t0) : 0;
        const size_t tok0 = seq0 + t0;
        if (part < nin) {
            if (e == 0) {
                const int slot = TI ? part + 2 : part;   // staging slots: abar, pbar, k, q
                const uint16_t* src = slot == 0 ? a : slot == 1 ? p : slot == 2 ? k : q;
                const uint32_t kbytes = nt > 0 ? (uint32_t)((nt - 1) * H * DK + 16) * 2 : 0u;
                uint16_t* stg = reinterpret_cast<uint16_t*>(wb + Cfg::STG) + (bb * 4 + slot) * kC * 16;
                buf_ld128_lds(make_rsrc(src + (tok0 * H + h) * DK + n0w, kbytes), stg,
                              (uint32_t)(lane >> 1) * tok_k + (lane & 1) * 16);
            } else if (part == 0) {
                const rsrc_t rr = make_rsrc(r + tok0 * H + h, nt > 0 ? (uint32_t)((nt - 1) * H + 1) * 2 : 0u);
                buf_ld16_lds(rr, wb + Cfg::RW + bb * 256, (uint32_t)lane * H * 2);
            } else if (part == 2) {
                const rsrc_t rv = make_rsrc(g.dyvar + tok0 * H + h, nt > 0 ? (uint32_t)((nt - 1) * H + 1) * 4 : 0u);
                buf_ld32_lds(rv, wb + Cfg::GV + bb * 256, (uint32_t)lane * H * 4);
            } else {
                // lanes 16 i + l: row i of the saved walk state (lam_0, lam_16, P_16) for slot n0w + l
                const rsrc_t rl = make_rsrc(saved_lam + (row_c0 + (in ? cn : 0)) * kLamRows * DK + n0w,
                                            in ? (uint32_t)(2 * DK + 16) * 4 : 0u);
                buf_ld32_lds(rl, wb + Cfg::LW + bb * 256, (uint32_t)((lane >> 4) * DK + (lane & 15)) * 4);
            }
        } else if (part < nparts) {
            const int m = (part - nin) >> 1, i = wave + NW * m, sel = (part - nin) & 1;
            const uint32_t vbytes = nt > 0 ? (uint32_t)((nt - 1) * H * DV + DV) * 2 : 0u;
            const rsrc_t rv = make_rsrc((sel ? vv : dy) + (tok0 * H + h) * DV, vbytes);
            const int row = i * Cfg::TPV + lane / Cfg::CPR, pch = lane % Cfg::CPR;
            const uint32_t off = (uint32_t)row * tok_v + (uint32_t)((pch ^ (row % Cfg::CPR)) * 16);
            buf_ld128_lds(rv, smem + (bb * 2 + sel) * Cfg::TILE + i * 1024, off);
        }
    };
    wait_vm_all();   // the carries and G^T are complete before the request stream starts
    if (nchunk > 0)
        for (int part = 0; part < nparts; ++part) issue_part(nchunk - 1, 0, part);

    for (int it = 0; it < nchunk; ++it) {
        const int c = nchunk - 1 - it, bb = it & 1;
        const int nt = min(kC, T - c * kC);
        const size_t row0 = seq0 + (size_t)c * kC;

        // the round's work for wave E of the pair; FULL: all kC tokens valid (no per-token guards)
        auto round_body = [&](auto full_tag, auto role_tag) {
            constexpr bool FULL = decltype(full_tag)::value;
            constexpr int E = decltype(role_tag)::value;
            // saved chunk-start state rows H0[n0w + l16][32 ks + 8 g4 .. + 7] (wave 0, for X)
            float4 h0[KSD][2];
            if constexpr (E == 0) {
                const float* H0 = saved_H + ((slot_c0 + c) * DK + n0w + l16) * DV;
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    h0[ks][0] = *reinterpret_cast<const float4*>(H0 + 32 * ks + 8 * g4);
                    h0[ks][1] = *reinterpret_cast<const float4*>(H0 + 32 * ks + 8 * g4 + 4);
                }
                // this chunk's requests (issued last round) have landed: younger are only the
                // last round's NST stores and the 2 KSD state loads just issued
                if (it == 0)
                    wait_vm_le<2 * KSD>();
                else
                    wait_vm_le<NST + 2 * KSD>();
            } else {
                if (it == 0)
                    wait_vm_le<0>();
                else
                    wait_vm_le<NST>();
            }
            barrier_lds();   // every wave's share of the dY / V tiles and staging is in

            const uint16_t* sDY = reinterpret_cast<const uint16_t*>(smem + bb * 2 * Cfg::TILE);
            const uint16_t* sV = sDY + kC * DV;
            const uint16_t* stg = reinterpret_cast<const uint16_t*>(wb + Cfg::STG) + bb * 4 * kC * 16;
            const uint32_t* rw = reinterpret_cast<const uint32_t*>(wb + Cfg::RW) + bb * 64;
            uint16_t* sQH = reinterpret_cast<uint16_t*>(wb + Cfg::QH);
            uint16_t* sQL = reinterpret_cast<uint16_t*>(wb + Cfg::QL);
            uint16_t* sKH = reinterpret_cast<uint16_t*>(wb + Cfg::KH);
            uint16_t* sKL = reinterpret_cast<uint16_t*>(wb + Cfg::KL);
            float* sX = reinterpret_cast<float*>(wb + Cfg::XT);
            float* sY = reinterpret_cast<float*>(wb + Cfg::YT);
            float* sPC = reinterpret_cast<float*>(wb + Cfg::PC);
            float* sWT = reinterpret_cast<float*>(wb + Cfg::WT);   // [2][16]: sum_t Qp X0, sum_j Kn Yg
            float* qs = reinterpret_cast<float*>(wb + Cfg::QS);
            // the lane's four tokens 4 gg .. 4 gg + 3, read again in each phase that uses them (one
            // transposing read per tensor; kept, they would cost nine registers across the phases).
            // Written out with their wait: for the builtin the compiler would also wait for every
            // request and store in flight, as the staging area is filled by direct loads.
            struct Toks {
                uint2 a, p, k, q;
                uint4 r;
            };
            const uint32_t tok_at = lds_addr(stg + (4 * gg + (nl >> 2)) * 16 + 4 * (nl & 3));
            const uint32_t r_at = lds_addr(rw + 4 * gg);
            static_assert(kC * 16 * 2 == 1024, "staged tensors 1 KiB apart");
            auto read_toks = [&](auto with_q) {
                Toks w;
                uint64_t xa, xp, xk, xq;
                u32x4_t xr;
                if constexpr (!TI && decltype(with_q)::value) {
                    asm volatile(
                        "ds_read_b64_tr_b16 %0, %5\n\tds_read_b64_tr_b16 %1, %5 offset:1024\n\t"
                        "ds_read_b64_tr_b16 %2, %5 offset:2048\n\tds_read_b64_tr_b16 %3, %5 offset:3072\n\t"
                        "ds_read_b128 %4, %6\n\ts_waitcnt lgkmcnt(0)"
                        : "=&v"(xa), "=&v"(xp), "=&v"(xk), "=&v"(xq), "=&v"(xr) : "v"(tok_at), "v"(r_at) : "memory");
                    w.q = __builtin_bit_cast(uint2, xq);
                } else if constexpr (!TI) {
                    asm volatile(
                        "ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:1024\n\t"
                        "ds_read_b64_tr_b16 %2, %4 offset:2048\n\tds_read_b128 %3, %5\n\ts_waitcnt lgkmcnt(0)"
                        : "=&v"(xa), "=&v"(xp), "=&v"(xk), "=&v"(xr) : "v"(tok_at), "v"(r_at) : "memory");
                } else if constexpr (decltype(with_q)::value) {
                    asm volatile(
                        "ds_read_b64_tr_b16 %0, %3 offset:2048\n\tds_read_b64_tr_b16 %1, %3 offset:3072\n\t"
                        "ds_read_b128 %2, %4\n\ts_waitcnt lgkmcnt(0)"
                        : "=&v"(xk), "=&v"(xq), "=&v"(xr) : "v"(tok_at), "v"(r_at) : "memory");
                    w.q = __builtin_bit_cast(uint2, xq);
                } else {
                    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:2048\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                                 : "=&v"(xk), "=&v"(xr) : "v"(tok_at), "v"(r_at) : "memory");
                }
                if constexpr (!TI) {
                    w.a = __builtin_bit_cast(uint2, xa);
                    w.p = __builtin_bit_cast(uint2, xp);
                }
                w.k = __builtin_bit_cast(uint2, xk);
                w.r = uint4{xr[0], xr[1], xr[2], xr[3]};
                return w;
            };
            auto in_a = [&](const Toks& w, int j) { return TI ? ca : tok(w.a, j); };
            auto in_p = [&](const Toks& w, int j) { return TI ? cp : tok(w.p, j); };
            auto in_r = [&](const Toks& w, int j) { return __uint_as_float((&w.r.x)[j] << 16); };
            const float* gvw = reinterpret_cast<const float*>(wb + Cfg::GV) + bb * 64;

            // ================================================================ phase 1
            // wave 0: B^T[j, t] = V_j . dY_t (j <= t), tiles (0,0), (0,1), (1,1), as operands over j;
            // wave 1: B[t, j] = dY_t . V_j (j <= t), tiles (0,0), (1,0), (1,1), as operands over t
            bf16x8 boh[2], bol[2];
            {
                f32x4 c0 = zero4(), c1 = zero4(), c2 = zero4();
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    const bf16x8 ya0 = lds8_swz<DV>(sDY, l16, 32 * ks + 8 * g4);
                    const bf16x8 ya1 = lds8_swz<DV>(sDY, 16 + l16, 32 * ks + 8 * g4);
                    const bf16x8 v0 = lds8_swz<DV>(sV, l16, 32 * ks + 8 * g4);
                    const bf16x8 v1 = lds8_swz<DV>(sV, 16 + l16, 32 * ks + 8 * g4);
                    if constexpr (E == 0) {
                        c0 = mfma_bf16(v0, ya0, c0);
                        c1 = mfma_bf16(v0, ya1, c1);
                        c2 = mfma_bf16(v1, ya1, c2);
                    } else {
                        c0 = mfma_bf16(ya0, v0, c0);
                        c1 = mfma_bf16(ya1, v0, c1);
                        c2 = mfma_bf16(ya1, v1, c2);
                    }
                }
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    // B^T: row j = 4 g4 + rr, column t = l16; B: row t = 4 g4 + rr, column j = l16
                    const bool drop = E == 0 ? 4 * g4 + rr > l16 : l16 > 4 * g4 + rr;
                    if (drop) {
                        c0[rr] = 0.f;
                        c2[rr] = 0.f;
                    }
                }
                // rows {4g..}, {16+4g..} of the contraction
                if constexpr (E == 0) {
                    split8(c0, zero4(), boh[0], bol[0]);
                    split8(c1, c2, boh[1], bol[1]);
                } else {
                    split8(c0, c1, boh[0], bol[0]);
                    split8(zero4(), c2, boh[1], bol[1]);
                }
            }
            // the transfer of this lane's group: (x, z) -> M (x, z) over its valid tokens, as the
            // images of (1, 0) and (0, 1), and the product of abar
            float tr[5];
            {
                float x0 = 1.f, z0 = 0.f, x1 = 0.f, z1 = 1.f, Aq = 1.f;
                const Toks w = read_toks(std::false_type{});
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = 4 * gg + j;
                    const float av = in_a(w, j), pv = in_p(w, j), kv = tok(w.k, j), rv = in_r(w, j);
                    const float a2 = av * av, phi = kv * kv * rv;
                    const float z0n = fmaf(pv, x0, a2 * z0), z1n = fmaf(pv, x1, a2 * z1);
                    const bool ok = FULL || t < nt;
                    x0 = ok ? fmaf(phi, z0n, x0) : x0;
                    x1 = ok ? fmaf(phi, z1n, x1) : x1;
                    z0 = ok ? z0n : z0;
                    z1 = ok ? z1n : z1;
                    Aq = ok ? Aq * av : Aq;
                }
                tr[0] = x0;
                tr[1] = z0;
                tr[2] = x1;
                tr[3] = z1;
                tr[4] = Aq;
            }
            __builtin_amdgcn_sched_barrier(0);   // keep the phases apart in the schedule (register pressure)

            // ================================================================ phase 2
            // chain the wave's earlier groups from the saved state at the start of its half:
            // (x, z, A) = (lam_0, 1, 1) for tokens 0..15, (lam_16, 1, P_16) for 16..31.  A
            // wave's four groups are its four 16-lane rows, so the transfers of the earlier rows
            // are read across lanes (ds_bpermute), with no LDS store and no barrier.
            const float* lws = reinterpret_cast<const float*>(wb + Cfg::LW) + bb * 64;
            float x = lws[16 * E + nl], z = 1.f, A = E == 0 ? 1.f : lws[32 + nl];
#pragma unroll
            for (int q2 = 0; q2 < NG / 2 - 1; ++q2) {
                auto pick = [&](int i) { return __shfl(tr[i], 16 * q2 + nl, 64); };   // row q2, same column
                const float m00 = pick(0), m10 = pick(1), m01 = pick(2), m11 = pick(3), aq = pick(4);
                const bool use = q2 < g4;
                const float xn = fmaf(m00, x, m01 * z), zn = fmaf(m10, x, m11 * z);
                x = use ? xn : x;
                z = use ? zn : z;
                A = use ? A * aq : A;
            }
            float izp = fast_rcp(z);              // 1 / z before the group's first token
            const float lamq = x * izp;           // lam before the group's first token
            // per token of the group: lam_t, P_t and, for the adjoint walk, 1/P_t, 1/lam_t,
            // rho_t, 1/rho_t = abar^2 + pbar lam_{t-1}, 1/abar
            float lam_r[4], P_r[4], iP_r[4], il_r[4], rho_r[4], den_r[4], ia_r[4];
            uint2 qh, ql, kh, kl;   // the four tokens' Qp, Kn
            const Toks w2 = read_toks(std::true_type{});
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) {
                float qp2[2], kn2[2];
#pragma unroll
                for (int e2 = 0; e2 < 2; ++e2) {
                    const int j = 2 * j2 + e2, t = 4 * gg + j;
                    const float av = in_a(w2, j), pv = in_p(w2, j), kv = tok(w2.k, j), qv = tok(w2.q, j), rv = in_r(w2, j);
                    const float kr = kv * rv;
                    const float zn = fmaf(pv, x, av * av * z);
                    const float xn = fmaf(kr * kv, zn, x);
                    const float An = A * av;
                    const float R = fast_rcp(xn * An);
                    const float iz = fast_rcp(zn);
                    const float AR = An * R, XR = xn * R;   // 1 / x_t, 1 / A_t
                    const bool ok = FULL || t < nt;
                    qp2[e2] = ok ? (qv * An) * AR : 0.f;
                    kn2[e2] = ok ? (kr * zn) * XR : 0.f;
                    chk = fmaf(qp2[e2], kn2[e2], chk);
                    lam_r[j] = xn * iz;
                    P_r[j] = An * iz;
                    iP_r[j] = zn * XR;
                    il_r[j] = zn * AR;
                    rho_r[j] = z * iz;
                    den_r[j] = zn * izp;
                    ia_r[j] = A * XR;
                    izp = iz;
                    x = ok ? xn : x;
                    z = ok ? zn : z;
                    A = ok ? An : A;
                }
                split2(qp2[0], qp2[1], j2 ? qh.y : qh.x, j2 ? ql.y : ql.x);
                split2(kn2[0], kn2[1], j2 ? kh.y : kh.x, j2 ? kl.y : kl.x);
            }
            const int e0 = nt_off(nl, 4 * gg);
            st_b64(sQH + e0, qh.x, qh.y);
            st_b64(sQL + e0, ql.x, ql.y);
            st_b64(sKH + e0, kh.x, kh.y);
            st_b64(sKL + e0, kl.x, kl.y);
            if (gg == NG - 1) sPC[nl] = A * fast_rcp(z);   // the last group ends at the chunk end
            barrier_lds();   // Qp, Kn of every token and P_C are in

            // ================================================================ phase 3
            if constexpr (E == 0) {
                // X^T[n, t] = sum_d H0[n, d] dY^T[d, t] + sum_j Kn^T[n, j] B^T[j, t]
                f32x4 xacc[2] = {zero4(), zero4()};
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    bf16x8 hh, hl;
                    split8(f32x4{h0[ks][0].x, h0[ks][0].y, h0[ks][0].z, h0[ks][0].w},
                           f32x4{h0[ks][1].x, h0[ks][1].y, h0[ks][1].z, h0[ks][1].w}, hh, hl);
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)
                        xacc[tt] = mfma2a(hh, hl, lds8_swz<DV>(sDY, 16 * tt + l16, 32 * ks + 8 * g4), xacc[tt]);
                }
                {   // chunk total of Qp X0 per slot n = 4 g4 + rr (tokens past the end have Qp = 0)
                    float w[4];
                    uint2 th[2], tl[2];
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt) {
                        th[tt] = nt_tr4(sQH, 4 * g4, 16 * tt, l16);
                        tl[tt] = nt_tr4(sQL, 4 * g4, 16 * tt, l16);
                    }
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        w[rr] = 0.f;
#pragma unroll
                        for (int tt = 0; tt < 2; ++tt)
                            w[rr] = fmaf(tok(th[tt], rr) + tok(tl[tt], rr), xacc[tt][rr], w[rr]);
                        w[rr] = row_sum16f(w[rr]);
                    }
                    if (l16 == 0)
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) sWT[4 * g4 + rr] = w[rr];
                }
                const int o0 = nt_off(l16, 4 * g4), o1 = nt_off(l16, 16 + 4 * g4);
                const bf16x8 knh = lds4x2(sKH + o0, sKH + o1), knl = lds4x2(sKL + o0, sKL + o1);
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    xacc[tt] = mfma3(knh, knl, boh[tt], bol[tt], xacc[tt]);
                    *reinterpret_cast<float4*>(sX + (16 * tt + l16) * LX + 4 * g4) =
                        float4{xacc[tt][0], xacc[tt][1], xacc[tt][2], xacc[tt][3]};
                }
            } else {
                // Y^T[n, j] = sum_d Gs[n, d] V^T[d, j] + sum_t Qp^T[n, t] B[t, j]: the state part
                // first, whose chunk total is taken before the attention part is added
                f32x4 yacc[2] = {zero4(), zero4()};
                const float pcn = sPC[l16];
#pragma unroll
                for (int rd = 0; rd < NRD; ++rd)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) GT[rd][rr] *= pcn;   // Gs^T in place
#pragma unroll
                for (int ks = 0; ks < KSD; ++ks) {
                    bf16x8 gh, gl;
                    split8(GT[2 * ks], GT[2 * ks + 1], gh, gl);
#pragma unroll
                    for (int jt = 0; jt < 2; ++jt) {
                        const bf16x8 vb = lds4x2_swz<DV>(sV, 16 * jt + l16, 32 * ks + 4 * g4, 32 * ks + 16 + 4 * g4);
                        yacc[jt] = mfma2a(gh, gl, vb, yacc[jt]);
                    }
                }
                {   // chunk total of Kn Yg per slot n = 4 g4 + rr (tokens past the end have Kn = 0)
                    float w[4];
                    uint2 th[2], tl[2];
#pragma unroll
                    for (int jt = 0; jt < 2; ++jt) {
                        th[jt] = nt_tr4(sKH, 4 * g4, 16 * jt, l16);
                        tl[jt] = nt_tr4(sKL, 4 * g4, 16 * jt, l16);
                    }
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        w[rr] = 0.f;
#pragma unroll
                        for (int jt = 0; jt < 2; ++jt)
                            w[rr] = fmaf(tok(th[jt], rr) + tok(tl[jt], rr), yacc[jt][rr], w[rr]);
                        w[rr] = row_sum16f(w[rr]);
                    }
                    if (l16 == 0)
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) sWT[16 + 4 * g4 + rr] = w[rr];
                }
                const int o0 = nt_off(l16, 4 * g4), o1 = nt_off(l16, 16 + 4 * g4);
                const bf16x8 qth = lds4x2(sQH + o0, sQH + o1), qtl = lds4x2(sQL + o0, sQL + o1);
#pragma unroll
                for (int jt = 0; jt < 2; ++jt) yacc[jt] = mfma3(qth, qtl, boh[jt], bol[jt], yacc[jt]);
#pragma unroll
                for (int jt = 0; jt < 2; ++jt)
                    *reinterpret_cast<float4*>(sY + (16 * jt + l16) * LX + 4 * g4) =
                        float4{yacc[jt][0], yacc[jt][1], yacc[jt][2], yacc[jt][3]};
            }
            barrier_lds();   // X and Y of every token are in

            // ================================================================ phase 4
            // adjoint pass 1: the group's tokens in reverse; per token the affine step
            //   (c, S) -> (alpha (c - w) - beta (S + u), S + u)
            // composed into c_out = Am c_in + Bm S_in + Cm, S_out = S_in + Dm
            float u_[4], w_[4], al_[4], be_[4], dq_[4], rdk_[4], kr2_[4], ia_[4], a2r2_[4], lp_[4], den_[4], lpr2_[4],
                kdk_[4], kk_[4];
            float Am = 1.f, Bm = 0.f, Cm = 0.f, Dm = 0.f;
            const Toks w4 = read_toks(std::true_type{});
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const int t = 4 * gg + j;
                const float av = in_a(w4, j), pv = in_p(w4, j), kv = tok(w4.k, j), qv = tok(w4.q, j), rv = in_r(w4, j);
                const float lam_p = j > 0 ? lam_r[j - 1] : lamq;
                const float Xv = sX[t * LX + nl], Yv = sY[t * LX + nl];
                const float rho = rho_r[j], ilam = il_r[j], ia = ia_r[j], den = den_r[j];
                const float dqt = P_r[j] * Xv, dkh = Yv * iP_r[j];
                const float kh = rv * kv;
                const float qi = qv * ilam, qg = YG ? qv * gvw[t] : 0.f;
                const bool ok = FULL || t < nt;
                const float u = ok ? qi * dqt - kh * dkh : 0.f;
                const float w = ok ? qi * (dqt + qg) * ilam : 0.f;
                const float rho2 = rho * rho;
                const float al = ok ? av * av * rho2 : 1.f;
                const float be = ok ? pv * rho : 0.f;
                u_[j] = u;
                w_[j] = w;
                al_[j] = al;
                be_[j] = be;
                if constexpr (SPLIT) {
                    dq_[j] = ok ? dqt : 0.f;
                    kdk_[j] = ok ? dkh : 0.f;
                } else {
                    dq_[j] = fmaf(2.f, qg, dqt) * ilam;
                    rdk_[j] = rv * dkh;
                    kr2_[j] = 2.f * kh;
                    ia_[j] = ia;
                    a2r2_[j] = 2.f * av * rho2;
                    lp_[j] = lam_p;
                    den_[j] = den;
                    lpr2_[j] = lam_p * rho2;
                    kdk_[j] = kv * dkh;
                    kk_[j] = kv * kv;
                }
                Cm = al * Cm - be * Dm - (al * w + be * u);
                Bm = al * Bm - be;
                Am = al * Am;
                Dm = Dm + u;
                // the next chunk's requests, two per token: they go out only after the
                // transposing LDS reads above (which would otherwise wait for them)
                issue_part(c - 1, bb ^ 1, 2 * (3 - j));
                issue_part(c - 1, bb ^ 1, 2 * (3 - j) + 1);
            }
            if constexpr (E == 1) {
                // G^T <- dY^T Qp + Gs^T
                const bf16x8 qbh = nt_row8(sQH, l16, g4), qbl = nt_row8(sQL, l16, g4);
                auto at = [&](int row, int rd) {
                    return lds_addr(swz<DV>(sDY, row + (l16 >> 2), 16 * rd + 4 * (l16 & 3)));
                };
                static_assert(NRD % 2 == 0, "row tiles in pairs");
#pragma unroll
                for (int rd = 0; rd < NRD; rd += 2) {
                    bf16x8 y0, y1;
                    tr8x2(at(8 * g4, rd), at(8 * g4 + 4, rd), at(8 * g4, rd + 1), at(8 * g4 + 4, rd + 1), y0, y1);
                    GT[rd] = mfma2b(y0, qbh, qbl, GT[rd]);
                    GT[rd + 1] = mfma2b(y1, qbh, qbl, GT[rd + 1]);
                }
            }
            float* qw = qs + (gg * 16 + nl) * 4;   // the last chunk's summaries were read before two barriers
            qw[0] = Am;
            qw[1] = Bm;
            qw[2] = Cm;
            qw[3] = Dm;
            barrier_lds();   // the group summaries are in

            if constexpr (SPLIT) {
                // dqt, dkh of the lane's tokens, and the chunk's composed step: A, B from wave 0, C and
                // the change of S from wave 1
                float* xo = xy + (win_c0 + c) * 2 * kC * DK;
                const rsrc_t rx = make_rsrc(xo, 2 * kC * DK * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t vo = (uint32_t)((4 * gg + j) * DK + n0w + nl) * 4;
                    buf_st32s(dq_[j], rx, vo, 0);
                    buf_st32s(kdk_[j], rx, vo, kC * DK * 4);
                }
                float Ac = 1.f, Bc = 0.f, Cc = 0.f, Dc = 0.f;
#pragma unroll
                for (int q2 = NG - 1; q2 >= 0; --q2) {
                    const float* m = qs + (q2 * 16 + nl) * 4;
                    const float m0 = m[0], m1 = m[1];
                    Cc = fmaf(m0, Cc, fmaf(m1, Dc, m[2]));
                    Bc = fmaf(m0, Bc, m1);
                    Ac *= m0;
                    Dc += m[3];
                }
                const rsrc_t rc = make_rsrc(coef + (win_c0 + c) * 4 * DK, 4 * DK * 4);
                const uint32_t vo = g4 == 0 ? (uint32_t)(2 * E * DK + n0w + nl) * 4 : 4 * DK * 4;   // other lanes: dropped
                buf_st32s(E == 0 ? Ac : Cc, rc, vo, 0);
                buf_st32s(E == 0 ? Bc : sWT[nl] - sWT[16 + nl], rc, vo, DK * 4);
                return;
            }
            // ================================================================ phase 5
            // carries into this group (through the later groups) and out of the chunk; S leaves
            // the chunk with the chunk's exact total, not the sum of its tokens' terms
            const float S_out = ST + (sWT[nl] - sWT[16 + nl]);
            float c_in = 0.f, S_in = 0.f;
#pragma unroll
            for (int q2 = NG - 1; q2 >= 0; --q2) {
                if (q2 == gg) {
                    c_in = cT;
                    S_in = ST;
                }
                const float* m = qs + (q2 * 16 + nl) * 4;
                const float cn = fmaf(m[0], cT, fmaf(m[1], ST, m[2]));
                ST += m[3];
                cT = cn;
            }
            ST = S_out;
            // pass 2: gradients of the group's tokens
            uint16_t* so = s_out + pr * 4 * kC * 16;
            float dk4[4], da4[4], dp4[4], dr4[4];
            float cc = c_in, SS = S_in;
#pragma unroll
            for (int j = 3; j >= 0; --j) {
                const int t = 4 * gg + j;
                SS += u_[j];
                const float gl = cc - w_[j];
                const float dkv = fmaf(kr2_[j], gl, rdk_[j]);
                const float drho = fmaf(gl, lp_[j], SS * den_[j]);
                const float dav = fmaf(-a2r2_[j], drho, SS * ia_[j]);
                const float dpv = -lpr2_[j] * drho;
                dr4[j] = fmaf(kk_[j], gl, kdk_[j]);
                cc = fmaf(al_[j], gl, -be_[j] * SS);
                dk4[j] = dkv;
                if constexpr (TI) {
                    if (FULL || t < nt) {
                        sum_da += dav;
                        sum_dp += dpv;
                    }
                } else {
                    da4[j] = dav;
                    dp4[j] = dpv;
                }
            }
            auto put = [&](int x, const float (&v)[4]) {
                st_b64(so + x * kC * 16 + nt_off(nl, 4 * gg), cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
            };
            put(0, dq_);
            put(1, dk4);
            if constexpr (!TI) {
                put(2, da4);
                put(3, dp4);
            }

            // ---- stores of this wave's 16 tokens: rows of 16 slots of dq, dk, dabar, dpbar (lanes
            // < 32: t = 16 E + lane % 16, 8 slots each) and the pair's dr partial over its 16 slots
            // (lane j < 4 of a group: its token j); the other lanes address the end of the range and
            // are dropped, as are tokens past the sequence end
            {
                const int hs = 8 * (g4 & 1);
                const uint32_t kbytes = (uint32_t)((nt - 1) * H * DK + 16) * 2;
                const size_t ek = (row0 * H + h) * DK + n0w;
                const uint32_t koff = lane < 32 ? (uint32_t)(16 * E + l16) * tok_k + hs * 2 : kbytes;
                const uint32_t oa = lds_addr(so + nt_off(hs + (l16 >> 2), 16 * E + 4 * (l16 & 3)));
                const uint32_t ob = lds_addr(so + nt_off(hs + 4 + (l16 >> 2), 16 * E + 4 * (l16 & 3)));
                constexpr uint32_t TB = kC * 16 * 2;   // bytes of one gradient tile
                auto store2 = [&](int x, void* d0, void* d1) {
                    bf16x8 v0, v1;
                    tr8x2(oa + x * TB, ob + x * TB, oa + (x + 1) * TB, ob + (x + 1) * TB, v0, v1);
                    buf_st128(__builtin_bit_cast(uint4, v0), make_rsrc(static_cast<uint16_t*>(d0) + ek, kbytes), koff);
                    buf_st128(__builtin_bit_cast(uint4, v1), make_rsrc(static_cast<uint16_t*>(d1) + ek, kbytes), koff);
                };
                store2(0, g.dq, g.dk);
                if constexpr (!TI) store2(2, g.da, g.dp);
#pragma unroll
                for (int j = 0; j < 4; ++j) dr4[j] = row_sum16f(dr4[j]);
                const float acc = nl & 2 ? (nl & 1 ? dr4[3] : dr4[2]) : (nl & 1 ? dr4[1] : dr4[0]);
                float* dst = dr_part + (size_t)(ntile * NP + pr) * nbt + row0 * H + h;
                const uint32_t dbytes = (uint32_t)((nt - 1) * H + 1) * 4;
                buf_st32(acc, make_rsrc(dst, dbytes), nl < 4 ? (uint32_t)(4 * gg + nl) * H * 4 : dbytes);
            }
        };
        if (e == 0) {
            if (nt == kC)
                round_body(std::true_type{}, std::integral_constant<int, 0>{});
            else
                round_body(std::false_type{}, std::integral_constant<int, 0>{});
        } else {
            if (nt == kC)
                round_body(std::true_type{}, std::integral_constant<int, 1>{});
            else
                round_body(std::false_type{}, std::integral_constant<int, 1>{});
        }
    }
    wait_vm_all();   // the requests for the chunk before the first have landed before exit
    if (g.range_flag && !(fabsf(chk) <= 3.0e38f)) *g.range_flag = 1;
    if (SPLIT) return;
    if (g.dlam0 && e == 0 && g4 == 0) g.dlam0[(size_t)bh * DK + n0w + nl] = cT;
    if constexpr (TI) {   // part e * B + b of the token sums: the wave's four token groups added
        sum_da += __shfl_xor(sum_da, 16, 64);
        sum_da += __shfl_xor(sum_da, 32, 64);
        sum_dp += __shfl_xor(sum_dp, 16, 64);
        sum_dp += __shfl_xor(sum_dp, 32, 64);
        if (g4 == 0) {
            const size_t np = (size_t)2 * s.B * H * DK;
            const size_t o = ((size_t)(e * s.B + b) * H + h) * DK + n0w + nl;
            float* part = static_cast<float*>(g.ou_part);
            part[o] = sum_da;
            part[np + o] = sum_dp;
        }
    }
}

// dr = sum of the per-pair partials, stored in the input dtype
__global__ void dr_combine_kernel(const float* __restrict__ part, int nparts, size_t n, uint16_t* __restrict__ dr) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float acc = 0.f;
    for (int t = 0; t < nparts; ++t) acc += part[(size_t)t * n + i];
    dr[i] = f32_to_bf16(acc);
}

template <int DK, int DV, bool TI, bool YG>
hipError_t launch_dk(const Shape& s, const BwdArgs& a, const float* saved_lam, const float* saved_H, float* dr_part,
                     hipStream_t st) {
    using Cfg = DkCfg<DK, DV>;
    auto kern = bwd_dk_kernel<DK, DV, TI, YG, false>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::BYTES);
    if (attr != hipSuccess) return attr;
    const int nct = (s.T + kC - 1) / kC;
    hipError_t e = launch_backward_dv(s, 1, nct, 0, 1, false, a, saved_lam, nullptr, nullptr, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(s.B * s.H * Cfg::NNT)), dim3(Cfg::NTHR), Cfg::BYTES, st, s, Seg{1, nct, 1},
                       a, saved_lam, saved_H, dr_part, nullptr, nullptr, nullptr);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t n = (size_t)s.B * s.T * s.H;
    if (n > 0) {
        hipLaunchKernelGGL(dr_combine_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, dr_part,
                           Cfg::NNT * Cfg::NP, n, static_cast<uint16_t*>(a.dr));
        e = hipGetLastError();
    }
    return e;
}

// ---- the segment-parallel backward of few sequences
// A window of segments (all of them where their buffers fit), last window first:
//   1. every segment's but the first's own contribution to the adjoint of the state before it
//      (bwd_dv_kernel without dV), 2. their scan to the adjoint of every segment's last state,
//   3. dV and, in 4., the contractions of the key side over the window's segments at once (SPLIT),
//   5. a scan of the chunks' adjoint steps for (c, S) at the chunk ends, 6. the gradients.
// The adjoints of the state and of lam, S and the OU sums are carried from window to window as
// the scans hold them, so the windows do not show in the results.
struct BwdCut {
    int ns, lc;   // segments of lc chunks
    int w;        // segments per window
};

// What the segments may use of device memory however long the sequences: 280 bytes per chunk, head
// and key slot for the chunks of a window, 4 (dv + 1) per segment, head and slot.  Past it the
// windows' additional kernels cost 2 to 7%: 65536 tokens of 16 heads of 128 x 128 in one window
// (1.2 GB) 3.50 ms, in five 3.56; 3500 of 64 heads 723 us in one, 777 in two.
constexpr size_t kSegWork = 256u << 20;

size_t pad256(size_t bytes) { return (bytes + 255) / 256 * 256; }

// Buffers of a window of w segments of lc chunks, and the carries between windows.
struct SegBufs {
    float *gend, *pseg, *xy, *coef, *ous, *cg;
    double* ccs;
    size_t bytes;
    SegBufs(const Shape& s, int w, int lc, void* ws) {
        const size_t nbh = (size_t)s.B * s.H, nc = (size_t)w * lc;
        bytes = 0;
        auto carve = [&](auto*& p, size_t count) {   // ws may be absent: only the bytes are asked for
            p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<uintptr_t>(ws) + bytes);
            bytes += pad256(count * sizeof(*p));
        };
        carve(gend, nbh * w * s.dk * s.dv);
        carve(pseg, nbh * w * s.dk);
        carve(xy, nbh * nc * 2 * kC * s.dk);
        carve(coef, nbh * nc * 4 * s.dk);
        carve(ous, nbh * nc * 2 * s.dk);
        carve(cg, nbh * s.dk * s.dv);
        carve(ccs, nbh * 2 * s.dk);
    }
};
size_t seg_bytes(const Shape& s, int w, int lc) { return SegBufs(s, w, lc, nullptr).bytes; }

// Microseconds per chunk round at 128 x 128: value side 3.3 (3.8 wide), its state-only pass 2.0,
// key side 7.4 (SPLIT 6.6); the gradient kernel 1.1 ns per token and head; the other kernels and
// launches of a window 40.  With dk = 128 and dv <= 64 the contractions take less of it all and the
// rest more, 1.6 ns and 28 (with the figures of 128 x 128, 80 heads of 128 x 32 over 2048 tokens took
// three segments, 472 us against 419).  One workgroup per CU, as in the forward.  ns and lc do not depend on
// limit (bytes the windows may use), so that the results do not; under a limit that cuts the
// windows too short to fill the chip the whole walk may be left as the faster one.
BwdCut bwd_cut(const Shape& s, size_t limit) {
    const int nct = (s.T + kC - 1) / kC, bh = s.B * s.H, nnt = s.dk / 64 > 0 ? s.dk / 64 : 1, ntile = s.dv == 128 ? 2 : 1;
    const BwdCut whole{1, nct, 1};
    if (nct < 4) return whole;
    auto rounds = [](int wg) { return (wg + 255) / 256; };
    auto dv_us = [&](int ns) { return chunked_wide(s, ns) ? 3.8 * rounds(bh * ns) : 3.3 * rounds(bh * ns * ntile); };
    const bool lean = s.dk == 128 && s.dv <= 64;
    const double grad_us = lean ? 1.6e-3 : 1.1e-3, fixed_us = lean ? 28.0 : 40.0;
    auto cost = [&](const BwdCut& c) {
        const int full = c.ns / c.w, rest = c.ns % c.w;
        auto window = [&](int w) { return c.lc * (2.0 + dv_us(w) + 6.6 * rounds(bh * w * nnt)) + fixed_us; };
        return full * window(c.w) + (rest ? window(rest) : 0.0) + grad_us * bh * s.T * s.dk / 128;
    };
    const double walk = 0.92 * nct * (dv_us(1) + 7.4 * rounds(bh * nnt));
    double best = walk;
    BwdCut cut = whole;
    for (int wg : {256 / (bh * ntile), 256 / (bh * nnt), 256 / bh}) {
        if (wg < 2) continue;
        // as many windows of wg segments as the bound asks for, in equal parts
        const size_t seg = seg_bytes(s, wg, 0), chunk = (size_t)bh * wg * s.dk * (2 * kC + 6) * sizeof(float);
        if (seg + chunk > kSegWork) continue;
        const int most = (int)std::min<size_t>((kSegWork - seg) / chunk, nct);
        const int nw = ((nct + wg - 1) / wg + most - 1) / most;
        const int lc = (nct + wg * nw - 1) / (wg * nw), ns = (nct + lc - 1) / lc;
        if (ns < 2) continue;
        const BwdCut c{ns, lc, std::min(ns, wg)};
        const double t = cost(c);
        if (t < best) {
            best = t;
            cut = c;
        }
    }
    if (cut.ns > 1 && seg_bytes(s, cut.w, cut.lc) > limit) {
        int w = cut.w - 1;
        while (w > 0 && seg_bytes(s, w, cut.lc) > limit) --w;
        if (w == 0) return whole;
        const int nw = (cut.ns + w - 1) / w;
        cut.w = (cut.ns + nw - 1) / nw;
        if (cost(cut) > walk) return whole;
    }
    return cut;
}

// Per element: the adjoint of the last state of every segment of a window (its w segments from s0
// on), in place of the segments' own contributions, from detaT (last window) or carry; carry
// receives the adjoint of the state before the window.
__global__ __launch_bounds__(256) void bwd_state_scan_kernel(int nbh, int DK, int DV, int s0, int w, bool last,
                                                             const float* __restrict__ pseg,
                                                             const float* __restrict__ detaT, float* __restrict__ g,
                                                             float* __restrict__ carry) {
    const size_t per = (size_t)DK * DV, i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)nbh * per) return;
    const size_t e = i % per, bh = i / per;
    const int n = (int)(e / DV);
    float x = !last ? carry[i] : detaT ? detaT[i] : 0.f;
    float* o = g + bh * w * per + e;
    const float* pn = pseg + bh * w * DK + n;
    const int lo = s0 > 0 ? 0 : min(1, w - 1);   // the sequence's first segment has no contribution
    constexpr int U = 8;
    for (int j0 = w - 1; j0 >= 0; j0 -= U) {
        float u[U], p[U];
#pragma unroll
        for (int m = 0; m < U; ++m) {
            const int j = max(j0 - m, lo);
            u[m] = o[(size_t)j * per];
            p[m] = pn[(size_t)j * DK];
        }
#pragma unroll
        for (int m = 0; m < U; ++m)
            if (j0 - m >= 0) {
                o[(size_t)(j0 - m) * per] = x;
                x = fmaf(p[m], x, u[m]);
            }
    }
    if (s0 > 0) carry[i] = x;
}

// (c, S) at the end of every chunk of a window, into rows 0 and 1 of its coef, carried in fp64
// along the sequence; from dlamT and sum_d detaT H_T (hT: the final states, hseq floats apart) in
// the last window, else from carry [B H][2][dk].  One thread per (b, h, slot); the steps of U
// chunks are loaded while those of the U after are applied.
__global__ __launch_bounds__(64) void bwd_carry_kernel(int nbh, int DK, int DV, int nc, bool last,
                                                       float* __restrict__ coef, double* __restrict__ carry,
                                                       const float* __restrict__ hT, size_t hseq,
                                                       const float* __restrict__ dlamT,
                                                       const float* __restrict__ detaT, float* __restrict__ dlam0) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbh * DK) return;
    const int n = i % DK, bh = i / DK;
    double* cr = carry + (size_t)bh * 2 * DK + n;
    double c = 0.0, S = 0.0;
    if (!last) {
        c = cr[0];
        S = cr[DK];
    } else {
        if (dlamT) c = (double)dlamT[i];
        if (detaT) {
            const float* h = hT + (size_t)bh * hseq + (size_t)n * DV;
            const float* d = detaT + (size_t)i * DV;
            for (int m = 0; m < DV; m += 4) {
                const float4 x = *reinterpret_cast<const float4*>(h + m), y = *reinterpret_cast<const float4*>(d + m);
                S += (double)x.x * y.x + (double)x.y * y.y + (double)x.z * y.z + (double)x.w * y.w;
            }
        }
    }
    float* cf = coef + (size_t)bh * nc * 4 * DK + n;
    constexpr int U = 8;
    float b[U][4], nx[U][4];
    auto load = [&](float (&d)[U][4], int j0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) d[u][r] = cf[((size_t)max(j0 - u, 0) * 4 + r) * DK];
    };
    load(nx, nc - 1);
    for (int j0 = nc - 1; j0 >= 0; j0 -= U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) b[u][r] = nx[u][r];
        load(nx, j0 - U);   // rows of other chunks than those written below
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 - u >= 0) {
                float* o = cf + (size_t)(j0 - u) * 4 * DK;
                o[0] = (float)c;
                o[DK] = (float)S;
                c = fma((double)b[u][0], c, fma((double)b[u][1], S, (double)b[u][2]));
                S += b[u][3];
            }
    }
    cr[0] = c;
    cr[DK] = S;
    if (dlam0) dlam0[i] = (float)c;
}

// The gradients of one chunk's tokens from dqt, dkh and (c, S) at its end: phases 1, 2, 4 and 5
// of bwd_dk_kernel for lanes = (slot, group of 8 tokens), one workgroup per (b, h, chunk), so
// dr is complete here.  HBM bound: 24 bytes per (token, slot) with per-token gates.  The
// window's nc chunks from c0 on; xy, coef and ous as in bwd_dk_kernel.
// TI: the chunk's sums of the gate gradients go to ous [B H][window's chunk][2][dk].
template <int DK, bool TI, bool YG>
__global__ __launch_bounds__(4 * DK) void bwd_grad_kernel(Shape s, int c0, int nc, BwdArgs g,
                                                          const float* __restrict__ saved_lam,
                                                          const float* __restrict__ xy,
                                                          const float* __restrict__ coef, float* __restrict__ ous) {
    constexpr int NG = 4, TPG = 8, NT = NG * DK;
    __shared__ float qs[NG][4][DK];
    __shared__ float sR[kC][DK + 1];
    const int nct = (s.T + kC - 1) / kC, c = c0 + blockIdx.x % nc, bh = blockIdx.x / nc;
    const int H = s.H, b = bh / H, h = bh % H, tid = threadIdx.x, n = tid % DK, gq = tid / DK;
    const int nt = min(kC, s.T - c * kC);
    const size_t tok0 = (size_t)b * s.T + (size_t)c * kC, row = blockIdx.x;   // row of xy, coef, ous
    const size_t k0 = (tok0 * H + h) * DK;
    const uint32_t kbytes = (uint32_t)((nt - 1) * H * DK + DK) * 2;
    const rsrc_t rk = make_rsrc(static_cast<const uint16_t*>(g.k) + k0, kbytes);
    const rsrc_t rq = make_rsrc(static_cast<const uint16_t*>(g.q) + k0, kbytes);
    const uint32_t gbytes = TI ? 0u : kbytes;   // of the per-token gates and their gradients
    const rsrc_t ra = make_rsrc(static_cast<const uint16_t*>(TI ? g.k : g.a) + k0, gbytes);
    const rsrc_t rp = make_rsrc(static_cast<const uint16_t*>(TI ? g.k : g.p) + k0, gbytes);
    const rsrc_t rr = make_rsrc(static_cast<const uint16_t*>(g.r) + tok0 * H + h, (uint32_t)((nt - 1) * H + 1) * 2);
    const rsrc_t rg = make_rsrc(YG ? g.dyvar + tok0 * H + h : nullptr, YG ? (uint32_t)((nt - 1) * H + 1) * 4 : 0u);
    float ca = 0.f, cp = 0.f;
    if constexpr (TI) ou_gates(g.ou_a[h * DK + n], g.ou_p[h * DK + n], g.ou_d[h * DK + n], ca, cp);
    // the lane's tokens; past the sequence end they enter as the identity step
    float av[TPG], pv[TPG], kv[TPG], qv[TPG], rv[TPG], gv[TPG], dqt[TPG], dkh[TPG];
    const float* xo = xy + row * 2 * kC * DK;
#pragma unroll
    for (int j = 0; j < TPG; ++j) {
        const int t = gq * TPG + j;
        const uint32_t vo = (uint32_t)(t * H * DK + n) * 2;
        const bool ok = t < nt;
        av[j] = ok ? (TI ? ca : bf16_to_f32(buf_ld16(ra, vo, 0))) : 1.f;
        pv[j] = TI ? (ok ? cp : 0.f) : bf16_to_f32(buf_ld16(rp, vo, 0));
        kv[j] = bf16_to_f32(buf_ld16(rk, vo, 0));
        qv[j] = bf16_to_f32(buf_ld16(rq, vo, 0));
        rv[j] = bf16_to_f32(buf_ld16(rr, (uint32_t)(t * H) * 2, 0));
        gv[j] = YG ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, (uint32_t)(t * H) * 4, 0, 0)) : 0.f;
        dqt[j] = xo[t * DK + n];
        dkh[j] = xo[(kC + t) * DK + n];
    }
    const float* lw = saved_lam + ((size_t)bh * nct + c) * kLamRows * DK + n;
    const bool half = gq >= 2;
    float x = half ? lw[DK] : lw[0], z = 1.f;
    float cc = coef[row * 4 * DK + n], SS = coef[(row * 4 + 1) * DK + n];
    // the transfer of the lane's group, handed to the next group of its half
    {
        float x0 = 1.f, z0 = 0.f, x1 = 0.f, z1 = 1.f;
#pragma unroll
        for (int j = 0; j < TPG; ++j) {
            const float a2 = av[j] * av[j], phi = kv[j] * kv[j] * rv[j];
            const float z0n = fmaf(pv[j], x0, a2 * z0), z1n = fmaf(pv[j], x1, a2 * z1);
            x0 = fmaf(phi, z0n, x0);
            x1 = fmaf(phi, z1n, x1);
            z0 = z0n;
            z1 = z1n;
        }
        qs[gq][0][n] = x0;
        qs[gq][1][n] = z0;
        qs[gq][2][n] = x1;
        qs[gq][3][n] = z1;
    }
    __syncthreads();
    if (gq & 1) {
        const float m00 = qs[gq - 1][0][n], m10 = qs[gq - 1][1][n], m01 = qs[gq - 1][2][n], m11 = qs[gq - 1][3][n];
        const float xn = fmaf(m00, x, m01 * z), zn = fmaf(m10, x, m11 * z);
        x = xn;
        z = zn;
    }
    __syncthreads();   // the transfers are read
    float lp[TPG], il[TPG], rho[TPG], den[TPG];
    {
        float izp = fast_rcp(z), lam = x * izp;
#pragma unroll
        for (int j = 0; j < TPG; ++j) {
            const float kr = kv[j] * rv[j];
            const float zn = fmaf(pv[j], x, av[j] * av[j] * z);
            const float xn = fmaf(kr * kv[j], zn, x);
            const float iz = fast_rcp(zn);
            lp[j] = lam;
            lam = xn * iz;
            il[j] = zn * fast_rcp(xn);
            rho[j] = z * iz;
            den[j] = zn * izp;
            izp = iz;
            x = xn;
            z = zn;
        }
    }
    // pass 1
    float Am = 1.f, Bm = 0.f, Cm = 0.f, Dm = 0.f, u_[TPG], w_[TPG];
#pragma unroll
    for (int j = TPG - 1; j >= 0; --j) {
        const float qi = qv[j] * il[j], qg = YG ? qv[j] * gv[j] : 0.f, rho2 = rho[j] * rho[j];
        const float u = qi * dqt[j] - rv[j] * kv[j] * dkh[j], w = qi * (dqt[j] + qg) * il[j];
        const float al = av[j] * av[j] * rho2, be = pv[j] * rho[j];
        u_[j] = u;
        w_[j] = w;
        Cm = al * Cm - be * Dm - (al * w + be * u);
        Bm = al * Bm - be;
        Am = al * Am;
        Dm = Dm + u;
    }
    qs[gq][0][n] = Am;
    qs[gq][1][n] = Bm;
    qs[gq][2][n] = Cm;
    qs[gq][3][n] = Dm;
    __syncthreads();
#pragma unroll
    for (int g2 = NG - 1; g2 >= 1; --g2) {   // through the later groups
        const bool use = g2 > gq;
        const float cn = fmaf(qs[g2][0][n], cc, fmaf(qs[g2][1][n], SS, qs[g2][2][n]));
        cc = use ? cn : cc;
        SS = use ? SS + qs[g2][3][n] : SS;
    }
    // pass 2
    const rsrc_t oq = make_rsrc(static_cast<uint16_t*>(g.dq) + k0, kbytes);
    const rsrc_t ok_ = make_rsrc(static_cast<uint16_t*>(g.dk) + k0, kbytes);
    const rsrc_t oa = make_rsrc(static_cast<uint16_t*>(TI ? g.dq : g.da) + k0, gbytes);
    const rsrc_t op = make_rsrc(static_cast<uint16_t*>(TI ? g.dq : g.dp) + k0, gbytes);
    float sum_da = 0.f, sum_dp = 0.f;
#pragma unroll
    for (int j = TPG - 1; j >= 0; --j) {
        const int t = gq * TPG + j;
        const float qg = YG ? qv[j] * gv[j] : 0.f, rho2 = rho[j] * rho[j];
        SS += u_[j];
        const float gl = cc - w_[j];
        const float drho = fmaf(gl, lp[j], SS * den[j]);
        const float dav = fmaf(-2.f * av[j] * rho2, drho, SS * fast_rcp(av[j]));
        const float dpv = -lp[j] * rho2 * drho;
        sR[t][n] = fmaf(kv[j] * kv[j], gl, kv[j] * dkh[j]);
        cc = fmaf(av[j] * av[j] * rho2, gl, -pv[j] * rho[j] * SS);
        const uint32_t vo = (uint32_t)(t * H * DK + n) * 2;   // tokens past the end fall outside
        __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(fmaf(2.f, qg, dqt[j]) * il[j]), oq, vo, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(fmaf(2.f * kv[j] * rv[j], gl, rv[j] * dkh[j])), ok_, vo, 0, 0);
        if constexpr (TI) {
            if (t < nt) {
                sum_da += dav;
                sum_dp += dpv;
            }
        } else {
            __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(dav), oa, vo, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(dpv), op, vo, 0, 0);
        }
    }
    if constexpr (TI) {
        __syncthreads();   // the summaries are read
        qs[gq][0][n] = sum_da;
        qs[gq][1][n] = sum_dp;
    }
    __syncthreads();
    {   // dr: the sum over the slots, NT / kC lanes per token
        constexpr int L = NT / kC;
        const int t = tid / L, l = tid % L;
        float acc = 0.f;
#pragma unroll
        for (int m = l; m < DK; m += L) acc += sR[t][m];
#pragma unroll
        for (int of = L / 2; of; of /= 2) acc += __shfl_xor(acc, of, 64);
        if (l == 0 && t < nt) static_cast<uint16_t*>(g.dr)[(tok0 + t) * H + h] = f32_to_bf16(acc);
    }
    if constexpr (TI)
        if (gq < 2) ous[(row * 2 + gq) * DK + n] = (qs[0][gq][n] + qs[1][gq][n]) + (qs[2][gq][n] + qs[3][gq][n]);
}

// The two OU parts of a batch row (chunked_ou_parts): the chunk sums of its even and odd chunks,
// later chunks first, those of a window (chunks c0 .. c0 + nc - 1) added to what the later windows left.
__global__ __launch_bounds__(64) void bwd_ou_kernel(int nbh, int H, int B, int DK, int c0, int nc, bool last,
                                                    const float* __restrict__ ous, float* __restrict__ part) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nbh * 4 * DK) return;
    const int n = i % DK, q = i / DK % 2, par = i / (2 * DK) % 2, bh = i / (4 * DK), b = bh / H, h = bh % H;
    float* o = part + (size_t)q * 2 * nbh * DK + ((size_t)(par * B + b) * H + h) * DK + n;
    float acc = last ? 0.f : *o;
    const int j1 = nc - 1 - ((c0 + nc - 1 - par) & 1);   // the window's last chunk of this parity
#pragma unroll 8
    for (int j = j1; j >= 0; j -= 2) acc += ous[(((size_t)bh * nc + j) * 2 + q) * DK + n];
    *o = acc;
}

template <int DK, int DV, bool TI, bool YG>
hipError_t launch_seg(const Shape& s, const BwdCut& cut, const BwdArgs& a, const float* saved_lam, const float* saved_H,
                      void* ws, hipStream_t st) {
    using Cfg = DkCfg<DK, DV>;
    auto kern = bwd_dk_kernel<DK, DV, TI, YG, true>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::BYTES);
    if (attr != hipSuccess) return attr;
    const int nbh = s.B * s.H, nct = (s.T + kC - 1) / kC;
    const SegBufs f(s, cut.w, cut.lc, ws);
    const size_t hseq = (size_t)(nct + 1) * DK * DV;
    hipError_t e;
    for (int s1 = cut.ns; s1 > 0; s1 -= cut.w) {   // the window's segments s0 .. s1 - 1
        const int s0 = std::max(s1 - cut.w, 0), w = s1 - s0;
        const int c0 = s0 * cut.lc, nc = std::min(w * cut.lc, nct - c0);
        const bool last = s1 == cut.ns;
        e = s1 > 1 ? launch_backward_dv(s, cut.ns, cut.lc, s0, w, true, a, saved_lam, f.gend, f.pseg, st) : hipSuccess;
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(bwd_state_scan_kernel, dim3((unsigned)(((size_t)nbh * DK * DV + 255) / 256)), dim3(256), 0, st,
                           nbh, DK, DV, s0, w, last, f.pseg, a.detaT, f.gend, f.cg);
        e = launch_backward_dv(s, cut.ns, cut.lc, s0, w, false, a, saved_lam, f.gend, f.pseg, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(nbh * w * Cfg::NNT)), dim3(Cfg::NTHR), Cfg::BYTES, st, s,
                           Seg{cut.ns, cut.lc, w, s0}, a, saved_lam, saved_H, nullptr, f.gend, f.xy, f.coef);
        hipLaunchKernelGGL(bwd_carry_kernel, dim3((unsigned)((nbh * DK + 63) / 64)), dim3(64), 0, st, nbh, DK, DV, nc, last,
                           f.coef, f.ccs, saved_H + (size_t)nct * DK * DV, hseq, a.dlamT, a.detaT,
                           s0 == 0 ? a.dlam0 : nullptr);
        hipLaunchKernelGGL((bwd_grad_kernel<DK, TI, YG>), dim3((unsigned)(nbh * nc)), dim3(4 * DK), 0, st, s, c0, nc, a,
                           saved_lam, f.xy, f.coef, f.ous);
        if (TI)
            hipLaunchKernelGGL(bwd_ou_kernel, dim3((unsigned)((nbh * 4 * DK + 63) / 64)), dim3(64), 0, st, nbh, s.H, s.B,
                               DK, c0, nc, last, f.ous, static_cast<float*>(a.ou_part));
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int DK, int DV, bool TI, bool YG>
hipError_t launch_either(const Shape& s, const BwdArgs& a, const float* saved_lam, const float* saved_H, void* ws,
                         size_t limit, hipStream_t st) {
    const BwdCut cut = bwd_cut(s, limit);
    if (cut.ns > 1) return launch_seg<DK, DV, TI, YG>(s, cut, a, saved_lam, saved_H, ws, st);
    return launch_dk<DK, DV, TI, YG>(s, a, saved_lam, saved_H, static_cast<float*>(ws), st);
}

}  // namespace

bool chunked_bwd_supported(const Shape& s) { return s.bf16 && s.dk >= 32 && s.dv >= 32; }

// one part per (wave of a pair, batch row)
int chunked_ou_parts(const Shape& s) { return 2 * s.B; }

// the segment-parallel form's buffers, or per-pair dr partials: dk / 16 of them per token
size_t chunked_bwd_workspace(const Shape& s, size_t limit) {
    const BwdCut cut = bwd_cut(s, limit);
    if (cut.ns > 1) return seg_bytes(s, cut.w, cut.lc);
    return (size_t)(s.dk / 16) * s.B * s.T * s.H * sizeof(float);
}

hipError_t launch_backward_chunked(const Shape& s, const BwdArgs& a, const void* saved, void* ws, size_t limit,
                                   hipStream_t st) {
    const size_t nchunk = (size_t)(s.T + kC - 1) / kC;
    const float* saved_lam = static_cast<const float*>(saved);
    const float* saved_H = saved_lam + (size_t)s.B * s.H * nchunk * kLamRows * s.dk;
#define KLA_DK_CASE(DK_, DV_)                                                    \
    if (s.dk == DK_ && s.dv == DV_) {                                            \
        if (a.dyvar)                                                             \
            return a.ou_a ? launch_either<DK_, DV_, true, true>(s, a, saved_lam, saved_H, ws, limit, st) \
                          : launch_either<DK_, DV_, false, true>(s, a, saved_lam, saved_H, ws, limit, st); \
        return a.ou_a ? launch_either<DK_, DV_, true, false>(s, a, saved_lam, saved_H, ws, limit, st)     \
                      : launch_either<DK_, DV_, false, false>(s, a, saved_lam, saved_H, ws, limit, st);    \
    }
#define KLA_DK_ROW(DK_) KLA_DK_CASE(DK_, 32) KLA_DK_CASE(DK_, 64) KLA_DK_CASE(DK_, 128)
    KLA_DK_ROW(32) KLA_DK_ROW(64) KLA_DK_ROW(128)
#undef KLA_DK_ROW
#undef KLA_DK_CASE
    return hipErrorInvalidValue;
}

}  // namespace kla
