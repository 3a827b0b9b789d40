// Chunked forward of the KLA filter on MFMA (bf16 inputs, fp32 state).
//
// Per chunk of kC = 32 tokens, with Qp[t, n] = (q_t / lam_t) P_t and
// Kn[t, n] = (r_t k_t) / P_t from the precision walk (kla_chunk.hpp), the
// information-state recursion over the chunk is exactly
//   y    = mask(Qp Kn^T) V + Qp H                       (readout, Algorithm 1)
//   H   <- diag(P_C) (H + Kn^T V)                       (state at the chunk end)
// (the unrolled "attention matrix" of the paper's appendix, restricted to a
// chunk, plus the carried state).  The contractions run on
// v_mfma_f32_16x16x32_bf16 with split-bf16 operands for the fp32 factors
// (kla_mfma.hpp), accumulating in fp32.
//
// One workgroup per (batch, head, segment of the sequence, value tile): scan waves
// walk chunk c while MFMA waves (16 or 32 value channels each, the state H[dk, 16]
// in registers) consume chunk c - 1 -- attention tiles, readout, y, state
// update; operands that run across the rows of a tile (Kn^T, V) are read with
// transposing LDS reads (lds_tr8), so each tile is stored once.  The MFMA
// waves only store; all loads come from the scan waves.  TI: the gates come
// from OU parameters (time-invariant per key slot) instead of per-token tensors.
#include "kla_chunk.hpp"
#include "kla_internal.hpp"

namespace kla {
namespace {

// Start beliefs (lam0, eta0) are indexed by sequence, or with ns > 1 segments by
// bh * ns + segment; so are the states a NOY pass leaves in etaT.  Otherwise the last
// segment writes the final belief.
template <int DK, int DV, bool WIDE, bool YV, bool TI, bool NOY, bool SAVE>
__global__ __launch_bounds__((ChunkCfg<DK, DV, WIDE>::NTHR)) void fwd_chunk_kernel(Shape s, Seg sg, FwdArgs g,
                                                                               float* saved_lam, float* saved_H) {
    using Cfg = ChunkCfg<DK, DV, WIDE>;
    constexpr int DVT = Cfg::DVT, NTILE = Cfg::NTILE, DCW = Cfg::DCW, NDT = Cfg::NDT, NSW = Cfg::NSW;
    constexpr int SW = Cfg::SW, NRT = Cfg::NRT, KSN = Cfg::KSN;
    extern __shared__ __align__(16) unsigned char smem[];

    const uint16_t* q = static_cast<const uint16_t*>(g.q);
    const uint16_t* k = static_cast<const uint16_t*>(g.k);
    const uint16_t* v = static_cast<const uint16_t*>(g.v);
    const uint16_t* a = static_cast<const uint16_t*>(g.a);
    const uint16_t* p = static_cast<const uint16_t*>(g.p);
    const uint16_t* r = static_cast<const uint16_t*>(g.r);
    uint16_t* y = static_cast<uint16_t*>(g.y);

    int vi, tile;
    xcd_tile_map(blockIdx.x, s.B * s.H * sg.run, NTILE, vi, tile);
    const int bh = vi / sg.run, seg = sg.first + vi % sg.run;
    const int b = bh / s.H, h = bh % s.H;
    const int c0 = seg * sg.lc, nct = (s.T + kC - 1) / kC;   // this segment's first chunk, the sequence's chunks
    const int H = s.H, T = min(s.T - c0 * kC, sg.lc * kC);
    const size_t start = (size_t)bh * sg.ns + seg;           // row of the start belief
    const size_t out = NOY ? start : bh;
    const bool ends = NOY || seg == sg.ns - 1;               // leaves a final belief
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform role
    const int l16 = lane & 15, g4 = lane >> 4;
    const int nchunk = (T + kC - 1) / kC;
    const size_t seq0 = (size_t)b * s.T + (size_t)c0 * kC;   // token index of the first token

    if (wave < NSW) {
        // ================================================================ scan waves
        const ScanSrc sc{a, p, k, q, r, v, tile * DVT, seq0, H, h, T, nchunk, start, g.ou_a, g.ou_p, g.ou_d,
                         g.range_flag};
        const float x = scan_wave<Cfg, YV, false, TI, NOY>(smem, wave, lane, sc, g.lam0, SAVE);
        if (g.lamT && ends && lane < SW && tile == 0) g.lamT[out * DK + wave * SW + lane] = x;
    } else {
        // ================================================================ MFMA waves
        const int m = wave - NSW;
        const int dm0 = tile * DVT + m * DCW;   // first value channel of this wave
        const int dl0 = m * DCW;                // its first column within the value tile

        // state H[n, d] for n = 16 rt + 4 g4 + rr, d = dm0 + 16 dt + l16
        f32x4 Hs[NRT][NDT];
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
                    Hs[rt][dt][rr] =
                        g.eta0 ? g.eta0[(start * DK + 16 * rt + 4 * g4 + rr) * DV + dm0 + 16 * dt + l16] : 0.f;

        // state rows 16 rt .. 16 rt + 15 (this wave's columns) into the saved slot behind rs
        const uint32_t h_voff = (uint32_t)(4 * g4 * DV + dm0 + l16) * 4;
        auto save_rows = [&](rsrc_t rs, int rt) {
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
                    buf_st32s(Hs[rt][dt][rr], rs, h_voff, (uint32_t)((16 * rt + rr) * DV + 16 * dt) * 4);
        };
        auto slot_rsrc = [&](int slot) {
            return make_rsrc(saved_H + ((size_t)bh * (nct + 1) + c0 + slot) * DK * DV, DK * DV * 4);
        };
        // eta0 has arrived: without this the loop would wait for it at the first use of the state,
        // and with it, every round, for all stores of the round before (65536-token forward without
        // a saved context: 855 -> 808 us, together with its stores through buffers)
        wait_vm_all();
        for (int c = 0; c <= nchunk; ++c) {
            const int cc = c - 1;   // the chunk consumed in this round
            if (cc >= 0) {
                const int nt = min(kC, T - cc * kC);
                const size_t row0 = seq0 + (size_t)cc * kC;
                const unsigned char* buf = smem + (cc & 1) * Cfg::BUF;
                const uint16_t* sVS = reinterpret_cast<const uint16_t*>(buf + Cfg::VS);   // V [t][DVT]
                const uint16_t* sQH = reinterpret_cast<const uint16_t*>(buf + Cfg::QH);
                const uint16_t* sQL = reinterpret_cast<const uint16_t*>(buf + Cfg::QL);
                const uint16_t* sKH = reinterpret_cast<const uint16_t*>(buf + Cfg::KH);
                const uint16_t* sKL = reinterpret_cast<const uint16_t*>(buf + Cfg::KL);
                const float* sDec = reinterpret_cast<const float*>(buf + Cfg::DEC);

                if constexpr (!NOY) {   // the readout (skipped when only the final state is asked for)
                    // ---- S^T[j, i] = sum_n Kn[j, n] Qp[i, n], tiles (jt, it) = (0,0), (0,1), (1,1)
                    f32x4 S00 = zero4(), S01 = zero4(), S11 = zero4();
#pragma unroll
                    for (int ks = 0; ks < KSN; ++ks) {
                        const int n0 = 32 * ks + 8 * g4;
                        const bf16x8 k0h = nt_tr8(sKH, n0, n0 + 4, 0, l16), k0l = nt_tr8(sKL, n0, n0 + 4, 0, l16);
                        const bf16x8 k1h = nt_tr8(sKH, n0, n0 + 4, 16, l16), k1l = nt_tr8(sKL, n0, n0 + 4, 16, l16);
                        const bf16x8 q0h = nt_tr8(sQH, n0, n0 + 4, 0, l16), q0l = nt_tr8(sQL, n0, n0 + 4, 0, l16);
                        const bf16x8 q1h = nt_tr8(sQH, n0, n0 + 4, 16, l16), q1l = nt_tr8(sQL, n0, n0 + 4, 16, l16);
                        S00 = mfma3(k0h, k0l, q0h, q0l, S00);
                        S01 = mfma3(k0h, k0l, q1h, q1l, S01);
                        S11 = mfma3(k1h, k1l, q1h, q1l, S11);
                    }
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {   // causal mask j <= i inside the diagonal tiles
                        if (4 * g4 + rr > l16) {
                            S00[rr] = 0.f;
                            S11[rr] = 0.f;
                        }
                    }
                    // B operands over the 32-deep contraction j (rows {4g..4g+3} and {16+4g..16+4g+3})
                    bf16x8 sbh[2], sbl[2];
                    split8(S00, zero4(), sbh[0], sbl[0]);
                    split8(S01, S11, sbh[1], sbl[1]);

                    // ---- y^T[d, i] = sum_j V^T[d, j] S^T[j, i] + sum_n H^T[d, n] Qp^T[n, i]
                    f32x4 yacc[NDT][2];
#pragma unroll
                    for (int dt = 0; dt < NDT; ++dt) {
                        const bf16x8 va = lds_tr8(sVS, DVT, 4 * g4, 16 + 4 * g4, dl0 + 16 * dt, l16);
#pragma unroll
                        for (int it = 0; it < 2; ++it) yacc[dt][it] = mfma2b(va, sbh[it], sbl[it], zero4());
                    }
#pragma unroll
                    for (int ks = 0; ks < KSN; ++ks) {
                        bf16x8 qbh[2], qbl[2];
#pragma unroll
                        for (int it = 0; it < 2; ++it) {
                            const int n0 = 32 * ks + 4 * g4;
                            qbh[it] = nt_tr8(sQH, n0, n0 + 16, 16 * it, l16);
                            qbl[it] = nt_tr8(sQL, n0, n0 + 16, 16 * it, l16);
                        }
#pragma unroll
                        for (int dt = 0; dt < NDT; ++dt) {
                            bf16x8 hh, hl;
                            split8(Hs[2 * ks][dt], Hs[2 * ks + 1][dt], hh, hl);
#pragma unroll
                            for (int it = 0; it < 2; ++it) yacc[dt][it] = mfma3(hh, hl, qbh[it], qbl[it], yacc[dt][it]);
                        }
                        // the chunk-start state goes to the saved context a few rows at a time, between
                        // the products, so that the stores of all workgroups do not come in one burst
                        if constexpr (SAVE) {
                            const rsrc_t rs = slot_rsrc(cc);
                            save_rows(rs, 2 * ks);
                            save_rows(rs, 2 * ks + 1);
                        }
                    }
                    // y[t, d .. d+3] for t = 16 it + l16, d = dm0 + 16 dt + 4 g4; rows past the chunk's
                    // last token fall outside the buffer
                    const rsrc_t ry = make_rsrc(y + (row0 * H + h) * DV + dm0, (uint32_t)((nt - 1) * H * DV + DCW) * 2);
#pragma unroll
                    for (int it = 0; it < 2; ++it)
#pragma unroll
                        for (int dt = 0; dt < NDT; ++dt)
                            buf_st64(uint2{cvt_pk_bf16(yacc[dt][it][0], yacc[dt][it][1]),
                                           cvt_pk_bf16(yacc[dt][it][2], yacc[dt][it][3])},
                                     ry, (uint32_t)((16 * it + l16) * H * DV + 16 * dt + 4 * g4) * 2);
                }

                // ---- state: H <- diag(P_C) (H + Kn^T V)
                bf16x8 vb[NDT];   // V rows t = 8 g4 .. 8 g4 + 7 of column d
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) vb[dt] = lds_tr8(sVS, DVT, 8 * g4, 8 * g4 + 4, dl0 + 16 * dt, l16);
#pragma unroll
                for (int rt = 0; rt < NRT; ++rt) {
                    // Kn^T rows n = 16 rt + l16, tokens 8 g4 .. 8 g4 + 7
                    const bf16x8 kth = nt_row8(sKH, 16 * rt + l16, g4), ktl = nt_row8(sKL, 16 * rt + l16, g4);
                    const float4 dec = *reinterpret_cast<const float4*>(sDec + 16 * rt + 4 * g4);
#pragma unroll
                    for (int dt = 0; dt < NDT; ++dt) {
                        const f32x4 hacc = mfma2a(kth, ktl, vb[dt], Hs[rt][dt]);
                        Hs[rt][dt][0] = hacc[0] * dec.x;
                        Hs[rt][dt][1] = hacc[1] * dec.y;
                        Hs[rt][dt][2] = hacc[2] * dec.z;
                        Hs[rt][dt][3] = hacc[3] * dec.w;
                    }
                }

                // the chunk's walk state goes to the saved context (one value tile stores it)
                if (SAVE && tile == 0) {
                    constexpr int NV4 = kLamRows * DK / 4;
                    const float4* src = reinterpret_cast<const float4*>(buf + Cfg::MIDS);
                    float4* dst = reinterpret_cast<float4*>(saved_lam + ((size_t)bh * nct + c0 + cc) * kLamRows * DK);
                    for (int i = m * 64 + lane; i < NV4; i += Cfg::NMW * 64) dst[i] = src[i];
                }

                if (YV && tile == 0 && m == 0 && lane < nt) {
                    const float* yv = reinterpret_cast<const float*>(buf + Cfg::YVP);
                    float acc = 0.f;
#pragma unroll
                    for (int w2 = 0; w2 < NSW; ++w2) acc += yv[w2 * kC + lane];
                    g.yvar[(row0 + lane) * H + h] = acc;
                }
            }
            barrier_lds();
        }

        if (SAVE && ends) {   // the final state closes the saved sequence
            const rsrc_t rs = slot_rsrc(nchunk);
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt) save_rows(rs, rt);
        }
        if (g.etaT && ends) {
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
                        g.etaT[(out * DK + 16 * rt + 4 * g4 + rr) * DV + dm0 + 16 * dt + l16] = Hs[rt][dt][rr];
        }
    }
}

template <int DK, int DV, bool WIDE, bool YV, bool TI, bool NOY, bool SAVE>
hipError_t launch_fwd_v(const Shape& s, const Seg& sg, const FwdArgs& a, float* saved_lam, float* saved_H,
                        hipStream_t st) {
    using Cfg = ChunkCfg<DK, DV, WIDE>;
    auto kern = fwd_chunk_kernel<DK, DV, WIDE, YV, TI, NOY, SAVE>;
    // more than 64 KiB of LDS must be opted into once per kernel (thread-safe static init)
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::BYTES);
    if (attr != hipSuccess) return attr;
    const unsigned grid = (unsigned)(s.B * s.H * sg.run * Cfg::NTILE);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(Cfg::NTHR), Cfg::BYTES, st, s, sg, a, saved_lam, saved_H);
    return hipGetLastError();
}

// the readout variance adds a cross-lane sum per token and the saved context its stores,
// so they are separate instantiations, as are the time-invariant gates and the state-only
// pass (no y: the segment-parallel forward's first pass)
template <int DK, int DV, bool WIDE, bool TI>
hipError_t launch_fwd(const Shape& s, const Seg& sg, const FwdArgs& a, float* saved_lam, float* saved_H,
                      hipStream_t st) {
    if (!a.y) return launch_fwd_v<DK, DV, WIDE, false, TI, true, false>(s, sg, a, nullptr, nullptr, st);
    if (saved_H)
        return a.yvar ? launch_fwd_v<DK, DV, WIDE, true, TI, false, true>(s, sg, a, saved_lam, saved_H, st)
                      : launch_fwd_v<DK, DV, WIDE, false, TI, false, true>(s, sg, a, saved_lam, saved_H, st);
    return a.yvar ? launch_fwd_v<DK, DV, WIDE, true, TI, false, false>(s, sg, a, nullptr, nullptr, st)
                  : launch_fwd_v<DK, DV, WIDE, false, TI, false, false>(s, sg, a, nullptr, nullptr, st);
}

template <int DK, int DV, bool WIDE>
hipError_t launch_fwd_ti(const Shape& s, const Seg& sg, const FwdArgs& a, float* saved_lam, float* saved_H,
                         hipStream_t st) {
    return a.ou_a ? launch_fwd<DK, DV, WIDE, true>(s, sg, a, saved_lam, saved_H, st)
                  : launch_fwd<DK, DV, WIDE, false>(s, sg, a, saved_lam, saved_H, st);
}

}  // namespace

bool chunked_supported(const Shape& s) { return s.bf16 && s.dk >= 32; }

// Saved context: the precision walk's state of every chunk [BH][nchunk][kLamRows][dk]
// (lam at the chunk start, lam_16 and P_16 after its first 16 tokens), then the
// information state at every chunk start and after the last token
// [BH][nchunk+1][dk][dv].
size_t chunked_saved_bytes(const Shape& s) {
    const size_t nchunk = (size_t)(s.T + kC - 1) / kC;
    return (size_t)s.B * s.H * s.dk * (kLamRows * nchunk + (nchunk + 1) * (size_t)s.dv) * sizeof(float);
}

bool chunked_wide(const Shape& s, int groups) {
    // dv = 128 in one workgroup per (sequence, segment) instead of two: where that takes fewer
    // rounds of the chip's 256 CUs (each workgroup fills a CU), the walk's repetition is saved
    // (a wide round takes 3.6 us against 3.1)
    const int n = s.B * s.H * groups;
    return s.dv == 128 && s.dk >= 64 && (2 * n + 255) / 256 > (n + 255) / 256;
}

hipError_t launch_forward_chunked_seg(const Shape& s, int ns, int lc, int run, const FwdArgs& a, void* saved,
                                      hipStream_t st) {
    float* saved_lam = nullptr;
    float* saved_H = nullptr;
    if (saved) {
        const size_t nchunk = (size_t)(s.T + kC - 1) / kC;
        saved_lam = static_cast<float*>(saved);
        saved_H = saved_lam + (size_t)s.B * s.H * nchunk * kLamRows * s.dk;
    }
    const Seg sg{ns, lc, run};
    if (chunked_wide(s, run)) {
        if (s.dk == 64) return launch_fwd_ti<64, 128, true>(s, sg, a, saved_lam, saved_H, st);
        if (s.dk == 128) return launch_fwd_ti<128, 128, true>(s, sg, a, saved_lam, saved_H, st);
    }
#define KLA_FWD_CASE(DK_, DV_) \
    if (s.dk == DK_ && s.dv == DV_) return launch_fwd_ti<DK_, DV_, false>(s, sg, a, saved_lam, saved_H, st);
#define KLA_FWD_ROW(DK_) KLA_FWD_CASE(DK_, 16) KLA_FWD_CASE(DK_, 32) KLA_FWD_CASE(DK_, 64) KLA_FWD_CASE(DK_, 128)
    KLA_FWD_ROW(32) KLA_FWD_ROW(64) KLA_FWD_ROW(128)
#undef KLA_FWD_ROW
#undef KLA_FWD_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_forward_chunked(const Shape& s, const FwdArgs& a, void* saved, hipStream_t st) {
    return launch_forward_chunked_seg(s, 1, (s.T + kC - 1) / kC, 1, a, saved, st);
}

}  // namespace kla
