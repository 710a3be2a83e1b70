// Integer GEMM + dequantization epilogue + fp16 outlier GEMM for gfx950
// (Algorithm 1 of arXiv 2310.09259: "INTmatmul", "Dequantization", "FPmatmul" and
// the final add; epilogue fusion as in Section 3.4).
//
// Data path.  gfx950 has no 4-bit integer MFMA, so packed nibbles travel
// HBM -> LDS -> VGPR still packed and are widened to int8 in registers.  A dot
// product does not care in which order k is visited as long as both operands
// agree, so the high and the low nibbles of a packed word simply become two
// different operand registers (no re-interleaving).  Two widenings are used:
//   symmetric:  (w & 0xF0F0F0F0) and ((w << 4) & 0xF0F0F0F0) hold 16x the signed
//     nibbles; done to both operands every product is exactly 256x too large
//     (3 VALU operations per two operand registers).  Used by the raw-accumulator
//     hook when it is given no correction terms.
//   asymmetric: one AND per operand register.  (w & 0xF0F0F0F0) is 16x the signed
//     high nibble; ((w ^ 0x08080808) & 0x0F0F0F0F) is the low nibble plus 8 (an
//     unsigned value 0..15).  Activations keep element 2p in the high nibble,
//     weights in the low nibble, so every product pairs a "16x" register with a
//     "+8" register of the same k: even k gives 16*a*(b+8), odd k gives (a+8)*16*b,
//     and the accumulator holds 16*sum(a*b) + 128*sum_{even k} a + 128*sum_{odd k} b.
//     The two sums are per-token / per-channel integers computed once (by the
//     quantization kernel and by the weight preparation) and subtracted, exactly,
//     in the epilogue.
// Headroom: the raw accumulator stays below 2^31 for K_b < 131072.
//
// MFMA shape: v_mfma_i32_32x32x32_i8.  First operand = activations (32 token
// rows), second = weights (32 output channels).  Lane l supplies row/column l%32
// and the k-group l/32; it receives output column l%32 and rows
// 8*(r/4) + 4*(l/32) + r%4 in accumulator register r.  The fp16 outlier product
// uses v_mfma_f32_32x32x16_f16, whose accumulator has the same layout, so the
// dequantized tile is simply the C operand of the outlier stages.
//
// Mixed widths (4-bit weights under 8-bit activations): see MIXED in gemm_kernel.
//
// Pipeline.  A workgroup of four or eight waves owns a BM x BN output tile.  Operand panels
// are copied global -> LDS without passing through registers (buffer_load ... lds,
// 16 bytes per lane, BKB bytes of every row per stage, NST stage buffers).  Rows
// beyond T / N and bytes beyond the row end are out of range for the buffer
// descriptor and arrive as zeros.  The 16-byte slots of a row are XOR-swizzled so
// that the 32 rows a ds_read_b128 touches fall into distinct banks.  The int4
// stages and the fp16 outlier stages run through the same stage ring.  Inside a
// wave the work is software pipelined three deep and the order is pinned with
// scheduling barriers: while the MFMAs of sub-step q issue, the packed words of
// sub-step q+1 are widened and the LDS reads of sub-step q+2 are in flight.
// One workgroup barrier per stage; right after it the stage buffer it has just
// freed is refilled, the DMA instructions spread between MFMAs.
//
// Epilogue.  Per-row parameters (LDS) and per-column parameters (registers) are
// fetched before the first DMA.  After the int stages the accumulators are
// dequantized in place of the C operand of the fp16 outlier stages; the fp16
// result tile is parked in the dead stage ring and leaves the CU as 16-byte
// pieces, whole row segments per store instruction.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "quik_kernels.h"
#include "quik_gemm_device.h"

namespace quik {

namespace {

using namespace gemm_dev;

// BM x BN output tile per workgroup, WM x WN waves, BKB bytes of every packed row per
// stage, NST stage buffers, GM = m-tiles per group of the tile order (0: plain column sweep).
// MODE 0: fused epilogue (asymmetric widening for 4 bits); MODE 1: write raw INT32 accumulators,
// symmetric widening; MODE 2: raw accumulators, asymmetric widening plus correction terms.
// BITS: activation bits; WBITS: weight bits (equal, or 4-bit weights under 8-bit activations).
template <int BITS, int WBITS, int BM, int BN, int WM, int WN, int BKB, int NST, int OCC, int GM, int MODE>
__global__ __launch_bounds__(WM * WN * 64, OCC) void gemm_kernel(GemmArgs a) {
    constexpr bool RAW = MODE != 0;
    constexpr bool ASYM = (BITS == 4) && (MODE != 1);
    // Every form runs two waves per SIMD (WM * WN * OCC = 8 waves per CU, and the stage buffers leave no room
    // for more workgroups), so each claims the full 256 registers of its share: the top of the allocation is
    // then never a live register (the row-quantization kernel misread such a register on MI355X when its
    // allocation left part of the SIMD's file free).
    static_assert(WM * WN * OCC == 8, "two waves per SIMD");
    asm volatile("" ::: "v255");
    // Mixed layers: a stage still covers BKB activation bytes = BKB k, which is only BKB/2 packed
    // weight bytes.  The weight nibbles are widened to 16x int8 (even / odd k of a word in two
    // registers); the int8 activations are brought into the same k order with two byte permutes
    // per 8 elements.  Accumulators are exactly 16x the integer dot product.
    constexpr bool MIXED = (BITS == 8 && WBITS == 4);
    static_assert(WBITS == BITS || MIXED, "weights: same width as the activations, or 4 under 8");
    constexpr int NWAVES = WM * WN, NT = NWAVES * 64;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int CPR = BKB / 16, RPI = 64 / CPR;
    constexpr int A_INSTR = BM / RPI / NWAVES, B_INSTR = BN / RPI / NWAVES;
    static_assert(A_INSTR >= 1 && B_INSTR >= 1, "tile too small for the wave count");
    constexpr int LPS = A_INSTR + B_INSTR;
    constexpr int KSUB = BKB / 32;
    constexpr int SHIFT = (BITS == 4) ? (ASYM ? 4 : 8) : (MIXED ? 4 : 0);
    constexpr int A_BYTES = BM * BKB, B_BYTES = BN * BKB, ST_BYTES = A_BYTES + B_BYTES;
    // mixed int stages: weight rows of BKW bytes, RPW rows per DMA instruction, WI instructions
    // per wave; the remaining B_INSTR - WI slots of a stage are issued as empty (out-of-range)
    // loads so that every stage counts the same number of DMA instructions
    constexpr int BKW = BKB / 2, CPW = BKW / 16, RPW = 64 / CPW;
    constexpr int WI = MIXED ? BN / RPW / NWAVES : B_INSTR;
    static_assert(!MIXED || (WI >= 1 && BKB == 128), "mixed layers: tile too small for the wave count");
    constexpr int NF = TM + TN;
    constexpr int HALVES = (BITS == 4) ? 2 : 1;          // MFMAs per output tile per sub-step
    constexpr int SLOTS = TM * TN * HALVES;
    constexpr int WORDS = NF * 4;
    // LDS reads run LA sub-steps ahead of their MFMAs (3 and 4 were measured: no faster, so the cost of
    // the fragment reads is their throughput, not their latency)
    constexpr int LA = (2 < KSUB) ? 2 : KSUB - 1;
    constexpr int RD = (KSUB % LA == 0) ? LA : LA + 1;   // raw fragment sets (a divisor of KSUB: static indices)
    constexpr int BAR_KS = KSUB - LA;                    // stage barrier sits before this sub-step
    static_assert(KSUB % 2 == 0 && NST >= 2 && LA >= 1 && KSUB % RD == 0, "raw set index must be static");

    __shared__ __align__(1024) uint8_t lds[NST * ST_BYTES];
    __shared__ __align__(16) float lds_sa[BM];
    __shared__ __align__(16) float lds_sh[BM];
    __shared__ __align__(16) int lds_ct[BM];             // -128 * (per-token correction sum)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int wm = wave_u / WN, wn = wave_u % WN;
    const int l32 = lane & 31, g = lane >> 5;

    const int tiles_m = (a.T + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    const int id = xcd_contiguous_id(blockIdx.x, tiles_m * tiles_n);
    // Tile order inside an XCD's range: GM consecutive m-tiles form a group that is swept along n
    // (m fastest), so the group's activation panels stay in that XCD's L2 while weight panels stream.
    int tile_m, tile_n;
    if constexpr (GM > 0) {
        const int per_group = GM * tiles_n;
        const int grp = id / per_group, rem = id % per_group;
        const int first_m = grp * GM;
        const int gsz = min(GM, tiles_m - first_m);
        tile_m = first_m + rem % gsz;
        tile_n = rem / gsz;
    } else {
        tile_m = id % tiles_m;
        tile_n = id / tiles_m;
    }
    const int t0 = tile_m * BM, n0 = tile_n * BN;

    const int row_bytes = a.K_b * BITS / 8;
    const int int_bytes = (row_bytes + 15) & ~15;
    const int nk_int = a.fp_only ? 0 : (row_bytes + BKB - 1) / BKB;
    const int fp_bytes = a.n_out * 2;
    const int nk_fp = RAW ? 0 : (fp_bytes + BKB - 1) / BKB;
    const int nk = nk_int + nk_fp;
    const int lda_fp = a.ldo * 2, ldb_fp = a.ldwo * 2;

    const v4i rA = make_rsrc((const uint8_t*)a.xq + (size_t)t0 * a.ldq, (size_t)(a.T - t0) * a.ldq);
    const v4i rB = make_rsrc((const uint8_t*)a.w_q + (size_t)n0 * a.ldw, (size_t)(a.N - n0) * a.ldw);
    const v4i rAf = make_rsrc(a.n_out ? (const uint8_t*)a.x_out + (size_t)t0 * lda_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.T - t0) * lda_fp : 0);
    const v4i rBf = make_rsrc(a.n_out ? (const uint8_t*)a.w_out + (size_t)n0 * ldb_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.N - n0) * ldb_fp : 0);

    const int lrow = lane / CPR, lslot = lane % CPR;
    const uint32_t lds_base = lds_addr(lds);
    uint32_t voA[A_INSTR], voB[B_INSTR];
    int chA[A_INSTR], chB[B_INSTR], rwA[A_INSTR], rwB[B_INSTR];
#pragma unroll
    for (int i = 0; i < A_INSTR; ++i) {
        int row = (wave_u * A_INSTR + i) * RPI + lrow;
        int c = (lslot ^ swz<BKB>(row)) * 16;
        rwA[i] = row; chA[i] = c;
        voA[i] = (uint32_t)(row * a.ldq + c);
    }
#pragma unroll
    for (int i = 0; i < B_INSTR; ++i) {
        int row = (wave_u * B_INSTR + i) * RPI + lrow;
        int c = (lslot ^ swz<BKB>(row)) * 16;
        rwB[i] = row; chB[i] = c;
        voB[i] = (uint32_t)(row * a.ldw + c);
    }
    const uint32_t m0A = lds_base + wave_u * A_INSTR * 1024;
    const uint32_t m0B = lds_base + A_BYTES + wave_u * B_INSTR * 1024;
    // mixed int stages: geometry of the half-width weight rows
    uint32_t voW[WI];
    int chW[WI];
    if constexpr (MIXED) {
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            int row = (wave_u * WI + i) * RPW + lane / CPW;
            int c = ((lane % CPW) ^ swz<BKW>(row)) * 16;
            chW[i] = c;
            voW[i] = (uint32_t)(row * a.ldw + c);
        }
    }
    const uint32_t m0W = lds_base + A_BYTES + wave_u * WI * 1024;
    // where a mixed stage's empty loads land: this wave's 1 KB of the unused half of the B region
    const uint32_t m0D = lds_base + A_BYTES + BN * BKW + wave_u * 1024;
    static_assert(!MIXED || NWAVES * 1024 <= BN * BKW, "no room for the empty loads");

    // DMA instruction d of a full (unguarded) int stage
    auto issue_one = [&](int s, int d) {
        const uint32_t sb = (uint32_t)(s % NST) * ST_BYTES;
        const uint32_t so = (uint32_t)s * BKB;
        if (d < A_INSTR) {
            dma16(rA, m0A + sb + d * 1024, voA[d < A_INSTR ? d : 0], so);
        } else if constexpr (MIXED) {
            const int j = d - A_INSTR;
            if (j < WI) dma16(rB, m0W + sb + j * 1024, voW[j < WI ? j : 0], (uint32_t)s * BKW);
            else dma16(rB, m0D + sb, kOob, 0);
        } else {
            dma16(rB, m0B + sb + (d - A_INSTR) * 1024, voB[d >= A_INSTR ? d - A_INSTR : 0], so);
        }
    };
    // any stage: K tail of the int part, fp16 part, or past the end (all lanes out of range)
    auto issue_any = [&](int s) {
        const uint32_t sb = (uint32_t)(s % NST) * ST_BYTES;
        const bool fp = s >= nk_int;
        const int koff = (fp ? s - nk_int : s) * BKB;
        // integer stages stop at the 16-byte piece that holds a row's last packed byte: what lies beyond may
        // be anything in the weight matrix
        const int lima = s < nk ? (fp ? fp_bytes : int_bytes) : 0;
        const int limb = s < nk ? (fp ? fp_bytes : (MIXED ? (((a.K_b / 2) + 15) & ~15) : int_bytes)) : 0;
        const int lda = fp ? lda_fp : a.ldq, ldb = fp ? ldb_fp : a.ldw;
        const v4i ra_ = fp ? rAf : rA;
        const v4i rb_ = fp ? rBf : rB;
#pragma unroll
        for (int i = 0; i < A_INSTR; ++i) {
            uint32_t vo = (koff + chA[i] < lima) ? (uint32_t)(rwA[i] * lda + koff + chA[i]) : kOob;
            dma16(ra_, m0A + sb + i * 1024, vo, 0);
        }
        if (MIXED && !fp) {
            const int koffw = s * BKW;
#pragma unroll
            for (int i = 0; i < B_INSTR; ++i) {
                uint32_t vo = kOob;
                if (i < WI && koffw + chW[i < WI ? i : 0] < limb) vo = voW[i < WI ? i : 0] + (uint32_t)koffw;
                dma16(rb_, (i < WI ? m0W + i * 1024 : m0D) + sb, vo, 0);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < B_INSTR; ++i) {
            uint32_t vo = (koff + chB[i] < limb) ? (uint32_t)(rwB[i] * ldb + koff + chB[i]) : kOob;
            dma16(rb_, m0B + sb + i * 1024, vo, 0);
        }
    };

    // ---- epilogue parameters, fetched before the first DMA so that their (in-order) return does
    // not sit behind the stage loads: per token row (to LDS below) and per output column (registers)
    constexpr int RPT = (BM + NT - 1) / NT;              // token rows per thread
    float p_s[RPT], p_z[RPT];
    int p_c[RPT];
    float c_sw[TN], c_wr[TN], c_bv[TN];
    int c_nc[TN];
    if constexpr (!RAW) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int t = t0 + tid + q * NT;
            const bool ok = (tid + q * NT < BM) && t < a.T;
            p_s[q] = ok ? a.scale[t] : 0.0f;
            p_z[q] = ok ? a.zero[t] : 0.0f;
            p_c[q] = 0;
            if constexpr (ASYM) p_c[q] = (ok && !a.fp_only) ? a.code_sum[t] : 0;
        }
        const __half* __restrict__ wsc = static_cast<const __half*>(a.w_scale);
        const __half* __restrict__ bias = static_cast<const __half*>(a.bias);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = min(n0 + wn * TN * 32 + j * 32 + l32, a.N - 1);
            c_sw[j] = __half2float(wsc[n]) * (1.0f / (float)(1 << SHIFT));   // exact power-of-two factor
            c_bv[j] = bias ? __half2float(bias[n]) : 0.0f;
            c_wr[j] = a.w_reduced[n];
            c_nc[j] = 0;
            if constexpr (ASYM) c_nc[j] = a.fp_only ? 0 : -128 * a.w_code_sum[n];
            if (a.fp_only) { c_sw[j] = 0.0f; c_bv[j] = 0.0f; c_wr[j] = 0.0f; }
        }
    }

    // ---- prologue: fill every stage buffer
#pragma unroll
    for (int s = 0; s < NST; ++s) issue_any(s);

    if constexpr (!RAW) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = tid + q * NT;
            if (r < BM) {
                lds_sa[r] = p_s[q];                                          // scaleAct
                lds_sh[r] = p_z[q] + (float)(1 << (BITS - 1)) * p_s[q];      // zeroAct + halfRange * scaleAct
                if constexpr (ASYM) lds_ct[r] = -128 * p_c[q];               // in raw accumulator units
            }
        }
    }

    uint32_t rd[NF][KSUB];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        int r = (f < TM) ? (wm * TM * 32 + f * 32 + l32) : (wn * TN * 32 + (f - TM) * 32 + l32);
        uint32_t base = (f < TM ? 0 : A_BYTES) + r * BKB;
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) rd[f][ks] = base + (((ks * 2 + g) ^ swz<BKB>(r)) << 4);
    }

    uint4 R[RD][NF];
    v4i U[2][NF][HALVES];

    // mixed int stages: 8 bytes (16 nibbles = this lane's k-group) of a half-width weight row
    uint32_t rdw[MIXED ? TN : 1][KSUB];
    if constexpr (MIXED) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int r = wn * TN * 32 + j * 32 + l32;
#pragma unroll
            for (int ks = 0; ks < KSUB; ++ks) rdw[j][ks] = A_BYTES + r * BKW + ((ks ^ swz<BKW>(r)) << 4) + g * 8;
        }
    }
    auto read_frag = [&](int set, int f, const uint8_t* stage, int ks) {
        R[set][f] = *reinterpret_cast<const uint4*>(stage + rd[f][ks]);
    };
    // fragment f of sub-step ks of a stage that is an int stage (wide == false) or an fp16 stage
    auto read_any = [&](int set, int f, const uint8_t* stage, int ks, bool wide) {
        if constexpr (MIXED) {
            if (f >= TM && !wide) {
                const uint2 v = *reinterpret_cast<const uint2*>(stage + rdw[f >= TM ? f - TM : 0][ks]);
                R[set][f].x = v.x;
                R[set][f].y = v.y;
                return;
            }
        }
        read_frag(set, f, stage, ks);
    };
    auto widen_word = [&](int set, int rset, int w) {
        const int f = w >> 2, k = w & 3;
        const uint32_t x = (k == 0) ? R[rset][f].x : (k == 1) ? R[rset][f].y : (k == 2) ? R[rset][f].z : R[rset][f].w;
        if constexpr (BITS == 4) {
            // slot 0 of a word pair holds the even k of the word, slot 1 the odd k
            constexpr uint32_t M = 0xF0F0F0F0u;
            const bool act = f < TM;                     // activations: even k in the high nibble
            uint32_t hi, lo;
            if constexpr (ASYM) {
                hi = x & M;                              // 16 * signed high nibble
                lo = (x ^ 0x08080808u) & 0x0F0F0F0Fu;    // low nibble + 8
            } else {
                hi = x & M;
                lo = (x << 4) & M;                       // 16 * signed, both
            }
            U[set][f][k >> 1][(k & 1) * 2] = (int)(act ? hi : lo);
            U[set][f][k >> 1][(k & 1) * 2 + 1] = (int)(act ? lo : hi);
        } else if constexpr (MIXED) {
            if (f < TM) {
                // int8 activations k0..k15 -> [even k of the low 8 | odd | even of the high 8 | odd]
                const uint32_t lo = (k < 2) ? R[rset][f].x : R[rset][f].z, hi = (k < 2) ? R[rset][f].y : R[rset][f].w;
                U[set][f][0][k] = (int)__builtin_amdgcn_perm(hi, lo, (k & 1) ? 0x07050301u : 0x06040200u);
            } else {
                // packed weights: word k/2 holds 8 nibbles; even k (low nibbles) / odd k (high), 16x
                constexpr uint32_t M = 0xF0F0F0F0u;
                const uint32_t wv = (k < 2) ? R[rset][f].x : R[rset][f].y;
                U[set][f][0][k] = (int)((k & 1) ? (wv & M) : ((wv << 4) & M));
            }
        } else {
            U[set][f][0][k] = (int)x;
        }
    };

    // With the single-AND widening and the fused epilogue the accumulators start at
    // -128 * (code_sum[t] + w_code_sum[n]) instead of zero, so that the K loop ends on 16 x the integer dot
    // product (the widening leaves it plus 128 times these sums; two's complement, nothing overflows on the way).
    v16i acc[TM][TN];
    if constexpr (ASYM && !RAW) {
        __syncthreads();                                  // lds_ct is complete (the first stages are in flight)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const int4 ct4 = *reinterpret_cast<const int4*>(&lds_ct[wm * TM * 32 + i * 32 + 8 * rq + 4 * g]);
                const int ct_[4] = {ct4.x, ct4.y, ct4.z, ct4.w};
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) acc[i][j][rq * 4 + rr] = ct_[rr] + c_nc[j];
            }
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    }

    // stage barrier of iteration s: stage s+1 has landed for everybody, and nobody reads stage s any more
    auto stage_barrier = [&]() {
        wait_stage<(NST - 2) * LPS>();
        __syncthreads();
    };

    // sub-step ks of stage s.  PLAIN: the DMA into the freed buffer is a full int stage and is spread over
    // the MFMA slots that follow the barrier; otherwise it is issued in one go.
    auto substep = [&](int s, int ks, bool plain) {
        const int par = ks & 1;
        if (ks == BAR_KS) {
            stage_barrier();
            if (!plain) issue_any(s + NST);
        }
        const int ts = (ks + LA < KSUB) ? s : s + 1, tks = (ks + LA) % KSUB;
        const uint8_t* tgt = lds + (ts % NST) * ST_BYTES;
        const int rnext = (ks + 1) % RD, rload = (ks + LA) % RD;   // static: KSUB is a multiple of RD
        const bool wide = ts >= nk_int;                             // the look-ahead reaches the fp16 part
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < SLOTS; ++m) {
            const int h = m / (TM * TN), ij = m % (TM * TN), i = ij / TN, j = ij % TN;
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(U[par][i][h], U[par][TM + j][h], acc[i][j], 0, 0, 0);
            if (plain && ks == BAR_KS) {
                constexpr int PER = (SLOTS >= LPS) ? SLOTS / LPS : 1;
                if (m % PER == 0 && m / PER < LPS) issue_one(s + NST, m / PER);
                if (SLOTS < LPS && m == SLOTS - 1)
                    for (int d = SLOTS; d < LPS; ++d) issue_one(s + NST, d);
            }
#pragma unroll
            for (int w = 0; w < WORDS; ++w)
                if (w * SLOTS / WORDS == m) widen_word(par ^ 1, rnext, w);
            if (m < NF) read_any(rload, m, tgt, tks, wide);
            if (SLOTS < NF && m == SLOTS - 1)
                for (int f = SLOTS; f < NF; ++f) read_any(rload, f, tgt, tks, wide);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    wait_stage<(NST - 1) * LPS>();          // stage 0 landed
    __syncthreads();
#pragma unroll
    for (int q = 0; q < LA; ++q)
#pragma unroll
        for (int f = 0; f < NF; ++f) read_any(q, f, lds, q, nk_int == 0);
#pragma unroll
    for (int w = 0; w < WORDS; ++w) widen_word(0, 0, w);

    int s = 0;
    for (; s + NST < nk_int - 1; ++s) {
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) substep(s, ks, true);
    }
    for (; s < nk_int; ++s) {
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) substep(s, ks, false);
    }
    // here: R[0 .. LA-1] hold raw sub-steps 0 .. LA-1 of stage nk_int (fp16 data)

    const int tw = t0 + wm * TM * 32, nw = n0 + wn * TN * 32;
    if constexpr (RAW) {
        wait_vm<0>();                      // drain the look-ahead DMA before the wave ends
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                int n = nw + j * 32 + l32;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    int t = tw + i * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                    if (t < a.T && n < a.N) {
                        int v = acc[i][j][r] >> SHIFT;
                        if constexpr (ASYM) v -= 8 * (a.code_sum[t] + a.w_code_sum[n]);
                        a.acc[(size_t)t * a.ldacc + n] = v;
                    }
                }
            }
        return;
    }
    // Dequantization.  The accumulator is 2^SHIFT times the integer dot product and 2^-SHIFT rides on the weight
    // scale.  The conversion to binary32 is exact with 4-bit activations (at most 24 significant bits); sums over
    // 8-bit ones can be longer and are rounded once (relative error 2^-24).
    v16f cf[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            const int lr = wm * TM * 32 + i * 32 + 8 * rq + 4 * g;
            const float4 sa4 = *reinterpret_cast<const float4*>(&lds_sa[lr]);
            const float4 sh4 = *reinterpret_cast<const float4*>(&lds_sh[lr]);
            const float sa_[4] = {sa4.x, sa4.y, sa4.z, sa4.w}, sh_[4] = {sh4.x, sh4.y, sh4.z, sh4.w};
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int r = rq * 4 + rr;
                    cf[i][j][r] = __builtin_fmaf((float)acc[i][j][r], sa_[rr] * c_sw[j],
                                                 __builtin_fmaf(sh_[rr], c_wr[j], c_bv[j]));
                }
        }

    for (; s < nk; ++s) {
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) {
            if (ks == BAR_KS) { stage_barrier(); issue_any(s + NST); }
            const int ts = (ks + LA < KSUB) ? s : s + 1, tks = (ks + LA) % KSUB;
            const uint8_t* tgt = lds + (ts % NST) * ST_BYTES;
            v8h fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = __builtin_bit_cast(v8h, R[ks % RD][i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = __builtin_bit_cast(v8h, R[ks % RD][TM + j]);
#pragma unroll
            for (int f = 0; f < NF; ++f) read_frag((ks + LA) % RD, f, tgt, tks);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    cf[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], cf[i][j], 0, 0, 0);
        }
    }

    wait_vm<0>();                          // drain the look-ahead DMA before the wave ends
    __half* __restrict__ y = static_cast<__half*>(a.y);
    // Output through LDS: a lane owns one column of sixteen rows of every 32 x 32 block, so direct
    // stores would be 2 bytes per lane.  Each wave instead parks its fp16 tile in its own slice of
    // the (now dead) stage ring and writes it out as 16-byte pieces, whole 64/128-byte row
    // segments per instruction.  Needs 16-byte aligned output rows; otherwise the direct path below.
    // bytes per parked row: padded against bank conflicts where the ring has the room
    constexpr int WROW = (NWAVES * TM * 32 * (TN * 64 + 16) <= NST * ST_BYTES) ? TN * 64 + 16 : TN * 64;
    constexpr int WBUF = TM * 32 * WROW;
    static_assert(NWAVES * WBUF <= NST * ST_BYTES, "stage ring too small to park the output tile");
    const bool vec_ok = !a.fp_only && ((reinterpret_cast<uintptr_t>(a.y) & 15u) == 0) && (a.ldy % 8 == 0);
    if (vec_ok) {
        __syncthreads();                   // every wave is past its last read of the stage ring
        uint8_t* wbuf = lds + wave_u * WBUF;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = i * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                    *reinterpret_cast<__half*>(wbuf + row * WROW + (j * 32 + l32) * 2) = __float2half(cf[i][j][r]);
                }
        constexpr int CH = TN * 4;                       // 16-byte pieces per row
        constexpr int RPS = 64 / CH;                     // rows per store instruction (lanes >= RPS * CH idle)
        const int prow = lane / CH, pch = lane % CH;
#pragma unroll
        for (int p = 0; p < (TM * 32 + RPS - 1) / RPS; ++p) {
            const int row = p * RPS + prow;
            if (prow >= RPS || row >= TM * 32) continue;
            const uint4 v = *reinterpret_cast<const uint4*>(wbuf + row * WROW + pch * 16);
            const int t = tw + row, n = nw + pch * 8;
            if (t < a.T) {
                __half* dst = y + (size_t)t * a.ldy + n;
                if (n + 8 <= a.N) {
                    store16_through(dst, v);
                } else {
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (n + e < a.N)
                            reinterpret_cast<uint16_t*>(dst)[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int n = nw + j * 32 + l32;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int t = tw + i * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (t < a.T && n < a.N) {
                    if (a.fp_only) reinterpret_cast<float*>(a.y)[(size_t)t * a.ldy + n] = cf[i][j][r];
                    else y[(size_t)t * a.ldy + n] = __float2half(cf[i][j][r]);
                }
            }
        }
}

template <int BITS, int WBITS, int BM, int BN, int WM, int WN, int BKB, int NST, int OCC, int GM, int MODE>
hipError_t launch_cfg(const GemmArgs& a, hipStream_t stream) {
    int tiles = ((a.T + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    hipLaunchKernelGGL((gemm_kernel<BITS, WBITS, BM, BN, WM, WN, BKB, NST, OCC, GM, MODE>), dim3(tiles),
                       dim3(WM * WN * 64), 0, stream, a);
    return hipGetLastError();
}

// The rules look at T, N, K_b and the widths alone, so the accumulator hook (every MODE) runs the tiles of the
// fused call.  One workgroup of eight waves per CU unless said otherwise: a launch takes ceil(tiles / cus) rounds.
inline long tiles_of(int T, int N, int bm, int bn) { return (long)((T + bm - 1) / bm) * ((N + bn - 1) / bn); }
inline long rounds_of(int T, int N, int bm, int bn, int cus) { return (tiles_of(T, N, bm, bn) + cus - 1) / cus; }

int basic_tile_4bit(int T, int N, int K_b, int cus) {
    if (T <= 128 || tiles_of(T, N, 256, 128) < cus) {
        // Fewer than one 256 x 128 tile per CU: the smallest tile that still goes through in one round, so that
        // all CUs have work.  64 x 64 runs two workgroups of four waves per CU.  us at 64 x 32 / 64 x 64 / 128 x 64 /
        // 128 x 128, weights from HBM (in brackets from the last-level cache); before, 128 x 64 served 65 to 128
        // tokens and 128 x 128 more:
        //   K=4096  N=4096  T=128:  9.5 / 10.8 / 14.0 / 17.4 (9.9 / 11.0 / 13.1 / 17.2);  T=192: 18.5 / 11.0 / 15.9 / 19.0
        //                   T=333: 26.8 / 13.7 / 15.7 / 18.8 (26.1 / 13.3 / 13.4 / 17.3);  T=512: ( - / 13.6 / 13.5 / 17.5)
        //   K=11008 N=4096  T=128: 15.7 / 20.7 / 38.2 / 42.5;  T=333: 41.3 / 27.7 / 37.6 / 42.4
        //   K=4096  N=11008 T=128: 29.0 / 16.9 / 18.8 / 21.7 (26.5 / 13.5 / 13.9 / 17.8)
        //   K=5120  N=15360 T=128: (37.9 / 16.2 / 17.6 / 21.1)
        // The four K groups of 64 x 32 cost two barriers and a pass through LDS at the end: at K = 1024 it takes
        // 7.2 where 64 x 64 takes 6.5, at K = 2048 7.8 against 8.0.  Beyond two 64 x 64 tiles per CU, 128 x 64 has
        // the edge over 128 x 128 only while weights are cached (T=66 K=4240 N=28296: 19.9 : 21.3, from HBM 28.9 : 27.9;
        // T=128 K=8192 N=28672 from HBM 43.1 : 40.0).
        if (tiles_of(T, N, 64, 32) <= cus && K_b >= 1792) return kTile64x32;
        if (T <= 64 || tiles_of(T, N, 64, 64) <= 2L * cus) return kTile64x64Pair32;
        return T <= 128 ? kTile128x64Pair32 : kTile128x128Pair32;
    }
    // Tiles of 1.5x the area (64 x 96 or 96 x 64 per wave: 17 % fewer LDS fragment reads and widening
    // operations per MFMA, a third fewer per-tile prologues and epilogues) take 1.42x as long per round
    // (measured); they win whenever they save enough rounds.
    const double cost_a = (double)rounds_of(T, N, 256, 128, cus);
    const double cost_b = 1.42 * (double)rounds_of(T, N, 256, 192, cus);
    const double cost_c = 1.42 * (double)rounds_of(T, N, 192, 256, cus);
    if (cost_b < cost_a && cost_b <= cost_c) return kTile256x192;
    if (cost_c < cost_a) return kTile192x256;
    // 256 x 128 runs on the 16 x 16 matrix instructions, under which the chip keeps its clock: 2 - 6 % faster.
    // The larger tiles do not fit the register file in that form.
    return kTile256x128;
}

// 8-bit activations: the tile whose launch is estimated to be the shortest.  One workgroup of eight waves per CU:
// rounds * (fixed + per_stage * stages), a stage being 128 k.  Workgroups of four waves go two to a CU
// (pair_fixed > 0): up to one per CU they take the same line; when some CUs hold two, pair_fixed + (pair_per_stage +
// pair_more * share of CUs that do) * stages, the launch lasting as long as such a CU but slowed by how many there
// are; every further two per CU that again, and a remainder `rest` of what it would take by itself, as the CUs have
// drifted apart by then.  (pair_more of a tile of eight waves: see kCost4; 0 here.)
// Measured lines behind it (us; integer stages; both from HBM unless said otherwise, N = 4096 .. 28672):
//   integer stages              4      6     14     30     84
//   W8A8  64 x 32             5.5    5.8    7.0   10.2   18.5 - 22.8
//         64 x 64             6.1    5.9    8.0   13.4   26 - 30
//         two of 64 x 64      4.8    4.1    6.5   11.3      -         (per 256 tiles)
//         128 x 64            8.9    8.9   11.4   18.6   32.2
//         128 x 128          10.1   10.0   15.1   26.5   44 - 57
//         256 x 128          15     14.5   21.3   34.2   88          256 x 192 (gemm_kernel): 50.8 at 30
//   W4A8  64 x 32             5.9    6.3    8.0   10.7   17.5 - 20.7
//         64 x 64             6.7    6.5    8.9   12.8   22 - 27
//         two of 64 x 64      5.2    4.9    7.1   11.0      -
//         128 x 64            9.5    9.0   12.0   17.7   33 - 37
//         128 x 128          13.8   12.3   17.2   26.6   54
//         256 x 128          15.8   15.6   22.0   36     79
//   128 x 128 in pairs (gemm_kernel; weights cached / from HBM), tiles on 256 CUs:
//   W8A8  256        10.0/11.7   10.7/13.2   14.3/19.6   27.7/32.9
//         272        12.6/13.2   13.9/14.8   20.4/21.4   30.0/35.0       (256 x 128: 13.7/14.2, 15.2/16.0, 20.9/22.1, 32.1/36.6)
//         500        13.9/15.7   16.1/18.4   24.0/28.6   39.8/49.2       (256 x 128: 14.7/15.8, 16.2/17.7, 23.4/25.0, 36.1/40.7)
//   W4A8  256        11.4/12.2   12.4/13.5   16.5/18.7   27.6/29.8
//         272        14.0/14.2   15.6/15.5   20.7/21.5   33.9/32.6       (256 x 128: 14.7/14.8, 16.4/16.5, 22.5/22.9, 36.4/36.6)
//         500        15.0/16.3   17.1/18.9   24.7/27.1   41.0/43.1       (256 x 128: 16.0/15.7, 17.3/17.7, 24.2/24.9, 39.4/40.1)
// The figures of the table are fitted, with cached weights and from HBM alike, to what loses least against the best
// tile over 900 shapes with every tile measured (T 33 .. 4096, K 512 .. 11008, N 512 .. 28672): they rank the tiles of
// a shape rather than predict its time.  Against the fastest tile the choice costs 0.9 % (W8A8) and 0.4 % (W4A8) in the
// mean.  With lines through the times from HBM alone and without the workgroups of four waves on 32 x 32 instructions,
// shapes like these took (cached / from HBM): W4A8 T=384 K=1024 N=24000 31.4/32.0 (now 26.4/30.4), T=120 K=1008 N=16448
// 13.5/14.2 (10.1/13.2), T=512 K=4096 N=8704 36.4/36.7 (34.8/33.0), T=508 K=592 N=5260 14.0/14.5 (11.1/11.6); W8A8
// T=947 K=1520 N=4232 18.8/21.6 (18.3/19.8), T=333 K=960 N=11008 13.9/14.6 (12.6/13.7).  Where the two states disagree
// the fit takes the middle: W8A8 T=200 K=960 N=21100 18.2/20.6 (17.6/22.0).
struct TileCost { int tile, bm, bn; double fixed, per_stage, pair_fixed, pair_per_stage, pair_more, rest; };
constexpr TileCost kCost8[] = {{kTile64x32, 64, 32, 5.44, 0.126, 0, 0, 0, 0},
                               {kTile64x64, 64, 64, 5.79, 0.218, 0, 0, 0, 0},
                               {kTile64x64Pair, 64, 64, 3.87, 0.311, 4.51, 0.605, 0, 0.71},
                               {kTile64x64Pair32, 64, 64, 2.61, 0.493, 3.54, 0.631, 0.117, 0.79},
                               {kTile128x64, 128, 64, 6.71, 0.281, 0, 0, 0, 0},
                               {kTile128x128Pair32, 128, 128, 7.17, 0.778, 6.51, 0.913, 0.405, 0.93},
                               {kTile128x128, 128, 128, 6.95, 0.415, 0, 0, 0, 0},
                               {kTile256x128, 256, 128, 9.89, 0.65, 0, 0, 0, 0},
                               {kTile256x192, 256, 192, 11.0, 0.897, 0, 0, 0, 0},
                               {kTile192x256, 192, 256, 11.0, 0.897, 0, 0, 0, 0}};
constexpr TileCost kCost8w4[] = {{kTile64x32, 64, 32, 6.12, 0.118, 0, 0, 0, 0},
                                 {kTile64x64, 64, 64, 6.6, 0.203, 0, 0, 0, 0},
                                 {kTile64x64Pair, 64, 64, 4.07, 0.406, 5.17, 0.485, 0, 0.88},
                                 {kTile128x64Pair32, 128, 64, 6.12, 0.569, 5.67, 0.692, 0.106, 0.99},
                                 {kTile128x64, 128, 64, 8.11, 0.288, 0, 0, 0, 0},
                                 {kTile128x128Pair32, 128, 128, 7.5, 0.736, 9.6, 0.649, 0.322, 0.743},
                                 {kTile128x128, 128, 128, 10.52, 0.487, 0, 0, 0, 0},
                                 {kTile256x128, 256, 128, 10.33, 0.82, 0, 0, 0, 0}};

double launch_cost(const TileCost& t, long tiles, int cus, int stages) {
    const double alone = t.fixed + t.per_stage * stages;
    if (t.pair_fixed == 0) return (double)((tiles + cus - 1) / cus) * alone + t.pair_more * stages * (double)tiles / cus;
    auto up_to_two = [&](long n) {
        return n <= cus ? alone : t.pair_fixed + (t.pair_per_stage + t.pair_more * (double)(n - cus) / cus) * stages;
    };
    if (tiles <= 2L * cus) return up_to_two(tiles);
    const long full = tiles / (2L * cus), left = tiles % (2L * cus);
    return (double)full * up_to_two(2L * cus) + (left ? t.rest * up_to_two(left) : 0.0);
}

// 4-bit operands beyond the smallest tiles: the same estimate, a stage being 256 k, fitted to 469 shapes with every tile
// measured (T 33 .. 4096, K 1808 .. 11008, N 512 .. 28672, cached weights and from HBM, mean of both).  A round of one
// workgroup per CU takes pair_more * stages longer when it is full than when it is empty: with rounds of one length 256 x
// 128 tiles were preferred to 128 x 128 for one nearly full round (T=905 K=8320 N=7384, 232 : 464 tiles, 58.0 : 54.8 us;
// T=1204 K=7712 N=6136 57.4 : 53.9).  It predicts a tile's time to 6 - 9 %, so the tile of basic_tile_4bit is left only
// for one that is estimated 7 % shorter; over those shapes that makes the launch 8 % shorter in the mean, on two of them
// 4 - 5 % longer.  GEMM, us, before : now, cached and from HBM alike:
//   T=333 K=4096 N=11008, 258 tiles of 128 x 128 on 256 CUs, now 460 of 96 x 96, two per CU          28.8 : 23.4
//   T=92 K=7552 N=18626 (128 x 64) 35.8 : 28.4;  T=143 K=9984 N=20644 56.0 : 43.2;  T=1360 K=7040 N=1628 29.8 : 25.0
//   T=512 K=4096 N=11008, 344 tiles, now 232 of 128 x 192                                              29.4 : 26.7
//   T=2325 K=5344 N=2444 39.2 : 33.4;  T=1365 K=8368 N=5514, 174 tiles of 256 x 192, now 484 of 128 x 128  73.9 : 59.5
constexpr TileCost kCost4[] = {{kTile128x64Pair32, 128, 64, 0.975, 0.777, 6.956, 0.769, 0.195, 0.891},
                               {kTile128x128Pair32, 128, 128, 8.110, 0.753, 10.168, 1.169, 0.318, 0.829},
                               {kTile96x96Pair, 96, 96, 7.771, 0.604, 8.613, 0.979, -0.039, 0.823},
                               {kTile96x128Pair, 96, 128, 8.225, 0.725, 9.431, 1.103, 0.128, 0.765},
                               {kTile128x192, 128, 192, 8.920, 0.926, 0, 0, 0.244, 0},
                               {kTile256x128, 256, 128, 9.991, 1.101, 0, 0, 0.328, 0},
                               {kTile256x192, 256, 192, 12.301, 1.329, 0, 0, 0.702, 0},
                               {kTile192x256, 192, 256, 12.180, 1.343, 0, 0, 0.657, 0}};
constexpr int kModelK4 = 1792;        // below, the fixed parts decide and the measurements behind basic_tile_4bit hold
constexpr double kModelGain4 = 0.93;

// estimate of a 4-bit tile; 0 where the table has no line for it
double tile_estimate_4bit(int tile, int T, int N, int K_b, int cus) {
    for (const TileCost& c : kCost4)
        if (c.tile == tile) return launch_cost(c, tiles_of(T, N, c.bm, c.bn), cus, (K_b + 255) / 256);
    return 0.0;
}

int choose_tile_4bit(int T, int N, int K_b, int cus) {
    const int basic = basic_tile_4bit(T, N, K_b, cus);
    if (K_b < kModelK4 || basic == kTile64x32 || basic == kTile64x64Pair32) return basic;
    int best = basic;
    double least = kModelGain4 * tile_estimate_4bit(basic, T, N, K_b, cus);
    for (const TileCost& c : kCost4) {
        const double e = tile_estimate_4bit(c.tile, T, N, K_b, cus);
        if (e < least) { best = c.tile; least = e; }
    }
    return best;
}

int choose_tile_8bit(int T, int N, int K_b, bool mixed, int cus) {
    const int stages = (K_b + 127) / 128;
    const TileCost* list = mixed ? kCost8w4 : kCost8;
    const int count = mixed ? (int)(sizeof(kCost8w4) / sizeof(TileCost)) : (int)(sizeof(kCost8) / sizeof(TileCost));
    int best = 0;
    double least = 0.0;
    for (int i = 0; i < count; ++i) {
        const double c = launch_cost(list[i], tiles_of(T, N, list[i].bm, list[i].bn), cus, stages);
        if (i == 0 || c < least) { best = i; least = c; }
    }
    return list[best].tile;
}

int choose_tile(int T, int N, int K_b, int bits, bool mixed, int cus) {
    return bits == 4 ? choose_tile_4bit(T, N, K_b, cus) : choose_tile_8bit(T, N, K_b, mixed, cus);
}

template <int BITS, int WBITS, int MODE>
hipError_t launch_tile(const GemmArgs& a, int tile, hipStream_t stream) {
    switch (tile) {
    case kTile64x64Pair32:
        if constexpr (BITS == WBITS) return launch_cfg<BITS, WBITS, 64, 64, 2, 2, 128, 4, 2, 0, MODE>(a, stream);
        else break;
    case kTile128x64Pair32:
        if constexpr (WBITS == 4) return launch_cfg<BITS, WBITS, 128, 64, 2, 2, 128, 2, 2, 0, MODE>(a, stream);
        else break;
    case kTile128x128Pair32: return launch_cfg<BITS, WBITS, 128, 128, 2, 2, 128, 2, 2, 8, MODE>(a, stream);
    case kTile256x192:
        if constexpr (BITS == WBITS) return launch_cfg<BITS, WBITS, 256, 192, 4, 2, 128, 2, 1, 4, MODE>(a, stream);
        else break;
    case kTile192x256:
        if constexpr (BITS == WBITS) return launch_cfg<BITS, WBITS, 192, 256, 2, 4, 128, 2, 1, 4, MODE>(a, stream);
        else break;
    default: return launch_gemm_tiles16(a, tile, stream);
    }
    return hipErrorInvalidValue;
}

// one wave per output channel; lanes stride over the packed row
template <int BITS>
__global__ __launch_bounds__(kThreads) void weight_reduce_kernel(WeightReduceArgs a) {
    const int lane = threadIdx.x & 63;
    const int n = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (n >= a.N) return;
    const uint8_t* row = static_cast<const uint8_t*>(a.w_q) + (size_t)n * a.ldw;
    const int row_bytes = a.K_b * BITS / 8;
    int s = 0, s_odd = 0;                  // all codes; codes at odd positions (high nibbles)
    for (int p = lane; p < row_bytes; p += 64) {
        int b = row[p];
        if constexpr (BITS == 4) {
            int hi = ((b >> 4) ^ 8) - 8;
            s += ((b & 0xF) ^ 8) - 8 + hi;
            s_odd += hi;
        } else {
            s += (int)(int8_t)b;
        }
    }
    if constexpr (BITS == 4) {
        // The GEMM reads a row up to the end of the 16-byte piece that holds its last packed byte.  Against
        // the zero bytes the activations have there, the single-AND widening turns whatever the weight
        // matrix holds in those pad bytes into 128 x (their high nibbles); counting them in the side data
        // makes the epilogue's correction remove exactly that, so pad bytes may hold anything.
        const int padded = min((row_bytes + 15) & ~15, a.ldw);
        for (int p = row_bytes + lane; p < padded; p += 64) s_odd += (((int)row[p] >> 4) ^ 8) - 8;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        s_odd += __shfl_xor(s_odd, o, 64);
    }
    if (lane == 0) {
        a.w_reduced[n] = __half2float(static_cast<const __half*>(a.w_scale)[n]) * (float)s;
        if (a.w_code_sum) a.w_code_sum[n] = s_odd;
    }
}

}  // namespace

// compute units of the current device (looked up once per device)
int compute_units() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        cached[dev] = n;
    }
    return cached[dev];
}

// Estimated time of the per-tile kernels' launch for a 4-bit [T, N] output on `cus` compute units, in the
// unit of plan_gemm_stream's estimate (one 32-channel block of a 256-row tile through the K loop): the
// rounds and relative round times of choose_tile_4bit.  (It knows the 256-row tiles only; the persistent kernel, whose
// own tiles have 256 rows, is not compared with the smaller ones.)
static double tiles_estimate(int T, int N, int cus) {
    auto rounds = [&](int bm, int bn) { return (double)((((long)(T + bm - 1) / bm) * ((N + bn - 1) / bn) + cus - 1) / cus); };
    const double a = 4.0 * rounds(256, 128), b = 4.0 * 1.42 * rounds(256, 192), c = 4.0 * 1.42 * rounds(192, 256);
    return a < b ? (a < c ? a : c) : (b < c ? b : c);
}

static int g_gemm_path = 0;     // 0: automatic; 1: the persistent kernel wherever it can run; 2: never
void set_gemm_path(int mode) { g_gemm_path = mode; }

// 0: the persistent kernel cannot run this shape; 1: it can and is the automatic choice; 2: it can, but
// the per-tile kernels are estimated to be at least as fast.  Measured on the LLaMA shapes, in the unit of
// tiles_estimate: a block of the persistent kernel costs 0.91 - 0.95 where its tiles are five or six blocks
// wide (its K loop runs on the 16 x 16 x 64 matrix instruction, under which the chip keeps its clock; whole
// rounds of fixed 256 x 192 tiles cost 0.947 per block, so it also wins 4 % where those balance perfectly),
// and 1.04 where the tiles are four blocks wide (a wave then holds two column blocks: more fragment reads
// and widening per MFMA than the per-tile 256 x 128 form) or K is shallow (its longer per-tile epilogue).
// From kModelK4 base columns on a fitted estimate of its launch (the persistent kernel forced onto 60 of the shapes behind
// kCost4; per tile of the busiest CU, and per block and stage of 256 k; good to 6 %) also gives it what it is estimated
// 7 % ahead on: T=2445 K=2160 N=10388 (256 x 128) 84 : 73, T=1945 K=3424 N=19666 145 : 125.
int choose_gemm_stream(int T, int N, int K_b, int cus, StreamPlan* plan) {
    if (!plan_gemm_stream(T, N, K_b, cus, plan)) return 0;
    const long tiles = (long)plan->tiles_m * plan->tn;
    const long r = (tiles + cus - 1) / cus;
    const double blocks = (double)(r * plan->base + (r * plan->rem + plan->tn - 1) / plan->tn);
    const bool rule = T > kRowsTokens && K_b >= 2048 && plan->base >= 5 && 0.94 * blocks <= tiles_estimate(T, N, cus);
    if (rule || T <= kRowsTokens || K_b < kModelK4) return rule ? 1 : 2;
    const double there = tile_estimate_4bit(choose_tile_4bit(T, N, K_b, cus), T, N, K_b, cus);
    const double here = 4.983 + 8.323 * (double)r + blocks * (0.33 * ((K_b + 255) / 256) + 0.099);
    return (here < kModelGain4 * there) ? 1 : 2;      // (`there` is 0 where the smallest tiles run)
}

// Few tokens go to gemm_rows_kernel, except 17 to 32 tokens of W4A8 layers with more than one pair of 16-channel blocks
// per CU: two activation lines per weight line and 32 rows of them fill the rings so far that a CU holds one
// workgroup, and its rounds do not overlap.  us, weights cached / from HBM, this kernel against 64 x 64 tiles, T = 32:
// N = 8192, K = 1280 5.2/5.2 : 8.3/8.3;  N = 14464, K = 768 8.5/9.1 : 7.2/7.6, K = 4352 14.6/15.1 : 13.2/13.9;
// N = 27520, K = 768 15.2/16.8 : 8.8/9.6, K = 4352 27.2/27.9 : 19.3/23.2.
static bool rows_take(int T, int N, int bits, int w_bits, int cus) {
    if (T <= 16) return true;
    return T <= kRowsTokens && !(bits == 8 && w_bits == 4 && N > 32L * (cus < 1 ? 256 : cus));
}

hipError_t launch_gemm(const GemmArgs& a, hipStream_t stream) {
    const int cus = compute_units(), path = g_gemm_path;
    if (a.bits == 4 && !a.fp_only && (path == 1 || (path == 0 && a.T > kRowsTokens))) {
        StreamPlan plan;
        const int c = choose_gemm_stream(a.T, a.N, a.K_b, cus, &plan);
        if (c == 1 || (c == 2 && path == 1)) return launch_gemm_stream(a, plan, stream);
    }
    if (rows_take(a.T, a.N, a.bits, a.w_bits, cus)) return launch_gemm_rows(a, cus, stream);
    return launch_gemm_tiles(a, cus, stream);
}

// one workgroup per output tile (every shape the persistent kernel does not take)
hipError_t launch_gemm_tiles(const GemmArgs& a, int cus, hipStream_t stream) {
    const bool raw = a.y == nullptr;
    if (cus < 1) cus = 256;              // the count could not be read: any value gives a working choice
    const bool mixed = a.bits == 8 && a.w_bits == 4;
    const int tile = choose_tile(a.T, a.N, a.K_b, a.bits, mixed, cus);
    if (mixed) return raw ? launch_tile<8, 4, 1>(a, tile, stream) : launch_tile<8, 4, 0>(a, tile, stream);
    if (a.bits == 8) return raw ? launch_tile<8, 8, 1>(a, tile, stream) : launch_tile<8, 8, 0>(a, tile, stream);
    if (!raw) return launch_tile<4, 4, 0>(a, tile, stream);
    return (a.code_sum && a.w_code_sum) ? launch_tile<4, 4, 2>(a, tile, stream) : launch_tile<4, 4, 1>(a, tile, stream);
}

GemmForm choose_gemm_form(int T, int N, int K_b, int bits, int w_bits, int cus) {
    const bool mixed = bits == 8 && w_bits == 4;
    StreamPlan plan;
    if (bits == 4 && T > kRowsTokens && choose_gemm_stream(T, N, K_b, cus, &plan) == 1)
        return GemmForm{4, kStreamRows, plan.base * 32, 8, 1};
    if (rows_take(T, N, bits, w_bits, cus)) return choose_rows_form(T, N, K_b, bits, w_bits, cus);
    switch (choose_tile(T, N, K_b, bits, mixed, cus)) {
    case kTile64x32: return GemmForm{3, 64, 32, 8, 4};
    case kTile64x64: return GemmForm{3, 64, 64, 8, 2};
    case kTile64x64Pair: return GemmForm{3, 64, 64, 4, 1};
    case kTile128x64: return GemmForm{3, 128, 64, 8, 2};
    case kTile128x128: return GemmForm{3, 128, 128, 8, mixed ? 2 : 1};
    case kTile256x128: return GemmForm{3, 256, 128, 8, 1};
    case kTile96x96Pair: return GemmForm{3, 96, 96, 4, 1};
    case kTile96x128Pair: return GemmForm{3, 96, 128, 4, 1};
    case kTile128x192: return GemmForm{3, 128, 192, 8, 1};
    case kTile64x64Pair32: return GemmForm{2, 64, 64, 4, 1};
    case kTile128x64Pair32: return GemmForm{2, 128, 64, 4, 1};
    case kTile128x128Pair32: return GemmForm{2, 128, 128, 4, 1};
    case kTile256x192: return GemmForm{2, 256, 192, 8, 1};
    default: return GemmForm{2, 192, 256, 8, 1};
    }
}

hipError_t launch_weight_reduce(const WeightReduceArgs& a, hipStream_t stream) {
    int blocks = (a.N + 3) / 4;
    if (a.bits == 4)
        hipLaunchKernelGGL(weight_reduce_kernel<4>, dim3(blocks), dim3(kThreads), 0, stream, a);
    else
        hipLaunchKernelGGL(weight_reduce_kernel<8>, dim3(blocks), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

}  // namespace quik
