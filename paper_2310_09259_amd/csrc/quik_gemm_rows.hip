// Integer GEMM + dequantization epilogue + fp16 outlier GEMM for few tokens (T <= 32), gfx950
// (Algorithm 1 of arXiv 2310.09259: "INTmatmul", "Dequantization", "FPmatmul" and the final add).
//
// What bounds it: the weights are read once and hardly anything is computed on them, so the time is that of
// streaming N * (K_b * wbits / 8 + 2 * n_out) bytes from HBM plus the fixed latencies around it.
//  - A workgroup owns CB blocks of 16 output channels and its waves split K: a row's 128-byte lines -- the packed
//    integer part, then the fp16 outlier part -- are dealt to the waves in contiguous ranges, so that every wave
//    streams the same number of bytes and the outlier weights ride in the same pipeline.  No barrier until the
//    waves add up their partial sums (INT32 exactly, the fp32 partials in wave order) through LDS.
//  - A wave copies its lines global -> LDS (16 bytes per lane, eight whole lines per instruction) into a private
//    ring of NST stages, the weights mostly with the non-temporal hint (see `once` below): they are read once, and
//    without it their lines evict the activations and wait for the evictions.  A copy-only loop over 47 MB of such rows in HBM takes 8.3 us
//    with the hint (5.7 TB/s, launch included), 9.9 us without, 9.3 us into registers instead of LDS, and 10.8 us
//    into registers in the matrix instruction's lane order (lane = row: four lines per quad of lanes).
//  - The activations of the same k (at most 32 rows, resident in every L2) come through the same ring.
// The 16-byte pieces of a row go from LDS into v_mfma_i32_16x16x64_i8 as they are: a dot product does not care
// about the order of k as long as both operands agree, so the 32 nibbles (or 16 bytes) of a piece are whatever k
// they are.  Operand widenings, accumulator corrections and epilogue arithmetic are those of quik_gemm.hip (see
// its header); the accumulator layout is the 16 x 16 form's: channel l of token rows 4g .. 4g + 3 in lane
// (l = lane % 16, g = lane / 16).
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "quik_kernels.h"
#include "quik_gemm_device.h"

namespace quik {

namespace {

using namespace gemm_dev;

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kLine = 128;                               // bytes of a row per stage
// More threads than any launch has: the bound makes the compiler keep to 128 registers (four waves per SIMD), which
// a bound on the waves alone does not where LDS allows fewer.
constexpr int kBoundThreads = 1024;

// XB / WB: activation / weight bits (4 + 4, 8 + 8, or 8 + 4).  TB: 16-token blocks.  CB: 16-channel blocks per
// workgroup.  NW: waves.  NST: stages of a wave's ring.  MODE as in quik_gemm.hip: 0 fused epilogue, 1 raw INT32 accumulators
// with the symmetric widening, 2 raw accumulators with the single-AND widening and its correction.  ONCE: weights
// are copied with the hint that their lines are read once.
template <int XB, int WB, int TB, int CB, int NW, int NST, int MODE, bool ONCE>
__global__ __launch_bounds__(kBoundThreads) void gemm_rows_kernel(GemmArgs a) {
    constexpr bool RAW = MODE != 0;
    constexpr bool ASYM = XB == 4 && MODE != 1;
    constexpr bool MIXED = XB == 8 && WB == 4;
    static_assert(XB == WB || MIXED, "weights: same width as the activations, or 4 under 8");
    constexpr int SHIFT = (XB == 4) ? (ASYM ? 4 : 8) : (MIXED ? 4 : 0);
    constexpr int AX = MIXED ? 2 : 1;                    // activation lines per weight line
    constexpr int OPS = (WB == 4) ? 2 : 1;               // matrix instructions per 16-byte weight piece
    constexpr int B_BYTES = CB * 16 * kLine, A_BYTES = TB * 16 * kLine * AX, ST_BYTES = B_BYTES + A_BYTES;
    constexpr int LPS = ST_BYTES / 1024;                 // copy instructions per stage
    static_assert((NST - 1) * LPS < 64, "vmcnt range");
    // the whole share of the register file (four waves per SIMD), so that its top is never a live register (see
    // quik_gemm.hip)
    asm volatile("" ::: "v127");

    // rings; then the partial sums.  Static: dynamic LDS beyond 64 KB needs a host call per launch
    constexpr int RING = NW * NST * ST_BYTES, RED = NW * TB * CB * 1024 * (RAW ? 1 : 2);
    __shared__ __align__(1024) uint8_t lds[RING > RED ? RING : RED];
    __shared__ float prm_sa[TB * 16], prm_sh[TB * 16];
    __shared__ int prm_ct[TB * 16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int n0 = xcd_contiguous_id(blockIdx.x, gridDim.x) * (CB * 16);

    const int wlim = (a.K_b * WB / 8 + 15) & ~15;        // up to the 16-byte piece that holds the last packed byte
    const int xlim = (a.K_b * XB / 8 + 15) & ~15;
    const int fplim = RAW ? 0 : a.n_out * 2;
    const int nint = a.fp_only ? 0 : (wlim + kLine - 1) / kLine;
    const int lines = nint + (fplim + kLine - 1) / kLine;
    const int first = (int)((long)lines * wave / NW), last = (int)((long)lines * (wave + 1) / NW);

    const v4i rA = make_rsrc(a.xq, (size_t)a.T * a.ldq);
    const v4i rB = make_rsrc((const uint8_t*)a.w_q + (size_t)n0 * a.ldw, (size_t)(a.N - n0) * a.ldw);
    const v4i rAf = make_rsrc(a.n_out ? a.x_out : a.xq, a.n_out ? (size_t)a.T * a.ldo * 2 : 0);
    const v4i rBf = make_rsrc(a.n_out ? (const uint8_t*)a.w_out + (size_t)n0 * a.ldwo * 2 : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.N - n0) * a.ldwo * 2 : 0);

    // ---- the epilogue's parameters are requested before the stream starts and used after it
    float p_sc = 0.0f, p_z = 0.0f, c_sw = 0.0f, c_wr = 0.0f, c_bv = 0.0f;
    int p_c = 0, c_nc = 0;
    const int fin_c = wave % CB, fin_t = wave / CB;      // the block this wave finishes (waves below TB * CB)
    const int n = min(n0 + fin_c * 16 + l16, a.N - 1);
    if constexpr (!RAW) {
        if (tid < TB * 16) {
            const int t = min(tid, a.T - 1);
            p_sc = a.scale[t];
            p_z = a.zero[t];
            if constexpr (ASYM) p_c = a.fp_only ? 0 : a.code_sum[t];
        }
        if (wave < TB * CB && !a.fp_only) {
            c_sw = __half2float(static_cast<const __half*>(a.w_scale)[n]);
            c_wr = a.w_reduced[n];
            if (a.bias) c_bv = __half2float(static_cast<const __half*>(a.bias)[n]);
            if constexpr (ASYM) c_nc = a.w_code_sum[n];
        }
    }

    uint8_t* const ring = lds + wave * (NST * ST_BYTES);
    const uint32_t ring_addr = lds_addr(ring);
    const int lrow = lane >> 3;
    // line `s` of this wave's range, or past its end (all lanes out of range): eight rows per instruction, the
    // 16-byte pieces of a row exchanged so that sixteen rows' pieces of one k fall into distinct LDS banks
    auto issue = [&](int s, int slot) {
        const uint32_t dst = ring_addr + (uint32_t)slot * ST_BYTES;
        const bool fp = s >= nint;
        const int k = (fp ? s - nint : s) * kLine;
        const int blim = s < last ? (fp ? fplim : wlim) : 0, alim = s < last ? (fp ? fplim : xlim) : 0;
        const int ldb = fp ? a.ldwo * 2 : a.ldw, lda = fp ? a.ldo * 2 : a.ldq;
        const v4i rb = fp ? rBf : rB, ra = fp ? rAf : rA;
#pragma unroll
        for (int i = 0; i < CB * 2; ++i) {
            const int row = i * 8 + lrow, c = k + (((lane & 7) ^ swz<kLine>(row)) << 4);
            const uint32_t vo = c < blim ? (uint32_t)(row * ldb + c) : kOob;
            if constexpr (ONCE) dma16_once(rb, dst + i * 1024, vo);
            else dma16(rb, dst + i * 1024, vo, 0);
        }
#pragma unroll
        for (int p = 0; p < AX; ++p)
#pragma unroll
            for (int i = 0; i < TB * 2; ++i) {
                const int row = i * 8 + lrow, c = (fp ? k : k * AX + p * kLine) + (((lane & 7) ^ swz<kLine>(row)) << 4);
                const int lim = (fp && p > 0) ? 0 : alim;
                dma16(ra, dst + B_BYTES + (p * TB * 2 + i) * 1024, c < lim ? (uint32_t)(row * lda + c) : kOob, 0);
            }
    };
    // 16-byte piece `piece` of row l of 16-row block `blk` in a panel of stage lines
    auto frag = [&](const uint8_t* panel, int blk, int piece) {
        return *reinterpret_cast<const uint4*>(panel + (blk * 16 + l16) * kLine + ((piece ^ swz<kLine>(l16)) << 4));
    };

    v4i acc[TB][CB];
    v4f cf[TB][CB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int c = 0; c < CB; ++c) { acc[t][c] = v4i{0, 0, 0, 0}; cf[t][c] = v4f{0.0f, 0.0f, 0.0f, 0.0f}; }

    constexpr uint32_t M = 0xF0F0F0F0u;
    auto hi = [](uint32_t x) { return (int)(x & M); };                           // 16 * signed high nibble
    auto lo = [](uint32_t x) {                                                   // low nibble + 8, or 16 * signed low nibble
        return ASYM ? (int)((x ^ 0x08080808u) & 0x0F0F0F0Fu) : (int)((x << 4) & M);
    };
    auto int_line = [&](const uint8_t* st) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            v4i ub[CB][OPS], ua[TB][OPS];
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const uint4 w = frag(st, c, kk * 4 + g);
                if constexpr (WB == 4) {                 // weights: even k in the low nibble
                    ub[c][0] = v4i{lo(w.x), hi(w.x), lo(w.y), hi(w.y)};
                    ub[c][OPS - 1] = v4i{lo(w.z), hi(w.z), lo(w.w), hi(w.w)};
                } else {
                    ub[c][0] = __builtin_bit_cast(v4i, w);
                }
            }
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                if constexpr (MIXED) {                   // bytes into the weights' order: even k, then odd k of every 8
#pragma unroll
                    for (int p = 0; p < OPS; ++p) {
                        const uint4 v = frag(st + B_BYTES + kk * (TB * 16 * kLine), t, 2 * g + p);
                        ua[t][p] = v4i{(int)__builtin_amdgcn_perm(v.y, v.x, 0x06040200u), (int)__builtin_amdgcn_perm(v.y, v.x, 0x07050301u),
                                       (int)__builtin_amdgcn_perm(v.w, v.z, 0x06040200u), (int)__builtin_amdgcn_perm(v.w, v.z, 0x07050301u)};
                    }
                } else {
                    const uint4 x = frag(st + B_BYTES, t, kk * 4 + g);
                    if constexpr (XB == 4) {             // activations: even k in the high nibble
                        ua[t][0] = v4i{hi(x.x), lo(x.x), hi(x.y), lo(x.y)};
                        ua[t][OPS - 1] = v4i{hi(x.z), lo(x.z), hi(x.w), lo(x.w)};
                    } else {
                        ua[t][0] = __builtin_bit_cast(v4i, x);
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < OPS; ++o)
#pragma unroll
                for (int t = 0; t < TB; ++t)
#pragma unroll
                    for (int c = 0; c < CB; ++c) acc[t][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ua[t][o], ub[c][o], acc[t][c], 0, 0, 0);
        }
    };
    auto fp_line = [&](const uint8_t* st) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            v8h fa[TB];
#pragma unroll
            for (int t = 0; t < TB; ++t) fa[t] = __builtin_bit_cast(v8h, frag(st + B_BYTES, t, kk * 4 + g));
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const v8h fb = __builtin_bit_cast(v8h, frag(st, c, kk * 4 + g));
#pragma unroll
                for (int t = 0; t < TB; ++t) cf[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[t], fb, cf[t][c], 0, 0, 0);
            }
        }
    };

#pragma unroll
    for (int i = 0; i < NST - 1; ++i) issue(first + i, i);
    int slot = 0, fill = NST - 1;                        // stage being read / stage being filled
    auto next_stage = [&](int s) {
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): the reads of the stage about to be refilled are done
        issue(s + NST - 1, fill);
        wait_vm<(NST - 1) * LPS>();                      // line s has landed (this wave's own copies)
        const uint8_t* st = ring + slot * ST_BYTES;
        slot = slot + 1 == NST ? 0 : slot + 1;
        fill = fill + 1 == NST ? 0 : fill + 1;
        return st;
    };
    int s = first;
    for (; s < min(last, nint); ++s) int_line(next_stage(s));
    for (; s < last; ++s) fp_line(next_stage(s));
    wait_vm<0>();

    // ---- add the waves' partial sums; wave w < TB * CB finishes one 16 x 16 block
    if constexpr (!RAW) {
        if (tid < TB * 16) {
            prm_sa[tid] = p_sc;                                                  // scaleAct
            prm_sh[tid] = p_z + (float)(1 << (XB - 1)) * p_sc;                   // zeroAct + halfRange * scaleAct
            prm_ct[tid] = -128 * p_c;                                            // in raw accumulator units
        }
    }
    __syncthreads();                                     // every ring is dead
    int4* red = reinterpret_cast<int4*>(lds);
    float4* redf = reinterpret_cast<float4*>(lds) + NW * TB * CB * 64;
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const int e = (wave * TB * CB + t * CB + c) * 64 + lane;
            red[e] = make_int4(acc[t][c][0], acc[t][c][1], acc[t][c][2], acc[t][c][3]);
            if constexpr (!RAW) redf[e] = make_float4(cf[t][c][0], cf[t][c][1], cf[t][c][2], cf[t][c][3]);
        }
    __syncthreads();
    if (wave >= TB * CB) return;
    int sum[4] = {0, 0, 0, 0};
    float sumf[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
    for (int w = 0; w < NW; ++w) {
        const int e = (w * TB * CB + wave) * 64 + lane;
        const int4 v = red[e];
        sum[0] += v.x; sum[1] += v.y; sum[2] += v.z; sum[3] += v.w;
        if constexpr (!RAW) {
            const float4 f = redf[e];
            sumf[0] += f.x; sumf[1] += f.y; sumf[2] += f.z; sumf[3] += f.w;
        }
    }
    if (n0 + fin_c * 16 + l16 >= a.N) return;
    c_sw *= 1.0f / (float)(1 << SHIFT);                  // exact power-of-two factor
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int t = fin_t * 16 + 4 * g + r;
        if (t >= a.T) continue;
        if constexpr (RAW) {
            int v = sum[r] >> SHIFT;
            if constexpr (ASYM) v -= 8 * (a.code_sum[t] + a.w_code_sum[n]);
            a.acc[(size_t)t * a.ldacc + n] = v;
        } else {
            int ai = sum[r];
            if constexpr (ASYM) ai += prm_ct[t] - 128 * c_nc;
            const float v = __builtin_fmaf((float)ai, prm_sa[t] * c_sw, __builtin_fmaf(prm_sh[t], c_wr, c_bv)) + sumf[r];
            if (a.fp_only) static_cast<float*>(a.y)[(size_t)t * a.ldy + n] = v;
            else static_cast<__half*>(a.y)[(size_t)t * a.ldy + n] = __float2half(v);
        }
    }
}

// Whether weights carry the read-once hint.  Rows that are not whole 128-byte lines share lines, and the second reader
// of a shared line should find it in a cache; the hint lets go of it.  Beyond what the L2s (8 x 4 MB) can hold beside
// the rest that costs as much from HBM as the hint brings there, or more.  GEMM, us, weights cached / from HBM, with and
// without the hint:
//   whole lines   K = 5120, N = 15360, T = 1 7.9/9.9 : 9.8/10.8;  K = 10624, N = 7488, 8-bit, T = 10 14.8/15.6 : 15.1/17.4
//   shared lines  92 MB (K = 6368, N = 13952, 8-bit, T = 19) 26.7/28.2 : 18.2/25.6;  107 MB (K = 4512, N = 22350, 8-bit,
//                 T = 1) 23.3/25.3 : 18.3/21.0;  30 MB (K = 5328, N = 10048, W4A8, T = 13) 13.6/14.5 : 8.6/14.1;
//                 26 MB (K = 6336, N = 3968, 8-bit, T = 3) 7.6/7.9 : 5.6/8.1;  15 MB (K = 1888, N = 11076, T = 3) 6.2/6.4 : 5.1/6.7
// Where the rule keeps the hint, a layer that is called by itself over and over, so that its weights stay in the L2s
// (or, from 17 tokens on, 80 MB and more in the last-level cache), would be faster without it: K = 4096, N = 11008, T = 24
// 9.6/9.8 : 7.6/10.0;  K = 8192, N = 28672, T = 24 26.9/27.8 : 24.3/28.8.  In a model the weights come from HBM.
bool once(const GemmArgs& a) {
    return a.ldw % kLine == 0 || (size_t)a.N * ((size_t)a.ldw + 2 * (size_t)a.n_out) <= (24u << 20);
}

// (the accumulator hook writes the same integers either way and has one form)
template <int XB, int WB, int TB, int CB, int NW, int NST, int MODE>
hipError_t launch_cfg(const GemmArgs& a, hipStream_t stream) {
    const dim3 groups((a.N + CB * 16 - 1) / (CB * 16)), threads(NW * 64);
    if constexpr (MODE == 0) {
        if (!once(a)) {
            hipLaunchKernelGGL((gemm_rows_kernel<XB, WB, TB, CB, NW, NST, 0, false>), groups, threads, 0, stream, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((gemm_rows_kernel<XB, WB, TB, CB, NW, NST, MODE, true>), groups, threads, 0, stream, a);
    return hipGetLastError();
}

// How a launch is cut.  Measured per launch in us (weights from HBM), best against the runner-up:
//  - up to one 16-channel block per CU, blocks stay single and eight waves split K where a row has the lines for
//    it (K = 11008, N = 4096, 16 tokens: 7.7 against 9.4 with pairs and four waves; 8-bit 11.3 against 14.4),
//    four with 17 - 32 tokens, whose activations fill the ring (8.4 against 8.9);
//  - beyond that pairs of blocks and four waves: half the activation traffic per weight byte (K = 5120,
//    N = 15360, 16 tokens: 10.7 against 12.0; N = 28672, K = 8192, 8 tokens: 23.7 against 24.9), except where single
//    blocks leave the busiest CU with less to do (K = 4096, N = 11008, 8-bit: 12.5 against 13.0; not with 8-bit
//    activations under 4-bit weights, whose activation traffic is twice as heavy).  Two stages there: what a third
//    brings in bytes in flight it costs in resident workgroups (N = 15360, one token: 9.9 against 10.1).
struct RowsForm { int cb, nst, waves; };
RowsForm rows_form(int N, int K_b, bool mixed, int w_bits, int tb, int cus) {
    const int blocks = (N + 15) / 16, lines = (K_b * w_bits / 8 + kLine - 1) / kLine;
    auto busiest = [&](int cb) { return (blocks + cb * cus - 1) / (cb * cus) * cb; };
    if (blocks <= cus) {
        if (tb == 1 && lines >= 16) return {1, 3, 8};
        return {1, (tb == 2 && mixed) ? 2 : 3, 4};
    }
    if (!mixed && blocks <= 4 * cus && busiest(1) < busiest(2)) return {1, 2, 4};
    return {2, 2, 4};
}

template <int XB, int WB, int TB, int MODE>
hipError_t launch(const GemmArgs& a, int cus, hipStream_t stream) {
    const RowsForm f = rows_form(a.N, a.K_b, XB != WB, WB, TB, cus);
    if (f.cb == 2) return launch_cfg<XB, WB, TB, 2, 4, 2, MODE>(a, stream);
    if constexpr (TB == 1) {
        if (f.waves == 8) return launch_cfg<XB, WB, 1, 1, 8, 3, MODE>(a, stream);
    }
    if (f.nst == 2) return launch_cfg<XB, WB, TB, 1, 4, 2, MODE>(a, stream);
    if constexpr (XB == WB || TB == 1) return launch_cfg<XB, WB, TB, 1, 4, 3, MODE>(a, stream);
    else return hipErrorInvalidValue;        // (rows_form gives two stages there)
}

template <int XB, int WB, int MODE>
hipError_t dispatch(const GemmArgs& a, int cus, hipStream_t stream) {
    return a.T <= 16 ? launch<XB, WB, 1, MODE>(a, cus, stream) : launch<XB, WB, 2, MODE>(a, cus, stream);
}

}  // namespace

GemmForm choose_rows_form(int T, int N, int K_b, int bits, int w_bits, int cus) {
    const int tb = T <= 16 ? 1 : 2;
    const RowsForm f = rows_form(N, K_b, bits == 8 && w_bits == 4, w_bits, tb, cus);
    return GemmForm{1, tb * 16, f.cb * 16, f.waves, f.waves};
}

hipError_t launch_gemm_rows(const GemmArgs& a, int cus, hipStream_t stream) {
    const bool raw = a.y == nullptr;
    if (a.bits == 4) {
        if (!raw) return dispatch<4, 4, 0>(a, cus, stream);
        return (a.code_sum && a.w_code_sum) ? dispatch<4, 4, 2>(a, cus, stream) : dispatch<4, 4, 1>(a, cus, stream);
    }
    if (a.w_bits == 4) return raw ? dispatch<8, 4, 1>(a, cus, stream) : dispatch<8, 4, 0>(a, cus, stream);
    return raw ? dispatch<8, 8, 1>(a, cus, stream) : dispatch<8, 8, 0>(a, cus, stream);
}

}  // namespace quik
