// QUIK-4B linear layer with the integer product computed on the FP6 matrix pipe of gfx950
// (Algorithm 1 of arXiv 2310.09259: "INTmatmul", "Dequantization", "FPmatmul", final add; the
// epilogue fusion of Section 3.4).  The signed 4-bit codes travel as E3M2 patterns (see
// quik_fp6_device.h: exact, and the fp32 accumulators hold the exact integer dot products), so the
// K loop is DMA -> LDS -> registers -> v_mfma_f32_16x16x128_f8f6f4 with no widening work at all, at
// twice the int8 rate of the matrix pipe.
//
// A workgroup of WM x WN waves owns a BM x BN output tile.  The operands are stored panel by panel of 64
// columns (quik_fp6_device.h), so a tile's rows of a panel are one contiguous run of BM * 48 (BN * 48) bytes
// that 16-byte-per-lane copies bring global -> LDS as it is, into one slot of a ring.  A step of the K loop is
// two panels = one matrix instruction per 16 x 16 block and wave.
//
// What bounds it: the supply of operand bytes (at 70B sizes the loop takes 0.9 us a step with them and 0.6 with
// copies that fetch nothing; the matrix instructions alone 0.5).  What it needs for that:
//  - whole lines per copy.  Splitting a panel's 16-byte and 8-byte parts into planes of LDS, for reads without bank
//    conflicts, made the copies touch every line twice: 256 x 192, K = 4096, N = 11008, T = 2048 72.6 us against 71.2,
//    70B 256 x 256 580 against 528;
//  - large tiles: 256 x 256 fetches 48 KB for 2 x 256 x 256 x 128 operations, 256 x 192 42 KB for three quarters of them;
//  - copies in flight: two block rows before the end of a step all its fragments have been read, so the one barrier
//    of a step sits there, frees the step's own slots and leaves all slots but four flying.  With the barrier at the
//    step's start (two slots landed but not yet read) 70B took 668 us instead of 580.
// The 16 x 16 x 128 instruction sustains 7.1 POP/s on operands like these, the 32 x 32 x 64 one 6.4 (the chip lowers its
// clock).  GEMM, us, 32 x 32 x 64 kernel with a step of one panel : this one, one box, weights cached: 7B up-projection,
// 2048 tokens 83.2 : 75.4;  70B, 4096 tokens 671 : 542;  13B QKV, 1024 tokens 77.8 : 53.3;  7B down-projection 68.9 : 66.6;
// T = 333, N = 11008, K = 4096 29.1 : 22.8;  T = 16, K = N = 4096 21.7 : 12.3.  Over 100 drawn shapes it takes 0.65 of
// that kernel's time with cached weights, 0.68 from HBM.
//
// The fp16 outlier columns run as stages of 32 columns (64-byte rows) through slots of their own over the same
// memory, copied while the tile is dequantized, with the dequantized integer part as the C operand of
// v_mfma_f32_16x16x32_f16, whose accumulator layout is the same.  Rows beyond T / N are out of range
// for the panel descriptors and arrive as zeros (the E3M2 pattern of 0); columns beyond K_b are zero padding.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "quik_kernels.h"
#include "quik_gemm_device.h"
#include "quik_fp6_device.h"

namespace quik {

namespace {

using namespace gemm_dev;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));

// place of a 16-byte piece in a 64-byte stage row: an LDS instruction serves lanes 0 - 3, 12 - 15, 20 - 27 together (and so
// on); with this the sixteen rows of a block meet 64 different banks in every such group
__device__ __forceinline__ int swz_f(int r) { return -(r >> 2) & 3; }

// MODE 0: fused epilogue, fp16 output; MODE 1: the integer accumulators as INT32.  IB x JB accumulator blocks of 16 x 16
// per wave, WM x WN waves; OCC: workgroups per CU; NST: ring slots of 64 columns; GM: as in quik_gemm.hip.
template <int IB, int JB, int WM, int WN, int NST, int OCC, int GM, int MODE>
__global__ __launch_bounds__(WM * WN * 64, OCC * WM * WN / 4) void gemm_fp6_kernel(GemmArgs a) {
    constexpr bool RAW = MODE != 0;
    constexpr int NWAVES = WM * WN;
    // claim the whole register budget of the launch bounds, so that the highest allocated register is
    // never a live one (see the note in the row-quantization kernel)
    if constexpr (OCC * NWAVES <= 8) asm volatile("" ::: "v255");
    else asm volatile("" ::: "v127");
    constexpr int BM = WM * IB * 16, BN = WN * JB * 16;
    // a slot: the 48-byte blocks of the tile's token rows, then of its channels, as they lie in memory
    constexpr int A_BYTES = BM * 48, SLOT = (BM + BN) * 48;
    // copy instructions of a slot (1 KB each); wave w issues instructions w, w + NWAVES, ...; one that does not exist is
    // issued empty so that every wave counts the same number
    constexpr int I_A = A_BYTES / 1024, INSTR = SLOT / 1024;
    constexpr int LPS = (INSTR + NWAVES - 1) / NWAVES;
    static_assert(BM % 64 == 0 && BN % 64 == 0 && IB % 4 == 0, "geometry");
    static_assert(NST >= 4 && NST * LPS < 64, "a step is read while the next lands");
    constexpr int RING = NST * SLOT, DUMMY = RING;       // 1 KB that empty copies clear
    // outlier stages: 32 columns, 64 bytes of every row, in slots of their own over the same memory
    constexpr int FSLOT = (BM + BN) * 64, FNST = RING / FSLOT, F_A = BM / 16, F_B = BN / 16, FLPS = (F_A + F_B + NWAVES - 1) / NWAVES;
    static_assert(FNST >= 3 && FNST * FLPS < 64, "outlier ring");
    constexpr int PARK_ROW = JB * 32 + 16, PARK = 16 * PARK_ROW;
    static_assert(NWAVES * PARK <= RING, "stage ring too small to park the output tile");

    __shared__ __align__(1024) uint8_t lds[RING + 1024];
    __shared__ __align__(16) float lds_sa[BM];
    __shared__ __align__(16) float lds_sh[BM];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;            // (the waves of a SIMD, 4 apart, differ in the channels)
    const int l16 = lane & 15, g = lane >> 4;

    const int tiles_m = (a.T + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    const int id = xcd_contiguous_id(blockIdx.x, tiles_m * tiles_n);
    const int per_group = GM * tiles_n;
    const int grp = id / per_group, rem = id % per_group;
    const int gsz = min(GM, tiles_m - grp * GM);
    const int t0 = (grp * GM + rem % gsz) * BM, n0 = (rem / gsz) * BN;

    const int S = fp6::stages(a.K_b);                    // slots of 64 columns
    const int nk = (S + 1) / 2;                          // steps of 128 columns; an odd last slot is filled with zeros
    const int fp_bytes = a.n_out * 2;
    const int nkf = RAW ? 0 : (fp_bytes + 63) / 64;
    const int lda_fp = a.ldo * 2, ldb_fp = a.ldwo * 2;
    const uint32_t lds_base = lds_addr(lds);

    // ---- copies.  Panel s of an operand with R rows begins s * R * 48 bytes into its buffer; the descriptor of a slot
    // covers the rest of the panel from the tile's first row on, so rows beyond R arrive as zeros.
    const uint64_t pA = (uint64_t)(uintptr_t)a.xq + (uint64_t)t0 * 48u, pB = (uint64_t)(uintptr_t)a.w_q + (uint64_t)n0 * 48u;
    const uint32_t nA = (uint32_t)(a.T - t0) * 48u, nB = (uint32_t)(a.N - n0) * 48u;
    const uint64_t strideA = (uint64_t)a.T * 48u, strideB = (uint64_t)a.N * 48u;
    uint32_t vo[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int i = wave + NWAVES * j;                 // instruction of the slot (wave-uniform)
        vo[j] = i < INSTR ? (uint32_t)((i < I_A ? i : i - I_A) * 1024 + lane * 16) : kOob;
    }
    int ring_f = 0;                                      // ring slot that is filled next
    uint32_t next = 0;                                   // panel that goes into it
    auto issue_one = [&](int j) __attribute__((always_inline)) {
        const int i = wave + NWAVES * j;
        const bool isb = i >= I_A;
        const uint64_t base = isb ? pB + next * strideB : pA + next * strideA;
        const uint32_t n = (int)next < S ? (isb ? nB : nA) : 0u;
        v4i r = v4i{(int)(uint32_t)base, (int)(uint32_t)(base >> 32), (int)n, 0x00020000};
        r = v4i{__builtin_amdgcn_readfirstlane(r[0]), __builtin_amdgcn_readfirstlane(r[1]), __builtin_amdgcn_readfirstlane(r[2]), r[3]};
        const uint32_t dst = i < INSTR ? (uint32_t)(ring_f * SLOT + i * 1024) : (uint32_t)DUMMY;
        dma16(r, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + dst)), vo[j], 0);
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ring_f = ring_f + 1 == NST ? 0 : ring_f + 1;
        ++next;
    };

    // ---- epilogue parameters of the token rows, requested before the first copy
    constexpr int NT = NWAVES * 64, RPT = (BM + NT - 1) / NT;
    float p_s[RPT], p_z[RPT];
    if constexpr (!RAW) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int t = min(t0 + tid + q * NT, a.T - 1);
            p_s[q] = a.scale[t];
            p_z[q] = a.zero[t];
        }
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) {
#pragma unroll
        for (int j = 0; j < LPS; ++j) issue_one(j);
        advance();
    }
    if constexpr (!RAW) {
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = tid + q * NT;
            if (r < BM) {
                lds_sa[r] = p_s[q];                      // scaleAct
                lds_sh[r] = p_z[q] + 8.0f * p_s[q];      // zeroAct + halfRange * scaleAct
            }
        }
    }

    // ---- fragments: lane (l, g) supplies 32 codes for row (channel) l of a 16-row block: half g / 2 of the row's block in
    // panel g % 2 of the step's two, 16 bytes at 16 (g / 2) and 8 at 32 + 8 (g / 2).  Both operands read alike, so which
    // columns a group holds does not matter; this assignment lets the lanes that LDS serves together (0 - 3, 12 - 15,
    // 20 - 27 and so on) read the same part of sixteen different rows, and twelve dwords a row spread these over all banks.
    const uint32_t rdP = (uint32_t)(l16 * 48 + (g >> 1) * 16), rdQ = (uint32_t)(l16 * 48 + 32 + (g >> 1) * 8);
    const uint32_t aP = rdP + wm * IB * 768, bP = rdP + A_BYTES + wn * JB * 768;
    const uint32_t aQ = rdQ + wm * IB * 768, bQ = rdQ + A_BYTES + wn * JB * 768;
    v8i fa[4], fb[JB];
    auto rd6 = [&](uint32_t P, uint32_t Q) __attribute__((always_inline)) -> v8i {
        const uint4 x = *reinterpret_cast<const uint4*>(lds + P);
        const uint2 y = *reinterpret_cast<const uint2*>(lds + Q);
        return v8i{(int)x.x, (int)x.y, (int)x.z, (int)x.w, (int)y.x, (int)y.y, 0, 0};
    };
    auto read_a = [&](int i, uint32_t so) __attribute__((always_inline)) { fa[i & 3] = rd6(so + aP + i * 768, so + aQ + i * 768); };
    auto read_b = [&](int j, uint32_t so) __attribute__((always_inline)) { fb[j] = rd6(so + bP + j * 768, so + bQ + j * 768); };
    // LDS offset of this lane's slot of the step whose first slot is `r`
    auto slot_of = [&](int r) __attribute__((always_inline)) {
        const int r1 = r + 1 == NST ? 0 : r + 1;
        return (uint32_t)(((g & 1) ? r1 : r) * SLOT);
    };

    v4f acc[IB][JB];
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    // A step: 128 columns.  Two block rows before its end every fragment of the step has been read, so the barrier there
    // frees the step's own two slots -- refilled right away, beside the last matrix instructions -- and lets everybody
    // read the next step's, which must have landed; all other slots (NST - 4 at the wait) are in flight.
    constexpr int SLOTS = IB * JB, LAST_READ = (IB - 2) * JB - 1;
    int cur = 0;
    auto step = [&]() __attribute__((always_inline)) {
        const int nxt = cur + 2 >= NST ? cur + 2 - NST : cur + 2;
        const uint32_t so = slot_of(cur), so1 = slot_of(nxt);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < SLOTS; ++m) {
            const int i = m / JB, j = m % JB;
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[i & 3], fb[j], acc[i][j], 3, 3, 0, 0, 0, 0);
            if (j == 0 && i + 2 < IB) read_a(i + 2, so);
            if (m == LAST_READ) {
                wait_stage<(NST - 4) * LPS>();
                __syncthreads();
            }
            if (j == 0 && i + 2 >= IB) read_a(i + 2 - IB, so1);
            if (i == IB - 1) read_b(j, so1);
#pragma unroll
            for (int d = 0; d < 2 * LPS; ++d)
                if (m > LAST_READ && d * (SLOTS - 1 - LAST_READ) / (2 * LPS) == m - LAST_READ - 1) {
                    issue_one(d % LPS);
                    if (d % LPS == LPS - 1) advance();
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    };
    // (always true, yet it keeps this wait in a block of its own: without the test the compiler schedules the first step
    // so that 256 x 192 and 128 x 256 tiles take 2 - 3 % longer: 7B up-projection, 2048 tokens 71.0 : 73.0 us)
    if (nk > 0) {
        wait_stage<(NST - 2) * LPS>();                   // the first step's two slots have landed
        __syncthreads();
        const uint32_t so = slot_of(0);
#pragma unroll
        for (int j = 0; j < JB; ++j) read_b(j, so);
        read_a(0, so);
        read_a(1, so);
    }
    for (int s = 0; s < nk; ++s) step();

    const int tw = t0 + wm * IB * 16, nw = n0 + wn * JB * 16;
    wait_stage<0>();
    __syncthreads();                                     // every copy and every read of the ring is done
    if constexpr (RAW) {
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                const int n = nw + j * 16 + l16;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = tw + i * 16 + 4 * g + r;
                    if (t < a.T && n < a.N) a.acc[(size_t)t * a.ldacc + n] = (int)acc[i][j][r];
                }
            }
        return;
    }

    // ---- outlier stages on the way while the tile is dequantized.  Instruction i of a stage: 16 rows, 16-byte pieces
    // exchanged so that the four rows of an LDS pass that share banks differ in their place.
    const v4i rAf = make_rsrc(a.n_out ? (const uint8_t*)a.x_out + (size_t)t0 * lda_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.T - t0) * lda_fp : 0);
    const v4i rBf = make_rsrc(a.n_out ? (const uint8_t*)a.w_out + (size_t)n0 * ldb_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.N - n0) * ldb_fp : 0);
    const int fc = ((lane & 3) ^ swz_f(lane >> 2)) << 4;
    auto issue_fp = [&](int f) __attribute__((always_inline)) {
        const uint32_t sb = (uint32_t)(f % FNST) * FSLOT;
        const bool live = f * 64 + fc < fp_bytes;
#pragma unroll
        for (int j = 0; j < FLPS; ++j) {
            const int i = wave + NWAVES * j;
            const bool isb = i >= F_A;
            const int row = (isb ? i - F_A : i) * 16 + (lane >> 2);
            const uint32_t v = live && i < F_A + F_B ? (uint32_t)(row * (isb ? ldb_fp : lda_fp) + fc) : kOob;
            const v4i r_ = isb ? rBf : rAf;
            dma16(r_, lds_base + (i < F_A + F_B ? sb + i * 1024 : (uint32_t)DUMMY), v, (uint32_t)f * 64u);
        }
    };
    float c_sw[JB], c_wr[JB], c_bv[JB];
    {
        const __half* __restrict__ wsc = static_cast<const __half*>(a.w_scale);
        const __half* __restrict__ bias = static_cast<const __half*>(a.bias);
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int n = min(nw + j * 16 + l16, a.N - 1);
            c_sw[j] = __half2float(wsc[n]);
            c_bv[j] = bias ? __half2float(bias[n]) : 0.0f;
            c_wr[j] = a.w_reduced[n];
        }
    }
    // (the parameters first: the compiler's wait for them would otherwise be one for the copies)
#pragma unroll
    for (int j = 0; j < JB; ++j) asm volatile("" : "+v"(c_sw[j]), "+v"(c_bv[j]), "+v"(c_wr[j]));
    if (nkf > 0) {
#pragma unroll
        for (int f = 0; f < FNST; ++f) issue_fp(f);
    }
    // Dequantization: the accumulators are exact integers already in binary32.
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int lr = wm * IB * 16 + i * 16 + 4 * g;
        const float4 sa4 = *reinterpret_cast<const float4*>(&lds_sa[lr]);
        const float4 sh4 = *reinterpret_cast<const float4*>(&lds_sh[lr]);
        const float sa_[4] = {sa4.x, sa4.y, sa4.z, sa4.w}, sh_[4] = {sh4.x, sh4.y, sh4.z, sh4.w};
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[i][j][r] = __builtin_fmaf(acc[i][j][r], sa_[r] * c_sw[j], __builtin_fmaf(sh_[r], c_wr[j], c_bv[j]));
    }
    if (nkf > 0) {
        const uint32_t rdF = (uint32_t)(l16 * 64 + ((g ^ swz_f(l16)) << 4));
        const uint32_t aF = rdF + wm * IB * 1024, bF = rdF + BM * 64 + wn * JB * 1024;
        v8h ha[4], hb[JB];
        auto read_ha = [&](int i, uint32_t fo) __attribute__((always_inline)) { ha[i & 3] = *reinterpret_cast<const v8h*>(lds + fo + aF + i * 1024); };
        auto read_hb = [&](int j, uint32_t fo) __attribute__((always_inline)) { hb[j] = *reinterpret_cast<const v8h*>(lds + fo + bF + j * 1024); };
        wait_stage<(FNST - 1) * FLPS>();
        __syncthreads();
#pragma unroll
        for (int j = 0; j < JB; ++j) read_hb(j, 0);
        read_ha(0, 0);
        read_ha(1, 0);
        for (int f = 0; f < nkf; ++f) {
            const uint32_t fo = (uint32_t)(f % FNST) * FSLOT, fo1 = (uint32_t)((f + 1) % FNST) * FSLOT;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < SLOTS; ++m) {
                const int i = m / JB, j = m % JB;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i & 3], hb[j], acc[i][j], 0, 0, 0);
                if (j == 0 && i + 2 < IB) read_ha(i + 2, fo);
                if (m == (IB - 2) * JB - 1) {
                    // every read of this stage has been issued: behind the barrier its slot is free, the next has landed
                    wait_stage<(FNST - 2) * FLPS>();
                    __syncthreads();
                    issue_fp(f + FNST);
                }
                if (j == 0 && i + 2 >= IB) read_ha(i + 2 - IB, fo1);
                if (i == IB - 1) read_hb(j, fo1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        wait_stage<0>();
        __syncthreads();                                 // the stage memory is dead
    }
    __half* __restrict__ y = static_cast<__half*>(a.y);
    // Output through LDS: a wave parks sixteen rows of its tile and writes them out as 16-byte pieces, whole row segments
    // per store; needs 16-byte aligned output rows.
    const bool vec_ok = ((reinterpret_cast<uintptr_t>(a.y) & 15u) == 0) && (a.ldy % 8 == 0);
    if (vec_ok) {
        uint8_t* wbuf = lds + wave * PARK;
        constexpr int CH = JB * 2, RPS = 64 / CH;        // 16-byte pieces per row, rows per store instruction
        const int prow = lane / CH, pch = lane % CH;
#pragma unroll
        for (int i = 0; i < IB; ++i) {
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<__half*>(wbuf + (4 * g + r) * PARK_ROW + (j * 16 + l16) * 2) = __float2half(acc[i][j][r]);
#pragma unroll
            for (int q = 0; q < (16 + RPS - 1) / RPS; ++q) {
                const int row = q * RPS + prow;
                if (prow >= RPS || row >= 16) continue;
                const uint4 v = *reinterpret_cast<const uint4*>(wbuf + row * PARK_ROW + pch * 16);
                const int t = tw + i * 16 + row, n = nw + pch * 8;
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
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            const int n = nw + j * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = tw + i * 16 + 4 * g + r;
                if (t < a.T && n < a.N) y[(size_t)t * a.ldy + n] = __float2half(acc[i][j][r]);
            }
        }
}

// Signed 4-bit weights (two per byte, column 2p in the low nibble) -> FP6 panels.  One thread per
// (row, group of 32 columns).  Offline step.
__global__ __launch_bounds__(256) void weight_pack_fp6_kernel(const uint8_t* __restrict__ w_q, int ldw, int N, int K_b,
                                                              uint32_t* __restrict__ w6) {
    const int S = fp6::stages(K_b);
    const int groups = 2 * S;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)N * groups) return;
    const int n = (int)(idx / groups), G = (int)(idx % groups);
    const uint8_t* src = w_q + (size_t)n * ldw + G * 16;
    uint32_t cw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t v = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int col = G * 32 + i * 8 + b * 2;                 // first column of this byte
            uint32_t byte = (col < K_b) ? src[i * 4 + b] : 0u;      // columns at or beyond K_b: value 0
            if (col + 1 >= K_b) byte &= 0x0Fu;
            v |= byte << (8 * b);
        }
        cw[i] = v ^ 0x88888888u;                                    // two's complement -> unsigned code (value + 8)
    }
    // 32 columns = four 48-bit strings at bits 0, 48, 96, 144
    const uint64_t e0 = fp6::pack8(cw[0]), e1 = fp6::pack8(cw[1]), e2 = fp6::pack8(cw[2]), e3 = fp6::pack8(cw[3]);
    uint32_t d[6];
    d[0] = (uint32_t)e0;
    d[1] = (uint32_t)(e0 >> 32) | (uint32_t)(e1 << 16);
    d[2] = (uint32_t)(e1 >> 16);
    d[3] = (uint32_t)e2;
    d[4] = (uint32_t)(e2 >> 32) | (uint32_t)(e3 << 16);
    d[5] = (uint32_t)(e3 >> 16);
    uint32_t* blk = w6 + ((size_t)(G >> 1) * N + n) * 12;         // the row's 48-byte block of this stage
#pragma unroll
    for (int i = 0; i < 6; ++i) blk[fp6::block_dword(G & 1, i)] = d[i];
}

template <int IB, int JB, int WM, int WN, int NST, int OCC, int GM, int MODE>
hipError_t launch_cfg(const GemmArgs& a, hipStream_t stream) {
    constexpr int BM = WM * IB * 16, BN = WN * JB * 16;
    const int tiles = ((a.T + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    hipLaunchKernelGGL((gemm_fp6_kernel<IB, JB, WM, WN, NST, OCC, GM, MODE>), dim3(tiles), dim3(WM * WN * 64), 0, stream, a);
    return hipGetLastError();
}

// The tile whose launch is estimated to be the shortest, up to `occ` workgroups of it per CU: base + round * rounds +
// tile * tiles of the busiest CU + stages (of 128 columns) * (round_stage * rounds + tile_stage * tiles of the busiest CU).
// Fitted to 765 shapes with every tile measured (T 1 .. 4096, K 512 .. 11008, N 512 .. 28672, cached weights and from
// HBM, mean of both); good to 5 - 10 %, and the choice costs 0.2 % against the fastest tile in the mean.  The 256 x 256 tile
// needs a third fewer operand bytes per operation than 256 x 128 and wins wherever it fills the chip: K = 5120, N = 15360,
// T = 1024 in one round 49 us (256 x 192 in two 73, 128 x 128 64; the former kernel's 256 x 128 73).
// The last line is the 64 x 128 tile with eight ring slots instead of six, for up to 64 tokens: weights from HBM want more
// bytes in flight (us, cached / from HBM, six : eight: T=21 K=7200 N=19600 21.4/29.0 : 22.1/24.5, T=25 K=10272 N=23456
// 29.6/40.6 : 30.7/34.4; the former kernel 27.5/28.1 and 38.6/40.0), smaller layers and cached ones do not.  With more
// tokens it was ahead nowhere.  65 to 128 tokens of such layers run 128 x 128 tiles, whose rings have no room for
// more: from HBM up to 8 % behind the former kernel, cached as much ahead (T=76 K=5152 N=20360 22.7/23.7 there, 21.0/25.8).
struct TileCost6 { int bm, bn, occ; double base, round, tile, round_stage, tile_stage; };
constexpr TileCost6 kCost6[] = {{64, 64, 4, 1.495, 1.495, 1.396, 0.160, 0.092},
                                {64, 128, 2, 2.120, 1.115, 2.468, 0.137, 0.153},
                                {128, 128, 2, 1.548, 1.636, 4.019, 0.099, 0.250},
                                {128, 192, 1, -2.250, 9.384, 0, 0.409, 0},
                                {128, 256, 1, -4.435, 12.559, 0, 0.481, 0},
                                {256, 192, 1, -6.078, 17.534, 0, 0.558, 0},
                                {256, 256, 1, -6.037, 20.272, 0, 0.670, 0},
                                {64, 128, 2, 0.848, 0.849, 4.383, -0.014, 0.291}};
constexpr int kDeepRing = 7;             // the line of the eight-slot 64 x 128 tile

int choose_tile_fp6(int T, int N, int K_b, int cus) {
    const int stages = (K_b + 127) / 128;
    int best = 0;
    double least = 0.0;
    for (int i = 0; i < (int)(sizeof(kCost6) / sizeof(TileCost6)); ++i) {
        const TileCost6& c = kCost6[i];
        if (i == kDeepRing && T > 64) continue;
        const long tiles = (long)((T + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const double rounds = (double)((tiles + (long)c.occ * cus - 1) / ((long)c.occ * cus)), busiest = (double)((tiles + cus - 1) / cus);
        const double t = c.base + c.round * rounds + c.tile * busiest + stages * (c.round_stage * rounds + c.tile_stage * busiest);
        if (i == 0 || t < least) { best = i; least = t; }
    }
    return best;
}

// Six ring slots but for that line: a seventh under 256 x 192 cost 3 %, 128 x 128 and 256 x 256 have room for no more.
template <int MODE>
hipError_t dispatch6(const GemmArgs& a, hipStream_t stream) {
    int cus = compute_units();
    if (cus < 1) cus = 256;
    switch (choose_tile_fp6(a.T, a.N, a.K_b, cus)) {
    case 0: return launch_cfg<4, 1, 1, 4, 6, 4, 8, MODE>(a, stream);
    case 1: return launch_cfg<4, 2, 1, 4, 6, 2, 8, MODE>(a, stream);
    case 2: return launch_cfg<4, 4, 2, 2, 6, 2, 8, MODE>(a, stream);
    case 3: return launch_cfg<4, 3, 2, 4, 6, 1, 8, MODE>(a, stream);
    case 4: return launch_cfg<4, 4, 2, 4, 6, 1, 8, MODE>(a, stream);
    case 5: return launch_cfg<4, 6, 4, 2, 6, 1, 4, MODE>(a, stream);
    case 6: return launch_cfg<8, 4, 2, 4, 6, 1, 8, MODE>(a, stream);
    default: return launch_cfg<4, 2, 1, 4, 8, 2, 8, MODE>(a, stream);
    }
}

}  // namespace

void fp6_form(int T, int N, int K_b, int cus, int* rows, int* cols, int* slots) {
    const int i = choose_tile_fp6(T, N, K_b, cus);
    const TileCost6& c = kCost6[i];
    *rows = c.bm;
    *cols = c.bn;
    *slots = i == kDeepRing ? 8 : 6;
}

hipError_t launch_gemm_fp6(const GemmArgs& a, hipStream_t stream) {
    if (a.T <= 0 || a.N <= 0) return hipSuccess;
    return a.y ? dispatch6<0>(a, stream) : dispatch6<1>(a, stream);
}

hipError_t launch_weight_pack_fp6(const void* w_q, int ldw, int N, int K_b, void* w6, hipStream_t stream) {
    if (N <= 0 || K_b <= 0) return hipSuccess;
    const long total = (long)N * 2 * fp6::stages(K_b);
    hipLaunchKernelGGL(weight_pack_fp6_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const uint8_t*>(w_q), ldw, N, K_b, static_cast<uint32_t*>(w6));
    return hipGetLastError();
}

}  // namespace quik
