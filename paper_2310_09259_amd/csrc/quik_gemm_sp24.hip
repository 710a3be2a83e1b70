// QUIK-4B linear layer for 2:4-sparse weights, the integer product computed by the sparse int8 matrix
// instruction of gfx950 (Algorithm 1 of arXiv 2310.09259: "INTmatmul", "Dequantization", "FPmatmul",
// final add, with the epilogue fusion of Section 3.4; the weight format is the joint INT4 + 2:4 one of
// Section 4.3.2).  v_smfmac_i32_16x16x128_i8 runs at twice the dense int8 rate and accumulates exactly in
// INT32.  Operand formats: quik_sp24_device.h.
//
// The sparse operand is the instruction's first one, so it carries the weights: an accumulator register
// belongs to an output channel and a lane to a token, the transpose of the dense kernels' arrangement.
// Per-token parameters therefore belong to lanes and per-channel ones to registers, and a lane converts four
// neighbouring channels of its token at a time.
//
// A workgroup of WM x WN waves owns a BM (tokens) x BN (channels) output tile.  The operands are stored panel by
// panel of 64 columns, 32 bytes a row, so a tile's rows of a panel are two contiguous runs that
// 16-byte-per-lane copies bring global -> LDS, into one slot of a ring.  A step of the K loop is two panels = one
// matrix instruction per 16 x 16 block and wave.
//
// What bounds it: the issue of matrix and widening instructions, which hardly overlap (measured, ns per 16 x 16 x 128
// instruction and SIMD beside 0 / 1 / 2 / 3 / 4 / 6 vector instructions: 9.2 / 11.7 / 12.3 / 13.5 / 15.3 / 18.5).  A
// token block of a step takes 12 of these and a channel block 6, so a wave of IB x JB blocks has 12 / JB + 6 / IB of
// them per matrix instruction: 3 for 4 x 8 blocks, 4.5 for 4 x 4.  N = 15360, K = 5120, T = 1024 without outliers takes
// 45 us; 41 with copies that fetch nothing, and the issue alone is 35.  What it needs beside that:
//  - two workgroups of four waves of 4 x 8 blocks per CU (128 x 256 tiles): as little widening as under 256 x 256 with
//    eight waves and half the granularity, and one works through its prologue and epilogue beside the other's loop;
//  - a barrier two token blocks before the end of a step, when all its fragments have been read: it frees the step's
//    own slots and leaves all slots but four flying;
//  - no drain at the ends: the epilogue's parameters come by copies to LDS, and the fp16 outlier columns run as stages
//    of 32 columns (64-byte rows) through the same ring right behind the last panels, with the dequantized integer part
//    as the C operand of v_mfma_f32_16x16x32_f16 (weights first, so the accumulator layout is the same).  With
//    parameters loaded to registers and an outlier ring that starts when the loop has ended 128 x 128 tiles
//    took 64 us instead of 60 for the shape above with 256 outliers.
// GEMM, us, a 32 x 32 x 64 kernel with steps of one panel : this one with the tiles that the estimate below takes, one box,
// weights cached: 13B QKV, 1024 tokens 78.6 : 56.5; 4096 tokens 237 : 206; 7B up-projection, 2048 tokens 83.7 : 70.2; 7B
// down-projection 64.8 : 63.9; 70B, 4096 tokens 635 : 543; T = 333, N = 11008, K = 4096 28.7 : 24.6.  Over 150 drawn shapes
// of 1 to 4096 tokens it takes 0.74 of that kernel's time.
// Rows beyond T / N are out of range for the panel descriptors and arrive as zeros.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "quik_kernels.h"
#include "quik_gemm_device.h"
#include "quik_sp24_device.h"

namespace quik {

namespace {

using namespace gemm_dev;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int swz_f(int r) { return (r >> 3) & 1; }   // 32-byte rows, two pieces

// descriptor r moved forward by `bytes`
__device__ __forceinline__ v4i advance(v4i r, uint32_t bytes) {
    const uint64_t base = (((uint64_t)(uint32_t)r[1]) << 32 | (uint32_t)r[0]) + bytes;
    r[0] = (int)(uint32_t)base;
    r[1] = (int)(uint32_t)(base >> 32);
    return r;
}

// place of a 16-byte piece in a 64-byte fp16 stage row: an LDS instruction serves lanes 0 - 3, 12 - 15, 20 - 27 together
// (and so on); with this the sixteen rows of a block meet 64 different banks in every such group
__device__ __forceinline__ int swz_h(int r) { return -(r >> 2) & 3; }

__device__ __forceinline__ float h2f(uint32_t u) { return __half2float(__ushort_as_half((unsigned short)u)); }

// MODE 0: fused epilogue, fp16 output; MODE 1: the integer accumulators as INT32.  IB (tokens) x JB (channels) accumulator
// blocks of 16 x 16 per wave, WM x WN waves; OCC: workgroups per CU; NST: ring slots of 64 columns; GM: as in quik_gemm.hip.
template <int IB, int JB, int WM, int WN, int NST, int OCC, int GM, int MODE>
__global__ __launch_bounds__(WM * WN * 64, OCC * WM * WN / 4) void gemm_sp24_kernel(GemmArgs a) {
    constexpr bool RAW = MODE != 0;
    constexpr int NWAVES = WM * WN;
    // claim the whole register budget of the launch bounds, so that the highest allocated register is
    // never a live one (see the note in the row-quantization kernel)
    if constexpr (OCC * NWAVES <= 8) asm volatile("" ::: "v255");
    else asm volatile("" ::: "v127");
    constexpr int BM = WM * IB * 16, BN = WN * JB * 16;
    // a slot: the 32-byte rows of the tile's tokens, then of its channels
    constexpr int A_BYTES = BM * 32, SLOT = (BM + BN) * 32;
    // copy instructions of a slot (1 KB each); wave w issues instructions w, w + NWAVES, ...; one that does not exist is
    // issued empty so that every wave counts the same number
    constexpr int I_A = A_BYTES / 1024, INSTR = SLOT / 1024;
    constexpr int LPS = (INSTR + NWAVES - 1) / NWAVES;
    static_assert(sp24::kActBytes == 32 && sp24::kWgtBytes == 32, "every row of a panel is 32 bytes");
    static_assert(BM % 64 == 0 && BN % 64 == 0 && IB % 4 == 0, "geometry");
    static_assert(NST % 2 == 0 && NST >= 6 && NST * LPS < 64, "a step is read while the next lands");
    constexpr int RING = NST * SLOT, DUMMY = RING;       // 1 KB that empty copies clear
    // outlier stages: 32 columns, 64 bytes of every row, in the two slots of a step
    constexpr int FSLOT = 2 * SLOT, F_A = BM / 16, F_B = BN / 16;
    static_assert((F_A + F_B + NWAVES - 1) / NWAVES <= 2 * LPS, "an outlier stage takes no more copies than a step");
    constexpr int PARK_ROW = JB * 32 + 16, PARK = 16 * PARK_ROW;
    static_assert(NWAVES * PARK <= RING, "stage ring too small to park the output tile");

    __shared__ __align__(1024) uint8_t lds[RING + 1024];
    __shared__ __align__(16) float lds_s[BM], lds_z[BM], lds_wr[BN];
    __shared__ __align__(16) uint32_t lds_sw[BN], lds_bv[BN];       // binary16 patterns

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int l16 = lane & 15, g = lane >> 4;

    const int tiles_m = (a.T + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    const int id = xcd_contiguous_id(blockIdx.x, tiles_m * tiles_n);
    const int per_group = GM * tiles_n;
    const int grp = id / per_group, rem = id % per_group;
    const int gsz = min(GM, tiles_m - grp * GM);
    const int t0 = (grp * GM + rem % gsz) * BM, n0 = (rem / gsz) * BN;

    const int S = sp24::stages(a.K_b);                   // slots of 64 columns
    const int nk = (S + 1) / 2;                          // steps of 128 columns; an odd last slot is filled with zeros
    const int fp_bytes = a.n_out * 2;
    const int nkf = RAW ? 0 : (fp_bytes + 63) / 64;
    const int lda_fp = a.ldo * 2, ldb_fp = a.ldwo * 2;
    const uint32_t lds_base = lds_addr(lds);

    // ---- copies.  Panel s of an operand with R rows begins s * R * 32 bytes into its buffer; the descriptor of a slot
    // covers the rest of the panel from the tile's first row on, so rows beyond R arrive as zeros.  The two records of a
    // channel change places in odd panels (see the fragments below).
    const uint64_t pA = (uint64_t)(uintptr_t)a.xq + (uint64_t)t0 * 32u, pB = (uint64_t)(uintptr_t)a.w_q + (uint64_t)n0 * 32u;
    const uint32_t nA = (uint32_t)(a.T - t0) * 32u, nB = (uint32_t)(a.N - n0) * 32u;
    const uint64_t strideA = (uint64_t)a.T * 32u, strideB = (uint64_t)a.N * 32u;
    const v4i rAf = make_rsrc(a.n_out ? (const uint8_t*)a.x_out + (size_t)t0 * lda_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.T - t0) * lda_fp : 0);
    const v4i rBf = make_rsrc(a.n_out ? (const uint8_t*)a.w_out + (size_t)n0 * ldb_fp : (const uint8_t*)a.xq,
                              a.n_out ? (size_t)(a.N - n0) * ldb_fp : 0);
    uint32_t vo[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int i = wave + NWAVES * j;                 // instruction of the slot (wave-uniform)
        vo[j] = i < INSTR ? (uint32_t)((i < I_A ? i : i - I_A) * 1024 + lane * 16) : kOob;
    }
    // copy d of the 2 * LPS of step p, whose slots begin at LDS offset `at`
    auto issue_int = [&](int p, int d, int at) __attribute__((always_inline)) {
        const int i = wave + NWAVES * (d % LPS);
        const uint32_t odd = d / LPS, panel = 2u * (uint32_t)p + odd;
        const bool isb = i >= I_A;
        const uint64_t base = isb ? pB + panel * strideB : pA + panel * strideA;
        const uint32_t n = (int)panel < S ? (isb ? nB : nA) : 0u;
        v4i r = v4i{(int)(uint32_t)base, (int)(uint32_t)(base >> 32), (int)n, 0x00020000};
        r = v4i{__builtin_amdgcn_readfirstlane(r[0]), __builtin_amdgcn_readfirstlane(r[1]), __builtin_amdgcn_readfirstlane(r[2]), r[3]};
        const uint32_t dst = i < INSTR ? (uint32_t)at + odd * SLOT + i * 1024 : (uint32_t)DUMMY;
        dma16(r, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + dst)), isb ? vo[d % LPS] ^ (odd << 4) : vo[d % LPS], 0);
    };
    // the same of outlier stage f (beyond the last one: nothing is fetched).  An instruction copies 16 rows, whose 16-byte
    // pieces are exchanged so that the four rows of an LDS pass that share banks differ in their place.
    const int fc = ((lane & 3) ^ swz_h(lane >> 2)) << 4;
    auto issue_fp = [&](int f, int d, int at) __attribute__((always_inline)) {
        const int i = wave + NWAVES * d;
        const bool isb = i >= F_A;
        const int row = (isb ? i - F_A : i) * 16 + (lane >> 2);
        const uint32_t v = f * 64 + fc < fp_bytes && i < F_A + F_B ? (uint32_t)(row * (isb ? ldb_fp : lda_fp) + fc) : kOob;
        const v4i r = isb ? rBf : rAf;
        const uint32_t dst = i < F_A + F_B ? (uint32_t)at + i * 1024 : (uint32_t)DUMMY;
        dma16(r, (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_base + dst)), v, (uint32_t)f * 64u);
    };

    // ---- the epilogue's parameters, copied to LDS first of all: loads into registers would make the compiler wait for
    // everything requested since when they are used
    if constexpr (!RAW) {
        constexpr int PA = BM / 64, PB = BN / 64;        // instructions of 64 values
        const v4i rs = make_rsrc(a.scale + t0, (size_t)(a.T - t0) * 4), rz = make_rsrc(a.zero + t0, (size_t)(a.T - t0) * 4);
        const v4i rr = make_rsrc(a.w_reduced + n0, (size_t)(a.N - n0) * 4);
        const v4i rw_ = make_rsrc(static_cast<const __half*>(a.w_scale) + n0, (size_t)(a.N - n0) * 2);
        const v4i rb = make_rsrc(a.bias ? static_cast<const __half*>(a.bias) + n0 : a.w_scale, a.bias ? (size_t)(a.N - n0) * 2 : 0);
#pragma unroll
        for (int q = 0; q < (2 * PA + 3 * PB + NWAVES - 1) / NWAVES; ++q) {
            int k = wave + NWAVES * q;
            if (k < PA) dma4(rs, lds_addr(lds_s) + k * 256, (uint32_t)(k * 64 + lane) * 4u);
            else if ((k -= PA) < PA) dma4(rz, lds_addr(lds_z) + k * 256, (uint32_t)(k * 64 + lane) * 4u);
            else if ((k -= PA) < PB) dma4(rr, lds_addr(lds_wr) + k * 256, (uint32_t)(k * 64 + lane) * 4u);
            else if ((k -= PB) < PB) dma2(rw_, lds_addr(lds_sw) + k * 256, (uint32_t)(k * 64 + lane) * 2u);
            else if ((k -= PB) < PB) dma2(rb, lds_addr(lds_bv) + k * 256, (uint32_t)(k * 64 + lane) * 2u);
        }
    }
#pragma unroll
    for (int p = 0; p < NST / 2; ++p)
#pragma unroll
        for (int d = 0; d < 2 * LPS; ++d) {
            if (p < nk) issue_int(p, d, p * FSLOT);
            else issue_fp(p - nk, d, p * FSLOT);
        }

    // ---- fragments.  v_smfmac_i32_16x16x128_i8, measured: dense lane (l, g) holds 32 columns of token l, sparse lane
    // (l, g) the 16 kept values of channel l, of which the first eight meet bytes 16 (g / 2) .. of the dense lanes of group
    // 2 (g % 2) and the others the same bytes of group 2 (g % 2) + 1.  So token lanes take piece g % 2 of panel g / 2 of
    // the step's two, channel lanes record g / 2 of panel g % 2.  Lanes that LDS serves together (0 - 3, 12 - 15, 20 - 27
    // and so on) read 16 different pieces of sixteen rows: the tokens' because groups 0 and 1 read two pieces of one
    // panel, the channels' because the records of odd panels have changed places.
    const uint32_t oddA = (uint32_t)((g >> 1) * SLOT + l16 * 32 + ((g & 1) << 4) + wm * IB * 512);
    const uint32_t oddW = (uint32_t)((g & 1) * SLOT + l16 * 32 + (((g >> 1) ^ (g & 1)) << 4) + A_BYTES + wn * JB * 512);
    uint4 ra[2], rw[JB];                                 // packed words (rw.z: the index word)
    v8i ua[2];                                           // int8 operands, sixteen-fold
    v4i uw[JB];
    constexpr uint32_t M = 0xF0F0F0F0u;
    auto read_a = [&](int i, uint32_t so) __attribute__((always_inline)) { ra[i & 1] = *reinterpret_cast<const uint4*>(lds + so + oddA + i * 512); };
    auto read_w = [&](int j, uint32_t so) __attribute__((always_inline)) { rw[j] = *reinterpret_cast<const uint4*>(lds + so + oddW + j * 512); };
    auto widen_a = [&](int i, int d) __attribute__((always_inline)) {      // one word: columns 8 d .. 8 d + 3, 8 d + 4 .. 8 d + 7
        const uint32_t w = d == 0 ? ra[i & 1].x : d == 1 ? ra[i & 1].y : d == 2 ? ra[i & 1].z : ra[i & 1].w;
        ua[i & 1][2 * d] = (int)(w & M);
        ua[i & 1][2 * d + 1] = (int)((w << 4) & M);
    };
    auto widen_w = [&](int j) __attribute__((always_inline)) {
        uw[j] = v4i{(int)((rw[j].x << 4) & M), (int)(rw[j].x & M), (int)((rw[j].y << 4) & M), (int)(rw[j].y & M)};
    };
    v4i acc[IB][JB];
#pragma unroll
    for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int j = 0; j < JB; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // A step: 128 columns.  The words of token block i + 2 are read and those of block i + 1 widened beside the matrix
    // instructions of block i; the next step's channel words are read beside the last block, each after the last use of its
    // predecessor, and widened one instruction before their first use.  Two blocks before the end of a step everything of
    // it has been read, so the barrier there frees the step's own two slots -- refilled right away -- and lets everybody
    // read the next step's, which must have landed; all other slots (NST - 4 at the wait) are in flight.
    constexpr int SLOTS = IB * JB, LAST_READ = (IB - 2) * JB - 1;
    int at = 0;                                          // LDS offset of the step's slots
    auto step = [&](int s, bool tail) __attribute__((always_inline)) {
        const int nxt = at + FSLOT == RING ? 0 : at + FSLOT;
        const uint32_t so = (uint32_t)at, so1 = (uint32_t)nxt;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < SLOTS; ++m) {
            const int i = m / JB, j = m % JB;
            acc[i][j] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(uw[j], ua[i & 1], acc[i][j], (int)rw[j].z, 0, 0);
            if (j == 0 && i + 2 < IB) read_a(i + 2, so);
            if (m == LAST_READ) {
                wait_stage<(NST - 4) * LPS>();
                __syncthreads();
            }
            if (j == 0 && i + 2 >= IB) read_a(i + 2 - IB, so1);
            if (i == IB - 1) read_w(j, so1);
#pragma unroll
            for (int d = 0; d < 4; ++d)
                if (d * JB / 4 == j) widen_a(i + 1, d);
            if (i == 0 && j + 1 < JB) widen_w(j + 1);
            if (m == SLOTS - 1) widen_w(0);
#pragma unroll
            for (int d = 0; d < 2 * LPS; ++d)
                if (m > LAST_READ && d * (SLOTS - 1 - LAST_READ) / (2 * LPS) == m - LAST_READ - 1) {
                    if (!tail) issue_int(s + NST / 2, d, at);
                    else issue_fp(s + NST / 2 - nk, d, at);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        at = nxt;
    };
    wait_stage<(NST - 2) * LPS>();                       // the first step's two slots have landed
    __syncthreads();
    {
#pragma unroll
        for (int j = 0; j < JB; ++j) read_w(j, 0);
        read_a(0, 0);
        read_a(1, 0);
#pragma unroll
        for (int d = 0; d < 4; ++d) widen_a(0, d);
        widen_w(0);
    }
    int s = 0;
    for (; s + NST / 2 < nk; ++s) step(s, false);
    for (; s < nk; ++s) step(s, true);                   // the freed slots take the outlier stages

    // lane: token tw + 16 i + l16; register r of block j: channel nw + 16 j + 4 g + r
    const int tw = t0 + wm * IB * 16, nw = n0 + wn * JB * 16;
    if constexpr (RAW) {
        wait_vm<0>();                                    // drain the copies before the wave ends
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                const int t = tw + i * 16 + l16;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int n = nw + j * 16 + 4 * g + r;
                    if (t < a.T && n < a.N) a.acc[(size_t)t * a.ldacc + n] = acc[i][j][r] >> 8;   // exact: a multiple of 256
                }
            }
        return;
    }

    // first outlier fragments (the last step waited for the first stage)
    const uint32_t rdF = (uint32_t)(l16 * 64 + ((g ^ swz_h(l16)) << 4));
    const uint32_t aF = rdF + wm * IB * 1024, bF = rdF + BM * 64 + wn * JB * 1024;
    v8h ha[4], hb[JB];
    auto read_ha = [&](int i, uint32_t fo) __attribute__((always_inline)) { ha[i & 3] = *reinterpret_cast<const v8h*>(lds + fo + aF + i * 1024); };
    auto read_hb = [&](int j, uint32_t fo) __attribute__((always_inline)) { hb[j] = *reinterpret_cast<const v8h*>(lds + fo + bF + j * 1024); };
    float t_s[IB], t_h[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int lr = wm * IB * 16 + i * 16 + l16;
        t_s[i] = lds_s[lr];                              // scaleAct
        t_h[i] = lds_z[lr] + 8.0f * t_s[i];              // zeroAct + halfRange * scaleAct
    }
    // Dequantization: the accumulators are 256 times the integer dot products (the factor rides on the weight scale); the
    // conversion to binary32 is exact (at most 24 significant bits).
    v4f cf[IB][JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        const int lc = wn * JB * 16 + j * 16 + 4 * g;
        const uint4 sw4 = *reinterpret_cast<const uint4*>(&lds_sw[lc]);
        const float4 wr4 = *reinterpret_cast<const float4*>(&lds_wr[lc]);
        const uint4 bv4 = *reinterpret_cast<const uint4*>(&lds_bv[lc]);
        const float wr_[4] = {wr4.x, wr4.y, wr4.z, wr4.w}, bv_[4] = {h2f(bv4.x), h2f(bv4.y), h2f(bv4.z), h2f(bv4.w)};
        constexpr float k = 1.0f / 256.0f;               // an exact power-of-two factor
        const float sw_[4] = {h2f(sw4.x) * k, h2f(sw4.y) * k, h2f(sw4.z) * k, h2f(sw4.w) * k};
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                cf[i][j][r] = __builtin_fmaf((float)acc[i][j][r], t_s[i] * sw_[r], __builtin_fmaf(t_h[i], wr_[r], bv_[r]));
    }
    if (nkf > 0) {
#pragma unroll
        for (int j = 0; j < JB; ++j) read_hb(j, (uint32_t)at);
        read_ha(0, (uint32_t)at);
        read_ha(1, (uint32_t)at);
        for (int f = 0; f < nkf; ++f) {
            const int nxt = at + FSLOT == RING ? 0 : at + FSLOT;
            const uint32_t fo = (uint32_t)at, fo1 = (uint32_t)nxt;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < SLOTS; ++m) {
                const int i = m / JB, j = m % JB;
                cf[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb[j], ha[i & 3], cf[i][j], 0, 0, 0);
                if (j == 0 && i + 2 < IB) read_ha(i + 2, fo);
                if (m == LAST_READ) {
                    // every read of this stage has been issued: behind the barrier its slot is free, the next has landed
                    wait_stage<(NST - 4) * LPS>();
                    __syncthreads();
#pragma unroll
                    for (int d = 0; d < 2 * LPS; ++d) issue_fp(f + NST / 2, d, at);
                }
                if (j == 0 && i + 2 >= IB) read_ha(i + 2 - IB, fo1);
                if (i == IB - 1) read_hb(j, fo1);
                __builtin_amdgcn_sched_barrier(0);
            }
            at = nxt;
        }
    }
    wait_stage<0>();
    __syncthreads();                                     // the stage memory is dead
    __half* __restrict__ y = static_cast<__half*>(a.y);
    // Output through LDS: a wave parks sixteen rows of its tile, four channels = 8 bytes per lane and write, and writes them
    // out as 16-byte pieces, whole row segments per store; needs 16-byte aligned output rows.
    const bool vec_ok = ((reinterpret_cast<uintptr_t>(a.y) & 15u) == 0) && (a.ldy % 8 == 0);
    if (vec_ok) {
        uint8_t* wbuf = lds + wave * PARK;
        constexpr int CH = JB * 2, RPS = 64 / CH;        // 16-byte pieces per row, rows per store instruction
        const int prow = lane / CH, pch = lane % CH;
#pragma unroll
        for (int i = 0; i < IB; ++i) {
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                uint2 v;
                v.x = __builtin_bit_cast(uint32_t, __floats2half2_rn(cf[i][j][0], cf[i][j][1]));
                v.y = __builtin_bit_cast(uint32_t, __floats2half2_rn(cf[i][j][2], cf[i][j][3]));
                *reinterpret_cast<uint2*>(wbuf + l16 * PARK_ROW + (j * 16 + 4 * g) * 2) = v;
            }
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
            const int t = tw + i * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = nw + j * 16 + 4 * g + r;
                if (t < a.T && n < a.N) y[(size_t)t * a.ldy + n] = __float2half(cf[i][j][r]);
            }
        }
}

// Few tokens: the layer is bound by streaming the weights, so the point is many bytes in flight per CU and many
// workgroups.  A workgroup owns a 32 TM (tokens) x 32 (channels) output tile and its four waves split K: every wave
// streams its own quarter of the panels (1 KB of weights and TM KB of activations each, one DMA instruction per KB)
// through a private ring, with no workgroup barrier in the main loop (a wave waits only for its own DMA), into
// v_smfmac_i32_32x32x64_i8.  The four partial INT32 accumulators are summed exactly through LDS; wave 0 then dequantizes,
// adds the fp16 outlier product (every wave takes every fourth 16-column step, operands straight from global memory,
// requested before the weight stream starts) and stores.
// TM = 2 reads the weights once for 33 to 64 tokens.  It is ahead of 32 x 32 and of the general kernel's 64 x 64 tiles
// where its launch gives the busiest CU two workgroups, or three, and K is deep.  GEMM, us, cached / from HBM,
// 32 x 32 : 64 x 64 : this: T=50 K=5600 N=15968 20.1/20.2 : 17.6/17.8 : 14.7/16.8;  T=44 K=8320 N=10104 19.0/19.2 :
// 23.5/23.7 : 16.6/17.0;  T=39 K=5856 N=10616 16.4/16.5 : 18.3/18.4 : 15.0/15.8;  with fewer workgroups 32 x 32 is ahead
// (T=34 K=8640 N=7616 15.2 : 23.5 : 15.3), with more 64 x 64 (T=60 K=4544 N=29936 28.3 : 17.4 : 25.6).
template <int TM, int NST, int MODE>
__global__ __launch_bounds__(256) void gemm_sp24_split(GemmArgs a) {
    constexpr bool RAW = MODE != 0;
    constexpr int BM = 32 * TM, A_BYTES = BM * 32, ST_BYTES = A_BYTES + 1024, RING = NST * ST_BYTES, LPS = TM + 1;
    constexpr int RED_BYTES = 2 * TM * 16 * 64 * 4;        // one wave's INT32 accumulators + fp32 outlier partials
    constexpr int LDS_BYTES = (4 * RING > 3 * RED_BYTES) ? 4 * RING : 3 * RED_BYTES;
    static_assert((NST - 1) * LPS < 64, "vmcnt range");
    __shared__ __align__(1024) uint8_t lds[LDS_BYTES];
    __shared__ float prm_sw[32], prm_wr[32], prm_bv[32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int tiles_m = (a.T + BM - 1) / BM;
    const int t0 = (blockIdx.x % tiles_m) * BM, n0 = (blockIdx.x / tiles_m) * 32;

    const int nk = sp24::stages(a.K_b);
    const int s_begin = (int)((long)nk * wave / 4), s_end = (int)((long)nk * (wave + 1) / 4);   // this wave's stages
    const uint32_t strideA = (uint32_t)a.T * sp24::kActBytes, strideB = (uint32_t)a.N * sp24::kWgtBytes;
    const v4i rA = make_rsrc((const uint8_t*)a.xq + (size_t)t0 * sp24::kActBytes, (size_t)(a.T - t0) * sp24::kActBytes);
    const v4i rB = make_rsrc((const uint8_t*)a.w_q + (size_t)n0 * sp24::kWgtBytes, (size_t)(a.N - n0) * sp24::kWgtBytes);

    uint8_t* ring = lds + wave * RING;
    const uint32_t ring_addr = lds_addr(ring);
    // 32 rows of 32 bytes per instruction, pieces exchanged in every second group of eight rows
    const uint32_t vo = (uint32_t)((lane >> 1) * 32 + (((lane & 1) ^ ((lane >> 4) & 1)) * 16));
    auto issue = [&](int s) __attribute__((always_inline)) {   // stage s of this wave's range (or beyond: nothing is read)
        const uint32_t sb = (uint32_t)((s - s_begin) % NST) * ST_BYTES;
        const bool live = s < s_end;
        v4i ra = advance(rA, (uint32_t)s * strideA), rb = advance(rB, (uint32_t)s * strideB);
        ra = v4i{__builtin_amdgcn_readfirstlane(ra[0]), __builtin_amdgcn_readfirstlane(ra[1]),
                 __builtin_amdgcn_readfirstlane(ra[2]), __builtin_amdgcn_readfirstlane(ra[3])};
        rb = v4i{__builtin_amdgcn_readfirstlane(rb[0]), __builtin_amdgcn_readfirstlane(rb[1]),
                 __builtin_amdgcn_readfirstlane(rb[2]), __builtin_amdgcn_readfirstlane(rb[3])};
#pragma unroll
        for (int i = 0; i < TM; ++i)
            dma16(ra, (uint32_t)__builtin_amdgcn_readfirstlane((int)(ring_addr + sb + i * 1024)), live ? vo + i * 1024 : kOob, 0);
        dma16(rb, (uint32_t)__builtin_amdgcn_readfirstlane((int)(ring_addr + sb + A_BYTES)), live ? vo : kOob, 0);
    };
    const uint32_t rd = (uint32_t)(l32 * 32 + ((g ^ swz_f(l32)) << 4));   // this lane's piece of its row

    // ---- everything the epilogue needs is requested before the weight stream starts
    constexpr int PF = TM == 1 ? 4 : 2;                    // prefetched outlier steps per wave
    float t_s[TM], t_z[TM];
    uint4 pfa[PF][TM], pfb[PF];
    const int fsteps = (a.n_out + 15) >> 4;                // 16-column steps of the outlier product
    const __half* __restrict__ xo = static_cast<const __half*>(a.x_out);
    const __half* __restrict__ wo = static_cast<const __half*>(a.w_out);
    const int n2 = min(n0 + l32, a.N - 1);
    // this lane's 8 outlier columns from kk on, of its channel and of its token in block i
    auto wgt8 = [&](int kk, bool live) __attribute__((always_inline)) {
        return live ? *reinterpret_cast<const uint4*>(wo + (size_t)n2 * a.ldwo + kk) : make_uint4(0, 0, 0, 0);
    };
    auto act8 = [&](int i, int kk, bool live) __attribute__((always_inline)) {
        const int t2 = min(t0 + i * 32 + l32, a.T - 1);
        return live ? *reinterpret_cast<const uint4*>(xo + (size_t)t2 * a.ldo + kk) : make_uint4(0, 0, 0, 0);
    };
    if constexpr (!RAW) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int t = t0 + i * 32 + l32;
            t_s[i] = t < a.T ? a.scale[t] : 0.0f;
            t_z[i] = t < a.T ? a.zero[t] : 0.0f;
        }
        if (tid < 32) {
            const int n = min(n0 + tid, a.N - 1);
            const __half* __restrict__ wsc = static_cast<const __half*>(a.w_scale);
            const __half* __restrict__ bias = static_cast<const __half*>(a.bias);
            prm_sw[tid] = __half2float(wsc[n]) * (1.0f / 256.0f);   // exact power-of-two factor
            prm_wr[tid] = a.w_reduced[n];
            prm_bv[tid] = bias ? __half2float(bias[n]) : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const int kk = (wave + 4 * q) * 16 + g * 8;    // first of this lane's 8 outlier columns
            const bool live = (wave + 4 * q) < fsteps && kk < a.n_out;
#pragma unroll
            for (int i = 0; i < TM; ++i) pfa[q][i] = act8(i, kk, live);
            pfb[q] = wgt8(kk, live);
        }
    }

    v16i acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;

#pragma unroll
    for (int s = 0; s < NST - 1; ++s) issue(s_begin + s);
    for (int s = s_begin; s < s_end; ++s) {
        issue(s + NST - 1);
        wait_vm<(NST - 1) * LPS>();                        // stage s has landed (this wave's own loads)
        const uint8_t* st = ring + ((s - s_begin) % NST) * ST_BYTES;
        constexpr uint32_t M = 0xF0F0F0F0u;
        const uint4 ww = *reinterpret_cast<const uint4*>(st + A_BYTES + rd);
        const v4i uw = v4i{(int)((ww.x << 4) & M), (int)(ww.x & M), (int)((ww.y << 4) & M), (int)(ww.y & M)};
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint4 wa = *reinterpret_cast<const uint4*>(st + i * 1024 + rd);
            const v8i ua = v8i{(int)(wa.x & M), (int)((wa.x << 4) & M), (int)(wa.y & M), (int)((wa.y << 4) & M),
                               (int)(wa.z & M), (int)((wa.z << 4) & M), (int)(wa.w & M), (int)((wa.w << 4) & M)};
            acc[i] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(uw, ua, acc[i], (int)ww.z, 0, 0);
        }
        // the buffer read here is refilled NST - 1 iterations later by this same wave: the LDS reads above
        // have returned (their data fed the matrix instructions) before that DMA is issued
    }
    wait_vm<0>();

    // ---- this wave's share of the fp16 outlier product (weights first: same accumulator layout)
    v16f cf[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) cf[i][r] = 0.0f;
    if constexpr (!RAW) {
        auto fp_step = [&](uint4 fb, uint4 fa, int i) __attribute__((always_inline)) {
            cf[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, fb), __builtin_bit_cast(v8h, fa), cf[i], 0, 0, 0);
        };
#pragma unroll
        for (int q = 0; q < PF; ++q)
#pragma unroll
            for (int i = 0; i < TM; ++i) fp_step(pfb[q], pfa[q][i], i);
        for (int stp = wave + 4 * PF; stp < fsteps; stp += 4) {     // the outlier columns beyond the prefetched ones
            const int kk = stp * 16 + g * 8;
            const uint4 fb = wgt8(kk, kk < a.n_out);
#pragma unroll
            for (int i = 0; i < TM; ++i) fp_step(fb, act8(i, kk, kk < a.n_out), i);
        }
    }
    __syncthreads();                                       // rings are dead: reuse LDS for the reduction

    // ---- sum the four partial results: waves 1..3 publish, wave 0 adds (INT32 exactly; the fp32 outlier
    // partials in wave order)
    int* red = reinterpret_cast<int*>(lds);
    float* redf = reinterpret_cast<float*>(lds) + 3 * TM * 16 * 64;
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int slot = (((wave - 1) * TM + i) * 16 + r) * 64 + lane;
                red[slot] = acc[i][r];
                if constexpr (!RAW) redf[slot] = cf[i][r];
            }
    }
    __syncthreads();
    if (wave > 0) return;
    // one block: all 96 loads at once, 0.5 us faster than one partial result after the other, at 60 registers; two blocks:
    // one after the other, all at once would halve the occupancy
    constexpr int AT_ONCE = TM == 1 ? 3 : 1;
#pragma unroll AT_ONCE
    for (int w = 0; w < 3; ++w)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int slot = ((w * TM + i) * 16 + r) * 64 + lane;
                acc[i][r] += red[slot];
                if constexpr (!RAW) cf[i][r] += redf[slot];
            }

    // lane: token t0 + 32 i + l32; register r: channel n0 + 8 (r / 4) + 4 g + r % 4
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int t = t0 + i * 32 + l32;
        if constexpr (RAW) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int n = n0 + 8 * (r >> 2) + 4 * g + (r & 3);
                if (t < a.T && n < a.N) a.acc[(size_t)t * a.ldacc + n] = acc[i][r] >> 8;   // exact: a multiple of 256
            }
        } else {
            __half* __restrict__ y = static_cast<__half*>(a.y);
            const float t_h = t_z[i] + 8.0f * t_s[i];      // zeroAct + halfRange * scaleAct
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = 8 * (r >> 2) + 4 * g + (r & 3), n = n0 + c;
                const float v = __builtin_fmaf((float)acc[i][r], t_s[i] * prm_sw[c], __builtin_fmaf(t_h, prm_wr[c], prm_bv[c])) + cf[i][r];
                if (t < a.T && n < a.N) y[(size_t)t * a.ldy + n] = __float2half(v);
            }
        }
    }
}

// Signed 4-bit weights (two per byte, column 2p in the low nibble) -> the weight format of
// quik_sp24_device.h.  One thread per (row, stage).  A group of four with more than two nonzero values
// is counted in *violations (if not null) and keeps its first two.  Offline step.
__global__ __launch_bounds__(256) void weight_pack_sp24_kernel(const uint8_t* __restrict__ w_q, int ldw, int N, int K_b,
                                                               uint32_t* __restrict__ w24, int* __restrict__ violations) {
    const int S = sp24::stages(K_b);
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)N * S) return;
    const int n = (int)(idx / S), s = (int)(idx % S);
    const uint8_t* src = w_q + (size_t)n * ldw + s * 32;
    uint64_t vals[2] = {0, 0};
    uint32_t ind[2] = {0, 0};
    int bad = 0;
    for (int kappa = 0; kappa < 16; ++kappa) {
        int v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int col = s * 64 + kappa * 4 + p;
            int nib = 0;
            if (col < K_b) {
                const uint32_t byte = src[(kappa * 4 + p) >> 1];
                nib = (int)((p & 1) ? (byte >> 4) : (byte & 0xFu));
            }
            v[p] = nib;                                   // two's complement nibble; 0 = value 0
        }
        // kept positions: the nonzero ones (at most two count), then the lowest unused ones, ascending
        int keep[2], nk = 0, nz = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (v[p] != 0) { if (nk < 2) keep[nk++] = p; ++nz; }
        if (nz > 2) ++bad;
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (nk < 2 && v[p] == 0) keep[nk++] = p;
        if (keep[0] > keep[1]) { const int tmp = keep[0]; keep[0] = keep[1]; keep[1] = tmp; }
        const int hg = sp24::half_of_group(kappa), q = sp24::pair_of_group(kappa);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int c = 2 * q + e;
            const int bit = 32 * (c >> 3) + 8 * (c & 3) + 4 * ((c >> 2) & 1);
            vals[hg] |= (uint64_t)(uint32_t)v[keep[e]] << bit;
            ind[hg] |= (uint32_t)keep[e] << (2 * c);
        }
    }
    uint4* blk = reinterpret_cast<uint4*>(w24) + ((size_t)s * N + n) * 2;
    blk[0] = make_uint4((uint32_t)vals[0], (uint32_t)(vals[0] >> 32), ind[0], 0u);
    blk[1] = make_uint4((uint32_t)vals[1], (uint32_t)(vals[1] >> 32), ind[1], 0u);
    if (bad && violations) atomicAdd(violations, bad);
}

template <int IB, int JB, int WM, int WN, int NST, int OCC, int GM, int MODE>
hipError_t launch_cfg(const GemmArgs& a, hipStream_t stream) {
    constexpr int BM = WM * IB * 16, BN = WN * JB * 16;
    const int tiles = ((a.T + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    hipLaunchKernelGGL((gemm_sp24_kernel<IB, JB, WM, WN, NST, OCC, GM, MODE>), dim3(tiles), dim3(WM * WN * 64), 0, stream, a);
    return hipGetLastError();
}

// The tile whose launch is estimated to be the shortest, up to `occ` workgroups of it per CU: base + round * rounds +
// tile * tiles of the busiest CU + steps * (round_step * rounds + tile_step * tiles of the busiest CU), an outlier stage
// counting as half a step.  Fitted to 976 shapes with all or most tiles measured (T 1 .. 4096, K 512 .. 11008, N 512 ..
// 28672, cached weights and from HBM, mean of both), those with output rows of whole 16-byte pieces counted threefold; the
// choice costs 0.3 % against the fastest tile in the mean.  A fit to fewer shapes of few tokens gave them 64 x 64 tiles
// where the K-split kernel is ahead (us, cached / from HBM: T=8 K=1376 N=8720 7.4/7.7, now 6.2/6.6; T=48 K=3296 N=8448
// 11.9/12.3, now 9.0/10.7), and took 256 x 192 tiles for T=2048 K=4096 N=11008 (68.1/70.7, now 128 x 256 with 64.9/68.8) and
// 128 x 128 ones for T=2048 K=11008 N=4096 (65.6/65.1, now 60.7/63.3).
// The first entry is the K-split kernel: it wins up to 64 tokens nearly always; beyond 256 its line does not hold.  The
// last one is its 64-token form, for the tokens that it reads the weights once for and two or three workgroups on the
// busiest CU: with one 32 x 32 is ahead, with more 64 x 64 (T=60 K=13312 N=26626 40.9/44.6 with 64 x 64, 46.8/64.2 with it).
// The 64 x 64 tile is left out beyond two rounds of it: the fit holds for cached operands, from HBM it fetches them too
// often there (T = 920, N = 21928, K = 576: 52 us, 128 x 256 27).
struct TileCost24 { int bm, bn, waves, occ; double base, round, tile, round_step, tile_step; };
constexpr TileCost24 kCost24[] = {{32, 32, 4, 3, 2.727, 1.520, 0.415, 0.024, 0.061},
                                  {64, 64, 4, 4, 3.614, -0.131, 0.752, 0.235, 0.060},
                                  {128, 128, 8, 2, 2.775, 1.632, 1.210, 0.091, 0.282},
                                  {128, 192, 8, 1, 0.530, 7.213, 0, 0.468, 0},
                                  {256, 192, 8, 1, 2.246, 8.223, 0, 0.671, 0},
                                  {128, 256, 4, 2, 4.382, 4.385, 1.162, 0.196, 0.324},
                                  {128, 192, 4, 2, 4.342, 4.285, 0.973, 0.288, 0.228},
                                  {128, 128, 4, 2, 2.660, 3.109, 0.655, 0.235, 0.161},
                                  {64, 32, 4, 3, 0.1, 0, 4.3, -0.011, 0.072}};
constexpr int kSplitTokens = 256;

int choose_tile_sp24(int T, int N, int K_b, int n_out, int cus) {
    const double steps = (K_b + 127) / 128 + 0.5 * ((n_out + 31) / 32);
    int best = -1;
    double least = 0.0;
    for (int i = 0; i < (int)(sizeof(kCost24) / sizeof(TileCost24)); ++i) {
        const TileCost24& c = kCost24[i];
        const long tiles = (long)((T + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const long rounds = (tiles + (long)c.occ * cus - 1) / ((long)c.occ * cus), busiest = (tiles + cus - 1) / cus;
        if ((i == 0 && T > kSplitTokens) || (i == 1 && rounds > 2)) continue;
        if (i == 8 && (T <= 32 || T > 64 || busiest < 2 || busiest > 3)) continue;
        const double t = c.base + c.round * rounds + c.tile * busiest + steps * (c.round_step * rounds + c.tile_step * busiest);
        if (best < 0 || t < least) { best = i; least = t; }
    }
    return best;
}

template <int MODE>
hipError_t dispatch24(const GemmArgs& a, hipStream_t stream) {
    int cus = compute_units();
    if (cus < 1) cus = 256;
    switch (choose_tile_sp24(a.T, a.N, a.K_b, MODE ? 0 : a.n_out, cus)) {
    case 0:
        // (ring depth: 4 and 6 measured alike, 8 to 16 up to 15 % slower)
        hipLaunchKernelGGL((gemm_sp24_split<1, 4, MODE>), dim3(((a.T + 31) / 32) * ((a.N + 31) / 32)), dim3(256), 0, stream, a);
        return hipGetLastError();
    case 1: return launch_cfg<4, 1, 1, 4, 8, 4, 8, MODE>(a, stream);
    case 2: return launch_cfg<4, 2, 2, 4, 6, 2, 8, MODE>(a, stream);
    case 3: return launch_cfg<4, 3, 2, 4, 8, 1, 8, MODE>(a, stream);
    case 4: return launch_cfg<4, 6, 4, 2, 6, 1, 8, MODE>(a, stream);
    case 5: return launch_cfg<4, 8, 2, 2, 6, 2, 8, MODE>(a, stream);
    case 6: return launch_cfg<4, 6, 2, 2, 6, 2, 8, MODE>(a, stream);
    case 7: return launch_cfg<4, 4, 2, 2, 8, 2, 8, MODE>(a, stream);
    default:
        hipLaunchKernelGGL((gemm_sp24_split<2, 4, MODE>), dim3(((a.T + 63) / 64) * ((a.N + 31) / 32)), dim3(256), 0, stream, a);
        return hipGetLastError();
    }
}

}  // namespace

void sp24_form(int T, int N, int K_b, int n_out, int cus, int* form) {
    const TileCost24& c = kCost24[choose_tile_sp24(T, N, K_b, n_out, cus)];
    form[0] = c.bm;
    form[1] = c.bn;
    form[2] = c.waves;
}

hipError_t launch_gemm_sp24(const GemmArgs& a, hipStream_t stream) {
    if (a.T <= 0 || a.N <= 0) return hipSuccess;
    return a.y ? dispatch24<0>(a, stream) : dispatch24<1>(a, stream);
}

hipError_t launch_weight_pack_sp24(const void* w_q, int ldw, int N, int K_b, void* w24, int* violations,
                                   hipStream_t stream) {
    if (N <= 0 || K_b <= 0) return hipSuccess;
    const long total = (long)N * sp24::stages(K_b);
    hipLaunchKernelGGL(weight_pack_sp24_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const uint8_t*>(w_q), ldw, N, K_b, static_cast<uint32_t*>(w24), violations);
    return hipGetLastError();
}

}  // namespace quik
