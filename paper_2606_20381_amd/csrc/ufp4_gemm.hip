// Block-scaled 4-bit NT GEMM on CDNA4 matrix cores (Sec. 2.2: Y_hat = Q(XH') Q(WH')^T; the three training
// GEMMs fwd_y, bwd_dx, bwd_dw all take this form once both operands are stored reduction-contiguous).
//
//   C[i, j] = sum_b  sA[i,b] * sB[j,b] * D_b[i, j],   D_b[i, j] = sum_{k in block b} A[i,k] * B[j,k]
//
// Every 16-element K-block has its own fp32 scale on both sides, so D_b is formed per block by one MFMA with
// K = 16 (the codes of either grid made exact fp8 numbers) and folded into an fp32 accumulator with the scale
// product of the block: acc += D_b * (sA * sB). The design is described at gemm_f32_kernel.
//
// Grouped (MoE) problems: ragged M (fwd_y, bwd_dx: token rows split into groups) resolves its group
// from the tile index with a wave-wide prefix sum over the group sizes; ragged K (bwd_dw: the reduction
// runs over each group's padded token range) takes the group from the grid's z index.

#include "ufp4_device.h"
#include "ufp4_internal.h"

#include <math.h>

namespace ufp4 {

// Tile configuration of gemm_f32_kernel: WM x WN x WK waves. A wave owns WTM x WTN MFMA tiles of 32 x 32 outputs, its
// row (column) tiles WM (WN) tiles apart; the WK wave groups split every stage's K-blocks between them and add their
// partial sums through LDS at the end. A stage holds SKB blocks per group.
template <int WTM_, int WTN_, int WM_, int WN_, int WK_, int SKB_>
struct TileCfg {
    static constexpr int WTM = WTM_, WTN = WTN_, WM = WM_, WN = WN_, WK = WK_, SKB = SKB_;
    static constexpr int BM = 32 * WTM * WM, BN = 32 * WTN * WN;
    static constexpr int kWaves = WM * WN * WK, kThreads = 64 * kWaves;
    static constexpr int kStageBlocks = SKB * WK;
    // staging units (64 rows of one block) of A and B in a stage, dealt round robin to the waves
    static constexpr int kUnitsA = kStageBlocks * BM / 64, kUnitsB = kStageBlocks * BN / 64;
    static_assert(BM % 64 == 0 && BN % 64 == 0, "a staging unit lies in one operand");
    static_assert(kUnitsA == kWaves && kUnitsB <= kWaves, "one unit of A and at most one of B per wave and stage");
};

// Offsets of (row, block) in the panel layout, the row counted from a tile's first row (row0 within its panel).
__device__ __forceinline__ int64_t code_off(int row0, int row, int64_t kb, int64_t pld) {
    const int r = row0 + row;
    return (int64_t)(r / kPanelRows) * pld + kb * kPanelBlockBytes + (int64_t)(r % kPanelRows) * 8;
}
__device__ __forceinline__ int64_t scale_off(int row0, int row, int64_t kb, int64_t pld) {
    const int r = row0 + row;
    return (int64_t)(r / kPanelRows) * pld + kb * kPanelBlockScales + (r % kPanelRows);
}
struct GemmArgs {
    GemmJob j;
};

// The problem one workgroup works on, with pointers already advanced to its tile / group.
// A workgroup's operand tiles. Operands are in the panel layout (panels of 128 rows, block b of a panel at
// b * 1024 bytes / b * 128 floats); a/as (b/bs) point at the panel holding the tile's first row, already
// advanced to the tile's first K-block, and a_row0 (b_row0) is that row's index within its panel (nonzero
// only for ragged-M groups, whose tiles start anywhere).
struct Tile {
    const uint8_t* a;
    const float* as;
    const uint8_t* b;
    const float* bs;
    int a_row0, b_row0;
    int mrows, nrows;  // valid rows of the tile in A and B
    int64_t nkb;       // reduction blocks
    int64_t c_off;     // element offset of the tile's (0, 0) in C
};

// Ragged-M: find the group owning global m-tile t. Wave 0 runs a prefix sum over per-group tile counts,
// 64 groups at a time; the result goes through LDS. Returns false for tiles past the last group.
template <int BM>
__device__ bool resolve_ragged_m(const GemmJob& j, int32_t* grp, int64_t t, int& g_out, int64_t& local_tile) {
    const int tid = threadIdx.x;
    if (tid == 0) grp[0] = -1;
    __syncthreads();
    if (tid < 64) {
        int64_t base = 0;
        for (int g0 = 0; g0 < j.G; g0 += 64) {
            const int g = g0 + tid;
            int64_t cnt = 0;
            if (g < j.G) cnt = (j.offsets[g + 1] - j.offsets[g] + BM - 1) / BM;
            if (cnt < 0) cnt = 0;  // offsets that decrease: an empty group
            int64_t incl = cnt;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t v = __shfl_up(incl, d, 64);
                if (tid >= d) incl += v;
            }
            const int64_t excl = incl - cnt;
            if (cnt > 0 && base + excl <= t && t < base + incl) {
                grp[0] = g;
                grp[1] = (int32_t)(t - base - excl);
            }
            base += __shfl(incl, 63, 64);
        }
    }
    __syncthreads();
    g_out = grp[0];
    local_tile = grp[1];
    return g_out >= 0;
}

// Grid position of a workgroup: tile column, tile row (ragged-M: global m-tile index) and group (ragged-K).
struct TilePos {
    int64_t tn, tm;
    int g;
};

// Workgroups are dealt to the 8 XCDs round robin (linear index L to XCD L % 8), each XCD with its own L2. On a
// single-problem grid the first 8 * floor(T / 8) workgroups are renumbered so that XCD k gets the contiguous
// range of tiles [k T/8, (k + 1) T/8); tiles are ordered in bands of kBandRows tile rows, column by column
// within a band, so the workgroups resident on one XCD share a few panels of A and of B instead of every XCD
// streaming every panel. The map is a bijection of the grid, so every tile is still computed exactly once.
constexpr int64_t kBandRows = 8;
__device__ __forceinline__ TilePos grid_pos() {
    if (gridDim.z != 1 || gridDim.y == 1) return {(int64_t)blockIdx.x, (int64_t)blockIdx.y, (int)blockIdx.z};
    const int64_t gx = gridDim.x, gy = gridDim.y, T = gx * gy, per = T / 8;
    const int64_t L = (int64_t)blockIdx.y * gx + blockIdx.x;
    const int64_t t = L < 8 * per ? (L % 8) * per + L / 8 : L;
    const int64_t band = t / (kBandRows * gx);
    const int64_t first = band * kBandRows;
    const int64_t rows = gy - first < kBandRows ? gy - first : kBandRows;
    const int64_t r = t - band * kBandRows * gx;
    return {r / rows, first + r % rows, 0};
}

// Padded start of group g along a ragged-K reduction: sum over h < g of the token counts rounded up to multiples
// of 16 (each group's tokens were zero-padded so; ufp4_quantize_grouped_t lays them out the same way). Wave 0
// sums, the result goes through LDS; every thread of the workgroup must call this.
__device__ int64_t padded_start(const int64_t* off, int g, int64_t* slot) {
    const int tid = threadIdx.x;
    if (tid < 64) {
        int64_t sum = 0;
        for (int h = tid; h < g; h += 64) {
            const int64_t c = off[h + 1] - off[h];
            sum += (c > 0 ? c + 15 : 0) / 16 * 16;
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if (tid == 0) *slot = sum;
    }
    __syncthreads();
    return *slot;
}

// Resolve the workgroup's output tile (dense, ragged-M group or ragged-K group). Returns false when the
// workgroup has nothing to do (a ragged-M tile index past the last group); all threads agree.
template <int BM, int BN>
__device__ bool resolve_tile(const GemmJob& j, int32_t* grp, int64_t* pad, const TilePos& pos, Tile& tl) {
    const int64_t tn = pos.tn;
    if (j.mode == kGemmRaggedM) {
        int g;
        int64_t lt;
        if (!resolve_ragged_m<BM>(j, grp, pos.tm, g, lt)) return false;
        const int64_t r0 = j.offsets[g] + lt * BM;
        const int64_t end = j.offsets[g + 1] < j.M ? j.offsets[g + 1] : j.M;  // offsets past M_total: ignored
        const int64_t rows_g = end - r0;
        if (rows_g <= 0) return false;
        tl.a = j.a + (r0 / kPanelRows) * j.a_pld;
        tl.as = j.as + (r0 / kPanelRows) * j.as_pld;
        tl.a_row0 = (int)(r0 % kPanelRows);
        const int64_t brow = g * j.b_group_rows + tn * BN;
        const int64_t bkb = g * j.b_group_kb;
        tl.b = j.b + (brow / kPanelRows) * j.b_pld + bkb * kPanelBlockBytes;
        tl.bs = j.bs + (brow / kPanelRows) * j.bs_pld + bkb * kPanelBlockScales;
        tl.b_row0 = (int)(brow % kPanelRows);
        tl.mrows = (int)(rows_g < BM ? rows_g : BM);
        const int64_t nr = j.N - tn * BN;
        tl.nrows = (int)(nr < BN ? nr : BN);
        tl.nkb = j.nkb;
        tl.c_off = r0 * j.ldc + tn * BN;
    } else {
        const int64_t tm = pos.tm;
        int64_t kb0 = 0, c_base = 0;
        tl.nkb = j.nkb;
        if (j.mode == kGemmRaggedK) {
            const int g = pos.g;
            // the group's padded token range, clamped to the operands' reduction length
            const int64_t c = j.offsets[g + 1] - j.offsets[g];
            const int64_t q0 = padded_start(j.offsets, g, pad);
            const int64_t q1 = q0 + (c > 0 ? c + 15 : 0) / 16 * 16;
            const int64_t p0 = q0 < j.red_total ? q0 : j.red_total;
            const int64_t p1 = q1 < j.red_total ? q1 : j.red_total;
            kb0 = p0 / 16;
            tl.nkb = p1 > p0 ? (p1 - p0) / 16 : 0;
            c_base = (int64_t)g * j.M * j.ldc;
        }
        // BM and BN divide the panel's 128 rows: a tile lies in one panel
        const int64_t pa = tm * BM / kPanelRows, pb = tn * BN / kPanelRows;
        tl.a = j.a + pa * j.a_pld + kb0 * kPanelBlockBytes;
        tl.as = j.as + pa * j.as_pld + kb0 * kPanelBlockScales;
        tl.b = j.b + pb * j.b_pld + kb0 * kPanelBlockBytes;
        tl.bs = j.bs + pb * j.bs_pld + kb0 * kPanelBlockScales;
        tl.a_row0 = (int)(tm * BM % kPanelRows);
        tl.b_row0 = (int)(tn * BN % kPanelRows);
        const int64_t mr = j.M - tm * BM, nr = j.N - tn * BN;
        tl.mrows = (int)(mr < BM ? mr : BM);
        tl.nrows = (int)(nr < BN ? nr : BN);
        tl.c_off = c_base + tm * BM * j.ldc + tn * BN;
    }

    return true;
}

// ================================================================================================
// The kernel.
//
// The per-block dot product D_b comes out of an MFMA already in fp32 and a second MFMA forms the outer
// product sA[:, b] x sB[:, b] in the same register layout, so the VALU does one FMA per output and block:
// acc += D_b * (sA sB)_b.
//
//  * D_b: the codes become fp8 e4m3 numbers while a stage is copied into LDS and go through
//    v_mfma_f32_32x32x16_fp8_fp8 (K = 16, one block): uniform code k -> the subnormal k * 2^-9, E2M1 level
//    -> the same value as an e4m3 normal (every level 0, 0.5, ..., 6 is one); both exact, so D_b is exact.
//  * (sA sB)_b: every fp32 scale is split exactly into three bf16 pieces s = s0 + s1 + s2 (top, middle and
//    low 8 significand bits) when staged, and stored directly as the operand of a v_mfma_f32_32x32x8_bf16
//    whose 8 K slots hold eight of the nine piece products (all but s2 * s2', below 2^-30 sA sB). Products
//    of two 8-bit significands are exact in fp32, so the MFMA returns sA sB up to fp32 accumulation
//    rounding. The bf16 MFMA co-executes with the VALU FMAs; an fp32 MFMA would not.
//  * Staging: global reads are buffer loads (out-of-range rows read as zero, so no branches) issued two
//    stages ahead into registers; the conversions happen once per workgroup when a stage is written to LDS.
// ================================================================================================

typedef float v16f __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));


// 8 uniform codes (one packed dword of sign-magnitude nibbles) -> 8 fp8 e4m3 bytes. The byte s000 0mmm is an
// e4m3 subnormal worth (-1)^s * m * 2^-9, so the code k becomes k * 2^-9 exactly (the product of two codes
// carries 2^-18, undone once at the store). Even codes go to the low dword, odd codes to the high one; both
// operands use the same order, so the K-slot permutation cancels in the dot product.
__device__ __forceinline__ uint2 uniform_to_e4m3(uint32_t d) {
    const uint32_t lo = (d & 0x07070707u) | ((d << 4) & 0x80808080u);
    const uint32_t hi = ((d >> 4) & 0x07070707u) | (d & 0x80808080u);
    return make_uint2(lo, hi);
}

// 8 E2M1 codes (sign-magnitude nibbles, magnitude = index of 0, 0.5, 1, 1.5, 2, 3, 4, 6) -> 8 fp8 e4m3 bytes of
// the same values: a byte-select table (v_perm_b32 picks byte m of {0x4C484440, 0x3C383000} for magnitude m:
// 0x00 0x30 0x38 0x3C 0x40 0x44 0x48 0x4C = 0, 0.5, 1, 1.5, 2, 3, 4, 6 in e4m3) and the sign in bit 7; even and
// odd codes split as for the uniform grid.
__device__ __forceinline__ uint2 e2m1_to_e4m3(uint32_t d) {
    const uint32_t lo = __builtin_amdgcn_perm(0x4C484440u, 0x3C383000u, d & 0x07070707u) | ((d << 4) & 0x80808080u);
    const uint32_t hi = __builtin_amdgcn_perm(0x4C484440u, 0x3C383000u, (d >> 4) & 0x07070707u) | (d & 0x80808080u);
    return make_uint2(lo, hi);
}

// Exact split x = p0 + p1 + p2 into three bf16 values, each returned in the top half of a dword (low half
// zero): truncations of the top, middle and low 8 significand bits; both differences are exact in fp32.
__device__ __forceinline__ void split_bf16x3(float x, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    p0 = __float_as_uint(x) & 0xFFFF0000u;
    const float r1 = x - __uint_as_float(p0);
    p1 = __float_as_uint(r1) & 0xFFFF0000u;
    p2 = __float_as_uint(r1 - __uint_as_float(p1));
}

// {lo: bf16 of x, hi: bf16 of y} from two split pieces
__device__ __forceinline__ uint32_t bf16_pair(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x07060302u); }

// Outer-product operands of one (row, block) scale. K slots 0-3 (lanes 0-31) and 4-7 (lanes 32-63) hold
//   A side: a0 a0 a0 a1 | a1 a1 a2 a2        B side: b0 b1 b2 b0 | b1 b2 b0 b1
// so the eight slot products are a0b0 a0b1 a0b2 a1b0 a1b1 a1b2 a2b0 a2b1.
struct ScaleOp {
    uint2 h0, h1;
};
__device__ __forceinline__ ScaleOp scale_op_a(float s) {
    uint32_t p0, p1, p2;
    split_bf16x3(s, p0, p1, p2);
    return {make_uint2(bf16_pair(p0, p0), bf16_pair(p0, p1)), make_uint2(bf16_pair(p1, p1), bf16_pair(p2, p2))};
}
__device__ __forceinline__ ScaleOp scale_op_b(float s) {
    uint32_t p0, p1, p2;
    split_bf16x3(s, p0, p1, p2);
    const uint32_t q01 = bf16_pair(p0, p1);
    return {make_uint2(q01, bf16_pair(p2, p0)), make_uint2(bf16_pair(p1, p2), q01)};
}

template <class C>
struct alignas(16) GemmStageSmem {
    // plane (block * 2 + half) holds one 8-byte entry per row: codes (8 e4m3 bytes) and outer-product scale operands
    uint2 a[2][C::kStageBlocks * 2][C::BM];
    uint2 b[2][C::kStageBlocks * 2][C::BN];
    uint2 as[2][C::kStageBlocks * 2][C::BM];
    uint2 bs[2][C::kStageBlocks * 2][C::BN];
};
template <class C>
struct GemmSmem {
    union {
        GemmStageSmem<C> st;
        // partial sums exchanged between the two wave groups: [group][wave of the group][half of the wave's
        // accumulators][lane]
        float part[C::WK > 1 ? 2 : 1][C::WM * C::WN][8 * C::WTM * C::WTN][64];
    };
    int32_t grp[2];
    int64_t pad;
};

// D_b of one 32 x 32 tile from the e4m3 bytes of a block (8 per lane: its K-half of the 16 codes).
__device__ __forceinline__ v16f block_dot(uint2 a, uint2 b) {
    const v16f z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    const long av = (long)(((uint64_t)a.y << 32) | a.x);
    const long bv = (long)(((uint64_t)b.y << 32) | b.x);
    return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(av, bv, z, 0, 0, 0);
}

__device__ __forceinline__ v16f scale_outer(uint2 a, uint2 b) {
    const v16f z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(v4s, a), __builtin_bit_cast(v4s, b), z, 0, 0,
                                                     0);
}

// Wave-uniform copies (SGPRs) of values the compiler cannot prove uniform, e.g. those read back from LDS.
__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    const uint64_t u = (uint64_t)v;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
    return reinterpret_cast<const T*>(uniform_i64((int64_t)(uintptr_t)p));
}

// Raw buffer resource over `bytes` bytes from `base`: loads at offsets past the end return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// One staging unit held by one lane: the codes and the scale of one (row, block).
struct Unit {
    uint2 c;
    uint32_t s;
};

// Work split (Tile128): 8 waves per 128 x 128 tile; wave (wm, wn) owns two 32 x 32 MFMA tiles. At <= 128 VGPRs two
// workgroups share a CU (four waves per SIMD), which is what lets MFMAs and VALU FMAs of different waves overlap: a
// single wave issues neither back to back.
template <int FMT, int OUT, class C>
__global__ __launch_bounds__(C::kThreads, 4) void gemm_f32_kernel(GemmArgs args) {
    __shared__ GemmSmem<C> sm;
    const GemmJob& j = args.j;
    const int tid = threadIdx.x;
    constexpr int BM = C::BM, BN = C::BN;

    Tile tl;
    if (!resolve_tile<BM, BN>(j, sm.grp, &sm.pad, grid_pos(), tl)) return;
    // the buffer resources below must live in SGPRs
    tl.a = uniform_ptr(tl.a);
    tl.b = uniform_ptr(tl.b);
    tl.as = uniform_ptr(tl.as);
    tl.bs = uniform_ptr(tl.bs);
    tl.a_row0 = __builtin_amdgcn_readfirstlane(tl.a_row0);
    tl.b_row0 = __builtin_amdgcn_readfirstlane(tl.b_row0);
    tl.mrows = __builtin_amdgcn_readfirstlane(tl.mrows);
    tl.nrows = __builtin_amdgcn_readfirstlane(tl.nrows);
    // 32-bit stage counters keep the loop (and the buffer loads' stage offsets) on the scalar unit
    const int nkb = __builtin_amdgcn_readfirstlane((int)tl.nkb);

    const int lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (C::WM * C::WN), wt = wave % (C::WM * C::WN);  // K group, tile of the wave
    const int wm = wt / C::WN, wn = wt % C::WN;
    // a wave whose outputs all lie past the problem's edge only helps staging
    const bool live = wm * 32 < tl.mrows && wn * 32 < tl.nrows;

    float acc[C::WTM][C::WTN][16];
#pragma unroll
    for (int a = 0; a < C::WTM; ++a)
#pragma unroll
        for (int b = 0; b < C::WTN; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    // Staging: in every stage wave w fetches unit w of A and (w < kUnitsB) unit w of B, a unit being 64 rows of one
    // block, i.e. contiguous runs of the panel layout. The resources end at the last valid byte of the tile, and a
    // block past the reduction gets an empty one: rows past the tile's last panel and blocks past the end read zeros.
    const int arow = (wave % (BM / 64)) * 64 + lane, ablk = wave / (BM / 64);
    const int brow = (wave % (BN / 64)) * 64 + lane, bblk = wave / (BN / 64);
    const bool has_b = C::kUnitsB == C::kWaves || wave < C::kUnitsB;
    const int64_t a_last = (tl.a_row0 + tl.mrows - 1) / kPanelRows, b_last = (tl.b_row0 + tl.nrows - 1) / kPanelRows;
    const int a_cbytes = (int)(a_last * j.a_pld + (int64_t)nkb * kPanelBlockBytes);
    const int a_sbytes = (int)((a_last * j.as_pld + (int64_t)nkb * kPanelBlockScales) * 4);
    const int b_cbytes = (int)(b_last * j.b_pld + (int64_t)nkb * kPanelBlockBytes);
    const int b_sbytes = (int)((b_last * j.bs_pld + (int64_t)nkb * kPanelBlockScales) * 4);
    const int voca = (int)code_off(tl.a_row0, arow, ablk, j.a_pld), vosa = (int)scale_off(tl.a_row0, arow, ablk, j.as_pld) * 4;
    const int vocb = (int)code_off(tl.b_row0, brow, bblk, j.b_pld), vosb = (int)scale_off(tl.b_row0, brow, bblk, j.bs_pld) * 4;

    auto fetch = [&](Unit& u, const uint8_t* cb, const float* sb, int cbytes, int sbytes, int voc, int vos, int blk, int s) {
        const int b0 = s * C::kStageBlocks;
        const bool in = b0 + blk < nkb;
        const int soc = __builtin_amdgcn_readfirstlane(b0 * (int)kPanelBlockBytes);
        const int sos = __builtin_amdgcn_readfirstlane(b0 * (int)kPanelBlockScales * 4);
        u.c = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(make_rsrc(cb, in ? cbytes : 0), voc, soc, 0));
        u.s = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(sb, in ? sbytes : 0), vos, sos, 0);
    };
    auto load = [&](Unit& a, Unit& b, int s) {
        fetch(a, tl.a, tl.as, a_cbytes, a_sbytes, voca, vosa, ablk, s);
        if (has_b) fetch(b, tl.b, tl.bs, b_cbytes, b_sbytes, vocb, vosb, bblk, s);
    };
    auto conv = [](uint32_t d) -> uint2 {
        if constexpr (FMT == kFmtUniform) return uniform_to_e4m3(d);
        else return e2m1_to_e4m3(d);
    };
    auto put_a = [&](int buf, const Unit& u) {
        sm.st.a[buf][2 * ablk][arow] = conv(u.c.x);
        sm.st.a[buf][2 * ablk + 1][arow] = conv(u.c.y);
        const ScaleOp o = scale_op_a(__uint_as_float(u.s));
        sm.st.as[buf][2 * ablk][arow] = o.h0;
        sm.st.as[buf][2 * ablk + 1][arow] = o.h1;
    };
    auto put_b = [&](int buf, const Unit& u) {
        if (!has_b) return;
        sm.st.b[buf][2 * bblk][brow] = conv(u.c.x);
        sm.st.b[buf][2 * bblk + 1][brow] = conv(u.c.y);
        const ScaleOp o = scale_op_b(__uint_as_float(u.s));
        sm.st.bs[buf][2 * bblk][brow] = o.h0;
        sm.st.bs[buf][2 * bblk + 1][brow] = o.h1;
    };
    auto block = [&](int buf, int kb) {
        const int pl = (C::SKB * wk + kb) * 2 + h;
#pragma unroll
        for (int b = 0; b < C::WTN; ++b) {
            const int col = (b * C::WN + wn) * 32 + l32;
            const uint2 bc = sm.st.b[buf][pl][col], bw = sm.st.bs[buf][pl][col];
#pragma unroll
            for (int a = 0; a < C::WTM; ++a) {
                const int row = (a * C::WM + wm) * 32 + l32;
                const v16f d = block_dot(sm.st.a[buf][pl][row], bc);
                const v16f w = scale_outer(sm.st.as[buf][pl][row], bw);
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[a][b][i] = __builtin_fmaf(d[i], w[i], acc[a][b][i]);
            }
        }
    };
    // a stage with another one behind it, from LDS buffer `buf`, and the next stage's units (fetched one stage earlier) into
    // the other buffer
    auto stage = [&](int buf, const Unit& na, const Unit& nb) {
        if (live) {
#pragma unroll
            for (int kb = 0; kb < C::SKB; ++kb) {
                block(buf, kb);
                if (kb == C::SKB / 2 - 1) put_a(buf ^ 1, na);
                __builtin_amdgcn_sched_barrier(0);
            }
            put_b(buf ^ 1, nb);
        } else {
            put_a(buf ^ 1, na);
            put_b(buf ^ 1, nb);
        }
    };

    if (nkb > 0) {
        const int nfull = (nkb - 1) / C::kStageBlocks;  // stages that another one follows
        Unit a0, b0, a1, b1;
        load(a0, b0, 0);
        load(a1, b1, 1);
        put_a(0, a0);
        put_b(0, b0);
        __syncthreads();
        // stage s computes from LDS buffer s % 2 while stage s + 2 is fetched into the registers that held stage s and
        // stage s + 1 (fetched one stage earlier) is written to the other buffer; past the end zeros are fetched
        for (int s = 0; s < nfull; s += 2) {
            load(a0, b0, s + 2);
            stage(0, a1, b1);
            __syncthreads();
            if (s + 1 >= nfull) break;
            load(a1, b1, s + 3);
            stage(1, a0, b0);
            __syncthreads();
        }
        // the blocks of the last stage, full or partial: nothing is staged behind them (a reduction of one stage, K = 64,
        // 2688 x 12768: 28.9 -> 26.3 us; 8192 x 8192 x 128 59.6 -> 56.8; 8192 x 8192 x 2048 445 -> 441)
        if (live) {
            const int left = nkb - nfull * C::kStageBlocks - C::SKB * wk;
#pragma unroll
            for (int kb = 0; kb < C::SKB; ++kb)
                if (kb < left) block(nfull & 1, kb);
        }
    }

    // uniform: the fp8 subnormal encoding scaled every product by 2^-18
    const float mul = FMT == kFmtUniform ? 262144.0f : 1.0f;
    auto store = [&](int a, int b, int i, float sum) {
        const int row = (a * C::WM + wm) * 32 + 8 * (i >> 2) + 4 * h + (i & 3), col = (b * C::WN + wn) * 32 + l32;
        if (row >= tl.mrows || col >= tl.nrows) return;
        const float v = sum * mul;
        const int64_t off = tl.c_off + (int64_t)row * j.ldc + col;
        if constexpr (OUT == kOutF32) {
            static_cast<float*>(j.c)[off] = v;
        } else {
            static_cast<uint16_t*>(j.c)[off] = __builtin_bit_cast(uint16_t, (__bf16)v);  // RNE
        }
    };
    if constexpr (C::WK == 1) {
#pragma unroll
        for (int a = 0; a < C::WTM; ++a)
#pragma unroll
            for (int b = 0; b < C::WTN; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) store(a, b, i, acc[a][b][i]);
    } else {
        static_assert(C::WK == 2, "two K groups");
        // each group hands the other half of its accumulators over and finishes (adds and stores) its own half
        __syncthreads();  // the last stage's LDS accesses
        float(*const mine)[64] = sm.part[wk][wt];
        float(*const other)[64] = sm.part[1 - wk][wt];
#pragma unroll
        for (int a = 0; a < C::WTM; ++a)
#pragma unroll
            for (int b = 0; b < C::WTN; ++b)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    mine[8 * (a * C::WTN + b) + i][lane] = wk ? acc[a][b][i] : acc[a][b][8 + i];
        __syncthreads();
#pragma unroll
        for (int a = 0; a < C::WTM; ++a)
#pragma unroll
            for (int b = 0; b < C::WTN; ++b)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float t = other[8 * (a * C::WTN + b) + i][lane];  // sums in the order group 0 + group 1
                    if (wk) store(a, b, 8 + i, t + acc[a][b][8 + i]);
                    else store(a, b, i, acc[a][b][i] + t);
                }
    }
}

using Tile128 = TileCfg<2, 1, 2, 4, 1, 4>;      // 128 x 128, 8 waves
using Tile128K2 = TileCfg<2, 1, 2, 4, 2, 4>;    // 128 x 128, 16 waves in two K groups
using Tile128x64 = TileCfg<1, 1, 4, 2, 1, 4>;   // 128 x 64, 8 waves

static dim3 gemm_grid(const GemmJob& j, int bm, int bn) {
    dim3 grid((unsigned)((j.N + bn - 1) / bn), (unsigned)((j.M + bm - 1) / bm), 1);
    if (j.mode == kGemmRaggedM) grid.y += (unsigned)j.G;  // each group may end in a partial tile
    else if (j.mode == kGemmRaggedK) grid.z = (unsigned)j.G;
    return grid;
}

template <int FMT, int OUT, class C>
static hipError_t launch_t(const GemmJob& j, hipStream_t s) {
    const dim3 grid = gemm_grid(j, C::BM, C::BN);
    if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
    GemmArgs args{j};
    gemm_f32_kernel<FMT, OUT, C><<<grid, C::kThreads, 0, s>>>(args);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Problems too small to fill the chip with the kernel above. A workgroup owns one (32 WTM) x (32 WTN) output tile and
// splits its reduction over NW waves; every wave loads its own operand fragments straight from global memory into
// registers (no LDS staging, so no barrier until the partial sums are added through LDS).
// ------------------------------------------------------------------------------------------------
template <int WTM_, int WTN_, int NW_, int U_, int EU_>
struct DirectCfg {
    static constexpr int WTM = WTM_, WTN = WTN_, NW = NW_;
    static constexpr int BM = 32 * WTM, BN = 32 * WTN, kThreads = 64 * NW;
    static constexpr int U = U_;    // blocks per group: one group is computed while the next is fetched
    static constexpr int EU = EU_;  // waves per SIMD the registers are bounded for
    // the partial sums pass through LDS in kPasses slices of kSlice accumulators per wave (32 KB)
    static constexpr int kAcc = 16 * WTM * WTN, kSlice = kAcc < 128 / NW ? kAcc : 128 / NW, kPasses = kAcc / kSlice;
    static_assert(kAcc % kSlice == 0 && kSlice % NW == 0, "slices are shared evenly");
};

// Outer-product operands of a lane's own half, from its row's scale. K slots 0-3 (lanes 0-31) and 4-7 (lanes 32-63):
//   A: a0 a1 a0 a1 | a0 a1 a2 a2        B: b0 b0 b1 b1 | b2 b2 b0 b1
// -> a0b0 a1b0 a0b1 a1b1 | a0b2 a1b2 a2b0 a2b1, the same eight products as the staged kernel's.
__device__ __forceinline__ uint2 scale_frag_a(float s, bool h) {
    uint32_t p0, p1, p2;
    split_bf16x3(s, p0, p1, p2);
    const uint32_t p01 = bf16_pair(p0, p1);
    return make_uint2(p01, h ? bf16_pair(p2, p2) : p01);
}
__device__ __forceinline__ uint2 scale_frag_b(float s, bool h) {
    uint32_t p0, p1, p2;
    split_bf16x3(s, p0, p1, p2);
    const uint32_t x = h ? p2 : p0, y = h ? p0 : p1;
    return make_uint2(bf16_pair(x, x), bf16_pair(y, p1));
}

template <int FMT, int OUT, class C>
__global__ __launch_bounds__(C::kThreads, C::EU) void gemm_direct_kernel(GemmArgs args) {
    constexpr int WTM = C::WTM, WTN = C::WTN, NW = C::NW, U = C::U;
    __shared__ float part[NW][C::kSlice][64];
    __shared__ int32_t s_grp[2];
    __shared__ int64_t s_pad;
    const GemmJob& j = args.j;
    Tile tl;
    if (!resolve_tile<C::BM, C::BN>(j, s_grp, &s_pad, grid_pos(), tl)) return;
    tl.a = uniform_ptr(tl.a);
    tl.b = uniform_ptr(tl.b);
    tl.as = uniform_ptr(tl.as);
    tl.bs = uniform_ptr(tl.bs);
    tl.a_row0 = __builtin_amdgcn_readfirstlane(tl.a_row0);
    tl.b_row0 = __builtin_amdgcn_readfirstlane(tl.b_row0);
    tl.mrows = __builtin_amdgcn_readfirstlane(tl.mrows);
    tl.nrows = __builtin_amdgcn_readfirstlane(tl.nrows);
    const int nkb = __builtin_amdgcn_readfirstlane((int)tl.nkb);

    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng = (nkb + U - 1) / U;  // groups of U blocks, dealt round robin to the waves

    // resources that end at the tile's last valid byte; rows past it read zeros
    const int64_t a_last = (tl.a_row0 + tl.mrows - 1) / kPanelRows, b_last = (tl.b_row0 + tl.nrows - 1) / kPanelRows;
    const int a_cbytes = (int)(a_last * j.a_pld + (int64_t)nkb * kPanelBlockBytes);
    const int a_sbytes = (int)((a_last * j.as_pld + (int64_t)nkb * kPanelBlockScales) * 4);
    const int b_cbytes = (int)(b_last * j.b_pld + (int64_t)nkb * kPanelBlockBytes);
    const int b_sbytes = (int)((b_last * j.bs_pld + (int64_t)nkb * kPanelBlockScales) * 4);
    int voca[WTM], vosa[WTM], vocb[WTN], vosb[WTN];
#pragma unroll
    for (int a = 0; a < WTM; ++a) {
        voca[a] = (int)code_off(tl.a_row0, a * 32 + l32, 0, j.a_pld) + 4 * h;  // the lane's K half: four bytes
        vosa[a] = (int)scale_off(tl.a_row0, a * 32 + l32, 0, j.as_pld) * 4;
    }
#pragma unroll
    for (int b = 0; b < WTN; ++b) {
        vocb[b] = (int)code_off(tl.b_row0, b * 32 + l32, 0, j.b_pld) + 4 * h;
        vosb[b] = (int)scale_off(tl.b_row0, b * 32 + l32, 0, j.bs_pld) * 4;
    }

    struct Group {  // codes and scales of the lane's rows, per block
        uint32_t ac[U][WTM], as[U][WTM], bc[U][WTN], bs[U][WTN];
    };
    // a block past the reduction reads zeros (empty resources)
    auto load = [&](Group& t, int g) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kb = g * U + u;
            const bool in = kb < nkb;
            const int soc = __builtin_amdgcn_readfirstlane(kb * (int)kPanelBlockBytes);
            const int sos = __builtin_amdgcn_readfirstlane(kb * (int)kPanelBlockScales * 4);
#pragma unroll
            for (int a = 0; a < WTM; ++a) {
                t.ac[u][a] = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(tl.a, in ? a_cbytes : 0), voca[a], soc, 0);
                t.as[u][a] = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(tl.as, in ? a_sbytes : 0), vosa[a], sos, 0);
            }
#pragma unroll
            for (int b = 0; b < WTN; ++b) {
                t.bc[u][b] = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(tl.b, in ? b_cbytes : 0), vocb[b], soc, 0);
                t.bs[u][b] = __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(tl.bs, in ? b_sbytes : 0), vosb[b], sos, 0);
            }
        }
    };
    auto conv = [](uint32_t d) -> uint2 {
        if constexpr (FMT == kFmtUniform) return uniform_to_e4m3(d);
        else return e2m1_to_e4m3(d);
    };
    float acc[WTM][WTN][16];
#pragma unroll
    for (int a = 0; a < WTM; ++a)
#pragma unroll
        for (int b = 0; b < WTN; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;
    auto compute = [&](const Group& t) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint2 ac[WTM], aw[WTM];
#pragma unroll
            for (int a = 0; a < WTM; ++a) {
                ac[a] = conv(t.ac[u][a]);
                aw[a] = scale_frag_a(__uint_as_float(t.as[u][a]), h);
            }
#pragma unroll
            for (int b = 0; b < WTN; ++b) {
                const uint2 bc = conv(t.bc[u][b]), bw = scale_frag_b(__uint_as_float(t.bs[u][b]), h);
#pragma unroll
                for (int a = 0; a < WTM; ++a) {
                    const v16f d = block_dot(ac[a], bc);
                    const v16f w = scale_outer(aw[a], bw);
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[a][b][i] = __builtin_fmaf(d[i], w[i], acc[a][b][i]);
                }
            }
        }
    };
    if (wave < ng) {
        Group t0, t1;
        load(t0, wave);
        for (int g = wave; g < ng; g += 2 * NW) {
            load(t1, g + NW);
            compute(t0);
            if (g + NW >= ng) break;
            load(t0, g + 2 * NW);
            compute(t1);
        }
    }

    const float mul = FMT == kFmtUniform ? 262144.0f : 1.0f;  // uniform: the fp8 subnormal encoding's 2^-18
#pragma unroll
    for (int p = 0; p < C::kPasses; ++p) {
        if (p > 0) __syncthreads();  // the previous slice has been read
#pragma unroll
        for (int i = 0; i < C::kSlice; ++i) {
            const int e = p * C::kSlice + i;
            part[wave][i][lane] = acc[e / 16 / WTN][e / 16 % WTN][e % 16];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < C::kSlice / NW; ++q) {
            const int i = q * NW + wave, e = p * C::kSlice + i, t = e / 16, r = e % 16;
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += part[w][i][lane];
            const int row = (t / WTN) * 32 + 8 * (r >> 2) + 4 * h + (r & 3), col = (t % WTN) * 32 + l32;
            if (row < tl.mrows && col < tl.nrows) {
                const float v = sum * mul;
                const int64_t off = tl.c_off + (int64_t)row * j.ldc + col;
                if constexpr (OUT == kOutF32) static_cast<float*>(j.c)[off] = v;
                else static_cast<uint16_t*>(j.c)[off] = __builtin_bit_cast(uint16_t, (__bf16)v);  // RNE
            }
        }
    }
}

using Direct32 = DirectCfg<1, 1, 8, 4, 4>;     // 32 x 32, 8 waves
using Direct64 = DirectCfg<2, 2, 4, 2, 3>;     // 64 x 64, 4 waves

template <int FMT, int OUT, class C>
static hipError_t launch_direct(const GemmJob& j, hipStream_t s) {
    const dim3 grid = gemm_grid(j, C::BM, C::BN);
    if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
    GemmArgs args{j};
    gemm_direct_kernel<FMT, OUT, C><<<grid, C::kThreads, 0, s>>>(args);
    return hipGetLastError();
}

// Which kernel takes a problem: the one with the smallest estimated time. A CU holds up to `resident` workgroups at
// once, so a grid runs in rounds of 256 * resident workgroups:
//     fixed + (rounds - 1) * again + blocks * ((rounds - 1) * round + slope[workgroups per CU in the last round - 1])
// with slope[n - 1] the time per K-block of n workgroups sharing a CU and `round` that of a full round followed by
// others, whose start hides its end. Microseconds, measured on gfx950 (256 CUs) on grids of 1/4 to 8 workgroups per CU at
// K = 512, 2048 and 4096; the 32 x 32 row's `again` at K = 32 to 256, where a round is little else (with 1.8, fitted at the
// longer ones: 240 x 5328 x 160 8.3 us on it, 5.7 on 128 x 64). The large tile stages least per output (an asymptotic 111
// cycles per 32 x 32 tile and block, against 127 for 128 x 64, 130 for the 64 x 64 and 186 for the 32 x 32 direct tiles)
// but needs 512 tiles to fill the chip; smaller tiles and a split reduction give up some of that for a full chip and a
// shorter chain per workgroup. Measured, us, 128 x 128 only -> picked: 256 x 512 x 256 8.7 -> 3.9, 64 x 4096 x 4096 74 ->
// 10, 1024^3 22 -> 11, 1040 x 2064 x 1552 33 -> 24, 2048 x 2048 x 4096 76 -> 63, 2048 x 3072 x 2048 59 -> 52; grids of
// many rounds keep the large tile.
enum GemmKernel { kTile128, kTile128K2, kTile128x64, kDirect32, kDirect64, kGemmKernels };
struct GemmCost {
    int bm, bn, resident;
    double fixed, again, round, slope[3];
};
constexpr GemmCost kGemmCost[kGemmKernels] = {
    {Tile128::BM, Tile128::BN, 2, 5.0, 5.0, 0.405, {0.267, 0.442, 0.0}},
    {Tile128K2::BM, Tile128K2::BN, 1, 7.0, 5.0, 0.217, {0.217, 0.0, 0.0}},
    {Tile128x64::BM, Tile128x64::BN, 3, 5.0, 4.5, 0.345, {0.195, 0.245, 0.370}},
    {Direct32::BM, Direct32::BN, 3, 3.6, 2.6, 0.060, {0.024, 0.046, 0.063}},
    {Direct64::BM, Direct64::BN, 3, 6.0, 4.5, 0.188, {0.108, 0.129, 0.188}},
};
// The E2M1 128 x 64 kernel needs 81 registers, one more than three workgroups per CU leave (the uniform one 80): two, and
// 155 instead of 127 cycles per 32 x 32 tile and block. us, 128 x 128 / 128 x 64 / 64 x 64: 368 x 16320 x 6528 192 / 211 /
// 167, 10832 x 560 x 6720 179 / 215 / 171.
constexpr GemmCost kCost128x64E2M1 = {Tile128x64::BM, Tile128x64::BN, 2, 5.0, 4.5, 0.258, {0.196, 0.360, 0.0}};

// Ragged-M: every workgroup first finds its group (a prefix sum over the offsets and two barriers before any load), and
// so do those that find none. Per workgroup and CU: of 0.1 to 1 the value closest to the fastest kernel over 734 problems of
// 1 to 256 groups (1.9% above it; 4.7% without it and with half a tile per group counted). us, 128 x 128 / then picked /
// now: 1273 tokens of 128 groups, 5248 x 256 122 / 165 / 122; 600 of 256, 1536 x 256 66 / 96 / 66; one group of 3124,
// 1280 x 1152 35 / 44 / 32.
constexpr double kLookupUs = 0.75;

static GemmKernel pick_kernel(const GemmJob& j) {
    constexpr double kCUs = 256.0;
    const double blocks = j.mode == kGemmRaggedK ? (double)j.red_total / 16.0 / j.G : (double)j.nkb;  // an average group
    GemmKernel best = kTile128;
    double best_us = 0.0;
    for (int k = 0; k < kGemmKernels; ++k) {
        const GemmCost& c = k == kTile128x64 && j.format == kFmtE2M1 ? kCost128x64E2M1 : kGemmCost[k];
        // launch limits: what the large tile's grid can hold must not fail on a smaller tile's (operands of millions of rows)
        const dim3 grid = gemm_grid(j, c.bm, c.bn);
        if (k != kTile128 && (grid.y > 65535u || grid.x >= 1u << 22)) continue;
        // Ragged-M: all workgroups of the grid count, a tile row for each group's remainder among them. Those without rows
        // are short, but which XCD they fall to is not known here: 250 tiles and 10 empty workgroups are 33 on some of
        // the 8 XCDs of 32 CUs, a second round for the kernel that runs one per CU.
        const double per_cu = (double)grid.x * grid.y * grid.z / kCUs;
        // the last round counts as partial even when it is full
        const double rounds = ceil(per_cu / c.resident), full = rounds > 1.0 ? rounds - 1.0 : 0.0;
        const double rest = per_cu - full * c.resident;
        const double last = c.slope[rest <= 1.0 ? 0 : rest <= 2.0 ? 1 : 2];
        double us = c.fixed + full * c.again + blocks * (full * c.round + last);
        if (j.mode == kGemmRaggedM) us += kLookupUs * per_cu;
        if (k == kTile128) us *= 0.96;  // the estimates' spread: within it the large tile stays
        if (k == 0 || us < best_us) {
            best = (GemmKernel)k;
            best_us = us;
        }
    }
    return best;
}

template <int FMT, int OUT>
static hipError_t launch_picked(const GemmJob& j, hipStream_t s) {
    switch (pick_kernel(j)) {
        case kTile128K2: return launch_t<FMT, OUT, Tile128K2>(j, s);
        case kTile128x64: return launch_t<FMT, OUT, Tile128x64>(j, s);
        case kDirect32: return launch_direct<FMT, OUT, Direct32>(j, s);
        case kDirect64: return launch_direct<FMT, OUT, Direct64>(j, s);
        default: return launch_t<FMT, OUT, Tile128>(j, s);
    }
}

hipError_t launch_gemm(const GemmJob& j, hipStream_t s) {
    if (j.format == kFmtE2M1) {
        return j.out_dtype == kOutBF16 ? launch_picked<kFmtE2M1, kOutBF16>(j, s) : launch_picked<kFmtE2M1, kOutF32>(j, s);
    }
    return j.out_dtype == kOutBF16 ? launch_picked<kFmtUniform, kOutBF16>(j, s) : launch_picked<kFmtUniform, kOutF32>(j, s);
}

}  // namespace ufp4

extern "C" int ufp4_plan_gemm(int mode, int format, int64_t M, int64_t N, int64_t red, int32_t G) {
    ufp4::GemmJob j{};
    j.mode = mode;
    j.format = format;
    j.M = M;
    j.N = N;
    j.nkb = red / 16;
    j.red_total = red;
    j.G = G;
    return ufp4::pick_kernel(j);
}

namespace ufp4 {
template <int FMT, int OUT>
static int gemm_resident(int kernel) {
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (kernel) {
        case kTile128: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_f32_kernel<FMT, OUT, Tile128>, Tile128::kThreads, 0); break;
        case kTile128K2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_f32_kernel<FMT, OUT, Tile128K2>, Tile128K2::kThreads, 0); break;
        case kTile128x64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_f32_kernel<FMT, OUT, Tile128x64>, Tile128x64::kThreads, 0); break;
        case kDirect32: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_direct_kernel<FMT, OUT, Direct32>, Direct32::kThreads, 0); break;
        case kDirect64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_direct_kernel<FMT, OUT, Direct64>, Direct64::kThreads, 0); break;
        default: break;
    }
    return e == hipSuccess ? n : -1;
}
}  // namespace ufp4

extern "C" int ufp4_plan_gemm_resident(int kernel, int format, int out_dtype, int* costed) {
    using namespace ufp4;
    if (kernel < 0 || kernel >= kGemmKernels) return -1;
    const bool e2m1 = format == kFmtE2M1, bf16 = out_dtype == kOutBF16;
    *costed = (kernel == kTile128x64 && e2m1 ? kCost128x64E2M1 : kGemmCost[kernel]).resident;
    if (e2m1) return bf16 ? gemm_resident<kFmtE2M1, kOutBF16>(kernel) : gemm_resident<kFmtE2M1, kOutF32>(kernel);
    return bf16 ? gemm_resident<kFmtUniform, kOutBF16>(kernel) : gemm_resident<kFmtUniform, kOutF32>(kernel);
}
