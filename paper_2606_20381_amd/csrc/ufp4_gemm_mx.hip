// Block-scaled 4-bit GEMM for the uniform grid with power-of-two 1x32 scales (the scale hierarchy of Sec. 4
// chosen for the hardware): C[i, j] = sum_k A[i,k] 2^(eA[i,k/32] - 127) B[j,k] 2^(eB[j,k/32] - 127), with the
// codes stored as FP6 E2M3 numbers and the scales as E8M0 bytes (quantizer: ufp4_quant.hip).
//
// The whole product runs on v_mfma_scale_f32_32x32x64_f8f6f4 with FP6 operands: each lane holds the 32 codes
// of one row and one 32-block (24 bytes, the storage format itself) and that block's E8M0 scale, and the
// matrix core applies both scales and accumulates in fp32. There is no per-block VALU work, unlike the fp32
// per-16 scales of the main recipe, so the kernel is bound by the matrix cores and by how fast operand tiles
// reach them.
//
// Tiling: a 256 x 256 output tile per 512-thread workgroup (8 waves of 128 x 64, 4 x 2 MFMA tiles of 32 x 32,
// two waves per SIMD, one workgroup per CU); problems with too few such tiles take 128 x 128 or 64 x 64 ones (four
// waves; see pick_mx). K advances 128 (four 32-blocks) per stage. A stage of one panel
// is a contiguous 12 KiB run (the panel layout puts the 128 rows of a 32-block together, each row's 24 bytes
// as three 8-byte units in three planes of 128 rows) plus 512 scale bytes; stages are copied unchanged from
// global memory into a three-deep LDS ring by direct-to-LDS loads issued two stages ahead, and a lane's
// operand is three 8-byte LDS reads that 32 consecutive rows make contiguous.

#include "ufp4_internal.h"

#include <math.h>

namespace ufp4 {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v8i __attribute__((ext_vector_type(8)));

constexpr int kMxStageBlocks = 4;  // 32-blocks per stage

// Tile configuration: WM x WN waves, each with WTM x WTN MFMA tiles of 32 x 32 outputs.
template <int WTM_, int WTN_, int WM_, int WN_>
struct MxCfg {
    static constexpr int WTM = WTM_, WTN = WTN_, WM = WM_, WN = WN_;
    static constexpr int BM = 32 * WTM * WM, BN = 32 * WTN * WN;
    static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
    // 1 KiB direct-to-LDS loads of a stage: 96 code bytes per row of A and B, dealt to the waves, and each
    // wave's share of the 4 scale bytes per row (16 bytes per lane)
    static constexpr int kLoadsA = BM * 3 / 32, kLoadsB = BN * 3 / 32;
    static constexpr int kWaveCodes = (kLoadsA + kLoadsB) / kWaves;
    static constexpr int kScaleLanes = (BM + BN) / 4 / kWaves;
    static constexpr int kWaveLoads = kWaveCodes + 1;
    static_assert((kLoadsA + kLoadsB) % kWaves == 0 && kScaleLanes <= 64 && kWaves % 2 == 0,
                  "every wave issues the same loads, and its scales belong to one operand");
};

template <class C>
struct MxStageSmem {
    uint8_t a[C::BM * 96];  // [panel][block][unit][row]: the panel layout, or its 64-row half
    uint8_t b[C::BN * 96];
    uint8_t s[C::BM * 4 + C::BN * 4];  // scale bytes of A, then of B: [panel][block][row]
};

// The 24 bytes of one row's 32-block: three 8-byte units PLANE bytes apart (planar layout, see the file
// header), so 32 lanes reading consecutive rows touch 256 contiguous bytes per unit.
template <int PLANE>
__device__ __forceinline__ v8i load_fp6_operand(const uint8_t* p) {
    const uint2 x0 = *reinterpret_cast<const uint2*>(p);
    const uint2 x1 = *reinterpret_cast<const uint2*>(p + PLANE);
    const uint2 x2 = *reinterpret_cast<const uint2*>(p + 2 * PLANE);
    const v8i v = {(int)x0.x, (int)x0.y, (int)x1.x, (int)x1.y, (int)x2.x, (int)x2.y, 0, 0};
    return v;
}

// 16 bytes per lane from global memory straight into LDS: lane i reads sbase + voff_i and its bytes land at
// lds_base + 16 i (sbase and lds_base wave-uniform, lds_base in M0). Written as inline assembly so that the
// compiler, which does not see these LDS writes, does not make every later LDS read wait for all of them; the
// kernel orders them itself (vmcnt waits and barriers).
__device__ __forceinline__ void dma16(uint32_t voff, const void* sbase, const void* lds_base) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(lds_base));
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(m0)
                 : "memory", "m0");
}

// Wait until at most N vector-memory operations are outstanding, and for all LDS operations (s_waitcnt immediate, gfx9
// encoding).
template <int N>
__device__ __forceinline__ void wait_vm_lgkm() {
    static_assert(N < 16, "low bits of vmcnt only");
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
}

// Workgroup -> output tile. Workgroups are dealt to the 8 XCDs round robin (workgroup L to XCD L % 8) and each
// XCD has its own L2, so the first 8 * floor(T / 8) workgroups are renumbered to give XCD k the contiguous
// range of tiles [k T/8, (k + 1) T/8); tiles are then ordered in bands of kGroupRows tile rows, column by
// column within a band, so that the workgroups running together on one XCD share a few A and B panels.
constexpr int kGroupRows = 8;
__device__ __forceinline__ void tile_of(int64_t L, int64_t gy, int64_t gx, int64_t& tm, int64_t& tn) {
    const int64_t T = gx * gy, per = T / 8;
    const int64_t t = L < 8 * per ? (L % 8) * per + L / 8 : L;
    const int64_t band = t / (kGroupRows * gx);
    const int64_t first = band * kGroupRows;
    const int64_t rows = gy - first < kGroupRows ? gy - first : kGroupRows;
    const int64_t r = t - band * kGroupRows * gx;
    tm = first + r % rows;
    tn = r / rows;
}

constexpr int64_t kMxBlock32 = 32;  // reduction values per scale block

// Wave-uniform copy (SGPRs) of a value the compiler cannot prove uniform, e.g. one read back from LDS.
__device__ __forceinline__ int64_t uniform_i64_mx(int64_t v) {
    const uint64_t u = (uint64_t)v;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Tile rows of the grid, for tiles of `bm` rows. Ragged-M: a bound over all groups (each may end in a partial tile).
__host__ __device__ inline int64_t mx_tile_rows(const MxGemmJob& j, int bm) {
    return j.mode == kGemmRaggedM ? (j.a_rows + bm - 1) / bm + j.G : (j.M + bm - 1) / bm;
}

// Ragged-M: the group and local tile of global m-tile t, with the group's padded row start (a multiple of 128)
// and its token rows. Wave 0 prefix-sums the per-group tile counts ceil(m_g / BM) and padded lengths
// pad128(m_g), 64 groups at a time; the result goes through LDS. Every thread calls this; false past the last tile.
struct MxGroupTile {
    int64_t g, lt, prow0, trow0, rows;
};
template <int BM>
__device__ bool resolve_mx_ragged_m(const MxGemmJob& j, int64_t t, int64_t* slot, MxGroupTile& r) {
    const int tid = threadIdx.x;
    if (tid == 0) slot[0] = -1;
    __syncthreads();
    if (tid < 64) {
        int64_t tbase = 0, pbase = 0;
        for (int g0 = 0; g0 < j.G; g0 += 64) {
            const int g = g0 + tid;
            int64_t m = 0;
            if (g < j.G) m = j.offsets[g + 1] - j.offsets[g];
            if (m < 0) m = 0;
            const int64_t cnt = (m + BM - 1) / BM, pad = (m + 127) / 128 * 128;
            int64_t ti = cnt, pi = pad;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t vt = __shfl_up(ti, d, 64), vp = __shfl_up(pi, d, 64);
                if (tid >= d) {
                    ti += vt;
                    pi += vp;
                }
            }
            const int64_t te = tbase + ti - cnt;  // first global tile of group g
            if (cnt > 0 && te <= t && t < te + cnt) {
                slot[0] = g;
                slot[1] = t - te;
                slot[2] = pbase + pi - pad;
                slot[3] = m;
            }
            tbase += __shfl(ti, 63, 64);
            pbase += __shfl(pi, 63, 64);
        }
    }
    __syncthreads();
    r.g = slot[0];
    if (r.g < 0) return false;
    r.lt = slot[1];
    r.prow0 = slot[2] + r.lt * BM;
    r.trow0 = j.offsets[r.g] + r.lt * BM;
    r.rows = slot[3] - r.lt * BM;
    return true;
}

// Padded start of group g along a ragged reduction (token counts rounded up to 32, summed over h < g) and the
// group's padded length, by wave 0 through LDS; every thread calls this.
__device__ void mx_padded_range(const int64_t* off, int g, int64_t* slot, int64_t& start, int64_t& len) {
    const int tid = threadIdx.x;
    if (tid < 64) {
        int64_t sum = 0;
        for (int h = tid; h < g; h += 64) {
            const int64_t c = off[h + 1] - off[h];
            sum += (c > 0 ? c + kMxBlock32 - 1 : 0) / kMxBlock32 * kMxBlock32;
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if (tid == 0) slot[0] = sum;
    }
    __syncthreads();
    start = slot[0];
    const int64_t c = off[g + 1] - off[g];
    len = (c > 0 ? c + kMxBlock32 - 1 : 0) / kMxBlock32 * kMxBlock32;
}

template <int OUT, class C>
__global__ __launch_bounds__(C::kThreads) void gemm_mx_kernel(MxGemmJob j) {
    // three separate LDS objects (not an array): the compiler then knows that loads in flight into one buffer
    // do not alias reads of another and does not make the reads wait for them
    __shared__ MxStageSmem<C> sm0, sm1, sm2;
    __shared__ int64_t s_slot[4];
    constexpr int BM = C::BM, BN = C::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: load addresses stay scalar
    const int h = lane >> 5, l32 = lane & 31;
    const int wm = (int)((unsigned)wave / C::WN), wn = (int)((unsigned)wave % C::WN);
    int64_t tm, tn;
    tile_of(blockIdx.x, mx_tile_rows(j, BM), (j.N + BN - 1) / BN, tm, tn);
    // What the tile covers: A rows from arow0 and B rows from brow0 of the operands, reduction blocks from a_kb0 /
    // b_kb0 (nkb of them), output rows out_row0 .. out_row0 + mrows - 1 (token rows for ragged-M) of the problem at
    // c_base.
    int64_t arow0 = tm * BM, brow0 = tn * BN, a_kb0 = 0, b_kb0 = 0, nkb64 = j.nkb;
    int64_t out_row0 = tm * BM, mrows = j.M - tm * BM, c_base = 0;
    if (j.mode == kGemmRaggedM) {
        MxGroupTile r;
        if (!resolve_mx_ragged_m<BM>(j, tm, s_slot, r)) return;  // the whole workgroup agrees
        arow0 = r.prow0;
        out_row0 = r.trow0;
        mrows = r.rows < j.M - r.trow0 ? r.rows : j.M - r.trow0;  // token rows past the output are not stored
        brow0 = r.g * j.b_group_rows + tn * BN;
        b_kb0 = r.g * j.b_group_kb;
    } else if (j.mode == kGemmRaggedK) {
        int64_t start, len;
        mx_padded_range(j.offsets, (int)blockIdx.y, s_slot, start, len);
        a_kb0 = b_kb0 = start / kMxBlock32;
        nkb64 = len / kMxBlock32;
        if (a_kb0 + nkb64 > j.nkb) nkb64 = j.nkb - a_kb0 > 0 ? j.nkb - a_kb0 : 0;  // clamped to the operands
        c_base = (int64_t)blockIdx.y * j.M * j.ldc;
    }
    arow0 = uniform_i64_mx(arow0);
    brow0 = uniform_i64_mx(brow0);
    a_kb0 = uniform_i64_mx(a_kb0);
    b_kb0 = uniform_i64_mx(b_kb0);
    nkb64 = uniform_i64_mx(nkb64);
    // The tile's panels (two of a 256-row tile) and, for a 64-row tile, its half of the panel. A panel past the
    // operand's last one (a tile over the edge) is replaced by the last panel: those rows only feed outputs that are
    // not stored.
    const int64_t pa_last = (j.a_rows - 1) / 128, pb_last = (j.b_rows - 1) / 128;
    int64_t pa0 = arow0 / 128, pb0 = brow0 / 128;
    if (pa0 > pa_last) pa0 = pa_last;  // only for offsets inconsistent with the operand: wrong values, no fault
    if (pb0 > pb_last) pb0 = pb_last;
    const int64_t pa1 = pa0 + 1 < pa_last ? pa0 + 1 : pa_last;
    const int64_t pb1 = pb0 + 1 < pb_last ? pb0 + 1 : pb_last;
    const int a_half = BM == 64 ? (int)((arow0 / 64) & 1) : 0, b_half = BN == 64 ? (int)((brow0 / 64) & 1) : 0;
    const uint8_t* const ga0 = j.a + pa0 * j.a_pld + a_kb0 * 3072 + a_half * 512;
    const uint8_t* const ga1 = j.a + pa1 * j.a_pld + a_kb0 * 3072;
    const uint8_t* const gb0 = j.b + pb0 * j.b_pld + b_kb0 * 3072 + b_half * 512;
    const uint8_t* const gb1 = j.b + pb1 * j.b_pld + b_kb0 * 3072;
    // This wave's scale run: chunks (16 bytes) kScaleLanes w .. of [A, B] x [panel][block][row]. The first half of the
    // waves take A's (square tiles).
    static_assert(BM == BN, "the waves' scale shares divide between the operands");
    const int sop = wave >= C::kWaves / 2;
    const int sc0 = (wave - sop * (C::kWaves / 2)) * C::kScaleLanes;  // first chunk within the operand
    constexpr int kBlkChunks = (BM < 128 ? BM : 128) / 16;                 // chunks of one block of a panel
    const int spanel = sc0 / (kBlkChunks * kMxStageBlocks);
    const uint8_t* const gs = sop == 0 ? j.as + (spanel ? pa1 : pa0) * j.as_pld + a_kb0 * 128 + a_half * 64
                                       : j.bs + (spanel ? pb1 : pb0) * j.bs_pld + b_kb0 * 128 + b_half * 64;
    const int64_t N = j.N, ldc = j.ldc;
    void* const cptr = j.c;
    const int nkb = (int)nkb64;
    const int nst = (nkb + kMxStageBlocks - 1) / kMxStageBlocks;
    const int kb_last = nkb - 1;

    // A stage with direct global-to-LDS loads: each wave instruction moves 64 x 16 bytes to 1024 contiguous LDS bytes
    // (the loads of A, then those of B, dealt round robin to the waves). Every wave issues the same number of
    // loads for every stage: blocks past the end of the reduction (partial last stage) are read from the last block
    // instead, and compute() gives them zero scales.
    auto issue = [&](int i, MxStageSmem<C>& d) {
        const int kb0 = i * kMxStageBlocks;
#pragma unroll
        for (int q = 0; q < C::kWaveCodes; ++q) {
            const int Lall = q * C::kWaves + wave;
            const bool isb = C::kLoadsA % C::kWaves == 0 ? q >= C::kLoadsA / C::kWaves : Lall >= C::kLoadsA;
            const int L = isb ? Lall - C::kLoadsA : Lall;
            const uint8_t* const g0 = isb ? gb0 : ga0;
            const uint8_t* const g1 = isb ? gb1 : ga1;
            uint8_t* const dst = (isb ? d.b : d.a) + L * 1024;
            if constexpr (BM >= 128) {  // whole panels: a load lies in one block
                const int p = L / 12, cp0 = (L - p * 12) * 64, blk = cp0 / 192;
                const int kb = kb0 + blk < kb_last ? kb0 + blk : kb_last;
                const int64_t off = (int64_t)kb * 3072 + (cp0 - blk * 192) * 16;
                dma16((uint32_t)lane * 16, (p ? g1 : g0) + off, dst);
            } else {  // half a panel: a load is two 512-byte runs (one unit of one block each)
                const int run = 2 * L + h, blk = run / 3, unit = run - blk * 3;
                const int kb = kb0 + blk < kb_last ? kb0 + blk : kb_last;
                dma16((uint32_t)kb * 3072u + (uint32_t)(unit * 1024 + l32 * 16), g0, dst);
            }
        }
        if (lane < C::kScaleLanes) {
            const int cc = sc0 % (kBlkChunks * kMxStageBlocks) + lane, blk = cc / kBlkChunks;  // chunk within the panel
            const int kb = kb0 + blk < kb_last ? kb0 + blk : kb_last;
            dma16((uint32_t)(kb * 128 + (cc % kBlkChunks) * 16), gs, d.s + sop * BM * 4 + sc0 * 16);
        }
    };

    v16f acc[C::WTM][C::WTN];
#pragma unroll
    for (int a = 0; a < C::WTM; ++a)
#pragma unroll
        for (int b = 0; b < C::WTN; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    constexpr int kPlane = BM < 128 ? BM * 8 : 1024, kRowsP = BM < 128 ? BM : 128;  // LDS panel (or half panel)
    static_assert(kRowsP % (32 * C::WTM) == 0 && kRowsP % (32 * C::WTN) == 0, "a wave's rows lie in one LDS panel");
    const unsigned arow = (unsigned)wm * C::WTM * 32, bcol = (unsigned)wn * C::WTN * 32;  // first tile row and column
    auto compute = [&](const MxStageSmem<C>& d, int valid) {
#pragma unroll
        for (int ks = 0; ks < kMxStageBlocks / 2; ++ks) {
            const int kk = 2 * ks + h;  // this lane's 32-block: lanes 0-31 hold K 0-31 of the step, 32-63 K 32-63
            const bool live = kk < valid;  // blocks past the end get scale 2^-127 on both sides: products 0
            v8i av[C::WTM], bv[C::WTN];
            int sa[C::WTM], sb[C::WTN];
#pragma unroll
            for (int b = 0; b < C::WTN; ++b) {
                const unsigned p = bcol / kRowsP, r = bcol % kRowsP + b * 32 + l32;
                bv[b] = load_fp6_operand<kPlane>(d.b + (p * kMxStageBlocks + kk) * 3 * kPlane + r * 8);
                sb[b] = live ? d.s[BM * 4 + (p * kMxStageBlocks + kk) * kRowsP + r] : 0;
            }
#pragma unroll
            for (int a = 0; a < C::WTM; ++a) {
                const unsigned p = arow / kRowsP, r = arow % kRowsP + a * 32 + l32;
                av[a] = load_fp6_operand<kPlane>(d.a + (p * kMxStageBlocks + kk) * 3 * kPlane + r * 8);
                sa[a] = live ? d.s[(p * kMxStageBlocks + kk) * kRowsP + r] : 0;
#pragma unroll
                for (int b = 0; b < C::WTN; ++b)
                    // formats 2 = FP6 E2M3 for both operands; the scale bytes sit in byte 0 of sa / sb
                    acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av[a], bv[b], acc[a][b], 2, 2, 0,
                                                                                sa[a], 0, sb[b]);
            }
        }
    };

    // Stage i is computed from buffer i % 3 while stages i + 1 and i + 2 are in flight. A wave's own loads
    // of stage i are complete once at most those of stage i + 1 are outstanding; the barrier then makes every
    // wave's part visible, and it also orders the previous stage's reads of buffer (i + 2) % 3 before the
    // loads into it are issued.
    auto step = [&](int i, MxStageSmem<C>& cur, MxStageSmem<C>& next2) {
        if (i + 1 < nst) wait_vm_lgkm<C::kWaveLoads>();
        else wait_vm_lgkm<0>();
        __builtin_amdgcn_s_barrier();
        if (i + 2 < nst) issue(i + 2, next2);
        const int left = nkb - i * kMxStageBlocks;
        compute(cur, left < kMxStageBlocks ? left : kMxStageBlocks);
    };
    if (nst > 0) issue(0, sm0);
    if (nst > 1) issue(1, sm1);
    for (int i = 0; i < nst; i += 3) {
        step(i, sm0, sm2);
        if (i + 1 < nst) step(i + 1, sm1, sm0);
        if (i + 2 < nst) step(i + 2, sm2, sm1);
    }

    // Epilogue: lane (l32, h) holds rows 8q + 4h + t (q, t < 4) of column l32 of each 32 x 32 tile; a store
    // instruction writes two runs of 32 consecutive outputs. Tiles inside the output skip the bounds tests.
    const bool inside = mrows >= BM && (tn + 1) * BN <= N;
    auto store = [&](int64_t row, int64_t col, float v) {
        const int64_t off = c_base + row * ldc + col;
        if constexpr (OUT == kOutF32) {
            static_cast<float*>(cptr)[off] = v;
        } else {
            static_cast<uint16_t*>(cptr)[off] = __builtin_bit_cast(uint16_t, (__bf16)v);  // RNE
        }
    };
#pragma unroll
    for (int a = 0; a < C::WTM; ++a) {
#pragma unroll
        for (int b = 0; b < C::WTN; ++b) {
            const int64_t col = tn * BN + (wn * C::WTN + b) * 32 + l32;
            const int64_t lr0 = (wm * C::WTM + a) * 32 + 4 * h;  // tile row of acc element 0
            if (inside) {
#pragma unroll
                for (int i = 0; i < 16; ++i) store(out_row0 + lr0 + 8 * (i >> 2) + (i & 3), col, acc[a][b][i]);
            } else if (col < N) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int64_t lr = lr0 + 8 * (i >> 2) + (i & 3);
                    if (lr < mrows) store(out_row0 + lr, col, acc[a][b][i]);
                }
            }
        }
    }
}

using MxTile256 = MxCfg<4, 2, 2, 4>;  // 256 x 256, 8 waves of 128 x 64, two per SIMD, one workgroup per CU
using MxTile128 = MxCfg<2, 2, 2, 2>;  // 128 x 128, 4 waves, two workgroups per CU
using MxTile64 = MxCfg<1, 1, 2, 2>;   // 64 x 64, 4 waves, four workgroups per CU

// Workgroups of the (x) grid for square tiles of `bm`.
static int64_t mx_grid_tiles(const MxGemmJob& j, int bm) { return ((j.N + bm - 1) / bm) * mx_tile_rows(j, bm); }

template <int OUT, class C>
static hipError_t launch_mx_cfg(const MxGemmJob& j, hipStream_t s) {
    const int64_t tiles = mx_grid_tiles(j, C::BM);
    if (tiles == 0) return hipSuccess;
    const dim3 grid((unsigned)tiles, j.mode == kGemmRaggedK ? (unsigned)j.G : 1u);
    gemm_mx_kernel<OUT, C><<<grid, C::kThreads, 0, s>>>(j);
    return hipGetLastError();
}

// Which tile takes a problem: the one with the smallest estimated time. A CU holds `resident` workgroups at once, so a
// grid runs in rounds of 256 * resident workgroups:
//     fixed + (rounds - 1) * again + stages * ((rounds - 1) * round + slope[workgroups per CU in the last round - 1])
// with slope[n - 1] the time per stage (128 of the reduction) of n workgroups sharing a CU and `round` that of a full
// round followed by others. Microseconds, measured on gfx950 (256 CUs) on grids of 1/4 to 16 workgroups per CU at K =
// 512, 2048 and 4096. The 256 x 256 tile moves the fewest operand bytes per output, and wins once its tiles fill the
// chip; a smaller grid runs faster on more, smaller tiles with their shorter stages. Measured, us, 256 x 256 only ->
// picked: 256 x 512 x 256 8.2 -> 3.8, 1024 x 3072 x 1024 15.1 -> 8.4, 1024 x 1024 x 3072 30.5 -> 9.7, 2048 x 2048 x
// 8192 70.6 -> 33.4, 4096 x 2048 x 2048 24.5 -> 17.8; 4096^3 (45.5; 52.9 on 128 x 128) and larger keep the large tile.
enum MxKernel { kMxTile256, kMxTile128, kMxTile64, kMxKernels };
struct MxCost {
    int tile, threads, resident;
    double fixed, again, round, slope[4];
};
constexpr MxCost kMxCost[kMxKernels] = {
    {MxTile256::BM, MxTile256::kThreads, 1, 7.5, 7.3, 1.19, {1.20, 0.0, 0.0, 0.0}},
    {MxTile128::BM, MxTile128::kThreads, 2, 5.0, 5.0, 0.66, {0.467, 0.700, 0.0, 0.0}},
    {MxTile64::BM, MxTile64::kThreads, 4, 3.5, 2.3, 0.62, {0.262, 0.326, 0.523, 0.647}},
};

// Ragged-M: every workgroup first finds its group, those that find none included. Per workgroup and CU: of 0.1 to 1 the value
// closest to the fastest tile over 366 problems of 1 to 256 groups (1.2% above it; 4.1% without it and with half a tile per
// group counted). us, 256 x 256 / then picked / now: 12759 tokens of 64 groups, 512 x 2432 35 / 38 / 35; 31445 of 8, 384 x
// 1664 42 / 42 / 30; 17081 of 32, 1408 x 2560 93 / 92 / 75.
constexpr double kMxLookupUs = 0.25;

static MxKernel pick_mx(const MxGemmJob& j) {
    constexpr double kCUs = 256.0;
    const double blocks = j.mode == kGemmRaggedK ? (double)j.nkb / j.G : (double)j.nkb;  // ragged-K: an average group
    const double stages = ceil(blocks / kMxStageBlocks);
    MxKernel best = kMxTile256;
    double best_us = 0.0;
    for (int k = 0; k < kMxKernels; ++k) {
        const MxCost& c = kMxCost[k];
        if (k == kMxTile64 && j.nkb >= (int64_t(1) << 20)) continue;  // its load offsets are 32-bit
        // a grid holds fewer than 2^32 threads in x: what fits with the large tile must not fail on a smaller tile's grid
        const int64_t tiles = mx_grid_tiles(j, c.tile);
        if (k != kMxTile256 && tiles * c.threads > int64_t(UINT32_MAX)) continue;
        // ragged-M: all workgroups of the grid count, a tile row for each group's remainder among them
        const double per_cu = (double)tiles * (j.mode == kGemmRaggedK ? j.G : 1) / kCUs;
        // the last round counts as partial even when it is full
        const double rounds = ceil(per_cu / c.resident), full = rounds > 1.0 ? rounds - 1.0 : 0.0;
        const double rest = per_cu - full * c.resident;
        const double last = c.slope[rest <= 1.0 ? 0 : rest <= 2.0 ? 1 : rest <= 3.0 ? 2 : 3];
        double us = c.fixed + full * c.again + stages * (full * c.round + last);
        if (j.mode == kGemmRaggedM) us += kMxLookupUs * per_cu;
        if (k == 0 || us < best_us) {
            best = (MxKernel)k;
            best_us = us;
        }
    }
    return best;
}

template <int OUT>
static hipError_t launch_mx_picked(const MxGemmJob& j, hipStream_t s) {
    switch (pick_mx(j)) {
        case kMxTile128: return launch_mx_cfg<OUT, MxTile128>(j, s);
        case kMxTile64: return launch_mx_cfg<OUT, MxTile64>(j, s);
        default: return launch_mx_cfg<OUT, MxTile256>(j, s);
    }
}

hipError_t launch_gemm_mx(const MxGemmJob& j, hipStream_t s) {
    return j.out_dtype == kOutBF16 ? launch_mx_picked<kOutBF16>(j, s) : launch_mx_picked<kOutF32>(j, s);
}

}  // namespace ufp4

extern "C" int ufp4_plan_gemm_mx(int mode, int64_t M, int64_t N, int64_t red, int32_t G, int64_t a_rows, int64_t* threads_x) {
    using namespace ufp4;
    MxGemmJob j{};
    j.mode = mode;
    j.M = M;
    j.N = N;
    j.nkb = red / 32;
    j.G = G;
    j.a_rows = a_rows;
    const MxKernel k = pick_mx(j);
    *threads_x = mx_grid_tiles(j, kMxCost[k].tile) * kMxCost[k].threads;
    return k;
}

namespace ufp4 {
template <int OUT>
static int mx_resident(int kernel) {
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (kernel) {
        case kMxTile256: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_mx_kernel<OUT, MxTile256>, MxTile256::kThreads, 0); break;
        case kMxTile128: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_mx_kernel<OUT, MxTile128>, MxTile128::kThreads, 0); break;
        case kMxTile64: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, gemm_mx_kernel<OUT, MxTile64>, MxTile64::kThreads, 0); break;
        default: break;
    }
    return e == hipSuccess ? n : -1;
}
}  // namespace ufp4

extern "C" int ufp4_plan_gemm_mx_resident(int kernel, int out_dtype, int* costed) {
    using namespace ufp4;
    if (kernel < 0 || kernel >= kMxKernels) return -1;
    *costed = kMxCost[kernel].resident;
    return out_dtype == kOutBF16 ? mx_resident<kOutBF16>(kernel) : mx_resident<kOutF32>(kernel);
}
