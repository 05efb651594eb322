// Matrix-core (MFMA) kernels of the matrix product for gfx950.
//
// Same contract as the VALU family (C = [C +] A B, row-major, any M, N, K),
// used where the product is a dense contraction in float32 or bfloat16:
//   float32:  v_mfma_f32_32x32x2_f32   (A 32x2, B 2x32, C 32x32 per wavefront)
//   bfloat16: v_mfma_f32_16x16x32_bf16 (A 16x32, B 32x16, float32 accumulate)
//
// Decomposition: a workgroup of WM x WN wavefronts owns a BM x BN output tile;
// each wavefront owns (BM/WM) x (BN/WN) of it, in blocks of 32 x 32 (float32) or
// 16 x 16 (bfloat16) accumulators.  K advances in steps through LDS.
//
// LDS holds a step's tiles as they lie in memory, A row by row (k contiguous)
// and B row by row (n contiguous), in chunks of 16 bytes without padding; the
// chunks of a row are permuted (a_swz, b_swz) so that the reads that feed the
// matrix unit fall in distinct banks (counted: no conflict cycles in any of
// them).
//
// Two ways bring the tiles there:
//   dma_tile   rows aligned for 16-byte loads: global_load_lds writes each
//              lane's chunk to LDS directly, no registers between.  NBUF
//              buffers; the loads of a step go out when its buffer's last
//              reader has passed a barrier, a whole step ahead at two buffers,
//              and no wait drains more than it must.  A program's LDS stage
//              budget decides: STAGES = 2 holds two buffers of BK; STAGES = 1,
//              the paper's one buffer, is cut into two of BK / 2.
//   regs_tile  other rows (and the programs of 1024 work-items, the
//              single-stage bfloat16 ones of K tile 32, too small to cut, and
//              large bfloat16 groups): chunks at element alignment through
//              registers, the next step's loads in flight while the current
//              step multiplies, STAGES buffers of BK.
// Against loads through registers with padded LDS (the earlier form of both),
// bfloat16 with 16 x 16 x 32 products: a float32 8192 x 3000 x 4096 product
// 1683 -> 1444 us (64 x 64 tiles), a bfloat16 product of order 4096 150 ->
// 122-127 us (1.1 PFLOP/s, operands from HBM), one of order 1024 14 -> 7.
// The 16 x 16 x 32 form draws less power than 32 x 32 x 16 at the same rate
// (half the accumulator traffic): a dense 4096^3 product runs at 2.2 GHz with
// it and 1.95 GHz without.
//
// Order of the sum: float32 products take k and k + 4 of each group of eight
// in one instruction (lanes 0-31 the first four k, 32-63 the last four),
// bfloat16 ones 32 consecutive k, both in ascending groups -- the same for
// every tile, step and way of loading, so results do not depend on alignment.
//
// Tiles crossing the matrix edge keep the 16-byte loads: they clamp the rows
// of A and the column chunks of B they read to the last in range (results
// outside C are never stored) and guard their stores.  In a step past the end
// of K, elements of A and rows of B at k >= K become zeros: dma_tile reads
// clamped addresses and zeroes its own chunks in LDS once they have arrived,
// regs_tile masks (or, across the end of an unaligned row, shifts) its chunks
// when they go to LDS.
//
// Workgroup -> tile map: workgroups are dispatched round-robin over the 8 XCDs
// (each with its own L2); blocks b and b+8 land on the same XCD, so the map
// first gives each XCD a contiguous range of tile indices and then walks that
// range in groups of GROUP_M tile rows, which keeps the A and B panels an XCD
// reads within its L2.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kargs.hpp"

namespace pkk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Pointers into global memory.  The grouped kernels read operand pointers
// from descriptors in memory, where the compiler cannot infer the address
// space and would emit flat accesses (which also wait on the LDS counter).
template <class T> using gptr = const __attribute__((address_space(1))) T *;
template <class T> using gmut = __attribute__((address_space(1))) T *;

// 16 bytes of a row: at a 16-byte boundary (rows aligned), or at any element
// of EB bytes (one global load of 16 bytes either way: gfx950 reads global
// memory at any byte address, a chunk that crosses a cache line as two).
template <int EB, bool ALIGNED> struct ChunkAt { typedef u32x4 type; };
template <> struct ChunkAt<4, false> { typedef unsigned int type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct ChunkAt<2, false> { typedef unsigned int type __attribute__((ext_vector_type(4), aligned(2))); };

// The elements of a chunk from element `s` on, zeros behind them (EB bytes an
// element; s is uniform over the workgroup, 0 <= s < 16 / EB).
template <int EB> __device__ __forceinline__ u32x4 chunk_from(u32x4 v, int s) {
    const int d = EB == 4 ? s : s >> 1;
    if (d & 1) v = u32x4{v[1], v[2], v[3], 0u};
    if (d & 2) v = u32x4{v[2], v[3], 0u, 0u};
    if (EB == 2 && (s & 1))
        v = u32x4{v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
    return v;
}

// the source of every element at k >= K (read only)
static __device__ __attribute__((aligned(16))) unsigned int kZeroBlock[4] = {0u, 0u, 0u, 0u};

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int cmin(int a, int b) { return a < b ? a : b; }

constexpr int XCDS = kXcds;
constexpr int GROUP_M = 8;

// tile (tm, tn) of linear workgroup b among tiles_m x tiles_n (below 2^31:
// a grid's workgroups; 64-bit divisions here would cost each workgroup the
// better part of a microsecond)
__device__ __forceinline__ void tile_of(uint32_t b, uint32_t tiles_m, uint32_t tiles_n, int *tm, int *tn) {
    const uint32_t q = tiles_m * tiles_n / XCDS;
    const uint32_t pid = b < q * XCDS ? (b % XCDS) * q + b / XCDS : b;
    const uint32_t group_rows = min(tiles_m, (uint32_t)GROUP_M);
    const uint32_t group = pid / (group_rows * tiles_n), in = pid - group * (group_rows * tiles_n);
    const uint32_t first_m = group * group_rows, gm = min(tiles_m - first_m, group_rows);
    *tn = (int)(in / gm);
    *tm = (int)(first_m + in - *tn * gm);
}

// ------------------------------------------------------------------ tiles in LDS
// A BM x BK tile of A and a BK x BN tile of B (EB bytes an element) for WM x WN
// wavefronts: chunks of 16 bytes, slots in LDS, the wavefront's operands and
// products.  The programs allocate what rows padded by 16 bytes (bfloat16 B: 64)
// would need, the case table's LDS symbol; the chunks need A_BYTES + B_BYTES a
// buffer, less by a tenth to a quarter.
constexpr int f32_lds(int bm, int bn, int bk, int stages) { return stages * 4 * (bm * (bk + 4) + bk * (bn + 4)); }
constexpr int bf16_lds(int bm, int bn, int bk, int stages) { return stages * 2 * (bm * (bk + 8) + bk * (bn + 32)); }

// The MFMA B operand of lanes [16g, 16g + 16) from a row-major tile in LDS:
// gfx950's transposing read hands lane i of each group of 16 element i % 4 of
// the 8 bytes addressed by lane 4j + i / 4, for j = 0..3.  With lane m of the
// group addressing row m / 4, columns 4 (m % 4) .. + 3, lane i receives
// column i of four consecutive rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ s16x4 lds_read_tr16(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
}

template <int EB, int BM, int BN, int BK, int WM, int WN> struct Tile {
    static constexpr bool F32 = EB == 4;
    static constexpr int NT = 64 * WM * WN;
    static constexpr int VE = 16 / EB;                        // elements per chunk
    static constexpr int AC = BK / VE, BC = BN / VE;          // chunks per row
    static constexpr int A_BYTES = BM * BK * EB, B_BYTES = BK * BN * EB;
    static constexpr int BYTES = A_BYTES + B_BYTES;
    // loads per work-item (a tile of fewer chunks than work-items is read by
    // the first of them and again, to the same slots, by the rest)
    static constexpr int AL = cmax(BM * AC / NT, 1), BL = cmax(BK * BC / NT, 1);
    static constexpr int RB = F32 ? 32 : 16;                  // block edge
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int TM = WTM / RB, TN = WTN / RB;        // blocks of a wavefront
    static constexpr int KG = F32 ? 8 : 32;                   // k of one group of products
    // Phases of a step: operands of one are read while the one before
    // multiplies.  A phase is half a group: of its k (float32: two of the four
    // pairs), or of the wavefront's columns (bfloat16) -- whole groups at once
    // would hold up to 48 registers more.  A's operands are read for a group,
    // in the two sets in turn (FLIP: a step ends on the other set).
    static constexpr int P = 2 * (BK / KG);
    static constexpr int FLIP = (BK / KG) & 1;
    typedef float acc_t __attribute__((ext_vector_type(RB * RB / 64)));
    static_assert(WTM % RB == 0 && WTN % RB == 0 && BK % KG == 0, "whole blocks and groups");
    static_assert(F32 || TN % 2 == 0, "two halves of columns");
    static_assert(AC == 2 || AC == 4 || AC == 8, "a_swz covers these row lengths");
    static_assert(F32 || BC == 8 || BC >= 16, "b_swz stays within a row");

    // Chunk c of A row r lies in slot r AC + (c ^ a_swz(r)).  A read of one
    // chunk by the lanes of a block's rows goes through in groups of lanes
    // 0-3, 12-15, 20-27 and so on; 256 / (16 AC) rows share a bank cycle, so
    // the permutation has to tell rows that far apart from each other.
    static __device__ __forceinline__ int a_swz(int r) {
        if (AC == 8) return (r >> 1) & 7;
        if (AC == 4) return (((r >> 2) ^ (r >> 3)) & 1) << 1 | ((r >> 3) & 1);
        return (r >> 3) & 1;
    }
    // Chunk c of B row k: slot k BC + (c ^ b_swz(k)).  float32 reads whole rows
    // (no permutation).  A bfloat16 transposing read touches 32 bytes of rows
    // k .. k + 3 and, by the next lanes, k + 8 .. k + 11: eight slots of 32
    // bytes of a 256-byte bank cycle.
    static __device__ __forceinline__ int b_swz(int k) {
        if (F32) return 0;
        return BC >= 16 ? ((k & 3) | ((k >> 3) & 1) << 2) << 1 : (((k >> 1) & 1) | ((k >> 3) & 1) << 1) << 1;
    }

    acc_t acc[TM][TN];
    typedef std::conditional_t<F32, f32x4, bf16x8> a_t;
    a_t af[2][TM];                         // a lane's k of a row: four (float32) or eight
    float bf32[2][TN][2];                  // float32: two k of a column
    bf16x8 bf16[2][cmax(TN / 2, 1)];       // bfloat16: eight k of a column
    int lane, wm, wn;

    __device__ __forceinline__ Tile() {
        lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        wm = wave / WN;
        wn = wave % WN;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < RB * RB / 64; ++v) acc[i][j][v] = 0.0f;
    }

    // requests phase p's operands from the tiles at `as` and `bs`
    __device__ __forceinline__ void read(const unsigned char *as, const unsigned char *bs, int p, int par) {
        if ((p & 1) == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i) read_a(as, i, p, par);
        }
        read_b(bs, p);
    }
    // block row i of A; the phase's part of B
    __device__ __forceinline__ void read_a(const unsigned char *as, int i, int p, int par) {
        const int r = lane % RB, h = lane / RB, g = p >> 1, row = wm * WTM + i * RB + r;
        af[(g + par) & 1][i] =
            *reinterpret_cast<const a_t *>(as + (row * AC + ((64 / RB * g + h) ^ a_swz(r))) * 16);
    }
    __device__ __forceinline__ void read_b(const unsigned char *bs, int p) {
        const int g = p >> 1, half = p & 1;
        if constexpr (F32) {
            const int r = lane & 31, h = lane >> 5;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    bf32[half][j][e] = *reinterpret_cast<const float *>(
                        bs + ((8 * g + 4 * h + 2 * half + e) * BN + wn * WTN + j * 32 + r) * 4);
        } else {
            const int m16 = lane & 15, kq = lane >> 4;
            const int k = 8 * kq + (m16 >> 2);  // and k + 4: both in one group of eight rows, of one b_swz
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) {
                const int col = wn * WTN + (half * (TN / 2) + j) * 16 + 4 * (m16 & 3);
                const unsigned char *b = bs + ((32 * g + k) * BC + ((col >> 3) ^ b_swz(k))) * 16 + (col & 7) * 2;
                const s16x4 lo = lds_read_tr16(b), hi = lds_read_tr16(b + 4 * BC * 16);
                bf16[half][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
    }

    // multiplies phase p's operands: block row i, or all
    __device__ __forceinline__ void mul_row(int i, int p, int par) {
        const int half = p & 1, q = ((p >> 1) + par) & 1;
        if constexpr (F32) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(half ? af[q][i][2 + e] : af[q][i][e],
                                                                     bf32[half][j][e], acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) {
                acc_t &c = acc[i][half * (TN / 2) + j];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[q][i], bf16[half][j], c, 0, 0, 0);
            }
        }
    }
    __device__ __forceinline__ void mul(int p, int par) {
#pragma unroll
        for (int i = 0; i < TM; ++i) mul_row(i, p, par);
    }

    // C at the tile's place: stored, added to (accumulate), or, for a share of
    // K, added atomically (C holds zeros or the other shares' sums).  float32:
    // value v of a block is row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane %
    // 32; bfloat16: row 4 (lane / 16) + v, column lane % 16.
    // BATCH: the rows that an accumulation loads at once (below)
    template <int BATCH> __device__ __forceinline__ void store(const MmArgs &a, int row0, int col0) const {
        const gmut<float> C = (gmut<float>)a.C;
        const bool interior = (row0 + BM <= a.M) && (col0 + BN <= a.N);
        // (the choices outside the loops: inside, every store would branch)
        // `put` of each value of rows [first, first + count) of the wavefront's
        // TM RB * RB / 64 of a lane, and whether it lies in C
        auto rows = [&](int first, int count, auto &&put) {
#pragma unroll
            for (int n = first; n < first + count; ++n) {
                const int i = n / (RB * RB / 64), v = n % (RB * RB / 64);
                const int gr = row0 + wm * WTM + i * RB + 4 * (lane / RB) + (F32 ? 8 * (v / 4) + v % 4 : v);
                const gmut<float> p = C + (int64_t)gr * a.ldc + col0 + wn * WTN + lane % RB;
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    put(n - first, j, interior || (gr < a.M && col0 + wn * WTN + j * RB + lane % RB < a.N), p + j * RB,
                        acc[i][j][v]);
            }
        };
        constexpr int ROWS = TM * RB * RB / 64;
        if (a.splits > 1)
            rows(0, ROWS, [](int, int, bool in, gmut<float> p, float x) { if (in) unsafeAtomicAdd((float *)p, x); });
        else if (a.accumulate) {
            // A load behind the store before it waits for memory row by row,
            // so several rows' loads go before their additions (and lanes
            // outside C load a zero: a branch around each load would put waits
            // between them).
            if constexpr (BATCH == 1) {
                rows(0, ROWS, [](int, int, bool in, gmut<float> p, float x) { if (in) *p += x; });
            } else {
                const gptr<float> zero = (gptr<float>)(const void *)kZeroBlock;
#pragma unroll
                for (int n = 0; n < ROWS; n += BATCH) {
                    float c[BATCH][TN];
                    rows(n, BATCH, [&](int k, int j, bool in, gmut<float> p, float) { c[k][j] = *(in ? (gptr<float>)p : zero); });
                    rows(n, BATCH, [&](int k, int j, bool in, gmut<float> p, float x) { if (in) *p = c[k][j] + x; });
                }
            }
        } else if (interior)
            rows(0, ROWS, [](int, int, bool in, gmut<float> p, float x) { if (in) *p = x; });
        else
            rows(0, ROWS, [](int, int, bool in, gmut<float> p, float x) { if (in) *p = x; });
    }

    // Rows an accumulation loads at once: four, or two of four blocks and more
    // (of 32 loads, programs of 512 and 1024 work-items spill).  Row by row
    // before, so now: bfloat16 4596 x 2027 x 40, 47 us and 27; float32 2883 x
    // 1126 x 3, 25 and 15; groups with rows padded to 8, bfloat16 700 of
    // 128-512, 418 and 244, 4096 of 16-512, 660 and 399, float32 798 and 626,
    // packed 857 and 682.  Grouped float32 kernels without `room`, registers
    // to hold the rows in, keep to one: aligned 64 x 128 tiles would take 104
    // for 96, two-stage unaligned 64 x 64 ones 142 for 128, and a workgroup
    // less would fit.
    static constexpr int batch(bool group, bool room) {
        return group && F32 && !room ? 1 : TN < 4 ? 4 : 2;
    }

    // a wavefront whose part of an edge tile lies wholly outside C has nothing
    // to multiply (it still loads its share of the operand tiles); skipping
    // its products frees the matrix unit for the other wavefronts
    __device__ __forceinline__ bool idle(const MmArgs &a, int row0, int col0) const {
        return row0 + wm * WTM >= a.M || col0 + wn * WTN >= a.N;
    }
};

// ------------------------------------------------------------------ loads straight to LDS
// 16 bytes a lane from `base` + voff to LDS, lane l's at `lds` + 16 l (`lds`
// uniform).  In asm because the compiler, which cannot tell the buffers apart,
// would wait for every such load before any LDS read; its one output is a
// scalar copy, and the waits are dma_tile's own (below).  A scalar pair that a
// vector instruction wrote must rest five states before a load may read it as
// its base, which the compiler sees to for its own loads but not in here: the
// load reads a copy by the scalar unit, which also is the state between the
// writing of m0 and its use.  (m0 is no register that the compiler allocates,
// hence its warning; the clobber tells it that a value of its own there is gone.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds16(uint32_t voff, const unsigned char *base, uint32_t lds) {
    uint64_t at;
    asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(at)
                 : "v"(voff), "s"(base), "s"(lds)
                 : "memory", "m0");
}
#pragma clang diagnostic pop
// The LDS from `p` on, as memory of an extent the compiler does not know: an
// address past the end of the object at `p`, in the LDS that a launch adds
// behind it, is then as defined as one inside.  (Taken from the object itself,
// such addresses are out of bounds, and the compiler may drop or reorder what
// reads there.)  The kernel has no other LDS object, so the added part follows.
__device__ __forceinline__ unsigned char *lds_pool(unsigned char *p) {
    uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)p;
    asm("" : "+s"(at));
    return (unsigned char *)(__attribute__((address_space(3))) unsigned char *)(uintptr_t)at;
}
// waits until at most N of the wavefront's memory operations are outstanding
// (they complete in order)
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// waits for the wavefront's LDS operations, then for the workgroup
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One BM x BN output tile at (row0, col0) over the K steps [kt0, kt1) of BK
// each, rows 16-byte aligned and a buffer's rows within kMaxDmaReach of its
// first (so that chunks' offsets fit 32 bits).  SBK: K extent of a buffer; a.depth of
// them from `object` on, two to MAX_DEPTH, the last ones perhaps in LDS that the
// launch adds (dma_depth in the host library).  The caller synchronises the workgroup
// before the call and before using the LDS otherwise.
//
// A step's last phase opens the next step: its loads have arrived in this
// wavefront's view (wait_loads) and, after the barrier, in all of them, and
// every wavefront has read the last of this step's buffer, which the loads of
// the step DEPTH further then fill.  What bounds it: at two buffers, the
// memory latency that one step of products does not cover when operands come
// from HBM (all workgroups of an XCD meet a panel's first touch together);
// bfloat16 of order 4096 on 128 x 256 x 32, 146 us with two and 124 with three.
template <int EB, int BM, int BN, int BK, int SBK, int WM, int WN, int MAX_DEPTH, bool GROUP>
__device__ __forceinline__ void dma_tile(const MmArgs &a, const int row0, const int col0, unsigned char *const object,
                                         const int kt0, const int kt1) {
    unsigned char *const lds = MAX_DEPTH > 2 ? lds_pool(object) : object;
    using T = Tile<EB, BM, BN, SBK, WM, WN>;
    constexpr int NT = T::NT, VE = T::VE, P = T::P;
    constexpr int LOADS = T::AL + T::BL;  // per work-item and step
    static_assert((MAX_DEPTH - 1) * LOADS < 64, "steps under way fit the wait's counter");
    static_assert(BM <= kLargestTile && SBK <= kLargestBuffer, "the host's rule for every program at once");
    T t;
    const int tid = threadIdx.x;
    const int K = min(kt1 * BK, a.K) - kt0 * BK;        // of this tile's share
    const int KF = K / SBK, KS = (K + SBK - 1) / SBK;   // whole steps, steps
    const unsigned char *ab = (const unsigned char *)a.A + ((int64_t)row0 * a.lda + (int64_t)kt0 * BK) * EB;
    const unsigned char *bb = (const unsigned char *)a.B + ((int64_t)kt0 * BK * a.ldb + col0) * EB;
    const int64_t bstep = (int64_t)SBK * a.ldb * EB;
    uint32_t va[T::AL], vb[T::BL];  // byte offsets of this work-item's chunks
#pragma unroll
    for (int u = 0; u < T::AL; ++u) {
        const int f = (tid + u * NT) % (BM * T::AC), r = f / T::AC, c = (f % T::AC) ^ T::a_swz(r);
        va[u] = ((uint32_t)min(r, a.M - 1 - row0) * (uint32_t)a.lda + c * VE) * EB;
    }
    const int clast = ((a.N - 1) & ~(VE - 1)) - col0;
#pragma unroll
    for (int u = 0; u < T::BL; ++u) {
        const int f = (tid + u * NT) % (SBK * T::BC), r = f / T::BC, c = (f % T::BC) ^ T::b_swz(r);
        vb[u] = ((uint32_t)r * (uint32_t)a.ldb + min(c * VE, clast)) * EB;
    }
    // this wavefront's part of the tiles' slots
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lbase = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds);
    auto a_slot = [&](int at, int u) { return lbase + at + ((wave * 64 + u * NT) % (BM * T::AC)) * 16; };
    auto b_slot = [&](int at, int u) { return lbase + at + T::A_BYTES + ((wave * 64 + u * NT) % (SBK * T::BC)) * 16; };
    // requests the next step (steps are requested in order) into the buffer
    // at byte `at` of the LDS
    auto load = [&](int at) {
#pragma unroll
        for (int u = 0; u < T::AL; ++u) load_lds16(va[u], ab, a_slot(at, u));
#pragma unroll
        for (int u = 0; u < T::BL; ++u) load_lds16(vb[u], bb, b_slot(at, u));
        ab += SBK * EB;
        bb += bstep;
    };
    // the same for a last step of `rest` < SBK k: chunks and rows past them
    // read the last one in range (its offset fits where theirs may not have:
    // all of this is modulo 2^32)
    const int rest = K - KF * SBK;
    auto load_rest = [&](int at) {
        const int kl = (rest - 1) & ~(VE - 1);
#pragma unroll
        for (int u = 0; u < T::AL; ++u) {
            const int f = (tid + u * NT) % (BM * T::AC), k = ((f % T::AC) ^ T::a_swz(f / T::AC)) * VE;
            load_lds16(va[u] - (uint32_t)max(k - kl, 0) * EB, ab, a_slot(at, u));
        }
#pragma unroll
        for (int u = 0; u < T::BL; ++u) {
            const int r = (tid + u * NT) % (SBK * T::BC) / T::BC;
            load_lds16(vb[u] - (uint32_t)max(r - (rest - 1), 0) * (uint32_t)a.ldb * EB, bb, b_slot(at, u));
        }
    };
    auto load_step = [&](int kt, int at) {
        if (kt < KF)
            load(at);
        else if (kt < KS)
            load_rest(at);
    };
    // zeros at k >= rest in this work-item's own chunks, which have arrived
    auto clear_rest = [&](int at) {
        unsigned char *const la = lds + at, *const lb = la + T::A_BYTES;
#pragma unroll
        for (int u = 0; u < T::AL; ++u) {
            const int f = (tid + u * NT) % (BM * T::AC), k = ((f % T::AC) ^ T::a_swz(f / T::AC)) * VE;
            if (k + VE > rest) {
                u32x4 v = *reinterpret_cast<const u32x4 *>(la + f * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if constexpr (T::F32)
                        v[e] = k + e < rest ? v[e] : 0u;
                    else  // word e holds k + 2e (low half) and k + 2e + 1 (high half)
                        v[e] &= k + 2 * e + 1 < rest ? 0xffffffffu : (k + 2 * e < rest ? 0x0000ffffu : 0u);
                *reinterpret_cast<u32x4 *>(la + f * 16) = v;
            }
        }
#pragma unroll
        for (int u = 0; u < T::BL; ++u) {
            const int f = (tid + u * NT) % (SBK * T::BC);
            if (f / T::BC >= rest) *reinterpret_cast<u32x4 *>(lb + f * 16) = u32x4{0u, 0u, 0u, 0u};
        }
    };
    const bool idle = t.idle(a, row0, col0);
    // (the code of a depth's own: buffers, waits and operand sets constant)
    auto run = [&](auto depth) {
        constexpr int DEPTH = decltype(depth)::value;
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) load_step(s, s * T::BYTES);
        if (KS >= DEPTH)
            wait_loads<(DEPTH - 1) * LOADS>();
        else
            wait_loads<0>();
        if (KF == 0) clear_rest(0);
        lds_barrier();
        t.read(lds, lds + T::A_BYTES, 0, 0);
        // step kt, in buffer buf, whose phase 0 is on its way.  FULL: all of
        // its k and of the next DEPTH steps' in range
        auto step = [&](int kt, int buf, int par, auto full) {
            constexpr bool FULL = decltype(full)::value;
            const int at = buf * T::BYTES, next = buf + 1 == DEPTH ? 0 : at + T::BYTES;
            const int kn = FULL ? SBK : min(K - kt * SBK, SBK);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (p + 1 < P) {
                    t.read(lds + at, lds + at + T::A_BYTES, p + 1, par);
                } else if (FULL || kt + 1 < KS) {
                    if (FULL || kt + DEPTH <= KS)
                        wait_loads<(DEPTH - 2) * LOADS>();
                    else
                        wait_loads<0>();
                    if (!FULL && kt + 1 >= KF) clear_rest(next);
                    lds_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                    t.read(lds + next, lds + next + T::A_BYTES, 0, par ^ T::FLIP);
                    if (FULL)
                        load(at);
                    else
                        load_step(kt + DEPTH, at);
                }
                __builtin_amdgcn_sched_barrier(0);
                // (groups past the end of K are zeros: nothing to multiply)
                if (FULL || (!idle && (p >> 1) * T::KG < kn)) t.mul(p, par);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // a round returns to the first buffer and operand set
        constexpr int ROUND = T::FLIP && DEPTH % 2 ? 2 * DEPTH : DEPTH;
        int kt = 0;
        if (!idle)
            for (; kt + ROUND - 1 + DEPTH < KF; kt += ROUND) {
#pragma unroll
                for (int s = 0; s < ROUND; ++s) step(kt + s, s % DEPTH, s & T::FLIP, std::true_type{});
            }
        int buf = 0;
        for (; kt < KS; kt += 2) {
            step(kt, buf, 0, std::false_type{});
            buf = buf + 1 == DEPTH ? 0 : buf + 1;
            if (kt + 1 < KS) step(kt + 1, buf, T::FLIP, std::false_type{});
            buf = buf + 1 == DEPTH ? 0 : buf + 1;
        }
    };
    if (KS > 0) {
        if (MAX_DEPTH == 2 || a.depth == 2)
            run(std::integral_constant<int, 2>{});
        else if (MAX_DEPTH == 3 || a.depth == 3)
            run(std::integral_constant<int, cmin(3, MAX_DEPTH)>{});
        else
            run(std::integral_constant<int, MAX_DEPTH>{});
    }
    t.template store<T::batch(GROUP, T::TN == 1 || T::TM > 1)>(a, row0, col0);
}

// ------------------------------------------------------------------ loads through registers
// The same tile with chunks through registers: STAGES buffers of BK at `lds`.
// WIDE: rows 16-byte aligned (else chunks are read at element alignment).
// EDGE_ADDR: edge chunks at chosen addresses; else (float32 twins whose fixups
// would spill at their register cap) guarded loads, element by element at the
// edges -- and everywhere in the large single-stage ones (CHUNKS false), where
// the wide form of the guards would spill.
template <int EB, int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE, bool EDGE_ADDR, bool GROUP>
__device__ __forceinline__ void regs_tile(const MmArgs &a, const int row0, const int col0, unsigned char *const lds,
                                          const int kt0, const int kt1) {
    using T = Tile<EB, BM, BN, BK, WM, WN>;
    constexpr int NT = T::NT, VE = T::VE, AC = T::AC, BC = T::BC, AL = T::AL, BL = T::BL;
    static_assert(BM * AC % NT == 0 && BK * BC % NT == 0, "whole loads");
    constexpr bool CHUNKS = WIDE || EDGE_ADDR || WM * WN >= 16;
    // one block row's operands at a time, where more would spill at the
    // register cap
    constexpr bool LEAN = NT >= 512 || (EB == 2 && BM * BN >= 128 * 128);
    using elem = std::conditional_t<EB == 4, uint32_t, unsigned short>;
    typedef elem elems __attribute__((ext_vector_type(VE)));
    typedef typename ChunkAt<EB, WIDE>::type chunk;
    T t;
    // the operands from this share's first K step on: its steps run from 0,
    // and K counts what is left of the product from there
    const gptr<elem> __restrict__ A = (gptr<elem>)a.A + kt0 * BK;
    const gptr<elem> __restrict__ B = (gptr<elem>)a.B + (int64_t)kt0 * BK * a.ldb;
    const int M = a.M, N = a.N, K = a.K - kt0 * BK;
    const int tid = threadIdx.x;
    const bool interior = (row0 + BM <= M) && (col0 + BN <= N);
    const bool idle = NT <= 512 && t.idle(a, row0, col0);  // (1024 work-items: registers at the limit)

    // the chunks of one K step
    struct Set {
        u32x4 a[AL], b[BL];
    };
    constexpr int SETS = STAGES == 1 || NT >= 512 ? 1 : AL + BL <= 4 ? (EB == 2 ? 4 : 2) : AL + BL <= 8 && EB == 2 ? 2 : 1;
    // row and first element of this work-item's u-th chunks
    auto a_row = [&](int u) { return (tid + u * NT) / AC; };
    auto a_k = [&](int u) { return (tid + u * NT) % AC * VE; };
    auto b_row = [&](int u) { return (tid + u * NT) / BC; };
    auto b_col = [&](int u) { return (tid + u * NT) % BC * VE; };
    const bool tiny = !WIDE && (a.K < VE || N < VE);
    const int sk = WIDE ? 0 : (VE - (K & (VE - 1))) & (VE - 1), sn = WIDE ? 0 : (VE - (N & (VE - 1))) & (VE - 1);
    const int klast = WIDE ? (K - 1) & ~(VE - 1) : K - VE, nlast = WIDE ? (N - 1) & ~(VE - 1) : N - VE;
    // A step all of whose k are in range, in a tile that lies inside the
    // operands or whose edge chunks are read at chosen addresses (see below):
    // no guards, so the loads issue back to back (guarded loads branch per
    // load, and the compiler then waits for each load before the next).
    auto gload_fast = [&](Set &set, int k0) {
#pragma unroll
        for (int u = 0; u < AL; ++u) {
            const int gr = row0 + a_row(u);
            set.a[u] = *reinterpret_cast<gptr<chunk>>(A + (int64_t)(EDGE_ADDR ? min(gr, M - 1) : gr) * a.lda + k0 + a_k(u));
        }
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const int gc = col0 + b_col(u);
            set.b[u] = *reinterpret_cast<gptr<chunk>>(B + (int64_t)(k0 + b_row(u)) * a.ldb + (EDGE_ADDR ? min(gc, nlast) : gc));
        }
    };
    // Any K step.  EDGE_ADDR: rows of A past M read row M - 1 and columns of B
    // past N a chunk inside N; rows of B at k >= K read a block of zeros.
    // Aligned rows: a chunk across k = K or column N is read whole (it holds
    // an element of the matrix, so it lies inside its aligned row).
    // Unaligned rows: such a chunk is read ending at the row's last element
    // and shifted down by sk (A) or sn (B) elements by fixup, when it goes to
    // LDS, so that the load stays in flight during the products.  Unaligned
    // rows shorter than a chunk (tiny): element loads.
    auto gload = [&](Set &set, int k0) {
        if constexpr (!EDGE_ADDR) {
            const bool kfull = (k0 + BK <= K);
#pragma unroll
            for (int u = 0; u < AL; ++u) {
                const int gr = row0 + a_row(u), gc = k0 + a_k(u);
                if (CHUNKS && kfull && gr < M) {
                    set.a[u] = *reinterpret_cast<gptr<chunk>>(A + (int64_t)gr * a.lda + gc);
                } else {
                    elems v;
#pragma unroll
                    for (int e = 0; e < VE; ++e)
                        v[e] = (gr < M && gc + e < K) ? A[(int64_t)gr * a.lda + gc + e] : elem(0);
                    set.a[u] = __builtin_bit_cast(u32x4, v);
                }
                if constexpr (LEAN) __builtin_amdgcn_sched_barrier(0);  // (one chunk's addresses at a time)
            }
#pragma unroll
            for (int u = 0; u < BL; ++u) {
                const int gr = k0 + b_row(u), gc = col0 + b_col(u);
                if (CHUNKS && gr < K && gc + VE <= N) {
                    set.b[u] = *reinterpret_cast<gptr<chunk>>(B + (int64_t)gr * a.ldb + gc);
                } else {
                    elems v;
#pragma unroll
                    for (int e = 0; e < VE; ++e)
                        v[e] = (gr < K && gc + e < N) ? B[(int64_t)gr * a.ldb + gc + e] : elem(0);
                    set.b[u] = __builtin_bit_cast(u32x4, v);
                }
                if constexpr (LEAN) __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        if (!tiny) {
#pragma unroll
            for (int u = 0; u < AL; ++u)
                set.a[u] = *reinterpret_cast<gptr<chunk>>(A + (int64_t)min(row0 + a_row(u), M - 1) * a.lda +
                                                       min(k0 + a_k(u), klast));
#pragma unroll
            for (int u = 0; u < BL; ++u) {
                const int k = k0 + b_row(u);
                set.b[u] = *(k < K ? reinterpret_cast<gptr<chunk>>(B + (int64_t)k * a.ldb + min(col0 + b_col(u), nlast))
                                : (gptr<chunk>)(const void *)kZeroBlock);
            }
            return;
        }
        const gptr<elem> zero = (gptr<elem>)(const void *)kZeroBlock;
#pragma unroll
        for (int u = 0; u < AL; ++u) {
            const gptr<elem> row = A + (int64_t)min(row0 + a_row(u), M - 1) * a.lda;
            elems v;
#pragma unroll
            for (int e = 0; e < VE; ++e) {
                const int k = k0 + a_k(u) + e;
                v[e] = *(k < K ? row + k : zero);
            }
            set.a[u] = __builtin_bit_cast(u32x4, v);
        }
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const int k = k0 + b_row(u);
            const gptr<elem> row = k < K ? B + (int64_t)k * a.ldb : nullptr;
            elems v;
#pragma unroll
            for (int e = 0; e < VE; ++e) v[e] = *(row ? row + min(col0 + b_col(u) + e, N - 1) : zero);
            set.b[u] = __builtin_bit_cast(u32x4, v);
        }
    };
    // what the chunks of an edge step at k0 become before they go to LDS
    auto fixup = [&](Set &set, int k0) {
        if constexpr (!EDGE_ADDR) return;
        if (tiny) return;
        if (k0 + BK > K) {
#pragma unroll
            for (int u = 0; u < AL; ++u) {
                const int k = k0 + a_k(u);
                if constexpr (!WIDE) {
                    const u32x4 s = chunk_from<EB>(set.a[u], sk);
#pragma unroll
                    for (int e = 0; e < 4; ++e) set.a[u][e] = k + VE <= K ? set.a[u][e] : k < K ? s[e] : 0u;
                } else if constexpr (EB == 4) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) set.a[u][e] = k + e < K ? set.a[u][e] : 0u;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)  // word e holds k + 2e (low half) and k + 2e + 1 (high half)
                        set.a[u][e] &= k + 2 * e + 1 < K ? 0xffffffffu : (k + 2 * e < K ? 0x0000ffffu : 0u);
                }
            }
        }
        if (!WIDE && sn && col0 + BN > N) {
#pragma unroll
            for (int u = 0; u < BL; ++u) {
                const u32x4 s = chunk_from<EB>(set.b[u], sn);
                const bool whole = col0 + b_col(u) + VE <= N;
#pragma unroll
                for (int e = 0; e < 4; ++e) set.b[u][e] = whole ? set.b[u][e] : s[e];
            }
        }
    };
    auto sstore = [&](const Set &set, int st) {
        unsigned char *const la = lds + st * T::BYTES, *const lb = la + T::A_BYTES;
#pragma unroll
        for (int u = 0; u < AL; ++u) {
            const int r = a_row(u);
            *reinterpret_cast<u32x4 *>(la + (r * AC + (a_k(u) / VE ^ T::a_swz(r))) * 16) = set.a[u];
        }
#pragma unroll
        for (int u = 0; u < BL; ++u) {
            const int r = b_row(u);
            *reinterpret_cast<u32x4 *>(lb + (r * BC + (b_col(u) / VE ^ T::b_swz(r))) * 16) = set.b[u];
        }
    };
    auto compute = [&](int st) {
        const unsigned char *const la = lds + st * T::BYTES, *const lb = la + T::A_BYTES;
        // (and operand addresses made anew each step, not held across it)
        if constexpr (LEAN) asm volatile("" : "+v"(t.lane));
#pragma unroll
        for (int p = 0; p < T::P; ++p) {
            if constexpr (LEAN) {
                t.read_b(lb, p);
#pragma unroll
                for (int i = 0; i < T::TM; ++i) {
                    t.read_a(la, i, p, 0);
                    t.mul_row(i, p, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                t.read(la, lb, p, 0);
                t.mul(p, 0);
            }
        }
    };
    const int KT = kt1 - kt0;
    const int KF = (EDGE_ADDR ? !tiny : CHUNKS && interior) ? min(K / BK, KT) : 0;  // leading steps without guards
    auto load = [&](Set &set, int kt) {
        if (kt < KF)
            gload_fast(set, kt * BK);
        else if (kt < KT)
            gload(set, kt * BK);
    };
    if constexpr (STAGES == 2 && NT >= 1024) {
        // at the register limit: step kt + 1's loads in flight while step kt
        // multiplies, no further ahead
        Set s0;
        load(s0, 0);
        if (KT > 0) {
            fixup(s0, 0);
            sstore(s0, 0);
        }
        lds_barrier();
        int kt = 0;
        for (; kt + 1 < KF; ++kt) {
            gload_fast(s0, (kt + 1) * BK);
            __builtin_amdgcn_sched_barrier(0);
            compute(kt & 1);
            sstore(s0, (kt + 1) & 1);
            lds_barrier();
        }
        for (; kt < KT; ++kt) {
            load(s0, kt + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(kt & 1);
            if (kt + 1 < KT) {
                fixup(s0, (kt + 1) * BK);
                sstore(s0, (kt + 1) & 1);
            }
            lds_barrier();
        }
    } else if constexpr (STAGES == 2) {
        // Step k's chunks are in set k mod SETS.  A step multiplies out of one
        // buffer, then stores the next step's chunks to the other and sends
        // out the loads of the step SETS further into their registers: with
        // one set a step's products do not cover the memory latency (packed
        // rows: float32 1531 x 777 x 1201 43.1 us with one set, 41.2 with two;
        // bfloat16 1021 x 3001 x 2047 39.6 with one, 36.9 with four).
        constexpr int U = SETS > 2 ? SETS : 2;  // steps of a round: static sets and buffers
        Set s0, s1, s2, s3;
        auto step = [&](Set &set, int kt, int cur, auto full_) {
            constexpr bool full = decltype(full_)::value;
            if (full || !idle) compute(cur);
            if (full || kt + 1 < KT) {
                fixup(set, (kt + 1) * BK);
                sstore(set, cur ^ 1);
                if constexpr (full)
                    gload_fast(set, (kt + 1 + SETS) * BK);
                else
                    load(set, kt + 1 + SETS);
            }
            lds_barrier();
        };
        auto round = [&](int kt, auto full_) {
            constexpr bool full = decltype(full_)::value;
            step(SETS > 1 ? s1 : s0, kt, 0, full_);
            if (full || kt + 1 < KT) step(SETS > 2 ? s2 : s0, kt + 1, 1, full_);
            if constexpr (U == 4) {
                if (full || kt + 2 < KT) step(s3, kt + 2, 0, full_);
                if (full || kt + 3 < KT) step(s0, kt + 3, 1, full_);
            }
        };
        if (KT > 0) {
            load(s0, 0);
            if constexpr (SETS > 1) load(s1, 1);
            if constexpr (SETS > 2) {
                load(s2, 2);
                load(s3, 3);
            }
            fixup(s0, 0);
            sstore(s0, 0);
            load(s0, SETS);
        }
        lds_barrier();
        int kt = 0;
        for (; kt + U + SETS < KF; kt += U) round(kt, std::true_type{});
        for (; kt < KT; kt += U) round(kt, std::false_type{});
    } else {
        // one LDS buffer: step kt + 1's loads are in flight (in registers)
        // while step kt multiplies out of LDS.  Left to itself, the compiler's
        // scheduler sinks them to the end of the step (shortening their
        // registers' lives) and the step then waits out a whole memory
        // latency: a scheduling barrier keeps them ahead of the products.
        Set s0;
        load(s0, 0);
        int kt = 0;
        for (; kt + 1 < KF; ++kt) {
            if constexpr (!WIDE) fixup(s0, kt * BK);
            __syncthreads();  // the previous step's LDS reads are done
            sstore(s0, 0);
            __syncthreads();
            gload_fast(s0, (kt + 1) * BK);
            __builtin_amdgcn_sched_barrier(0);
            compute(0);
        }
        for (; kt < KT; ++kt) {
            fixup(s0, kt * BK);
            __syncthreads();
            sstore(s0, 0);
            __syncthreads();
            load(s0, kt + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (!idle) compute(0);
        }
    }
    t.template store<T::batch(GROUP, STAGES == 1 || T::TN > 1)>(a, row0, col0);
}

// The tile by the way that its program and its rows' alignment take.
template <int EB, int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE, int MAX_DEPTH, bool GROUP = false>
__device__ __forceinline__ void mfma_tile(const MmArgs &a, int row0, int col0, unsigned char *lds, int kt0, int kt1) {
    constexpr int SBK = buffer_k(BK, STAGES == 1);
    constexpr bool DMA = WIDE && loads_directly(EB == 4, BK, STAGES == 1, WM, WN);
    // the largest tiles' guarded loads: see regs_tile
    constexpr bool EDGE = WM * WN < 16 && (EB == 2 || STAGES == 2 || BM * BN * BK <= 128 * 256 * 16);
    if constexpr (DMA)
        dma_tile<EB, BM, BN, BK, SBK, WM, WN, MAX_DEPTH, GROUP>(a, row0, col0, lds, kt0, kt1);
    else
        regs_tile<EB, BM, BN, BK, WM, WN, STAGES, WIDE, EDGE, GROUP>(a, row0, col0, lds, kt0, kt1);
}

// ------------------------------------------------------------------ single product
// Split along K (a.splits = S > 1): the grid holds S x tiles workgroups, share
// by share; workgroup b takes share b / tiles of tile b % tiles, the K steps
// [KT s / S, KT (s + 1) / S) of the product's KT = ceil(K / BK).  Programs of
// 1024 work-items are never split (kSplittableThreads): their registers are
// at the limit already.
template <int BK>
__device__ __forceinline__ void k_share(const MmArgs &a, uint32_t tiles, uint32_t *b, int *kt0, int *kt1) {
    const int KT = (a.K + BK - 1) / BK;
    *kt0 = 0;
    *kt1 = KT;
    if (a.splits > 1) {
        const uint32_t s = *b / tiles;
        *b -= s * tiles;
        *kt0 = (int)((uint32_t)KT * (uint64_t)s / (uint32_t)a.splits);
        *kt1 = (int)((uint32_t)KT * (uint64_t)(s + 1) / (uint32_t)a.splits);
    }
}

// WIDE: 16-byte loads along aligned rows; the element-load twin (WIDE =
// false: 16-byte loads at element alignment) is a kernel of its own, so
// neither carries the other's load path.  SPLIT: the kernel runs shares of K
// (a.splits > 1); the wide program's split form is a kernel of its own too,
// so the whole-product kernel carries none of it (the element-load twins
// split in place).
template <int EB, int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE, bool SPLIT>
__device__ __forceinline__ void mfma_product(const MmArgs &a0, unsigned char *lds) {
    MmArgs a = a0;
    if constexpr (!SPLIT || 64 * WM * WN > kSplittableThreads) a.splits = 0;
    int tm, tn;
    uint32_t b = blockIdx.x;
    const uint32_t tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
    int kt0, kt1;
    k_share<BK>(a, tiles_m * tiles_n, &b, &kt0, &kt1);
    tile_of(b, tiles_m, tiles_n, &tm, &tn);
    mfma_tile<EB, BM, BN, BK, WM, WN, STAGES, WIDE, max_depth(EB == 4, BM, BN, WM, WN)>(a, tm * BM, tn * BN, lds, kt0, kt1);
}

template <int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE = true, bool SPLIT = !WIDE>
__device__ __forceinline__ void mfma_f32(const MmArgs &a) {
    __shared__ __attribute__((aligned(256))) unsigned char lds[f32_lds(BM, BN, BK, STAGES)];
    mfma_product<4, BM, BN, BK, WM, WN, STAGES, WIDE, SPLIT>(a, lds);
}

template <int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE = true, bool SPLIT = !WIDE>
__device__ __forceinline__ void mfma_bf16(const MmArgs &a) {
    __shared__ __attribute__((aligned(256))) unsigned char lds[bf16_lds(BM, BN, BK, STAGES)];
    mfma_product<2, BM, BN, BK, WM, WN, STAGES, WIDE, SPLIT>(a, lds);
}

// ------------------------------------------------------------------ grouped (persistent)
// Many independent products in one launch; tile t belongs to group
// tile_group[t] and is tile t - tile_start of that group, numbered row-major
// over its tiles (a product's tiles are consecutive).  Workgroup b runs on XCD
// b % 8, so XCD x is given the tile range [bin_first[x], bin_first[x + 1]),
// which its workgroups stride over: a product's tiles then share one XCD's L2
// (striding over all tiles would spread them over every XCD and fetch the same
// panels into eight caches).  The host orders and cuts the ranges (by
// estimated cost, most expensive tiles first).  Grids of fewer than 8
// workgroups stride over all tiles.
struct GroupWalk {
    int64_t t, end, stride;
    __device__ __forceinline__ explicit GroupWalk(const GroupArgs &g) {
        const int64_t G = gridDim.x, b = blockIdx.x;
        if (G < kXcds) {
            t = b;
            end = g.total_tiles;
            stride = G;
        } else {
            const int x = (int)(b % kXcds);
            t = g.bin_first[x] + b / kXcds;
            end = g.bin_first[x + 1];
            stride = (G - x + kXcds - 1) / kXcds;  // workgroups on XCD x
        }
    }
};

// Runs tile(d, local) for each tile of the workgroup's walk: d the tile's
// product, local its tile index within the product (a product's tiles fit 32
// bits).  The loads a tile's setup waits on are requested a tile early: the
// next tile's descriptor and the product index of the tile after it are
// loaded before the current tile runs (their latency otherwise opens every
// tile, and tiles here run only a few K steps).  The indices are uniform
// over the workgroup and the map and descriptors do not change while the
// kernel runs, so they are read as constants (through the scalar cache).
__device__ __forceinline__ int32_t const_load(const int32_t *p) {
    return *(const __attribute__((address_space(4))) int32_t *)p;
}

__device__ __forceinline__ GroupDesc const_load(const GroupDesc *p) {
    struct Words {
        uint32_t w[sizeof(GroupDesc) / 4];
    } v;
    static_assert(sizeof(GroupDesc) % 4 == 0, "descriptor of whole words");
    const __attribute__((address_space(4))) uint32_t *q = (const __attribute__((address_space(4))) uint32_t *)p;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(GroupDesc) / 4); ++i) v.w[i] = q[i];
    return __builtin_bit_cast(GroupDesc, v);
}

template <class Tile>
__device__ __forceinline__ void walk_tiles(const GroupArgs &g, Tile &&tile) {
    GroupWalk w(g);
    if (w.t >= w.end) return;
    int gnext = const_load(g.tile_group + w.t);
    GroupDesc d = const_load(g.descs + gnext);
    if (w.t + w.stride < w.end) gnext = const_load(g.tile_group + w.t + w.stride);
    for (; w.t < w.end; w.t += w.stride) {
        const int64_t t2 = w.t + 2 * w.stride;
        const int gafter = t2 < w.end ? const_load(g.tile_group + t2) : gnext;
        const GroupDesc dn = const_load(g.descs + gnext);
        lds_barrier();  // the previous tile's LDS reads are done (its stores need not be)
        tile(d, (int)(w.t - d.tile_start));
        d = dn;
        gnext = gafter;
    }
}

// WIDE: every product of the launch has rows aligned for 16-byte loads (the
// host gives a launch only such products), so the kernel carries no
// element-load path -- fewer registers, one more resident wavefront per SIMD
// for the 64 x 64 programs; the element-load twin (WIDE = false) runs the
// products whose rows are not aligned.
// STREAM (bfloat16, single-stage, aligned rows): through registers all the
// same, for groups too large to stay in the memory-side cache.  What bounds
// those is HBM's latency and how its lines are used: direct loads fetch a row
// of A in pieces of half a K step, 64 bytes of a 128-byte line, and wait for
// each half; through registers a whole step's line is one request.  Fresh
// operands each run, 64 x 128 tiles, rows padded to 8: 2500 products of 16-400
// (295 MB) 97.7 us direct and 86.9 so, 4096 of 16-512 (683 MB) 220 and 203, 300
// of 300-512 (376 MB) 151 and 139; held in the cache, 300 products of 16-512
// (46 MB), 12.4 and 13.5.  Both halves of A's lines requested at once, in four
// half-step buffers, gave half of it (2500 products: 91); whole steps through
// two buffers as much as registers where operands come from HBM (90), but cost
// workgroups, and 10-25 % where they do not.
template <int EB, int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE, bool STREAM = false>
__device__ __forceinline__ void grouped_tile(const GroupArgs &g, const GroupDesc &d, int local, unsigned char *lds) {
    const int tm = local / d.tiles_n, tn = local % d.tiles_n;
    const MmArgs a{d.A, d.B, d.C, d.lda, d.ldb, d.ldc, d.M, d.N, d.K, g.accumulate, WIDE, 0, 2};
    if constexpr (STREAM)
        regs_tile<EB, BM, BN, BK, WM, WN, STAGES, WIDE, true, true>(a, tm * BM, tn * BN, lds, 0, (d.K + BK - 1) / BK);
    else
        mfma_tile<EB, BM, BN, BK, WM, WN, STAGES, WIDE, 2, true>(a, tm * BM, tn * BN, lds, 0, (d.K + BK - 1) / BK);
}

template <int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE>
__device__ __forceinline__ void grouped_f32(const GroupArgs &g) {
    __shared__ __attribute__((aligned(256))) unsigned char lds[f32_lds(BM, BN, BK, STAGES)];
    walk_tiles(g, [&](const GroupDesc &d, int local) { grouped_tile<4, BM, BN, BK, WM, WN, STAGES, WIDE>(g, d, local, lds); });
}

template <int BM, int BN, int BK, int WM, int WN, int STAGES, bool WIDE, bool STREAM = false>
__device__ __forceinline__ void grouped_bf16(const GroupArgs &g) {
    __shared__ __attribute__((aligned(256))) unsigned char lds[bf16_lds(BM, BN, BK, STAGES)];
    walk_tiles(g, [&](const GroupDesc &d, int local) {
        grouped_tile<2, BM, BN, BK, WM, WN, STAGES, WIDE, STREAM>(g, d, local, lds);
    });
}

// Mixed grouped kernels: each product's tiles run the program kMixedTile[prog]
// of its descriptor; one LDS allocation, the largest program's, serves all.
template <int EB, int STAGES> constexpr int mixed_lds() {
    int n = 0;
    for (int p = 0; p < kMixedPrograms; ++p)
        n = cmax(n, EB == 4 ? f32_lds(kMixedTile[p][0], kMixedTile[p][1], kMixedBk[0], STAGES)
                            : bf16_lds(kMixedTile[p][0], kMixedTile[p][1], kMixedBk[2], STAGES));
    return n;
}

template <int EB, int STAGES, bool WIDE, bool STREAM>
__device__ __forceinline__ void grouped_mixed(const GroupArgs &g) {
    static_assert(kMixedPrograms == 4, "one case per program");
    constexpr int BK = kMixedBk[EB == 4 ? 0 : 2];
    __shared__ __attribute__((aligned(256))) unsigned char lds[mixed_lds<EB, STAGES>()];
    walk_tiles(g, [&](const GroupDesc &d, int local) {
        switch (d.prog) {
        case 0: grouped_tile<EB, kMixedTile[0][0], kMixedTile[0][1], BK, 2, 2, STAGES, WIDE, STREAM>(g, d, local, lds); break;
        case 1: grouped_tile<EB, kMixedTile[1][0], kMixedTile[1][1], BK, 2, 2, STAGES, WIDE, STREAM>(g, d, local, lds); break;
        case 2: grouped_tile<EB, kMixedTile[2][0], kMixedTile[2][1], BK, 2, 2, STAGES, WIDE, STREAM>(g, d, local, lds); break;
        default: grouped_tile<EB, kMixedTile[3][0], kMixedTile[3][1], BK, 2, 2, STAGES, WIDE, STREAM>(g, d, local, lds); break;
        }
    });
}

template <int STAGES, bool WIDE> __device__ __forceinline__ void grouped_mixed_f32(const GroupArgs &g) {
    grouped_mixed<4, STAGES, WIDE, false>(g);
}
template <int STAGES, bool WIDE, bool STREAM = false> __device__ __forceinline__ void grouped_mixed_bf16(const GroupArgs &g) {
    grouped_mixed<2, STAGES, WIDE, STREAM>(g);
}

}  // namespace pkk
