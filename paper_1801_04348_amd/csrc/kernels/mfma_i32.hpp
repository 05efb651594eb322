// Wrapping int32 matrix product on the int8 matrix cores, for gfx950: the
// MFMA family's int32 programs (same contract as the float32 ones: C = [C +]
// A B, row-major, any M, N, K; the workgroup -> tile map and the 32 x 32
// block layout of mfma.hpp).
#pragma once

#include <type_traits>

#include "mfma.hpp"

namespace pkk {

// ------------------------------------------------------------------ int32
// The wrapping int32 product on the int8 matrix cores (v_mfma_i32_32x32x32_i8:
// A 32x32 and B 32x32 of int8, C 32x32 of int32 per wavefront).  Every int32 x
// has four signed base-256 digits, x = sum_p d_p 256^p (mod 2^32) with d_p in
// [-128, 127]: the bytes of y = x + 0x80808080 (each byte v of y stands for
// v - 128), i.e. the bytes of y ^ 0x80808080 read as int8.  So
//   a b = sum over p + q <= 3 of 256^(p+q) d_p(a) d_q(b)   (mod 2^32):
// ten int8 products per pair of operand blocks, summed into four int32
// accumulators by p + q.  Each accumulator wraps modulo 2^32 as the result
// does, so combining them at the end, acc0 + 2^8 acc1 + 2^16 acc2 + 2^24
// acc3, gives the wrapped product exactly for every K.
// LDS, per stage: the four digit planes of the A tile (BM rows of BK bytes,
// k contiguous, rows BK + 16 bytes apart) and of the B tile stored by column
// (BN columns of BK bytes, k contiguous): 4 (BM + BN) (BK + 16) bytes.  With
// rows BK + 16 bytes apart (48 or 80) the sixteen 16-byte reads of a quarter
// wavefront, one per row, cover 64 distinct banks.  The stores of the digits do
// not: a third of a conflict cycle per LDS cycle, with the LDS busy 19 % (order
// 1024) to 46 % (order 4096) of the time.
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

template <int BM, int BN, int BK, int STAGES> struct I32Lds {
    static constexpr int LD = BK + 16;                      // bytes per plane row
    static constexpr int A = 4 * BM * LD, B = 4 * BN * LD;  // bytes per stage
    static constexpr int bytes = STAGES * (A + B);
};

// The digit planes of four int32 values x[0..3] (consecutive k): byte e of
// plane word p is digit p of x[e].  A transposition of 4 x 4 bytes: eight
// permutations.
__device__ __forceinline__ i32x4 digit_planes(const i32x4 x) {
    uint32_t y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = ((uint32_t)x[e] + 0x80808080u) ^ 0x80808080u;
    // the low (l) and high (h) two digits of each pair of values
    const uint32_t l0 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400), h0 = __builtin_amdgcn_perm(y[1], y[0], 0x07030602);
    const uint32_t l1 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400), h1 = __builtin_amdgcn_perm(y[3], y[2], 0x07030602);
    return i32x4{(int)__builtin_amdgcn_perm(l1, l0, 0x05040100), (int)__builtin_amdgcn_perm(l1, l0, 0x07060302),
                 (int)__builtin_amdgcn_perm(h1, h0, 0x05040100), (int)__builtin_amdgcn_perm(h1, h0, 0x07060302)};
}

// int32 tile (the whole K range).  A is read in 16-byte chunks of four k along
// its rows, at element alignment; B element by element, four consecutive k of
// one column per work-item (lanes along the row: each load instruction reads
// 256 contiguous bytes).  Rows of A past M and columns of B past N read the
// last row / column (their results are never stored); elements at k >= K are
// zeros (whose digits are zeros).
//
// What bounds it: a wavefront's instructions, one every four cycles.  The
// matrix cores need 320 cycles for a 32 x 32 block of a K step of 32, and the
// step takes about 140 instructions beside (64 of them split the work-item's
// operands into digits), which only a second wavefront on the SIMD can overlap
// in full.  So everything a step waits for is under way before it: loads go
// out SETS + 1 steps ahead of their use, the digits of step k + 1 are made and
// stored while step k multiplies, and a barrier in the middle of the step lets
// its second half read the next step's first digits.  Order 1024 (a 64 x 64
// tile a compute unit): 28.2 us loading one step ahead, splitting after the
// products and with shifts instead of byte permutations, 20.6 so; order 2048:
// 123 and 93.
template <int BM, int BN, int BK, int WM, int WN, int STAGES>
__device__ __forceinline__ void mfma_i32_tile(const MmArgs &a, const int row0, const int col0,
                                              unsigned char *const As0, unsigned char *const Bs0) {
    constexpr int NT = 64 * WM * WN;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    using L = I32Lds<BM, BN, BK, STAGES>;
    constexpr int LD = L::LD;
    constexpr int AQ = BM * BK / 4 / NT;  // quads (four consecutive k) of A per work-item per step
    constexpr int BQ = BK * BN / 4 / NT;  // quads of B
    constexpr int SETS = TM * TN == 1 ? 2 : 1;       // register sets of loads in flight
    constexpr int BLOCKS = TM * TN * (BK / 32);       // 32 x 32 x 32 blocks of a wavefront's step
    static_assert(BLOCKS == 1 || BLOCKS == 2, "a step in two halves");
    static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be 32x32 blocks");
    static_assert(AQ >= 1 && BQ >= 1 && (BM * BK / 4) % NT == 0 && (BK * BN / 4) % NT == 0, "tile loads");
    static_assert(BK % 32 == 0, "BK: whole MFMA steps in each half of the tile");
    typedef int chunk __attribute__((ext_vector_type(4), aligned(4)));

    const gptr<int32_t> __restrict__ A = (gptr<int32_t>)a.A;
    const gptr<int32_t> __restrict__ B = (gptr<int32_t>)a.B;
    const gmut<int32_t> __restrict__ C = (gmut<int32_t>)a.C;
    const int M = a.M, N = a.N, K = a.K;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 31, h = lane >> 5;
    const bool interior = (row0 + BM <= M) && (col0 + BN <= N);

    i32x16 acc[4][TM][TN];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[s][i][j][v] = 0;

    // each work-item's rows of A, fixed for the tile (the 64-bit address
    // arithmetic done once, not per load and step)
    static_assert(NT % (BK / 4) == 0 && NT % BN == 0 && BN % 64 == 0, "a work-item's A column and B column stay fixed");
    const int akq = 4 * (tid % (BK / 4));  // k offset of the work-item's A quads in a step
    // (rows below the first as 32-bit distances: fewer registers)
    const int ar = min(row0 + tid / (BK / 4), M - 1);
    const gptr<int32_t> arow = A + (int64_t)ar * a.lda + akq;
    int down[AQ];
#pragma unroll
    for (int u = 0; u < AQ; ++u) down[u] = min(row0 + (tid + u * NT) / (BK / 4), M - 1) - ar;
    // B: a work-item's BQ quads are consecutive in k (4 BQ of them from bk0,
    // the same for its whole wavefront: rows at scalar addresses, the column
    // a 32-bit offset), so each digit plane takes one 4 BQ-byte LDS store per
    // step: with one four-byte store per quad, the 64 lanes' stores (one
    // column each, rows BK + 16 bytes apart) fell four to a bank
    const int bk0 = 4 * BQ * (wave * 64 / BN);
    const int64_t ldb = a.ldb;
    const gptr<int32_t> bcol = B + col0 + bk0 * ldb;
    const uint32_t bc = 4u * (uint32_t)min(tid % BN, N - 1 - col0);  // byte offset of its column
    auto bload = [&](gptr<int32_t> row) {
        uint32_t off = bc;
        asm("" : "+v"(off));  // extended here, where the load can take it as its 32-bit offset
        return *(gptr<int32_t>)((gptr<char>)row + off);
    };

    struct Set {
        i32x4 a[AQ], b[BQ];
    } s0, s1;  // step k's loads are in set k mod SETS
    // all of the step's k in range
    auto gload_fast = [&](Set &set, int k0) {
#pragma unroll
        for (int u = 0; u < AQ; ++u) set.a[u] = *reinterpret_cast<gptr<chunk>>(arow + down[u] * a.lda + k0);
        const gptr<int32_t> row = bcol + k0 * ldb;
#pragma unroll
        for (int u = 0; u < BQ; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) set.b[u][e] = bload(row + (4 * u + e) * ldb);
    };
    auto gload = [&](Set &set, int k0) {
        if (k0 + BK <= K) return gload_fast(set, k0);
#pragma unroll
        for (int u = 0; u < AQ; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) set.a[u][e] = k0 + akq + e < K ? (arow + down[u] * a.lda)[k0 + e] : 0;
        const gptr<int32_t> row = bcol + k0 * ldb;
#pragma unroll
        for (int u = 0; u < BQ; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) set.b[u][e] = k0 + bk0 + 4 * u + e < K ? bload(row + (4 * u + e) * ldb) : 0;
    };
    auto split = [&](Set &set) {
#pragma unroll
        for (int u = 0; u < AQ; ++u) set.a[u] = digit_planes(set.a[u]);
#pragma unroll
        for (int u = 0; u < BQ; ++u) set.b[u] = digit_planes(set.b[u]);
    };
    auto sstore = [&](const Set &set, int st) {
        unsigned char *as = As0 + st * L::A;
        unsigned char *bs = Bs0 + st * L::B;
#pragma unroll
        for (int u = 0; u < AQ; ++u) {
            const int f = tid + u * NT;
            const int rr = f / (BK / 4), kq = f % (BK / 4);
#pragma unroll
            for (int p = 0; p < 4; ++p) *reinterpret_cast<int *>(as + p * BM * LD + rr * LD + 4 * kq) = set.a[u][p];
        }
        static_assert(BQ == 2 || BQ == 4, "a B run of 8 or 16 bytes per plane");
        typedef int brun __attribute__((ext_vector_type(BQ)));
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            brun w;
#pragma unroll
            for (int u = 0; u < BQ; ++u) w[u] = set.b[u][p];
            *reinterpret_cast<brun *>(bs + p * BN * LD + (tid % BN) * LD + bk0) = w;
        }
    };
    // The digits of block b of a step: A's in fa, B's in fb, at slot 0 or 1.
    // Two blocks along one dimension share the other's digits, and those of a
    // single block outlive the reads of the next step's: these alternate with
    // the step's parity; the others take the block's slot.
    constexpr bool A_OWN = TM == 2 || BK == 64, B_OWN = TN == 2 || BK == 64;
    i32x4 fa[2][4], fb[2][4];
    auto read = [&](int st, auto block_, auto parity_) {
        constexpr int blk = decltype(block_)::value, parity = decltype(parity_)::value;
        constexpr int i = TM == 2 ? blk : 0, j = TN == 2 ? blk : 0, c = BK == 64 ? 16 * blk : 0;
        const unsigned char *as = As0 + st * L::A + (wm * WTM + r) * LD + h * (BK / 2) + i * 32 * LD + c;
        const unsigned char *bs = Bs0 + st * L::B + (wn * WTN + r) * LD + h * (BK / 2) + j * 32 * LD + c;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (A_OWN || blk == 0) fa[A_OWN ? blk : parity][p] = *reinterpret_cast<const i32x4 *>(as + p * BM * LD);
            if (B_OWN || blk == 0) fb[B_OWN ? blk : parity][p] = *reinterpret_cast<const i32x4 *>(bs + p * BN * LD);
        }
    };
    // half `half` of a step's products: a block's ten, or five of them
    auto multiply = [&](auto half_, auto parity_) {
        constexpr int half = decltype(half_)::value, parity = decltype(parity_)::value, blk = BLOCKS == 2 ? half : 0;
        constexpr int i = TM == 2 ? blk : 0, j = TN == 2 ? blk : 0;
        constexpr int fs = A_OWN ? blk : parity, gs = B_OWN ? blk : parity;
        int n = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; p + q < 4; ++q, ++n)
                if (BLOCKS == 2 || n / 5 == half)
                    acc[p + q][i][j] =
                        __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[fs][p], fb[gs][q], acc[p + q][i][j], 0, 0, 0);
    };
    // for each product of a half, in the order of its issue
    auto for_products = [&](auto &&f) {
#pragma unroll
        for (int n = 0; n < 5 * BLOCKS; ++n) f();
    };
    // vector instructions of the splitting per product it is spread over
    constexpr int VALU = ((AQ + BQ) * 18 + 5 * BLOCKS - 1) / (5 * BLOCKS);
    // Step kt.  First half: the second block's digits are read, the first
    // block multiplied, step kt + 1 (in `set`) split and stored to the other
    // buffer, and the loads of step kt + 1 + SETS sent out.  Second half,
    // behind the barrier: the first digits of step kt + 1 are read while the
    // second block is multiplied.  (Single-stage programs store between two
    // barriers: the one buffer must have been read by all.)
    constexpr bool EARLY = SETS == 2 && BLOCKS == 1;  // split in the half before the store
    constexpr bool LEAN = STAGES == 1 && TM == 2;  // short of registers for splitting beside the products
    const int KT = (K + BK - 1) / BK;
    typedef std::integral_constant<int, 0> zero;
    typedef std::integral_constant<int, 1> one;
    auto step = [&](Set &set, Set &other, int kt, auto parity_, auto full_) {
        constexpr bool full = decltype(full_)::value;
        constexpr int parity = decltype(parity_)::value;
        const int cur = STAGES == 2 ? parity : 0, next = STAGES == 2 ? parity ^ 1 : 0;
        const bool more = full || kt + 1 < KT;
        auto fill = [&]() {  // step kt + 1 to LDS, then loads into its registers
            if (!more) return;
            sstore(set, next);
            if (full)
                gload_fast(set, (kt + 1 + SETS) * BK);
            else if (kt + 1 + SETS < KT)
                gload(set, (kt + 1 + SETS) * BK);
        };
        if constexpr (EARLY) {
            if constexpr (STAGES == 1) lds_barrier();
            fill();
            multiply(zero(), parity_);
            if constexpr (full) {
                __builtin_amdgcn_sched_group_barrier(0x200, 4 * AQ + 4, 0);
                for_products([&]() {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
                });
            }
        } else {
            if constexpr (BLOCKS == 2 && !LEAN) read(cur, one(), parity_);
            multiply(zero(), parity_);
            if constexpr (LEAN) {
                __builtin_amdgcn_sched_barrier(0);
                read(cur, one(), parity_);
            }
            if (more) split(set);
            if constexpr (full && !LEAN) {
                __builtin_amdgcn_sched_group_barrier(0x100, 4 * (A_OWN + B_OWN), 0);
                for_products([&]() {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
                });
            }
            if constexpr (STAGES == 1) lds_barrier();
            fill();
        }
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (more) read(next, zero(), std::integral_constant<int, parity ^ 1>());
        multiply(one(), parity_);
        if (EARLY && (full || kt + 2 < KT)) split(other);
        if constexpr (full && !LEAN) {
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
            for_products([&]() {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if constexpr (EARLY) __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);
            });
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    if (KT > 0) {
        gload(s0, 0);
        split(s0);
        sstore(s0, 0);
        if (SETS == 2 && KT > 1) {
            gload(s1, BK);
            if (EARLY) split(s1);
        }
        if (KT > SETS) gload(s0, SETS * BK);
        lds_barrier();
        read(0, zero(), zero());
        const int KF = K / BK;  // steps all of whose k are in range
        Set &odd = SETS == 2 ? s1 : s0;
        int kt = 0;
        // steps whose loads (the last go SETS + 2 steps ahead) need no guards
        for (; kt + SETS + 2 < KF; kt += 2) {
            step(odd, s0, kt, zero(), std::true_type());
            step(s0, odd, kt + 1, one(), std::true_type());
        }
        for (; kt < KT; kt += 2) {
            step(odd, s0, kt, zero(), std::false_type());
            if (kt + 1 < KT) step(s0, odd, kt + 1, one(), std::false_type());
        }
    }

    // epilogue: value v of block (i, j) is row 8*(v/4) + 4*h + v%4, column r
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int gc = col0 + wn * WTN + j * 32 + r;
            auto each = [&](int first, int count, auto &&put) {
#pragma unroll
                for (int v = first; v < first + count; ++v) {
                    const int gr = row0 + wm * WTM + i * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                    const uint32_t x = (uint32_t)acc[0][i][j][v] + ((uint32_t)acc[1][i][j][v] << 8) +
                                       ((uint32_t)acc[2][i][j][v] << 16) + ((uint32_t)acc[3][i][j][v] << 24);
                    put(v - first, interior || (gr < M && gc < N), C + (int64_t)gr * a.ldc + gc, x);
                }
            };
            if (a.accumulate) {
                // four rows' loads before their additions: a load behind the
                // store before it waits for memory row by row (lanes outside C
                // load a zero: a branch around each load would put waits
                // between them)
                const gptr<int32_t> zero = (gptr<int32_t>)(const void *)kZeroBlock;
#pragma unroll
                for (int v = 0; v < 16; v += 4) {
                    uint32_t c[4];
                    each(v, 4, [&](int n, bool in, gmut<int32_t> p, uint32_t) { c[n] = (uint32_t)*(in ? (gptr<int32_t>)p : zero); });
                    each(v, 4, [&](int n, bool in, gmut<int32_t> p, uint32_t x) { if (in) *p = (int32_t)(c[n] + x); });
                }
            } else {
                each(0, 16, [](int, bool in, gmut<int32_t> p, uint32_t x) { if (in) *p = (int32_t)x; });
            }
        }
}

// int32 programs: one form serves aligned and unaligned rows, and none splits K.
template <int BM, int BN, int BK, int WM, int WN, int STAGES>
__device__ __forceinline__ void mfma_i32(const MmArgs &a) {
    using L = I32Lds<BM, BN, BK, STAGES>;
    __shared__ __attribute__((aligned(16))) unsigned char As[STAGES * L::A];
    __shared__ __attribute__((aligned(16))) unsigned char Bs[STAGES * L::B];
    int tm, tn;
    tile_of(blockIdx.x, (a.M + BM - 1) / BM, (a.N + BN - 1) / BN, &tm, &tn);
    mfma_i32_tile<BM, BN, BK, WM, WN, STAGES>(a, tm * BM, tn * BN, As, Bs);
}

}  // namespace pkk
