// Parametric polynomial division modulo a prime (Section 5, Fig. 8, Table 4),
// for gfx950.
//
// a holds the n coefficients of the dividend (a[i] multiplies x^i), b the M
// low coefficients of a monic divisor of degree M; residues in [0, P),
// P < 2^31.  One step (the body of the figure's while loop, one launch) with
// q = a[n-1]:
//     a[n-1-M+p] = (a[n-1-M+p] - q b[p]) mod P,   0 <= p < M,
// which eliminates the leading coefficient; its slot a[n-1] is not read
// again, and the host clears a[M .. N-1] once after the last step (clearing
// it inside a step would race with workgroups still reading q).  A workgroup
// of B work-items owns S * B consecutive p; work-item j takes p = j + k * B,
// k < S, so lanes touch consecutive addresses.
// polydiv_step_tiled (the figure's cache(a, b) programs): the tile's a and b
//   values and q are staged in LDS with coalesced loads first.  LDS bytes:
//   4 * (2 * S * B + 1).  After granularity reduction S = 1.
// polydiv_step_direct (no caching, decision (4b)): operands straight from
//   global memory; q is one address every lane reads (a cache broadcast).
// Products are reduced by Barrett's method with mu = floor(2^64 / P): for
// x < P^2 < 2^62 the estimate floor(x mu / 2^64) is the quotient or one less.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pkk {

struct PdArgs {
    uint32_t *a;
    const uint32_t *b;
    int32_t M;
    int32_t n;      // current number of dividend coefficients, n - 1 >= M
    uint32_t P;
    uint64_t mu;    // floor(2^64 / P)
};

__device__ __forceinline__ uint32_t mulmod(uint32_t x, uint32_t y, uint32_t P, uint64_t mu) {
    const uint64_t t = (uint64_t)x * y;
    const uint64_t q = __umul64hi(t, mu);
    uint64_t r = t - q * P;
    if (r >= P) r -= P;
    return (uint32_t)r;
}

__device__ __forceinline__ uint32_t submod(uint32_t x, uint32_t y, uint32_t P) {
    return x >= y ? x - y : x + (P - y);
}

template <int B, int S>
__device__ __forceinline__ void polydiv_step_tiled(const PdArgs &g) {
    constexpr int TW = S * B;
    __shared__ uint32_t sa[TW], sb[TW], sq;
    const int M = g.M, t = threadIdx.x;
    const int base = g.n - 1 - M;  // a index of p = 0
    const int tiles = (M + TW - 1) / TW;
    if (t == 0) sq = g.a[g.n - 1];
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int p0 = tile * TW;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int p = p0 + t + k * B;
            if (p < M) {
                sa[t + k * B] = g.a[base + p];
                sb[t + k * B] = g.b[p];
            }
        }
        __syncthreads();
        const uint32_t q = sq;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int p = p0 + t + k * B;
            if (p < M) g.a[base + p] = submod(sa[t + k * B], mulmod(q, sb[t + k * B], g.P, g.mu), g.P);
        }
        __syncthreads();
    }
}

template <int B, int S>
__device__ __forceinline__ void polydiv_step_direct(const PdArgs &g) {
    constexpr int TW = S * B;
    const int M = g.M, t = threadIdx.x;
    const int base = g.n - 1 - M;
    const int tiles = (M + TW - 1) / TW;
    const uint32_t q = g.a[g.n - 1];
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int p0 = tile * TW;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            const int p = p0 + t + k * B;
            if (p < M) g.a[base + p] = submod(g.a[base + p], mulmod(q, g.b[p], g.P, g.mu), g.P);
        }
    }
}

}  // namespace pkk

namespace pkk {

// The whole division in one launch (a program of this library, not one of
// the paper's): the K = n - M quotient coefficients first, then every
// remainder coefficient independently.  With top[j] the dividend coefficient
// at index n-1-j, step j of the division subtracts q_j b[M-d] from top[j+d]
// (1 <= d <= M), so q_k is top[k] after the steps before it -- a short
// sequential recurrence -- and the remainder is
//     r[x] = a[x] - sum_{0 <= j < K} q_j b[x - (K-1) + j]   (terms with a
//     b index below 0 vanish),
// K products per coefficient, no dependence between coefficients.
// Phase 1 (redundantly in every workgroup, so no grid-wide synchronisation is
// needed) is bound by the latency of the recurrence: it goes in blocks of 64
// quotient coefficients.  Within a block the first wavefront holds one
// coefficient per lane and takes a step per coefficient: a lane read, one
// product reduced by Shoup's method (the quotient estimated by the high word
// of x w', w' = floor(2^32 w / P) precomputed per divisor coefficient: three
// 32-bit multiplies instead of the six of a 64-bit Barrett reduction, two of
// them in the chain), a subtraction.  Then all wavefronts apply the block's
// 64 steps to the coefficients behind it, as one sum of products each.
// Sums of products (there and in phase 2) are kept whole: four products of
// residues below 2^31 fit 64 bits, and their 32-bit halves are summed apart
// and reduced once at the end, about 2 instructions a product instead of 16.
// Divisions modulo 2^31 - 1, M = 2^15: K = 100 33 -> 10.5 us (two launches'
// worth), K = 1000 71 us with 1024 work-items.
// Phase 2: each workgroup stages the b window of its tile of S * B remainder
// coefficients and reads the quotient from LDS.  Needs K <= 1024 and B >= 64.
// LDS bytes: 4 * (2 * 1024 + S * B + 1024).  a[M .. n-1] are left for the host
// to clear.
constexpr int kPdMaxK = 1024;
constexpr int kPdBlock = 64;  // quotient coefficients per block: one per lane

__device__ __forceinline__ uint32_t barrett(uint64_t t, uint32_t P, uint64_t mu) {
    const uint64_t q = __umul64hi(t, mu);
    uint64_t r = t - q * P;
    if (r >= P) r -= P;
    return (uint32_t)r;
}

// sum_{0 <= j < n} x[j] y[j] mod P over residues (n <= kPdMaxK): y[j] at
// y[j * DIR]
template <int DIR>
__device__ __forceinline__ uint32_t dot_mod(const uint32_t *x, const uint32_t *y, int n, uint32_t P, uint64_t mu) {
    uint64_t lo = 0, hi = 0;
    int j = 0;
    for (; j + 4 <= n; j += 4) {
        uint64_t t = 0;  // 4 (2^31 - 2)^2 < 2^64
#pragma unroll
        for (int e = 0; e < 4; ++e) t += (uint64_t)x[j + e] * y[(j + e) * DIR];
        lo += (uint32_t)t;
        hi += t >> 32;
    }
    uint64_t t = 0;
    for (; j < n; ++j) t += (uint64_t)x[j] * y[j * DIR];
    lo += (uint32_t)t;
    hi += t >> 32;
    // lo, hi < 2^41: hi mod P < 2^31, so the last sum stays below 2^64
    return barrett(((uint64_t)barrett(hi, P, mu) << 32) + lo, P, mu);
}

template <int B, int S>
__device__ __forceinline__ void polydiv_fused(const PdArgs &g) {
    static_assert(B % 64 == 0, "fused division: whole wavefronts");
    constexpr int TW = S * B;
    __shared__ uint32_t qs[kPdMaxK];              // top[j], turning into q_j
    __shared__ __attribute__((aligned(16))) uint32_t work[2 * kPdMaxK + TW];   // phase 1: divisor coefficients; phase 2: the b window
    // phase 1: bt[d - 1] = b[M - d] (zeros past the divisor's end), and the
    // first 64 of them as (w, w') pairs, with 64 zero pairs before
    uint32_t *const bt = work;
    uint2 *const pairs = reinterpret_cast<uint2 *>(work + kPdMaxK);
    static_assert(kPdMaxK + 4 * kPdBlock <= 2 * kPdMaxK, "phase 1 fits the window's space");
    const int M = g.M, n = g.n, K = n - M;
    const uint32_t P = g.P;
    const uint64_t mu = g.mu;
    const int t = threadIdx.x;
    for (int i = t; i < K; i += B) qs[i] = g.a[n - 1 - i];
    for (int i = t; i < K; i += B) bt[i] = i < M ? g.b[M - 1 - i] : 0u;
    for (int i = t; i < 2 * kPdBlock; i += B) {
        const int d = i - kPdBlock;
        uint32_t w = 0, ws = 0;
        if (d >= 0 && d < M) {
            w = g.b[M - 1 - d];
            const uint64_t x = (uint64_t)w << 32;
            uint64_t q = __umul64hi(x, mu);
            if (x - q * P >= P) ++q;
            ws = (uint32_t)q;
        }
        pairs[i] = make_uint2(w, ws);
    }
    __syncthreads();
    for (int kb = 0; kb < K; kb += kPdBlock) {
        const int kn = min(kPdBlock, K - kb);
        if (t < 64) {
            uint32_t top = t < kn ? qs[kb + t] : 0u;
            const uint2 *const pl = pairs + t;  // step i: d = t - i, pair d - 1 + 64
#pragma unroll
            for (int i0 = 0; i0 < kPdBlock; i0 += 16) {
                // (a step past kn - 1 within the 16 takes its q from a lane past
                // kn, which it subtracts from lanes further on only: none of
                // them is stored)
                if (i0 >= kn) break;
                uint2 w[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) w[i] = pl[kPdBlock - 1 - i0 - i];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)top, i0 + i);
                    uint32_t r = q * w[i].x - __umulhi(q, w[i].y) * P;  // in [0, 2P)
                    r = min(r, r - P);
                    top -= r;
                    top = min(top, top + P);
                }
            }
            if (t < kn) qs[kb + t] = top;
        }
        __syncthreads();
        if (kb + kPdBlock >= K) break;
        for (int j = kb + kPdBlock + t; j < K; j += B)
            qs[j] = submod(qs[j], dot_mod<-1>(qs + kb, bt + (j - kb - 1), kPdBlock, P, mu), P);
        __syncthreads();
    }
    const int tiles = (M + TW - 1) / TW;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int x0 = tile * TW;
        for (int i = t; i < TW + K - 1; i += B) {
            const int p = x0 - (K - 1) + i;
            work[i] = (p >= 0 && p < M) ? g.b[p] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int xl = t + s * B, x = x0 + xl;
            if (x < M) g.a[x] = submod(g.a[x], dot_mod<1>(qs, work + xl, K, P, mu), P);
        }
        __syncthreads();
    }
}

}  // namespace pkk
