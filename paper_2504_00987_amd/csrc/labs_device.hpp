// Device building blocks of liblabs (gfx950): counter-based RNG, wavefront
// primitives, sequence masks of up to 256 bits and the tabu walk.
//
// One tabu walk (Alg. 2 / Alg. 4 of arXiv:2504.00987) runs on one 64-lane
// wavefront; lane l owns neighbours j = l + 64h.  The score of neighbour j is
//
//     dE_j = 4 * ( sum_k t_jk^2  -  s_j * sum_k t_jk C_k ),
//     t_jk = s_{j+k} + s_{j-k}   (terms outside the sequence are 0)
//
// (flipping s_j changes C_k of Eq. 1 by -2 s_j t_jk).  Every lane keeps its
// neighbours' scores across moves: with the autocorrelations C_k and the
// pair sums Q_m = sum_{a+b=m} s_a s_b in LDS, a move changes each score by an
// expression in one C and one Q entry, so a step is O(N) instead of the
// O(N^2) of recomputing the sums (the paper's Sec. III.C updates are O(N) per
// neighbour).  All arithmetic is exact int32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

#include <type_traits>

#include "labs_internal.h"

namespace liblabs {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
// ---------------------------------------------------------------------------
enum : uint32_t {
    kTagStart = 1,  // random start of a stand-alone walk
    kTagStep = 2,   // per tabu step: tie-break word 0, tenure word 1
    kTagLen = 3,    // per walk: random walk length, word 0
    kTagInit = 4,   // per population member: initial sequence
    kTagGen = 5,    // per generation: crossover, parents, cut, replacement
    kTagMut = 6     // per generation: mutation words
};

struct Draw4 {
    uint32_t w0, w1, w2, w3;
};

__device__ __forceinline__ Draw4 philox10(uint32_t x0, uint32_t x1, uint32_t x2,
                                          uint32_t x3, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 64-bit product each instead of its halves apart: the multiplies
        // are quarter-rate and a call is one chain of ten rounds
        const uint64_t p2 = (uint64_t)0xCD9E8D57u * x2, p0 = (uint64_t)0xD2511F53u * x0;
        x0 = (uint32_t)(p2 >> 32) ^ x1 ^ k0;
        x2 = (uint32_t)(p0 >> 32) ^ x3 ^ k1;
        x1 = (uint32_t)p2;
        x3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return {x0, x1, x2, x3};
}

// Uniform integer in [0, range) from a 32-bit word: (u * range) >> 32.
__device__ __forceinline__ uint32_t below(uint32_t u, uint32_t range) {
    return __umulhi(u, range);
}

// ---------------------------------------------------------------------------
// Wavefront primitives (wave64).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() {
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) {
    return __builtin_amdgcn_ballot_w64(p);
}

__device__ __forceinline__ int readlane(int v, int l) {
    return __builtin_amdgcn_readlane(v, l);
}

__device__ __forceinline__ uint32_t readlane_u(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// A wave-uniform 64-bit value, read from the first lane into scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Orders this wavefront's LDS accesses across lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// DPP controls (GFX9 encoding).
#define LABS_DPP_QUAD_1032 0xB1
#define LABS_DPP_QUAD_2301 0x4E
#define LABS_DPP_ROW_MIRROR 0x140
#define LABS_DPP_ROW_HALF_MIRROR 0x141
#define LABS_DPP_ROW_BCAST15 0x142
#define LABS_DPP_ROW_BCAST31 0x143

// Minimum over the 64 lanes, returned wave-uniform: row minima by DPP, then
// rows combined with the row broadcasts (lane 63 ends with the total).
__device__ __forceinline__ int wave_min(int v) {
    // the first four patterns give every lane a source: no fill value
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_1032, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_2301, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_HALF_MIRROR, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_MIRROR, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, LABS_DPP_ROW_BCAST15, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, LABS_DPP_ROW_BCAST31, 0xc, 0xf, false));
    return readlane(v, 63);
}

// Sum over the 64 lanes, returned wave-uniform.
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, LABS_DPP_QUAD_1032, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, LABS_DPP_QUAD_2301, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, LABS_DPP_ROW_HALF_MIRROR, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, LABS_DPP_ROW_MIRROR, 0xf, 0xf, false);
    return readlane(v, 0) + readlane(v, 16) + readlane(v, 32) + readlane(v, 48);
}

// Next index of the persistent work queue, wave-uniform.  Every lane executes
// the atomic (lane 0 adds 1, the others add 0) so that the value read back
// with readlane is never produced under a lane-dependent branch: a
// lane-0-only fetch lets the optimiser thread that branch into the loop's
// other lane-0 branches, and lanes then reach the readlane before lane 0 has
// fetched, disagreeing on the index.
__device__ __forceinline__ uint32_t next_work(uint32_t *counter, uint32_t take = 1u) {
    const uint32_t v = atomicAdd(counter, lane_id() == 0 ? take : 0u);
    return readlane_u(v, 0);
}

// ---------------------------------------------------------------------------
// Sequence masks: 64-bit for N <= 64, 128-bit for N <= 128, 256-bit for
// N <= 256.
// ---------------------------------------------------------------------------
struct M128 {
    uint64_t lo, hi;
};

__device__ __forceinline__ uint64_t m_and(uint64_t a, uint64_t b) { return a & b; }
__device__ __forceinline__ uint64_t m_or(uint64_t a, uint64_t b) { return a | b; }
__device__ __forceinline__ uint64_t m_xor(uint64_t a, uint64_t b) { return a ^ b; }
__device__ __forceinline__ uint64_t m_not(uint64_t a) { return ~a; }
__device__ __forceinline__ int m_popc(uint64_t a) { return __popcll(a); }
// a >> sh for 0 <= sh <= 64 (64 gives 0).
__device__ __forceinline__ uint64_t m_shr(uint64_t a, int sh) {
    return sh >= 64 ? 0ull : (a >> sh);
}
// Bits [0, n) set, 0 <= n <= 64.
__device__ __forceinline__ uint64_t m_low(uint64_t, int n) {
    return n >= 64 ? ~0ull : ((1ull << n) - 1ull);
}
__device__ __forceinline__ int m_bit(uint64_t a, int i) { return (int)((a >> i) & 1ull); }

__device__ __forceinline__ M128 m_and(M128 a, M128 b) { return {a.lo & b.lo, a.hi & b.hi}; }
__device__ __forceinline__ M128 m_or(M128 a, M128 b) { return {a.lo | b.lo, a.hi | b.hi}; }
__device__ __forceinline__ M128 m_xor(M128 a, M128 b) { return {a.lo ^ b.lo, a.hi ^ b.hi}; }
__device__ __forceinline__ M128 m_not(M128 a) { return {~a.lo, ~a.hi}; }
__device__ __forceinline__ int m_popc(M128 a) { return __popcll(a.lo) + __popcll(a.hi); }
// a >> sh for 0 <= sh <= 128.
__device__ __forceinline__ M128 m_shr(M128 a, int sh) {
    M128 r;
    if (sh >= 64) {
        r.lo = sh >= 128 ? 0ull : (a.hi >> (sh - 64));
        r.hi = 0ull;
    } else if (sh == 0) {
        r = a;
    } else {
        r.lo = (a.lo >> sh) | (a.hi << (64 - sh));
        r.hi = a.hi >> sh;
    }
    return r;
}
__device__ __forceinline__ M128 m_low(M128, int n) {
    M128 r;
    if (n >= 128) {
        r.lo = ~0ull; r.hi = ~0ull;
    } else if (n >= 64) {
        r.lo = ~0ull; r.hi = (1ull << (n - 64)) - 1ull;
    } else {
        r.lo = (1ull << n) - 1ull; r.hi = 0ull;
    }
    return r;
}
__device__ __forceinline__ int m_bit(M128 a, int i) {
    return (int)(((i < 64 ? a.lo : a.hi) >> (i & 63)) & 1ull);
}

// 256-bit masks for N <= 256 (four words, selected by value so that a
// variable word index never forces the mask out of registers).
struct M256 {
    uint64_t w0, w1, w2, w3;
};

__device__ __forceinline__ uint64_t m_word(const M256 &a, int i) {
    return i == 0 ? a.w0 : i == 1 ? a.w1 : i == 2 ? a.w2 : i == 3 ? a.w3 : 0ull;
}
__device__ __forceinline__ M256 m_and(M256 a, M256 b) {
    return {a.w0 & b.w0, a.w1 & b.w1, a.w2 & b.w2, a.w3 & b.w3};
}
__device__ __forceinline__ M256 m_or(M256 a, M256 b) {
    return {a.w0 | b.w0, a.w1 | b.w1, a.w2 | b.w2, a.w3 | b.w3};
}
__device__ __forceinline__ M256 m_xor(M256 a, M256 b) {
    return {a.w0 ^ b.w0, a.w1 ^ b.w1, a.w2 ^ b.w2, a.w3 ^ b.w3};
}
__device__ __forceinline__ M256 m_not(M256 a) { return {~a.w0, ~a.w1, ~a.w2, ~a.w3}; }
__device__ __forceinline__ int m_popc(M256 a) {
    return __popcll(a.w0) + __popcll(a.w1) + __popcll(a.w2) + __popcll(a.w3);
}
// a >> sh for 0 <= sh <= 256.
__device__ __forceinline__ M256 m_shr(M256 a, int sh) {
    const int q = sh >> 6, r = sh & 63;
    auto out = [&](int i) {
        const uint64_t lo = m_word(a, i + q);
        return r == 0 ? lo : (lo >> r) | (m_word(a, i + q + 1) << (64 - r));
    };
    return {out(0), out(1), out(2), out(3)};
}
__device__ __forceinline__ M256 m_low(M256, int n) {
    auto word = [&](int i) {
        const int b = n - 64 * i;
        return b >= 64 ? ~0ull : b <= 0 ? 0ull : ((1ull << b) - 1ull);
    };
    return {word(0), word(1), word(2), word(3)};
}
__device__ __forceinline__ int m_bit(M256 a, int i) {
    return (int)((m_word(a, i >> 6) >> (i & 63)) & 1ull);
}

template <int NW> struct MaskOf;
template <> struct MaskOf<1> { using type = uint64_t; };
template <> struct MaskOf<2> { using type = M128; };
template <> struct MaskOf<3> { using type = M256; };
template <> struct MaskOf<4> { using type = M256; };

// Word h (0 <= h < 4) of a mask; words past its width are 0.
__device__ __forceinline__ uint64_t mask_word(uint64_t a, int h) { return h == 0 ? a : 0ull; }
__device__ __forceinline__ uint64_t mask_word(const M128 &a, int h) {
    return h == 0 ? a.lo : h == 1 ? a.hi : 0ull;
}
__device__ __forceinline__ uint64_t mask_word(const M256 &a, int h) { return m_word(a, h); }

// A mask of NW words from four words (words past NW are ignored).
template <int NW>
__device__ __forceinline__ typename MaskOf<NW>::type make_mask(uint64_t w0, uint64_t w1,
                                                               uint64_t w2 = 0ull,
                                                               uint64_t w3 = 0ull) {
    if constexpr (NW == 1) {
        return w0;
    } else if constexpr (NW == 2) {
        return M128{w0, w1};
    } else {
        return M256{w0, w1, w2, w3};
    }
}

// Mask of NW words stored at p[0 .. NW).
template <int NW>
__device__ __forceinline__ typename MaskOf<NW>::type load_mask(const uint64_t *p) {
    return make_mask<NW>(p[0], NW > 1 ? p[1] : 0ull, NW > 2 ? p[2] : 0ull, NW > 3 ? p[3] : 0ull);
}
template <int NW, typename Mask>
__device__ __forceinline__ void store_mask(uint64_t *p, const Mask &m) {
#pragma unroll
    for (int h = 0; h < NW; ++h) p[h] = mask_word(m, h);
}

// ---------------------------------------------------------------------------
// Walk schedule: maxIter and the tenure range.
// ---------------------------------------------------------------------------
struct Schedule {
    int T, lo, hi;
};

// `draw` is word 0 of the walk's LEN draw (unused where the rule draws none).
__device__ __forceinline__ Schedule make_schedule(const RuleParams &r, int N, uint32_t draw) {
    Schedule s;
    if (r.steps_rule == 0) {
        s.T = r.steps_a;
    } else if (r.steps_rule == 1) {
        s.T = r.steps_a * N;
    } else {
        // PAPER: floor(N/2) + U[0, N]; RANGE: U[lo, hi] from the same word
        int lo = N / 2, span = N + 1;
        if (r.steps_rule == 3) {
            lo = r.slo_num * N / r.slo_den;
            span = r.shi_num * N / r.shi_den - lo + 1;
        }
        s.T = lo + (int)below(draw, (uint32_t)span);
    }
    if (r.tenure_rule == 0) {
        s.lo = r.lo_num * N / r.lo_den + r.lo_add;
        s.hi = r.hi_num * N / r.hi_den + r.hi_add;
    } else {
        s.lo = s.T / 10;
        s.hi = 3 * s.T / 25;
    }
    return s;
}

// ---------------------------------------------------------------------------
// Energy of a sequence mask, computed by the whole wavefront (lane l owns
// lags l+1 and l+65): C_k = (N-k) - 2 * popcount((M ^ (M >> k)) & low(N-k)).
// ---------------------------------------------------------------------------
template <typename Mask>
__device__ __forceinline__ int lag_corr(Mask M, int N, int k) {
    return (N - k) - 2 * m_popc(m_and(m_xor(M, m_shr(M, k)), m_low(M, N - k)));
}

// a * b + c of 24-bit factors (signed), a full-rate instruction: the
// compiler turns products of spins into shifts, masks and the quarter-rate
// 32-bit multiply.
__device__ __forceinline__ int mad_i24(int a, int b, int c) {
    int d;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
template <int B>
__device__ __forceinline__ int mad_i24_const(int a, int c) {
    static_assert(B >= -16 && B <= 64, "an inline constant");
    int d;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "n"(B), "v"(c));
    return d;
}
__device__ __forceinline__ int mad_i24_s(int a, int b, int c) {  // b wave-uniform
    int d;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b), "v"(c));
    return d;
}
__device__ __forceinline__ int mul_i24(int a, int b) {
    int d;
    asm("v_mul_i32_i24 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ int mul_i24_s(int a, int b) {  // b wave-uniform
    int d;
    asm("v_mul_i32_i24 %0, %1, %2" : "=v"(d) : "s"(b), "v"(a));
    return d;
}

// popc(x) + acc in one instruction.
__device__ __forceinline__ int popc_add(uint32_t x, int acc) {
    int d;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(d) : "v"(x), "v"(acc));
    return d;
}

// Part of one row's energy in one lane: the lags k0, k0 + STEP, .. below
// nmax (>= N) except 0, with the row's mask in W words, 0 <= k0 < STEP:
//   C_k = (N - k) - 2 popc over k <= i < N of (M ^ (M << k)).
// M << k moves by STEP bits a lag; of lags in [32 b, 32 b + 32) the words
// below b hold no pair.  Lags past N add nothing (N - k saturates at 0, no
// bit of a word is at or above the lag), so a trip of the loop takes four
// lags: the shifted words' copies and the loop's own instructions were a
// third of a trip with one.
template <int W, int STEP>
__device__ __forceinline__ int lane_lags(const uint32_t *mask, int N, int nmax, int k0) {
    constexpr int kLags = 4;
    static_assert(32 % (STEP * kLags) == 0, "trips end with the words");
    uint32_t M[W], Y[W], V[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        M[w] = mask[w];
        const int n = N - 32 * w;  // valid bits of word w
        V[w] = n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u;
    }
#pragma unroll
    for (int w = W - 1; w >= 0; --w)
        Y[w] = w && k0 ? __builtin_amdgcn_alignbit(M[w], M[w - 1], (uint32_t)(32 - k0))
                       : M[w] << k0;
    int k = k0, e = k0 ? 0 : -N * N;  // the square of lag 0
    uint32_t left = (uint32_t)max(N - k0, 0);  // N - k
#pragma unroll
    for (int b = 0; b < W; ++b) {
        const int end = min(nmax, 32 * (b + 1));
        while (k < end) {
#pragma unroll
            for (int i = 0; i < kLags; ++i, k += STEP) {
                int pop = popc_add((M[b] ^ Y[b]) & (V[b] & (~0u << (k & 31))), 0);
#pragma unroll
                for (int w = b + 1; w < W; ++w) pop = popc_add((M[w] ^ Y[w]) & V[w], pop);
                const int c = mad_i24_const<-2>(pop, (int)left);
                e = mad_i24(c, c, e);
                left = __builtin_elementwise_sub_sat(left, (uint32_t)STEP);
#pragma unroll
                for (int w = W - 1; w > b; --w)
                    Y[w] = __builtin_amdgcn_alignbit(Y[w], Y[w - 1], 32 - STEP);
                Y[b] <<= STEP;
            }
        }
    }
    return e;
}

// lane_lags with the mask in `words` (wave-uniform) words.
template <int STEP>
__device__ __forceinline__ int lane_energy(int words, const uint32_t *mask, int N, int nmax,
                                           int k0) {
    switch (words) {
    case 1: return lane_lags<1, STEP>(mask, N, nmax, k0);
    case 2: return lane_lags<2, STEP>(mask, N, nmax, k0);
    case 3: return lane_lags<3, STEP>(mask, N, nmax, k0);
    case 4: return lane_lags<4, STEP>(mask, N, nmax, k0);
    case 5: return lane_lags<5, STEP>(mask, N, nmax, k0);
    case 6: return lane_lags<6, STEP>(mask, N, nmax, k0);
    case 7: return lane_lags<7, STEP>(mask, N, nmax, k0);
    default: return lane_lags<8, STEP>(mask, N, nmax, k0);
    }
}

// ---------------------------------------------------------------------------
// The tabu walk.
// ---------------------------------------------------------------------------
template <int NW>
struct WalkResult {
    typename MaskOf<NW>::type best;
    int best_e;
    int final_e;
};

// LDS of one walk of N <= SPAN: 2 C_k for k = 0 .. SPAN - 1 (entry 0 is
// scratch) and 2 Q_m for m = 0 .. 2 SPAN - 1 as int32, and the sequence as
// int8 with zeros around it, SP[q] = 4 s_q for 0 <= q < N and 0 for the other
// q in -SPAN .. 2 SPAN - 1, which covers every 2j - p and 2p - j of two
// positions j, p < SPAN.  (With these factors one number, -s_p, scales every
// term of a move.)  15 SPAN bytes: the registers bind occupancy, not the LDS (61
// VGPRs at N <= 64, eight wavefronts per SIMD; 77 to 80 beyond, six).  (Spins
// as whole words, with fewer loads for several neighbours per lane, cost 3
// to 8 % on full devices: the stride-two reads of 2j - p meet in the banks.)
template <int SPAN>
struct WalkTables {
    static constexpr int CT = 0;
    static constexpr int QT = CT + 4 * SPAN;
    static constexpr int SPLO = QT + 8 * SPAN, SP = SPLO + SPAN;
    static constexpr int BYTES = SP + 2 * SPAN;
    static_assert(BYTES % 16 == 0, "16-byte aligned walks");
};
template <int NW>
using WalkLds = WalkTables<64 * NW>;

// Lane l receives bit l of a wave-uniform 64-bit mask.
__device__ __forceinline__ bool lane_bit(uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask);
}

__device__ __forceinline__ int dot4(uint32_t a, uint32_t b, int acc) {
    return __builtin_amdgcn_sdot4((int)a, (int)b, acc, false);
}

// |a - b| + c in one instruction, a wave-uniform.
__device__ __forceinline__ uint32_t absdiff_add_s(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_sad_u32 %0, %1, %2, %3" : "=v"(d) : "s"(a), "v"(b), "v"(c));
    return d;
}

// LDS accesses by offset (the 32-bit address of the local address space, so
// that an offset computed in one instruction is the address).
typedef __attribute__((address_space(3))) int8_t lds_i8;
typedef __attribute__((address_space(3))) int32_t lds_i32;
__device__ __forceinline__ uint32_t lds_offset(const void *p) {
    return (uint32_t)(uintptr_t)(const lds_i8 *)p;
}
__device__ __forceinline__ int lds_load_i8(uint32_t a) { return *(const lds_i8 *)(uintptr_t)a; }
__device__ __forceinline__ int lds_load_i32(uint32_t a) { return *(const lds_i32 *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store_i32(uint32_t a, int v) {
    *(lds_i32 *)(uintptr_t)a = v;
}

// One neighbour's part of a move at p (see tabu_walk): c = 2 C_|p-j|,
// q = 2 Q_(p+j), y = 4 s_(2p-j), z = 4 s_(2j-p), nsp = -s_p, nsp4 = -4 s_p
// (wave-uniform) and x = 4 s_p s_j.  Adds the change of 4 D_j and returns
// e = 2 C_k - 4y; the entries' new values are e - x and q - 2x.
__device__ __forceinline__ void move_score(int c, int q, int y, int z, int nsp, int nsp4, int x,
                                           int &D, int &e) {
    e = mad_i24_s(y, nsp, c);
    D = mad_i24(x, c + e + q, D);
    D = mad_i24_s(z, nsp4, D);
}

// The moved position, the lane of `bit` (none if 0): -4 s_p (nr) stored as its
// new spin at LDS offset za + OFF and negated, x = 0, and D and tabu set to
// wave-uniform values.  (A masked block without a branch, so that the step
// stays one run of instructions.)
template <int OFF>
__device__ __forceinline__ void set_moved(uint64_t bit, uint32_t za, int d_new, int tabu_new,
                                          int &nr, int &x, int &D, int &tabu) {
    uint64_t all;
    asm volatile(
        "s_and_saveexec_b64 %0, %5\n\t"
        "ds_write_b8 %6, %1 offset:%9\n\t"
        "v_mov_b32 %2, 0\n\t"
        "v_mov_b32 %3, %7\n\t"
        "v_mov_b32 %4, %8\n\t"
        "v_sub_u32 %1, 0, %1\n\t"
        "s_mov_b64 exec, %0"
        : "=&s"(all), "+&v"(nr), "+&v"(x), "+&v"(D), "+&v"(tabu)
        : "s"(bit), "v"(za), "s"(d_new), "s"(tabu_new), "n"(OFF)
        : "memory", "scc");
}

// Runs one walk of sch.T steps from mask M0 (bits >= N must be clear) on one
// wavefront, lane l owning neighbours j = l + 64h, h < NW (64 (NW - 1) < N <=
// 64 NW).
//
// The step is O(N).  Neighbour j's key is d_j = 2 u_j - s_j v_j with
// v_j = sum_k t_jk C_k and 2 u_j = Q_2j - 1 (candE_j = E + 4 (N - 1) + 4 d_j).
// A move at p changes C_k by -2 s_p t_pk, so v_j changes by
// -2 s_p sum_k t_jk t_pk, and that sum has a closed form: the products
// s_(j+k) s_(p+k), s_(j-k) s_(p-k) over k >= 1 are those of C_|j-p| without
// s_j s_p, the products s_(j+k) s_(p-k), s_(j-k) s_(p+k) those of Q_(j+p)
// without s_j s_p:
//     sum_k t_jk t_pk = C_|j-p| + Q_(j+p) - 2 s_j s_p        (j != p).
// With x = s_p s_j, y = s_p s_(2p-j), z = s_p s_(2j-p) (old spins, zero
// outside the sequence), k = |p - j|, and the change of t_jk itself included:
//     d_j += 2x (2 C_k + Q_(p+j) - 2y) - 4z - 8,
//     C_k -= 2 (x + y),   Q_(p+j) -= 4x,
// and d_p = -d_p - 2 (N - 1) (undoing the move), Q_2p unchanged.  Lane j
// reads and writes exactly the entries C_|p-j| and Q_(p+j) (lanes j and
// 2p - j write the same value to C_k).  The common -8 is left out of the
// stored D_j and put back on the scalar unit.
// Lanes past the sequence have s_j = 0: they write back the Q they read, and
// the C they read or, where 2p - j lies in the sequence, what lane 2p - j
// writes; their D never falls to an aspiration threshold.
//
// Bound: the instructions a wavefront issues and, with few wavefronts, one
// chain of an LDS round trip, a wavefront minimum and the scalar pick.  So the
// moved position is dealt with while the entries are on their way, and the
// entries' new values are stored in the wait states of the minimum.  One
// wavefront per walk with NW neighbours per lane keeps the chain free of
// barriers.  Measured (MI355X, a call; recomputing v_j from packed int8
// products -> this): 4096 walks of N = 64 and 256 steps 131 -> 77 us, of
// N = 120 and 480 steps 717 -> 200 us, of N in 129..256 3.90 -> 0.49 ms.
//   lds    WalkLds<NW>::BYTES bytes of per-walk scratch, 16-aligned
//   trace  with TRACE: trace[t-1] = flipped index
//   AHEAD  the wavefront issues ahead of the others of its SIMD from the
//          minimum to the next reads (see the step)
// Every lane must call this with identical uniform inputs.
template <int NW, bool TRACE = false, bool AHEAD = false>
__device__ __forceinline__ WalkResult<NW> tabu_walk(const int N_in,
                                                    const typename MaskOf<NW>::type M0,
                                                    const Schedule sch_in, const int aspiration_in,
                                                    const uint32_t k0, const uint32_t k1,
                                                    const uint32_t entity, const uint32_t gen,
                                                    uint8_t *lds,
                                                    int16_t *__restrict__ trace) {
    static_assert(NW >= 1 && NW <= 4, "N <= 256");
    using Mask = typename MaskOf<NW>::type;
    using L = WalkLds<NW>;
    const int lane = lane_id();
    // Wave-uniform parameters, pinned to scalar registers so that the step
    // loop is controlled by scalar branches.
    const int N = __builtin_amdgcn_readfirstlane(N_in);
    const int aspiration = __builtin_amdgcn_readfirstlane(aspiration_in);
    Schedule sch;
    sch.T = __builtin_amdgcn_readfirstlane(sch_in.T);
    sch.lo = __builtin_amdgcn_readfirstlane(sch_in.lo);
    sch.hi = __builtin_amdgcn_readfirstlane(sch_in.hi);
    const Mask M = make_mask<NW>(uniform64(mask_word(M0, 0)), uniform64(mask_word(M0, 1)),
                                 uniform64(mask_word(M0, 2)), uniform64(mask_word(M0, 3)));
    // words of M and of its reversal (bit i of R is bit N-1-i of M)
    uint64_t Mw[NW], Rw[NW];
    {
        const int sh = 64 * NW - N;  // 0 .. 63
        uint64_t b[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            Mw[w] = mask_word(M, w);
            b[NW - 1 - w] = __builtin_bitreverse64(Mw[w]);
        }
#pragma unroll
        for (int w = 0; w < NW; ++w)
            Rw[w] = (b[w] >> sh) | (w + 1 < NW ? (b[w + 1] << 1) << (63 - sh) : 0ull);
    }
    int32_t *const CT = (int32_t *)(lds + L::CT);
    int32_t *const QT = (int32_t *)(lds + L::QT);
    int8_t *const SP = (int8_t *)(lds + L::SP);

    // C_s, Q_(N-1-s) and Q_(N-1+s) for s = lane + 64h from popcounts: with the
    // reversal R, over the N - s positions i < N - s,
    //   C_s pairs M_i, M_(i+s);  Q_(N-1-s) M_i, R_(i+s);  Q_(N-1+s) R_i, M_(i+s).
    // Bits i >= N - s of the first operand, which meet zeros, are taken off
    // again: the first s bits of R (of M where the operand is R).
    wave_sync();
    int C[NW], nr[NW];  // nr: -4 s_j, 0 past the sequence
    int sq_e = 0;       // sum of C_k^2 over this lane's lags
    int below_m = 0, below_r = 0;  // set bits of the words below
#pragma unroll
    for (int h = 0; h < NW; ++h) {
        const int j = lane + 64 * h;
        int pc = 0, pl = 0, ph = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            uint64_t xm = 0ull, xr = 0ull;  // words w of M >> j and R >> j
            if (w + h < NW) {
                xm = Mw[w + h] >> lane;
                xr = Rw[w + h] >> lane;
            }
            if (w + h + 1 < NW) {
                xm |= (Mw[w + h + 1] << 1) << (63 - lane);
                xr |= (Rw[w + h + 1] << 1) << (63 - lane);
            }
            pc += __popcll(Mw[w] ^ xm);
            pl += __popcll(Mw[w] ^ xr);
            ph += __popcll(Rw[w] ^ xm);
        }
        auto below = [&](uint64_t m, int from) {  // `from` + set bits of m below this lane
            return (int)__builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)from));
        };
        const int tm = below(Mw[h], below_m), tr = below(Rw[h], below_r);
        below_m += __popcll(Mw[h]);
        below_r += __popcll(Rw[h]);
        const bool in = j < N;
        C[h] = in && j > 0 ? N - j - 2 * (pc - tr) : 0;
        sq_e += C[h] * C[h];
        nr[h] = in ? (lane_bit(Mw[h]) ? 4 : -4) : 0;
        if (in) {
            QT[N - 1 - j] = 2 * (N - j - 2 * (pl - tr));
            QT[N - 1 + j] = 2 * (N - j - 2 * (ph - tm));
        }
        SP[j] = (int8_t)-nr[h];
        SP[j - 64 * NW] = 0;
        SP[j + 64 * NW] = 0;
    }

    // v_j = sum_i s_i C_|i-j|: C mirrored around zero as bytes (C_k >> 1 for
    // NW > 2, where |C_k| may reach 255), for now in the place of C; a lane's
    // window starts at any byte, so four dwords at a time are aligned.
    constexpr bool kHalfC = NW > 2;
    int8_t *const F = (int8_t *)CT;  // F[64 NW + k] = F[64 NW - k] = C_k, 0 at k = 0
    int8_t *const S8 = F + 128 * NW + 16;  // s_i as bytes, 0 past the sequence
    static_assert(128 * NW + 16 + 64 * NW <= L::QT - L::CT, "both fit");
#pragma unroll
    for (int h = 0; h < NW; ++h) {
        const int k = lane + 64 * h;
        const int8_t c = (int8_t)(kHalfC ? C[h] >> 1 : C[h]);
        F[64 * NW + k] = c;
        F[64 * NW - k] = c;
        S8[k] = (int8_t)(-nr[h] >> 2);
    }
    wave_sync();
    int D[NW], tabu[NW];
    {
        int v[NW];
        const uint32_t *win[NW];
        uint32_t last[NW];
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            win[h] = (const uint32_t *)F + ((64 * NW - 64 * h - lane) >> 2);
            last[h] = win[h][0];
            v[h] = 0;
        }
        const uint32_t shift = (uint32_t)(-lane) & 3u;
        const uint4 *const S16 = (const uint4 *)S8;
        for (int i = 0; i < N; i += 16) {
            const uint4 s = S16[i >> 4];
#pragma unroll
            for (int h = 0; h < NW; ++h) {
                const uint32_t *w = win[h] + (i >> 2);
                const uint32_t a = w[1], b = w[2], c = w[3], d = w[4];
                v[h] = dot4(__builtin_amdgcn_alignbyte(a, last[h], shift), s.x, v[h]);
                v[h] = dot4(__builtin_amdgcn_alignbyte(b, a, shift), s.y, v[h]);
                v[h] = dot4(__builtin_amdgcn_alignbyte(c, b, shift), s.z, v[h]);
                v[h] = dot4(__builtin_amdgcn_alignbyte(d, c, shift), s.w, v[h]);
                last[h] = d;
            }
        }
        // parity part of v_j where the products took C_k >> 1 = (C_k -
        // ((N - k) & 1)) / 2: the s_i with N - |i-j| odd are those of parity
        // q = (j + N - 1) mod 2, without s_j itself (counted when N is odd)
        int S0 = 0, S1 = 0;
        if constexpr (kHalfC) {
            constexpr uint64_t kEven = 0x5555555555555555ull;
            S0 = (N + 1) / 2;
            S1 = N / 2;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                S0 -= 2 * __popcll(Mw[w] & kEven);
                S1 -= 2 * __popcll(Mw[w] & ~kEven);
            }
        }
        const int Sq = ((lane + N - 1) & 1) ? S1 : S0;  // the same for lane + 64h
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            const int j = lane + 64 * h;
            if constexpr (kHalfC) v[h] = 2 * v[h] + Sq + ((N & 1) ? nr[h] >> 2 : 0);
            // 4 (Q_2j - 1 - s_j v_j); beyond the sequence never a minimum
            D[h] = j < N ? 2 * QT[2 * j] - 4 + nr[h] * v[h] : 0x3fffffff;
            // lanes past the sequence are never admissible: infinite tenure
            tabu[h] = j < N ? -1 : INT_MAX;
        }
    }
    wave_sync();
#pragma unroll
    for (int h = 0; h < NW; ++h) CT[lane + 64 * h] = 2 * C[h];
    wave_sync();

    const int E0 = wave_sum(sq_e);
    Mask best = M;
    // The best against E0, and how far the walk is above its best.
    // Aspiration: candE_j < bestE <=> 4 d_j < bestE - E - 4 (N - 1); without
    // it `asp` is kept far from every key.
    int best_d = 0, above = 0;
    const int asp0 = aspiration ? 0 : 1 << 29;
    int asp = asp0;
    // LDS addresses less their part in p
    const uint32_t base = lds_offset(lds), ct_base = base + (uint32_t)L::CT;
    uint32_t ct[NW];
#pragma unroll
    for (int h = 0; h < NW; ++h) ct[h] = (uint32_t)(4 * (lane + 64 * h));
    const uint32_t qt = base + (uint32_t)(L::QT + 4 * lane);  // + 4p: Q_(p + lane)
    const uint32_t sy = base + (uint32_t)(L::SP - lane - 64 * (NW - 1));  // + 2p: last word's SP[2p - j]
    const uint32_t sz = base + (uint32_t)(L::SP + 2 * lane);  // - p: SP[2 lane - p]

    // The least admissible key and the lanes that hold it, for the coming step.
    int m;
    uint64_t T[NW];
    auto keys = [&](int slot, int thr, int *key) {
        int kmin = INT_MAX;
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            key[h] = tabu[h] < slot || D[h] < thr ? D[h] : INT_MAX;
            kmin = h ? min(kmin, key[h]) : key[h];
        }
        return kmin;
    };
    {
        int key[NW];
        m = wave_min(keys(0, -4 * (N - 1) - asp, key));
#pragma unroll
        for (int h = 0; h < NW; ++h) T[h] = ballot(key[h] == m);
    }

    // Steps in blocks of 64: one Philox call per lane supplies the draws of
    // a block (read back with readlane), and the inner loop carries no
    // refill test.  Within a block the tenures count from its start, and
    // D_j = 4 d_j + 32 (moves made in the block).
    for (int t0 = 1; t0 <= sch.T; t0 += 64) {
        uint32_t dr0;
        int expire;  // lane l: slot l plus that step's tenure
        {
            const Draw4 d = philox10(entity, gen, (uint32_t)(t0 + lane), kTagStep, k0, k1);
            dr0 = d.w0;
            expire = lane + sch.lo + (int)below(d.w1, (uint32_t)(sch.hi - sch.lo + 1));
        }
        const int steps = __builtin_amdgcn_readfirstlane(min(sch.T - t0 + 1, 64));
        int off = -4 * (N - 1);  // 32 (moves made in the block) - 4 (N - 1)
        int slot = 0;
        do {
            // of several tied moves keep the r-th (ascending), r = (u0 * count) >> 32
            int c[NW], count = 0;
#pragma unroll
            for (int h = 0; h < NW; ++h) {
                c[h] = __popcll(T[h]);
                asm("" : "+s"(c[h]));  // 32-bit scalar arithmetic
                count += c[h];
            }
            if (__builtin_expect(count > 1, 0)) {
                int r = (int)below(readlane_u(dr0, slot), (uint32_t)count);
                bool found = false;
#pragma unroll
                for (int h = 0; h < NW; ++h) {
                    const bool here = !found && (h == NW - 1 || r < c[h]);
                    if (here) {
                        uint64_t t = T[h];
                        for (; r > 0; --r) t &= t - 1ull;  // drop the r lowest
                        T[h] = t & (0ull - t);
                    } else {
                        r -= found ? 0 : c[h];
                        T[h] = 0ull;
                    }
                    found |= here;
                }
            }
            const int gain = m - off;  // E' - E = 4 (N - 1 + d_p)
            off += 32;
            asm("" : "+s"(off));
            above += gain;
            asp += gain;
            if (__builtin_expect(above < 0, 0)) {
                best_d += above;
                above = 0;
                asp = asp0;
                uint64_t b[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
                for (int h = 0; h < NW; ++h) b[h] = ballot(nr[h] > 0) ^ T[h];
                best = make_mask<NW>(b[0], b[1], b[2], b[3]);
            }

            // All of the moved position p (the lane of T's one bit): its new
            // spin, its tenure and its key 4 (-d_p - 2 (N - 1)).  With x = 0
            // its entry Q_2p stays, and the update below changes its D by
            // z nsp4: -16 with the old spin (one neighbour per lane: set
            // while the entries are on their way), +16 with the new one
            // (several: branches, ahead of the reads).
            int x[NW], nsp4, nsp, p, tabu_new;  // tabu_new: slot + tenure
            uint32_t za;
            if constexpr (NW > 1) tabu_new = readlane(expire, slot);
            auto at = [&](auto H) {
                p = 64 * decltype(H)::value + __builtin_ctzll(T[decltype(H)::value]);
                za = sz - (uint32_t)p;
            };
            auto moved = [&](auto H) {
                constexpr int h = decltype(H)::value;
                if constexpr (NW == 1) tabu_new = readlane(expire, slot);
                const int d_new = off - gain + (NW == 1 ? 16 : -16);
                nsp4 = readlane(nr[h], p - 64 * h);
                nsp = nsp4 >> 2;
#pragma unroll
                for (int g = 0; g < NW; ++g) x[g] = mul_i24_s(nr[g], nsp);
                set_moved<128 * h>(T[h], za, d_new, tabu_new, nr[h], x[h], D[h], tabu[h]);
            };
            auto both = [&](auto H) {
                at(H);
                moved(H);
            };
            using std::integral_constant;
            if constexpr (NW == 1)
                at(integral_constant<int, 0>());
            else if (T[0] != 0ull)
                both(integral_constant<int, 0>());
            else if (NW == 2 || T[1] != 0ull)
                both(integral_constant<int, 1>());
            else if (NW == 3 || T[NW > 2 ? 2 : 0] != 0ull)
                both(integral_constant<int, NW == 2 ? 0 : 2>());
            else
                both(integral_constant<int, NW - 1>());

            // entries of the move (all reads before any write)
            const uint32_t qa = qt + 4u * (uint32_t)p;
            uint32_t ya = sy + 2u * (uint32_t)p;
            asm("" : "+v"(ya));  // one address, the words by offset
            uint32_t ca[NW];
            int cv[NW], qv[NW], yv[NW], zv[NW], e[NW];
#pragma unroll
            for (int h = 0; h < NW; ++h) {
                ca[h] = absdiff_add_s(4u * (uint32_t)p, ct[h], ct_base);
                cv[h] = lds_load_i32(ca[h]);
                qv[h] = lds_load_i32(qa + 256u * h);
                yv[h] = lds_load_i8(ya + 64u * (NW - 1 - h));
                zv[h] = lds_load_i8(za + 128u * h);
            }
            __builtin_amdgcn_sched_barrier(0);  // every load is out
            if constexpr (AHEAD) __builtin_amdgcn_s_setprio(0);
            if constexpr (NW == 1) moved(integral_constant<int, 0>());
            ++slot;
            asm("" : "+s"(slot));  // one register: the loop closes with one branch

#pragma unroll
            for (int h = 0; h < NW; ++h)
                move_score(cv[h], qv[h], yv[h], zv[h], nsp, nsp4, x[h], D[h], e[h]);
            // the next key; the wait states of the wavefront minimum take the
            // entries' new values
            int key[NW];
            int v = keys(slot, off - asp, key);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < NW; ++h) lds_store_i32(ca[h], e[h] - x[h]);
            __builtin_amdgcn_sched_barrier(0);
            v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_1032, 0xf, 0xf, true));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < NW; ++h) qv[h] = mad_i24_const<-2>(x[h], qv[h]);
            lds_store_i32(qa, qv[0]);
            __builtin_amdgcn_sched_barrier(0);
            v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_2301, 0xf, 0xf, true));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 1; h < NW; ++h) lds_store_i32(qa + 256u * h, qv[h]);
            __builtin_amdgcn_sched_barrier(0);
            v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_HALF_MIRROR, 0xf, 0xf, true));
            // AHEAD: from here to the next step's reads the wavefront issues
            // ahead of the others of its SIMD: the sooner its reads are out,
            // the more of their latency the others' work covers.  (In a wait
            // state of the minimum; before the minimum it gains 1 % more on
            // a full device and costs 1 % alone on a SIMD.)
            if constexpr (AHEAD) {
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_setprio(1);
                __builtin_amdgcn_sched_barrier(0);
            }
            v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_MIRROR, 0xf, 0xf, true));
            v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, LABS_DPP_ROW_BCAST15, 0xa, 0xf, false));
            v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, LABS_DPP_ROW_BCAST31, 0xc, 0xf, false));
            m = readlane(v, 63);
#pragma unroll
            for (int h = 0; h < NW; ++h) T[h] = ballot(key[h] == m);
            if constexpr (TRACE) trace[t0 + slot - 2] = (int16_t)p;  // uniform store
            wave_sync();
        } while (slot < steps);
        m -= 32 * 64;
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            D[h] -= 32 * 64;
            tabu[h] -= 64;
        }
    }

    WalkResult<NW> res;
    res.best = best;
    res.best_e = E0 + best_d;
    res.final_e = E0 + best_d + above;
    return res;
}

}  // namespace liblabs
