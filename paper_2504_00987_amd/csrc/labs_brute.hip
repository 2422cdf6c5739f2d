// Exhaustive minima of Eq. (2) over all sequences of one length, and over
// the skew-symmetric ones of an odd length (Sec. II.C), for gfx950, and
// their launchers.
#include <algorithm>

#include "labs_device.hpp"
#include "labs_internal.h"

namespace liblabs {

namespace {


// ---------------------------------------------------------------------------
// Exhaustive minimum.  Lane g of the grid evaluates the codes
// [g * per, (g + 1) * per) (code c <=> sequence mask c << 1, so s_0 = +1) by
// Eq. (1)-(2) through popcounts: C_k = (N - k) - 2 popc((M ^ M >> k) & low).
// Lengths below the branch and bound's: 32-bit masks.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int code_energy(uint32_t M, int N) {
    int e = 0;
    for (int k = 1; k < N; ++k) {
        const int c = (N - k) - 2 * __popc((M ^ (M >> k)) & (~0u >> (32 - (N - k))));
        e += c * c;
    }
    return e;
}

// A wavefront's part of the result: its minimum, the count and the smallest
// code attaining it.
__device__ __forceinline__ void write_part(int best, int64_t cnt, uint64_t best_code, uint64_t wave,
                                           int32_t *part_e, int64_t *part_count,
                                           uint64_t *part_code) {
    const int m = wave_min(best);
    const int32_t n_at = best == m ? (int32_t)cnt : 0;
    const uint64_t c_at = best == m ? best_code : ~0ull;
    int64_t tot = 0;
    uint64_t code = ~0ull;
    for (int l = 0; l < 64; ++l) {
        tot += (int64_t)readlane(n_at, l);
        const uint64_t cl = ((uint64_t)readlane_u((uint32_t)(c_at >> 32), l) << 32) |
                            readlane_u((uint32_t)c_at, l);
        code = cl < code ? cl : code;
    }
    part_e[wave] = m;  // uniform values, stored by every lane
    part_count[wave] = tot;
    part_code[wave] = code;
}

__global__ __launch_bounds__(256) void bruteforce_kernel(int N, uint64_t per, uint64_t total,
                                                         int32_t *part_e, int64_t *part_count,
                                                         uint64_t *part_code) {
    const int lane = lane_id();
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t wave = g >> 6;
    uint64_t c0 = g * per, c1 = c0 + per;
    if (c0 > total) c0 = total;
    if (c1 > total) c1 = total;
    int best = INT_MAX;
    int64_t cnt = 0;
    uint64_t best_code = ~0ull;
    for (uint64_t c = c0; c < c1; ++c) {
        const int e = code_energy((uint32_t)(c << 1), N);
        if (e < best) {
            best = e;
            cnt = 1;
            best_code = c;
        } else if (e == best) {
            ++cnt;
        }
    }
    write_part(best, cnt, best_code, wave, part_e, part_count, part_code);
}

// Skew-symmetric sequences of odd length N = 2c + 1: lane g evaluates codes
// [g * per, (g + 1) * per) of the c free spins s_1..s_c (s_0 = +1); the
// other half is s_{c+i} = (-1)^i s_{c-i}.  Their C_k vanish for odd k, so E
// sums C_k^2 over even k only.  The code written back is the free-spin
// pattern F (bit i set <=> s_i = -1, i = 0..c).
template <int NW>
__device__ __forceinline__ typename MaskOf<NW>::type skew_mask(uint64_t F, int c) {
    // R_i = F_{c-i}; bit c + i of the sequence is R_i ^ (i odd), i = 1..c
    const uint64_t R = __builtin_bitreverse64(F) >> (63 - c);
    const uint64_t hiF = ((c >= 63 ? ~0ull : ((1ull << (c + 1)) - 1ull)) & ~1ull);
    const uint64_t U = (R ^ 0xAAAAAAAAAAAAAAAAull) & hiF;
    const uint64_t lo = F | (U << c);
    if constexpr (NW == 1) {
        return lo;
    } else {
        const uint64_t hi = c == 0 ? 0ull : (U >> (64 - c));
        return make_mask<NW>(lo, hi);
    }
}

template <int NW>
__global__ __launch_bounds__(256) void skew_bruteforce_kernel(int N, uint64_t per, uint64_t total,
                                                              int32_t *part_e, int64_t *part_count,
                                                              uint64_t *part_code) {
    using Mask = typename MaskOf<NW>::type;
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t wave = g >> 6;
    const int c = (N - 1) / 2;
    uint64_t c0 = g * per, c1 = c0 + per;
    if (c0 > total) c0 = total;
    if (c1 > total) c1 = total;
    int best = INT_MAX;
    int64_t cnt = 0;
    uint64_t best_code = ~0ull;
    for (uint64_t code = c0; code < c1; ++code) {
        const uint64_t F = code << 1;
        const Mask M = skew_mask<NW>(F, c);
        int e = 0;
        for (int k = 2; k < N; k += 2) {
            const int ck = lag_corr(M, N, k);
            e += ck * ck;
        }
        if (e < best) {
            best = e;
            cnt = 1;
            best_code = F;
        } else if (e == best) {
            ++cnt;
        }
    }
    // the reduction shifts the code back
    write_part(best, cnt, best_code >> 1, wave, part_e, part_count, part_code);
}

// ---------------------------------------------------------------------------
// Branch and bound (unrestricted search).
// ---------------------------------------------------------------------------
// Spins are fixed from both ends, pair by pair: with the first m and last m
// known, the lags k >= N - m are known too (N - k pairs each), and every
// other lag with N - k odd adds at least 1.  A node whose known lags plus
// that exceed the least energy seen so far is dropped; ties are kept, so the
// count and the smallest code stay exact.
//
// Images with the same energy and s_0 = +1: alternating the signs of the odd
// positions flips s_1, so only s_1 = +1 is searched and every sequence counts
// twice.  Reversing (with the signs that restore s_0 = s_1 = +1) maps x to
//     x'_i = b (ab)^i x_{N-1-i},   a = x_{N-2}, b = x_{N-1},
// which is its own inverse; of x and x', the one with +1 where they first
// differ is searched and counts twice again.  That is decided at the roots:
// where the first m0 positions of both agree the whole subtree holds x and
// x' alike, and neither is dropped.  The smallest code is taken over all
// images.
//
// A node is 64 bits: the first m spins (bits 0..19) and the energy so far
// (bits 20..31; at most N (N - 1) / 2 <= 780, the mean over all sequences) in
// one word, the last m spins (bit j: s_{N-m+j}) in the other.  One wavefront
// takes 64 root nodes of depth m0 at a time from a queue and runs their
// subtrees in LDS: a stack per depth, always the deepest one that fills the
// wavefront, so every lane has a node until the queue is empty.  A node's
// children cost about ten vector instructions each.  Bound: the instructions of
// few wavefronts, as many scalar as vector ones: the stacks (15 KB at n = 33)
// leave two wavefronts per SIMD, each issuing on half of its cycles and waiting
// on 0.4, the VALU on 0.38 (0.43 at n = 36).  Against evaluating every code (a
// call): n = 26 235 -> 68 us, n = 30 3.3 -> 0.14 ms, n = 33 41 -> 0.33 ms; n = 36
// takes 2.3 ms, n = 40 54 ms.
constexpr uint32_t kTwice = 1u << 31;     // in a node's second word: x' is not searched
constexpr int kFirstLags = 2;              // evaluated before the leaves are gathered again
constexpr int kStackNodes = 64 + 4 * 64;  // below 64 when a batch's children come on top

// The queue of root batches is kQueues counters 256 bytes apart, each for the
// batches of one residue and taken from by the wavefronts of that residue:
// one counter serves a fetch-and-add in about 33 ns whatever its form, which
// would bound a queue of this many short entries.
constexpr uint32_t kQueues = 64, kQueueStride = 64;

// Odd lengths in [a, N - 1]: the least the lags of those lengths can add.
__device__ __forceinline__ int odd_lengths(int a, int N) { return N / 2 - a / 2; }

template <typename U>
__global__ __launch_bounds__(64) void search_kernel(int N, int m0, uint32_t batches,
                                                    uint32_t *queue, int32_t *bound,
                                                    int32_t *part_e, int64_t *part_count,
                                                    uint64_t *part_code) {
    extern __shared__ uint2 stack[];  // [N / 2 - m0 + 2][kStackNodes]
    const int lane = lane_id();
    const int half = N / 2;
    queue += kQueueStride * (blockIdx.x % kQueues);
    int held = 0;  // lane i: nodes on the stack of depth m0 + i
    int ub = __builtin_amdgcn_readfirstlane(*(volatile int32_t *)bound);
    bool roots = true;
    int best = INT_MAX;
    int64_t cnt = 0;
    uint64_t best_code = ~0ull;
    for (;;) {
        const uint64_t full = ballot(held >= 64);
        int level;
        if (full != 0ull) {
            level = 63 - __builtin_clzll(full);
        } else if (roots) {
            const uint32_t b = next_work(queue) * kQueues + blockIdx.x % kQueues;
            if (b >= batches) {
                roots = false;
                continue;
            }
            ub = min(ub, __builtin_amdgcn_readfirstlane(*(volatile int32_t *)bound));
            // an odd multiplier permutes the roots: a batch takes them from
            // all over the tree, so that batches are about equally large
            const uint32_t idx = ((b * 64u + (uint32_t)lane) * 0x9E3779B1u) & (64u * batches - 1u);
            const uint32_t l = (idx & ((1u << (m0 - 2)) - 1u)) << 2;  // s_0 = s_1 = +1
            const uint32_t h = idx >> (m0 - 2);
            int e = 0;
            for (int len = 1; len <= m0; ++len) {
                const int c = len - 2 * __popc((l ^ (h >> (m0 - len))) & ((1u << len) - 1u));
                e += c * c;
            }
            // the reversal: drop the root if its image comes first
            const uint32_t hr = __builtin_bitreverse32(h) >> (32 - m0);  // bit i: s_{N-1-i}
            const uint32_t flip = (hr & 1u ? ~0u : 0u) ^ ((hr ^ (hr >> 1)) & 1u ? 0xAAAAAAAAu : 0u);
            const uint32_t diff = (l ^ hr ^ flip) & ((1u << m0) - 1u);
            const bool first = diff == 0u || ((l & (diff & (0u - diff))) == 0u);
            const uint32_t twice = diff != 0u ? kTwice : 0u;
            const bool keep = first && e <= ub - odd_lengths(m0 + 1, N);
            const uint64_t kept = ballot(keep);
            const int at = readlane(held, 0);
            if (keep)
                stack[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u))] =
                    make_uint2(l | ((uint32_t)e << 20), h | twice);
            wave_sync();
            held += lane == 0 ? (int)__popcll(kept) : 0;
            continue;
        } else {
            const uint64_t some = ballot(held > 0);
            if (some == 0ull) break;
            level = __builtin_ctzll(some);
        }
        const int have = readlane(held, level);
        const int take = min(have, 64);
        held -= lane == level ? take : 0;
        const bool on = lane < take;
        const uint2 nd = stack[level * kStackNodes + have - take + (on ? lane : 0)];
        const uint32_t l = nd.x & 0xFFFFFu, h = nd.y & ~kTwice, twice = nd.y & kTwice;
        const int e = (int)(nd.x >> 20);
        const int m = m0 + level;
        wave_sync();
        if (m < half) {
            const uint32_t x = l ^ (h << 1);  // the pairs of lag N - 1 - m
            const int thr = ub - odd_lengths(m + 2, N);
            int at = readlane(held, level + 1);
            const int at0 = at;
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) {
                const uint32_t a = (uint32_t)(ch & 1) << m, b = (uint32_t)(ch >> 1);
                const int c = (m + 1) - 2 * __popc(x ^ a ^ b);
                const int e2 = mad_i24(c, c, e);
                const bool keep = on && e2 <= thr;
                const uint64_t kept = ballot(keep);
                if (keep)
                    stack[(level + 1) * kStackNodes + at +
                          __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u))] =
                        make_uint2(l | a | ((uint32_t)e2 << 20), (h << 1) | b | twice);
                at += (int)__popcll(kept);
            }
            held += lane == level + 1 ? at - at0 : 0;
            wave_sync();
            continue;
        }
        // all pairs fixed: the remaining lags 1 .. N - 1 - half, the longest
        // sums first.  C_k^2 added for k in [from, to); false once no lane
        // can reach the bound (the lengths still to come: half + 1 .. N - k - 1)
        auto lags = [&](U M, int from, int to, int &sum) {
            for (int k = from; k < to; ++k) {
                int p;
                if (sizeof(U) == 4 || N - k <= 32) {  // the pairs fit the low word
                    uint32_t x = (uint32_t)M >> k;
                    if constexpr (sizeof(U) == 8)
                        x = __builtin_amdgcn_alignbit((uint32_t)(M >> 32), (uint32_t)M, (uint32_t)k);
                    p = __popc(((uint32_t)M ^ x) & (~0u >> (32 - (N - k))));
                } else {
                    p = __popcll((M ^ (M >> k)) & (~0ull >> (64 - (N - k))));
                }
                const int c = (N - k) - 2 * p;
                sum = mad_i24(c, c, sum);
                if (ballot(on && sum <= ub - ((N - k) / 2 - (half + 1) / 2)) == 0ull) return false;
            }
            return true;
        };
        if (m == half) {
            // both values of an odd length's middle spin; what the first lags
            // leave (a fifth) is gathered again on the last stack
            const int thr = ub - ((N - kFirstLags) / 2 - (half + 1) / 2);
            int at = readlane(held, level + 1);
            const int at0 = at;
            for (uint32_t z = 0; z <= (uint32_t)(N & 1); ++z) {
                int sum = e;
                if (!lags((U)l | ((U)h << (N - half)) | ((U)z << half), 1, 1 + kFirstLags, sum))
                    continue;
                const bool keep = on && sum <= thr;
                const uint64_t kept = ballot(keep);
                if (keep)
                    stack[(level + 1) * kStackNodes + at +
                          __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u))] =
                        make_uint2(l | ((uint32_t)sum << 20), h | (z << 30) | twice);
                at += (int)__popcll(kept);
            }
            held += lane == level + 1 ? at - at0 : 0;
            wave_sync();
            continue;
        }
        const U M = (U)l | ((U)(h & 0xFFFFFu) << (N - half)) | ((U)(h >> 30) << half);
        int s = e;
        if (!lags(M, 1 + kFirstLags, N - half, s)) continue;
        if (on && s <= ub) {
            // the smallest code of the sequence and its images with s_0 = +1
            const uint64_t low = ~0ull >> (64 - N);
            const uint64_t X = (uint64_t)M;
            uint64_t R = __builtin_bitreverse64(X) >> (64 - N);
            R = R & 1ull ? ~R & low : R;
            auto least = [&](uint64_t v) {
                const uint64_t alt = (v ^ 0xAAAAAAAAAAAAAAAAull) & low;
                return alt < v ? alt : v;
            };
            const uint64_t cx = least(X), cr = least(R);
            const uint64_t code = (cr < cx ? cr : cx) >> 1;
            if (s < best) {
                best = s;
                cnt = 0;
                best_code = ~0ull;
            }
            if (s == best) {
                cnt += twice ? 4 : 2;
                best_code = code < best_code ? code : best_code;
            }
        }
        const int found = wave_min(on ? s : INT_MAX);
        if (found < ub) {
            ub = found;
            atomicMin(bound, found);  // one value from every lane
        }
    }
    write_part(best, cnt, best_code, (uint64_t)blockIdx.x, part_e, part_count, part_code);
}

// The search's start: its queue, and as the bound the least energy of W
// walks and of the mean over all sequences, N (N - 1) / 2.
constexpr int kStartThreads = 1024;
__global__ __launch_bounds__(kStartThreads) void search_start_kernel(const int32_t *best_e, int32_t W,
                                                                     int N, uint32_t *queue,
                                                                     int32_t *bound) {
    __shared__ int part[kStartThreads / 64];
    int m = N * (N - 1) / 2;
    for (int i = (int)threadIdx.x; i < W; i += kStartThreads) m = min(m, best_e[i]);
    if (threadIdx.x < kQueues) queue[kQueueStride * threadIdx.x] = 0u;
    part[threadIdx.x >> 6] = wave_min(m);  // uniform values, every lane
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int i = 0; i < kStartThreads / 64; ++i) m = min(m, part[i]);
    bound[0] = m;
}

// One workgroup: every thread a share of the wavefronts' parts, then thread 0
// the threads' (with one wavefront, 25 us for 4096 parts).
constexpr int kReduceThreads = 512;
__global__ __launch_bounds__(kReduceThreads) void bruteforce_reduce_kernel(int64_t waves,
                                                                          BruteParts p) {
    __shared__ int best_s[kReduceThreads / 64];
    __shared__ int64_t cnt_s[kReduceThreads / 64];
    __shared__ uint64_t code_s[kReduceThreads / 64];
    const int wave = (int)(threadIdx.x >> 6);
    int best = INT_MAX;
    int64_t cnt = 0;
    uint64_t code = ~0ull;
    for (int64_t w = threadIdx.x; w < waves; w += kReduceThreads) {
        const int e = p.part_e[w];
        const int64_t n = p.part_count[w];
        const uint64_t c = p.part_code[w];
        if (e < best) {
            best = e;
            cnt = 0;
            code = ~0ull;
        }
        if (e == best) {
            cnt += n;
            code = c < code ? c : code;
        }
    }
    const int m = wave_min(best);
    int64_t tot = 0;
    uint64_t cmin = ~0ull;
    // (a wavefront without parts, or whose parts hold no sequence, has no turn:
    // 64 of them took 4 us)
    for (uint64_t at = ballot(best == m && m != INT_MAX); at != 0ull; at &= at - 1ull) {
        const int l = __builtin_ctzll(at);
        tot += ((int64_t)readlane_u((uint32_t)(cnt >> 32), l) << 32) | readlane_u((uint32_t)cnt, l);
        const uint64_t cl = ((uint64_t)readlane_u((uint32_t)(code >> 32), l) << 32) |
                            readlane_u((uint32_t)code, l);
        cmin = cl < cmin ? cl : cmin;
    }
    best_s[wave] = m;  // uniform values, every lane
    cnt_s[wave] = tot;
    code_s[wave] = cmin;
    __syncthreads();
    if (threadIdx.x != 0) return;
    best = INT_MAX;
    for (int i = 0; i < kReduceThreads / 64; ++i) best = min(best, best_s[i]);
    tot = 0;
    cmin = ~0ull;
    for (int i = 0; i < kReduceThreads / 64; ++i)
        if (best_s[i] == best) {
            tot += cnt_s[i];
            cmin = code_s[i] < cmin ? code_s[i] : cmin;
        }
    p.out_e[0] = best;
    p.out_count[0] = 2 * tot;  // and the negations (s_0 = -1)
    p.out_code[0] = cmin << 1;
}

}  // namespace

// Lanes of the exhaustive search: every lane gets at least 64 codes, at
// most 2^18 lanes (4096 wavefronts) share the space.
static uint64_t brute_lanes(int n) {
    const uint64_t total = 1ull << (n - 1);
    uint64_t lanes = total >> 6;
    if (lanes < 64) lanes = 64;
    if (lanes > (1ull << 18)) lanes = 1ull << 18;
    return lanes;
}

int64_t brute_waves(int n) { return (int64_t)(brute_lanes(n) >> 6); }

// The skew-symmetric search has 2^c codes, c = (n - 1) / 2: the lane count
// of an exhaustive search over c + 1 spins.
int64_t skew_brute_waves(int n) { return brute_waves((n - 1) / 2 + 1); }

hipError_t launch_skew_bruteforce(int n, const BruteParts &p, hipStream_t s) {
    const int c = (n - 1) / 2;
    const uint64_t total = 1ull << c;
    const uint64_t lanes = brute_lanes(c + 1);
    const uint64_t per = (total + lanes - 1) / lanes;
    const unsigned blocks = (unsigned)(lanes / 256 > 0 ? lanes / 256 : 1);
    const unsigned threads = (unsigned)(lanes < 256 ? lanes : 256);
    if (n <= 64)
        hipLaunchKernelGGL(skew_bruteforce_kernel<1>, dim3(blocks), dim3(threads), 0, s, n, per,
                           total, p.part_e, p.part_count, p.part_code);
    else
        hipLaunchKernelGGL(skew_bruteforce_kernel<2>, dim3(blocks), dim3(threads), 0, s, n, per,
                           total, p.part_e, p.part_count, p.part_code);
    hipLaunchKernelGGL(bruteforce_reduce_kernel, dim3(1), dim3(kReduceThreads), 0, s, (int64_t)(lanes >> 6), p);
    return hipGetLastError();
}

// Wavefronts of the branch and bound: as many as its LDS lets a CU hold, and
// more to even out the subtrees.
constexpr int kSearchWaves = 4096;
int64_t search_waves() { return kSearchWaves; }
size_t search_queue_bytes() { return kQueues * kQueueStride * sizeof(uint32_t); }

hipError_t launch_search(int n, const BruteParts &p, const int32_t *walk_e, int32_t walks,
                         uint32_t *queue, int32_t *bound, hipStream_t s) {
    // roots of depth m0: 2^(2 m0 - 2) with s_0 = s_1 = +1
    // four pairs above the leaves: enough batches to balance, short stacks
    // (at n = 33 one pair more or less costs 10 to 25 %)
    const int m0 = std::min(n / 2 - 4, 13);
    const uint32_t batches = 1u << (2 * m0 - 8);
    const size_t lds = (size_t)(n / 2 - m0 + 2) * kStackNodes * sizeof(uint2);
    hipLaunchKernelGGL(search_start_kernel, dim3(1), dim3(kStartThreads), 0, s, walk_e, walks, n, queue, bound);
    if (n <= 32)
        hipLaunchKernelGGL(search_kernel<uint32_t>, dim3(kSearchWaves), dim3(64), lds, s, n, m0,
                           batches, queue, bound, p.part_e, p.part_count, p.part_code);
    else
        hipLaunchKernelGGL(search_kernel<uint64_t>, dim3(kSearchWaves), dim3(64), lds, s, n, m0,
                           batches, queue, bound, p.part_e, p.part_count, p.part_code);
    hipLaunchKernelGGL(bruteforce_reduce_kernel, dim3(1), dim3(kReduceThreads), 0, s, (int64_t)kSearchWaves, p);
    return hipGetLastError();
}

hipError_t launch_bruteforce(int n, const BruteParts &p, hipStream_t s) {
    const uint64_t total = 1ull << (n - 1);
    const uint64_t lanes = brute_lanes(n);
    const uint64_t per = (total + lanes - 1) / lanes;
    const unsigned blocks = (unsigned)(lanes / 256 > 0 ? lanes / 256 : 1);
    const unsigned threads = (unsigned)(lanes < 256 ? lanes : 256);
    hipLaunchKernelGGL(bruteforce_kernel, dim3(blocks), dim3(threads), 0, s, n, per, total,
                       p.part_e, p.part_count, p.part_code);
    hipLaunchKernelGGL(bruteforce_reduce_kernel, dim3(1), dim3(kReduceThreads), 0, s, (int64_t)(lanes >> 6), p);
    return hipGetLastError();
}

}  // namespace liblabs
