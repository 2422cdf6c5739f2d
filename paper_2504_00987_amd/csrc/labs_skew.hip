// Deviation from skew-symmetry d(S) (App. A of arXiv:2504.00987) for a batch
// of sequences, for gfx950, and its launcher.
//
// Skew-symmetry of an odd-length sequence t, m = 2c + 1 (Sec. II.C):
// t_{c+i} = (-1)^i t_{c-i} for i = 1..c; n_non-skew(t) counts the pairs that
// break it.  d(S) is the least n_non-skew over one rotation of S (its first
// r elements moved to the end) followed, for even N, by one deletion: odd N
// has N candidates, even N has N * N (rotation r, deleted position q).
//
// One wavefront per sequence, rotations over the lanes, everything on bit
// masks.  Let S2 be the mask repeated twice and R2 that of the reversed
// sequence, so the elements right and left of any point of any rotation are
// windows of S2 and R2.  A candidate's broken pairs are the set bits of
// right ^ left ^ (i odd).  For even N, deleting element q of rotation r
// leaves, with c = N / 2 - 1, the pairs
//   q <= c:  A_i (i <= c - q), B_i (i > c - q),
//   q >  c:  A'_i (i < q - c), B_i (i >= q - c),
// where A pairs elements c+1+i and c+1-i of the rotation, A' c+i and c-i, and
// B c+1+i and c-i.  So the least over q is sum B plus the least prefix sum
// of A - B or of A' - B: O(N) per rotation instead of O(N^2).  Bound: VALU (it
// issues on 0.75 of the cycles).  4096 rows of N = 120: 987 -> 13.3 us a call
// against comparing the pairs of all N^2 candidates byte by byte.
#include <algorithm>

#include "../../include/liblabs.h"
#include "labs_device.hpp"
#include "labs_internal.h"

namespace liblabs {

namespace {

// Words 0 .. W - 1 of the bits from `at` on.
template <int W>
__device__ __forceinline__ void bit_window(const uint32_t *bits, int at, uint32_t *out) {
    const uint32_t *p = bits + (at >> 5);
    uint32_t lo = p[0];
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t hi = p[w + 1];
        out[w] = __builtin_amdgcn_alignbit(hi, lo, (uint32_t)(at & 31));
        lo = hi;
    }
}

// Least broken-pair count over this lane's rotations lane, lane + 64, ..; W
// words hold the pairs i = 1 .. c of a candidate (bit i - 1).
template <int W>
__device__ __forceinline__ int least_broken(const uint32_t *S2, const uint32_t *R2, int N,
                                            int lane) {
    constexpr uint32_t kOdd = 0x55555555u;  // bit i - 1, i odd
    const int c = (N - 1) / 2;              // odd N: pairs; even N: N / 2 - 1 likewise
    int best = N;
    for (int r = lane; r < N; r += 64) {
        uint32_t H0[W], L0[W];
        int l0 = N - 1 - c - r;  // element r + c - i is bit l0 + i of R2
        l0 = l0 < 0 ? l0 + N : l0;
        bit_window<W>(S2, r + c + 1, H0);
        bit_window<W>(R2, l0 + 1, L0);
        if (N & 1) {
            int cnt = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int n = c - 32 * w;
                const uint32_t valid = n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u;
                cnt += __popc((H0[w] ^ L0[w] ^ kOdd) & valid);
            }
            best = min(best, cnt);
        } else {
            uint32_t H1[W], L1[W];
            int l1 = N - 2 - c - r;  // element r + c + 1 - i is bit l1 + i of R2
            l1 = l1 < 0 ? l1 + N : l1;
            bit_window<W>(S2, r + c + 2, H1);
            bit_window<W>(R2, l1 + 1, L1);
            int sum_b = 0, pa = 0, ma = 0, pc = 0, mc = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const uint32_t A = H1[w] ^ L1[w], B = H1[w] ^ L0[w], C = H0[w] ^ L0[w];
                const int n = c - 32 * w;
                const uint32_t valid = n >= 32 ? ~0u : n <= 0 ? 0u : (1u << n) - 1u;
                sum_b += __popc((B ^ kOdd) & valid);
                // A - B per pair is +1, -1 or 0: only where the bits differ,
                // +1 where A's (B ^ odd)'s complement is set
                const uint32_t b = B ^ kOdd, da = A ^ B, dc = C ^ B;
                const auto pair = [&](int i) {
                    const int sg = 1 - 2 * (int)((b >> i) & 1u);
                    pa += (int)((da >> i) & 1u) * sg;
                    pc += (int)((dc >> i) & 1u) * sg;
                    ma = min(ma, pa);
                    mc = min(mc, pc);
                };
                // all words but the last are full (unrolled: 4096 rows of
                // N = 120 14.4 us, as one rolled loop 18.4)
                if (w + 1 < W) {
#pragma unroll
                    for (int i = 0; i < 32; ++i) pair(i);
                } else {
#pragma unroll 1
                    for (int i = 0; i < n; ++i) pair(i);
                }
            }
            best = min(best, sum_b + min(ma, mc));
        }
    }
    return best;
}

// The same for N <= 32, lane r's rotation r, on masks in registers.
__device__ __forceinline__ int least_broken_short(uint64_t S2, uint64_t R2, int N, int lane) {
    const int c = (N - 1) / 2, r = min(lane, N - 1);
    const uint32_t valid = (1u << c) - 1u, odd = 0x55555555u;
    int l0 = N - 1 - c - r;
    l0 = l0 < 0 ? l0 + N : l0;
    const uint32_t H0 = (uint32_t)(S2 >> (r + c + 1)), L0 = (uint32_t)(R2 >> (l0 + 1));
    if (N & 1) return __popc((H0 ^ L0 ^ odd) & valid);
    int l1 = N - 2 - c - r;
    l1 = l1 < 0 ? l1 + N : l1;
    const uint32_t H1 = (uint32_t)(S2 >> (r + c + 2)), L1 = (uint32_t)(R2 >> (l1 + 1));
    const uint32_t B = H1 ^ L0, b = B ^ odd, da = L1 ^ L0, dc = H0 ^ H1;  // A ^ B, C ^ B
    int pa = 0, ma = 0, pc = 0, mc = 0;
    for (int i = 0; i < c; ++i) {
        const int sg = 1 - 2 * (int)((b >> i) & 1u);
        pa += (int)((da >> i) & 1u) * sg;
        pc += (int)((dc >> i) & 1u) * sg;
        ma = min(ma, pa);
        mc = min(mc, pc);
    }
    return __popc(b & valid) + min(ma, mc);
}

template <int WPG>
__global__ __launch_bounds__(64 * WPG) void skew_deviation_kernel(
    const int8_t *__restrict__ seqs, const int32_t *__restrict__ ns, int32_t n_uniform,
    int32_t stride, int64_t count, int32_t *__restrict__ out) {
    // 2 N <= 512 bits and the word after the last window
    constexpr int kWords = 2 * LABS_MAX_N / 32 + 4;
    __shared__ uint32_t bits[WPG][2][kWords];
    const int wave = threadIdx.x >> 6;
    const int lane = lane_id();
    const int64_t b = (int64_t)blockIdx.x * WPG + wave;
    if (b >= count) return;  // whole wavefronts only: no workgroup barrier below
    const int N = __builtin_amdgcn_readfirstlane(ns ? ns[b] : n_uniform);
    const int8_t *row = seqs + b * (int64_t)stride;
    uint32_t *S2 = bits[wave][0], *R2 = bits[wave][1];
    // N <= 32: the doubled masks in scalar registers, the row read once
    // (262144 rows of N = 8: 57 us a call; 75 through LDS and the loop below,
    // whose second trip waits for the memory again)
    if (N <= 32) {
        const uint64_t s = ballot(lane < N && row[lane < N ? lane : 0] < 0);
        const uint64_t r = __builtin_bitreverse64(s) >> (64 - N);
        out[b] = wave_min(least_broken_short(s | (s << N), r | (r << N), N, lane));  // every lane
        return;
    }
    for (int x0 = 0; x0 < 2 * N + 64; x0 += 64) {
        const int x = x0 + lane, k = x < N ? x : x - N;
        const bool in = x < 2 * N;
        const uint64_t f = ballot(in && row[in ? k : 0] < 0);
        const uint64_t r = ballot(in && row[in ? N - 1 - k : 0] < 0);
        if (x0 / 32 + 1 < kWords) {
            S2[x0 / 32] = (uint32_t)f;  // uniform values, every lane
            S2[x0 / 32 + 1] = (uint32_t)(f >> 32);
            R2[x0 / 32] = (uint32_t)r;
            R2[x0 / 32 + 1] = (uint32_t)(r >> 32);
        }
    }
    wave_sync();
    const int words = ((N - 1) / 2 + 31) / 32;
    int best;
    if (words <= 1)
        best = least_broken<1>(S2, R2, N, lane);
    else if (words == 2)
        best = least_broken<2>(S2, R2, N, lane);
    else if (words == 3)
        best = least_broken<3>(S2, R2, N, lane);
    else
        best = least_broken<4>(S2, R2, N, lane);
    out[b] = wave_min(best);  // uniform value, every lane
}

}  // namespace

hipError_t launch_skew_deviation(const int8_t *seqs, const int32_t *ns, int32_t n_uniform,
                                 int32_t stride, int64_t count, int32_t *out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    constexpr int WPG = 4;
    // at most 2^30 work-items per launch (a grid's x extent in work-items is
    // a 32-bit count): larger batches run as consecutive launches
    constexpr int64_t kRowsPerLaunch = (int64_t(1) << 30) / 64;
    for (int64_t b0 = 0; b0 < count; b0 += kRowsPerLaunch) {
        const int64_t n = std::min(kRowsPerLaunch, count - b0);
        hipLaunchKernelGGL(skew_deviation_kernel<WPG>, dim3((unsigned)((n + WPG - 1) / WPG)),
                           dim3(64 * WPG), 0, s, seqs + b0 * (int64_t)stride, ns ? ns + b0 : nullptr,
                           n_uniform, stride, n, out + b0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace liblabs
