// Walk kernels of liblabs for gfx950 and their launchers.
//
//   energy_kernel   Eq. (2) for a batch of +-1 rows, 64 rows per workgroup
//   tabu_kernel     independent tabu walks (Alg. 2 / Alg. 4), one walk per
//                   wave, either one wave per walk or a persistent grid
//                   draining a longest-first work queue
//   tabu_kernel_group  two or four walks of N <= 32 per wave
//   fill_u32_kernel device-side fill (queue heads, flags), capturable
//   order_by_length_kernel  longest-first processing order built on the
//                   device (the allocation-free entry point's lengths)
#include <algorithm>
#include <mutex>

#include "../../include/liblabs.h"
#include "labs_device.hpp"
#include "labs_internal.h"

namespace liblabs {

namespace {


// ---------------------------------------------------------------------------
// Energies.
// ---------------------------------------------------------------------------
// Sign bits of 16 bytes (bit i set <=> byte i < 0).
__device__ __forceinline__ uint32_t sign_bits16(const uint4 &v) {
    auto four = [](uint32_t w, uint32_t weights, uint32_t acc) {
        return (uint32_t)__builtin_amdgcn_udot4((w >> 7) & 0x01010101u, weights, acc, false);
    };
    const uint32_t lo = four(v.y, 0x80402010u, four(v.x, 0x08040201u, 0u));
    const uint32_t hi = four(v.w, 0x80402010u, four(v.z, 0x08040201u, 0u));
    return lo | (hi << 8);
}

// Sign bits of a workgroup's rows into LDS (bit i set <=> s_i = -1; bits past
// N clear): thread r * chunks + c takes bits [16 c, 16 c + 16) of row r, whose
// length is len(r).  Rows may have any alignment and stride: the 16 bytes are
// read at any address (global loads need no alignment on this target), and
// the last chunk of a row from its last 16 bytes, so nothing past N is read.
// A thread has kDeep reads in flight: a workgroup lives for little more than
// these reads' latency, which one after another is what bounds it.
constexpr int kEnergyWaves = 4, kEnergyThreads = 64 * kEnergyWaves;
constexpr int kRowWords = LABS_MAX_N / 32;
template <int ROWS, typename Len>
__device__ __forceinline__ void load_row_masks(uint32_t (*mask)[kRowWords + 1],
                                               const int8_t *__restrict__ seqs, int stride,
                                               int words, Len len) {
    constexpr int kDeep = 4;
    const uint32_t chunks = 2u * (uint32_t)words, total = ROWS * chunks;
    const uint32_t magic = 65536u / chunks + 1u;  // i / chunks, exact for i < 4096
    for (uint32_t base = 0; base < total; base += kDeep * kEnergyThreads) {
        uint4 v[kDeep];
        int n[kDeep];
        const auto at = [&](int j, uint32_t &r, uint32_t &c) {
            const uint32_t i = base + (uint32_t)j * kEnergyThreads + threadIdx.x;
            r = (i * magic) >> 16;
            c = i - r * chunks;
            return i < total;
        };
#pragma unroll
        for (int j = 0; j < kDeep; ++j) {
            uint32_t r, c;
            const bool in = at(j, r, c);
            n[j] = len((int)min(r, (uint32_t)ROWS - 1u));
            const int x = 16 * (int)c;
            if (in && x < n[j] && n[j] >= 16)
                __builtin_memcpy(&v[j], seqs + (int)r * (int64_t)stride + min(x, n[j] - 16), 16);
        }
#pragma unroll
        for (int j = 0; j < kDeep; ++j) {
            uint32_t r, c, bits = 0u;
            const bool in = at(j, r, c);
            const int x = 16 * (int)c, left = n[j] - x;
            if (in && left > 0) {
                if (n[j] >= 16) {
                    bits = sign_bits16(v[j]) >> max(16 - left, 0);
                } else {
                    const int8_t *row = seqs + (int)r * (int64_t)stride;
                    for (int i = 0; i < n[j]; ++i) bits |= (uint32_t)(row[i] < 0) << i;
                }
            }
            if (in) ((uint16_t *)mask[r])[c] = (uint16_t)bits;
        }
    }
}

// Eq. (2) for 64 rows per workgroup: lane l of every wavefront holds row l as
// a bit mask and the four wavefronts take every fourth lag.  Bound: VALU,
// three instructions per 32 pairs and lag and four per lag (row l in one lane
// needs no cross-lane sum, and a shift by a fixed number of bits is one
// instruction a word; a row per wavefront takes twice as many).  A group takes
// as long as its longest row; 256 rows ordered by length first are 8 % faster
// for a million rows and no faster for 262144.  262144 rows of N in 20..128
// (34 MB): 14.8 us a call (124 with a row per wavefront on 256-bit masks,
// 15.6 with one read in flight and a lag a trip); of N in 3..256 41.6 (48.9).
constexpr int kEnergyRows = 64;
__global__ __launch_bounds__(kEnergyThreads) void energy_kernel(
    const int8_t *__restrict__ seqs, const int32_t *__restrict__ ns, int32_t n_uniform,
    int32_t stride, int64_t count, int32_t *__restrict__ out) {
    // rows of 9 words: lanes read their rows' words without bank conflicts
    __shared__ uint32_t mask[kEnergyRows][kRowWords + 1];
    __shared__ int part[kEnergyWaves][kEnergyRows];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t r0 = (int64_t)blockIdx.x * kEnergyRows;
    const int rows = (int)min((int64_t)kEnergyRows, count - r0);
    const int N = lane < rows ? (ns ? ns[r0 + lane] : n_uniform) : 0;
    const int nmax = -wave_min(-N);
    const int words = (nmax + 31) >> 5;
    load_row_masks<kEnergyRows>(mask, seqs + r0 * (int64_t)stride, stride, words,
                                [&](int r) { return __shfl(N, r); });
    __syncthreads();
    int e = lane_energy<kEnergyWaves>(words, mask[lane], N, nmax, wave);
    part[wave][lane] = e;
    __syncthreads();
    if (wave == 0 && lane < rows) {
#pragma unroll
        for (int w = 1; w < kEnergyWaves; ++w) e += part[w][lane];
        out[r0 + lane] = e;
    }
}


// ---------------------------------------------------------------------------
// Batched tabu walks.
// ---------------------------------------------------------------------------
// Start mask of walk w: row w of the caller's starts, or the draws
// (w, 0, q, START) (bits 128 q .. 128 q + 127).
template <int NW>
__device__ __forceinline__ typename MaskOf<NW>::type walk_start(const TabuLaunchArgs &a,
                                                                int64_t w, int N) {
    const int lane = lane_id();
    uint64_t wd[4] = {0ull, 0ull, 0ull, 0ull};
    if (a.starts != nullptr) {
        const int8_t *row = a.starts + w * (int64_t)a.start_stride;
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            const int i = lane + 64 * h;
            wd[h] = ballot(i < N && row[i] < 0);
        }
    } else {
#pragma unroll
        for (int q = 0; q < (NW + 1) / 2; ++q) {
            const Draw4 d = philox10((uint32_t)w, 0u, (uint32_t)q, kTagStart, a.k0, a.k1);
            wd[2 * q] = (uint64_t)d.w0 | ((uint64_t)d.w1 << 32);
            if (2 * q + 1 < NW) wd[2 * q + 1] = (uint64_t)d.w2 | ((uint64_t)d.w3 << 32);
        }
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            const int b = N - 64 * h;  // bits of word h inside the sequence
            wd[h] &= b >= 64 ? ~0ull : b <= 0 ? 0ull : ((1ull << b) - 1ull);
        }
    }
    return make_mask<NW>(wd[0], wd[1], wd[2], wd[3]);
}

// Word 0 of the draw (walk, 0, 0, LEN), where the rule draws the length.
__device__ __forceinline__ uint32_t length_draw(const RuleParams &r, uint32_t k0, uint32_t k1,
                                                uint32_t walk) {
    return r.steps_rule >= 2 ? philox10(walk, 0u, 0u, kTagLen, k0, k1).w0 : 0u;
}

// One walk on one wavefront, NW neighbours per lane.
template <int NW, bool TRACE, bool AHEAD>
__device__ void run_tabu_item(const TabuLaunchArgs &a, int64_t w, int N, uint8_t *lds) {
    const int lane = lane_id();
    const auto M = walk_start<NW>(a, w, N);
    const Schedule sch = make_schedule(a.rule, N, length_draw(a.rule, a.k0, a.k1, (uint32_t)w));
    const WalkResult<NW> r =
        tabu_walk<NW, TRACE, AHEAD>(N, M, sch, a.rule.aspiration, a.k0, a.k1, (uint32_t)w, 0u, lds,
                             TRACE ? a.trace + w * (int64_t)a.trace_stride : nullptr);
    int8_t *out = a.best_seq + w * (int64_t)a.out_stride;
    for (int i = lane; i < a.out_stride; i += 64)
        out[i] = i < N ? (m_bit(r.best, i) ? (int8_t)-1 : (int8_t)1) : (int8_t)0;
    a.best_e[w] = r.best_e;  // uniform values, stored by every lane
    a.final_e[w] = r.final_e;
}

// ---------------------------------------------------------------------------
// Several walks per wavefront (N <= 32).
// ---------------------------------------------------------------------------
// A wavefront runs 64 / GL walks of N <= GL NL (GL = 16 or 32 lanes) at once,
// lane l of a group of GL owning neighbours j = l + GL h, h < NL.  The step is
// tabu_walk's, with every per-walk quantity (the sequence mask, the energy,
// the best, the chosen move, the schedule) held per lane for the lane's own
// walk instead of in scalar registers, and the minimum taken within each
// group of lanes.  Walks of different lengths share the step loop; a walk past
// its last step takes no move.  Bound: VALU on a full device (72 instructions
// a step of four walks), where 16 lanes with two neighbours each share the
// per-walk work over half the lanes of 32 with one; one step's chain of
// dependent instructions on a part-filled one, where the second neighbour
// lengthens it (group2_form).  16384 walks of N = 32 and 128 steps on 32 lanes
// 118 us a call, on 16 100; 64 walks 53 and 64.

// The values of the two 16-lane rows of each half wavefront, in every lane of
// the half.
__device__ __forceinline__ void row_pair(int v, int &a, int &b) {
    const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    a = (int)r[0];
    b = (int)r[1];
}

// Minimum and sum over each group of GL lanes, every lane receiving its
// group's value: rows of 16 by DPP, then two rows.
template <int GL>
__device__ __forceinline__ int group_min(int v) {
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_1032, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_2301, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_HALF_MIRROR, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_MIRROR, 0xf, 0xf, true));
    if constexpr (GL == 32) {
        int a, b;
        row_pair(v, a, b);
        v = min(a, b);
    }
    return v;
}

template <int GL>
__device__ __forceinline__ int group_sum(int v) {
    v += __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_1032, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, LABS_DPP_QUAD_2301, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_HALF_MIRROR, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, LABS_DPP_ROW_MIRROR, 0xf, 0xf, true);
    if constexpr (GL == 32) {
        int a, b;
        row_pair(v, a, b);
        v = a + b;
    }
    return v;
}

// |a - b| + c in one instruction, every operand per lane.
__device__ __forceinline__ uint32_t absdiff_add_v(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_sad_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// set_moved for the moved positions of all groups, the lanes of `at`, with
// per-lane values.
template <int OFF>
__device__ __forceinline__ void set_moved_v(uint64_t at, uint32_t za, int d_new, int tabu_new,
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
        : "s"(at), "v"(za), "v"(d_new), "v"(tabu_new), "n"(OFF)
        : "memory", "scc");
}

// Walks at processing-order positions pos0 .. pos0 + 64 / GL - 1 (those below
// `end`), all of N <= GL NL, on one wavefront; `lds` holds their tables.
// Results as the one-walk-per-wavefront form writes them.
template <int GL, int NL, bool TRACE>
__device__ void run_group_walks(const TabuLaunchArgs &a, int64_t pos0, int64_t end,
                                uint8_t *lds_wave) {
    constexpr int SPAN = GL * NL;
    static_assert((GL == 16 || GL == 32) && SPAN <= 32, "rows of lanes, one-word masks");
    constexpr uint32_t kGroupMask = GL == 32 ? ~0u : 0xffffu;
    using L = WalkTables<SPAN>;
    const int lane = lane_id();
    const int g = lane / GL, l = lane % GL;
    const int64_t pos = pos0 + g;
    const bool live = pos < end;
    const int64_t w = live ? (a.order ? (int64_t)a.order[pos] : pos) : 0;
    const int N = live ? (a.ns ? a.ns[w] : a.n_uniform) : 0;
    uint8_t *const lds = lds_wave + g * L::BYTES;
    int32_t *const CT = (int32_t *)(lds + L::CT);
    int32_t *const QT = (int32_t *)(lds + L::QT);
    int8_t *const SP = (int8_t *)(lds + L::SP);

    // start (bit i set <=> s_i = -1): the caller's row, or the low N bits
    // of the draw (w, 0, 0, START)
    uint32_t M = 0u;
    if (a.starts != nullptr) {
        const int8_t *row = a.starts + w * (int64_t)a.start_stride;
#pragma unroll
        for (int h = 0; h < NL; ++h) {
            const int j = l + GL * h;
            M |= ((uint32_t)(ballot(j < N && row[j] < 0) >> (GL * g)) & kGroupMask) << (GL * h);
        }
    } else {
        const Draw4 d = philox10((uint32_t)w, 0u, 0u, kTagStart, a.k0, a.k1);
        M = N > 0 ? d.w0 & (0xffffffffu >> (32 - N)) : 0u;
    }
    Schedule sch = make_schedule(a.rule, N, length_draw(a.rule, a.k0, a.k1, (uint32_t)w));
    if (!live) sch.T = 0;
    const uint32_t Mr = N > 0 ? __builtin_bitreverse32(M) >> (32 - N) : 0u;  // bit i: s_{N-1-i}

    // the tables (entries past the sequence 0)
    int sq_e = 0;
#pragma unroll
    for (int h = 0; h < NL; ++h) {
        const int k = l + GL * h;
        const int c = k > 0 && k < N ? (N - k) - 2 * __popc((M ^ (M >> k)) & ((1u << (N - k)) - 1u))
                                     : 0;
        CT[k] = 2 * c;
        sq_e += c * c;
    }
    auto pairs = [&](int m) -> int {  // Q_m
        if (m > 2 * N - 2) return 0;
        const bool low = m < N;
        const int cnt = low ? m + 1 : 2 * N - 1 - m;
        const uint32_t A = low ? Mr >> (N - 1 - m) : M >> (m - (N - 1));
        return cnt - 2 * __popc((A ^ (low ? M : Mr)) & (0xffffffffu >> (32 - cnt)));
    };
#pragma unroll
    for (int i = 0; i < 2 * NL; ++i) QT[l + GL * i] = 2 * pairs(l + GL * i);
#pragma unroll
    for (int i = 0; i < 3 * NL; ++i) {
        const int x = l + GL * i - SPAN;
        SP[x] = x >= 0 && x < N ? (((M >> x) & 1u) ? (int8_t)-4 : (int8_t)4) : (int8_t)0;
    }
    const int E0 = group_sum<GL>(sq_e);
    wave_sync();

    // D_j = Q_2j - 1 - s_j v_j, v_j = sum_i s_i C_|i-j|
    const uint32_t base = lds_offset(lds);
    int D[NL], nr[NL], tabu[NL];
#pragma unroll
    for (int h = 0; h < NL; ++h) {
        const int j = l + GL * h;
        int v = 0;  // 8 v_j
        for (int i = 0; i < SPAN; ++i) {
            const int k = i < j ? j - i : i - j;
            v += __mul24(SP[i], CT[k]);
        }
        nr[h] = j < N ? (((M >> j) & 1u) ? 4 : -4) : 0;
        // past the sequence: never a minimum, never admissible
        D[h] = j < N ? 4 * pairs(2 * j) - 4 + nr[h] * (v >> 3) : 0x3fffffff;
        tabu[h] = j < N ? 0 : INT_MAX;
    }
    uint32_t P = ~M;  // bit i set <=> s_i = +1
    uint32_t best = P;
    int ed = 0;  // E - E0
    int bd = 0;  // its minimum over the walk
    const int N4 = 4 * (N - 1);
    // minus N4, and far below every key without aspiration
    const int asp4 = -N4 - (a.rule.aspiration ? 0 : 1 << 29);
    int thr = asp4;  // aspiration threshold for D
    const uint32_t ct = base + (uint32_t)L::CT;
    const uint32_t qt = base + (uint32_t)(L::QT + 4 * l);
    const uint32_t sy = base + (uint32_t)(L::SP - (l + GL * (NL - 1)));
    const uint32_t sz = base + (uint32_t)(L::SP + 2 * l);
    uint32_t ct4[NL];
#pragma unroll
    for (int h = 0; h < NL; ++h) ct4[h] = 4u * (uint32_t)(l + GL * h);
    const uint32_t group_at = (uint32_t)(GL * g);  // of a ballot
    const int src0 = 4 * GL * g;                   // byte address of the group's first lane
    const int T_all = -wave_min(-sch.T);           // the longest walk of the wavefront
    // the shortest one: no walk ends before (a group without a walk runs
    // along in its own tables and stores nothing)
    const int T_each = wave_min(live ? sch.T : INT_MAX);

    for (int t0 = 1; t0 <= T_all; t0 += GL) {
        // lane l of a group: the draws of its walk's step t0 + l
        uint32_t dr0;
        int expire;
        {
            const Draw4 d = philox10((uint32_t)w, 0u, (uint32_t)(t0 + l), kTagStep, a.k0, a.k1);
            dr0 = d.w0;
            expire = t0 + l + sch.lo + (int)below(d.w1, (uint32_t)(sch.hi - sch.lo + 1));
        }
        auto step = [&](const int t, auto every) {
            const int src = src0 + 4 * (t - t0);  // the lane holding this step's draws
            const uint32_t dr = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)dr0);
            const int tabu_new = __builtin_amdgcn_ds_bpermute(src, expire);
            int key[NL];
#pragma unroll
            for (int h = 0; h < NL; ++h)
                key[h] = tabu[h] < t || D[h] < thr ? D[h] : INT_MAX;
            int kmin = key[0];
#pragma unroll
            for (int h = 1; h < NL; ++h) kmin = min(kmin, key[h]);
            const int m = group_min<GL>(kmin);
            // ties: the r-th lowest tied neighbour of the group, r from the
            // step's first draw
            uint32_t tied = (uint32_t)(ballot(key[0] == m) >> group_at);
            if constexpr (NL == 2)
                tied = __builtin_amdgcn_perm((uint32_t)(ballot(key[1] == m) >> group_at), tied,
                                             0x05040100u);
            else
                tied &= kGroupMask;
            int r = (int)below(dr, (uint32_t)__popc(tied));
            while (r > 0) {  // drop the r lowest
                tied &= tied - 1u;
                --r;
            }
            const uint32_t pick = (uint32_t)__builtin_ctz(tied);
            if (!decltype(every)::value && t > sch.T) return;

            const int nsp = __builtin_amdgcn_sbfe((int)P, pick, 1) | 1;  // -s_p
            const int nsp4 = 4 * nsp;
            P ^= 1u << pick;
            const uint32_t za = sz - pick;
            const int off = N4 - 32 * (t - 1);
            const int gain = m + off;  // E' - E
            // the moved position (as in tabu_walk): x = 0 keeps Q_2p, and
            // the update changes its D by +16 (its z is the new spin)
            const int d_new = 16 - gain - off;  // 4 (-d_p - 2 (N - 1)) + 32 t - 16
            int x[NL];
#pragma unroll
            for (int h = 0; h < NL; ++h) {
                x[h] = mul_i24(nr[h], nsp);
                const uint64_t at = ballot(l + GL * h == (int)pick);
                if (h == 0)
                    set_moved_v<0>(at, za, d_new, tabu_new, nr[h], x[h], D[h], tabu[h]);
                else
                    set_moved_v<2 * GL>(at, za, d_new, tabu_new, nr[h], x[h], D[h], tabu[h]);
            }
            const uint32_t qa = qt + 4u * pick;
            uint32_t ya = sy + 2u * pick;
            asm("" : "+v"(ya));  // one address, the words by offset
            uint32_t ca[NL];
            int cv[NL], qv[NL], yv[NL], zv[NL];
#pragma unroll
            for (int h = 0; h < NL; ++h) {
                ca[h] = absdiff_add_v(4u * pick, ct4[h], ct);
                cv[h] = lds_load_i32(ca[h]);
                qv[h] = lds_load_i32(qa + 4u * GL * h);
                yv[h] = lds_load_i8(ya + (uint32_t)(GL * (NL - 1 - h)));
                zv[h] = lds_load_i8(za + 2u * GL * h);
            }
            __builtin_amdgcn_sched_barrier(0);  // every load is out
            ed += gain;
            best = ed < bd ? P : best;
            bd = min(bd, ed);
            thr = bd - ed + (asp4 + 32 * t);
            if constexpr (TRACE) {
                if (l == 0 && live) a.trace[w * (int64_t)a.trace_stride + t - 1] = (int16_t)pick;
            }
#pragma unroll
            for (int h = 0; h < NL; ++h) {
                const int e = mad_i24(yv[h], nsp, cv[h]);
                D[h] = mad_i24(x[h], cv[h] + e + qv[h], D[h]);
                D[h] = mad_i24(zv[h], nsp4, D[h]);
                lds_store_i32(ca[h], e - x[h]);
                lds_store_i32(qa + 4u * GL * h, mad_i24_const<-2>(x[h], qv[h]));
            }
        };
        int t = t0;
        const int end = __builtin_amdgcn_readfirstlane(min(T_all, t0 + GL - 1));
        const int each = min(T_each, end);
        for (; t <= each; ++t) {
            step(t, std::true_type());
            wave_sync();
        }
        for (; t <= end; ++t) {
            step(t, std::false_type());
            wave_sync();
        }
    }
    if (live) {
        int8_t *out = a.best_seq + w * (int64_t)a.out_stride;
        for (int i = l; i < a.out_stride; i += GL)
            out[i] = i < N ? (((best >> i) & 1u) ? (int8_t)1 : (int8_t)-1) : (int8_t)0;
        if (l == 0) {
            a.best_e[w] = E0 + bd;
            a.final_e[w] = E0 + ed;
        }
    }
}

// Walks of N <= GL NL at positions [begin, end), G = 64 / GL per wavefront and
// WAVES wavefronts per workgroup.  PERSIST: a grid sized to the device takes G
// positions at a time from the queue head `counter`; otherwise one wavefront
// per G positions.
template <int GL, int NL, int WAVES, bool PERSIST, bool TRACE>
__global__ __launch_bounds__(64 * WAVES) void tabu_kernel_group(TabuLaunchArgs a, int64_t begin,
                                                                int64_t end, uint32_t *counter) {
    constexpr int G = 64 / GL;
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[WAVES][G * WalkTables<GL * NL>::BYTES];
    uint8_t *lds = lds_all[threadIdx.x >> 6];
    if constexpr (PERSIST) {
        for (int64_t pos = begin + next_work(counter, G); pos < end;
             pos = begin + next_work(counter, G))
            run_group_walks<GL, NL, TRACE>(a, pos, end, lds);
    } else {
        const int64_t pos = begin + ((int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6)) * G;
        if (pos < end) run_group_walks<GL, NL, TRACE>(a, pos, end, lds);
    }
}

// The walk at one position of the processing order, of N <= 64 NWMAX, on the
// fewest neighbours per lane that hold it.
template <int NWMAX, bool TRACE, bool AHEAD>
__device__ __forceinline__ void run_position(const TabuLaunchArgs &a, int64_t pos, uint8_t *lds) {
    const int64_t w = a.order ? (int64_t)a.order[pos] : pos;
    const int N = __builtin_amdgcn_readfirstlane(a.ns ? a.ns[w] : a.n_uniform);
    if (NWMAX >= 4 && N > 192)
        run_tabu_item<NWMAX >= 4 ? 4 : 1, TRACE, AHEAD>(a, w, N, lds);
    else if (NWMAX >= 4 && N > 128)
        run_tabu_item<NWMAX >= 4 ? 3 : 1, TRACE, AHEAD>(a, w, N, lds);
    else if (NWMAX >= 2 && N > 64)
        run_tabu_item<NWMAX >= 2 ? 2 : 1, TRACE, AHEAD>(a, w, N, lds);
    else
        run_tabu_item<1, TRACE, AHEAD>(a, w, N, lds);
}

// Walks of N <= 64 NWMAX at positions [begin, end) of the processing order,
// one per wavefront.  PERSIST: a grid sized to the device drains the range
// through the queue head `counter`; otherwise one wavefront per position.
// TRACE: record every walk's moves (a separate instantiation, so that the
// untraced kernel does not carry the registers of the traced one).  AHEAD: as
// in tabu_walk (untraced grids).
template <int NWMAX, int WPG, bool PERSIST, bool TRACE, bool AHEAD>
__global__ __launch_bounds__(64 * WPG) void tabu_kernel(TabuLaunchArgs a, int64_t begin,
                                                        int64_t end, uint32_t *counter) {
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[WPG][WalkLds<NWMAX>::BYTES];
    const int wave = threadIdx.x >> 6;
    uint8_t *lds = lds_all[wave];
    if constexpr (PERSIST) {
        for (int64_t pos = begin + next_work(counter); pos < end;
             pos = begin + next_work(counter))
            run_position<NWMAX, TRACE, AHEAD>(a, pos, lds);
    } else {
        const int64_t pos = begin + (int64_t)blockIdx.x * WPG + wave;
        if (pos < end) run_position<NWMAX, TRACE, AHEAD>(a, pos, lds);
    }
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

// Processing order of W walks, longest first, from their lengths in device
// memory (LABS_MIN_N <= ns[w] <= LABS_MAX_N, checked by the host): one
// workgroup counts the lengths in LDS, turns the counts into the first
// position of each length (descending N), then every walk takes the next
// position of its length.  Walks of one length land in an order that
// depends on the atomics' timing; results do not depend on the order.
constexpr int kOrderThreads = 1024;
__global__ __launch_bounds__(kOrderThreads) void order_by_length_kernel(
    const int32_t *__restrict__ ns, int64_t W, int32_t *__restrict__ order) {
    __shared__ int32_t next[LABS_MAX_N + 1];
    for (int n = threadIdx.x; n <= LABS_MAX_N; n += kOrderThreads) next[n] = 0;
    __syncthreads();
    for (int64_t w = threadIdx.x; w < W; w += kOrderThreads) atomicAdd(&next[ns[w]], 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t pos = 0;
        for (int n = LABS_MAX_N; n >= 0; --n) {
            const int32_t c = next[n];
            next[n] = pos;
            pos += c;
        }
    }
    __syncthreads();
    for (int64_t w = threadIdx.x; w < W; w += kOrderThreads)
        order[atomicAdd(&next[ns[w]], 1)] = (int32_t)w;
}

// Scratch of the allocation-free tabu batch: the queue heads
// (kNoAllocHeadBytes), then the per-walk lengths and the processing order
// (kNoAllocMaxWalks int32 each).  Each device holds its own copy for the
// life of the process; host code reaches it only through the address
// returned by noalloc_scratch_address, never through this name.
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

}  // namespace

hipError_t noalloc_scratch_address(int device, void **ptr) {
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        // the caller has made `device` current
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t launch_order_by_length(const int32_t *ns, int64_t W, int32_t *order, hipStream_t s) {
    if (W <= 0) return hipSuccess;
    hipLaunchKernelGGL(order_by_length_kernel, dim3(1), dim3(kOrderThreads), 0, s, ns, W, order);
    return hipGetLastError();
}

namespace {

// Work-items of one launch at most (a grid's x extent in work-items is a
// 32-bit count): a grid of one workgroup per few positions that would pass
// it runs as consecutive launches over sub-ranges of the positions.
constexpr int64_t kMaxLaunchItems = int64_t(1) << 30;

// launch(b, e, grid) for consecutive sub-ranges [b, e) of [begin, end), with
// `per_group` positions per workgroup of `lanes` lanes.
template <typename F>
hipError_t launch_in_ranges(int64_t begin, int64_t end, int per_group, int lanes, F &&launch) {
    const int64_t step = kMaxLaunchItems / lanes * per_group;
    for (int64_t b = begin; b < end; b += step) {
        const int64_t e = std::min(end, b + step);
        launch(b, e, (unsigned)((e - b + per_group - 1) / per_group));
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_energy(const int8_t *seqs, const int32_t *ns, int32_t n_uniform,
                         int32_t stride, int64_t count, int32_t *out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    return launch_in_ranges(0, count, kEnergyRows, kEnergyThreads,
                            [&](int64_t b, int64_t e, unsigned grid) {
        hipLaunchKernelGGL(energy_kernel, dim3(grid), dim3(kEnergyThreads), 0, s,
                           seqs + b * (int64_t)stride, ns ? ns + b : nullptr, n_uniform, stride,
                           e - b, out + b);
    });
}

namespace {

template <int NWMAX, int WPG, bool TRACE, bool AHEAD>
hipError_t launch_wave_t(const TabuLaunchArgs &a, int64_t begin, int64_t end, int groups,
                         uint32_t *counter, hipStream_t s) {
    if (groups > 0) {
        hipError_t e = launch_fill_u32(counter, 0u, 1, s);
        if (e != hipSuccess) return e;
        const int64_t need = (end - begin + WPG - 1) / WPG;
        hipLaunchKernelGGL((tabu_kernel<NWMAX, WPG, true, TRACE, false>),
                           dim3((unsigned)std::min<int64_t>(groups, need)), dim3(64 * WPG), 0, s, a,
                           begin, end, counter);
    } else {
        return launch_in_ranges(begin, end, WPG, 64 * WPG, [&](int64_t b, int64_t e, unsigned grid) {
            hipLaunchKernelGGL((tabu_kernel<NWMAX, WPG, false, TRACE, AHEAD>), dim3(grid), dim3(64 * WPG),
                               0, s, a, b, e, counter);
        });
    }
    return hipGetLastError();
}

template <int NWMAX, int WPG>
hipError_t launch_wave(const TabuLaunchArgs &a, int64_t begin, int64_t end, int groups,
                       int64_t ahead_from, uint32_t *counter, hipStream_t s) {
    if (end <= begin) return hipSuccess;
    if (a.trace != nullptr)
        return launch_wave_t<NWMAX, WPG, true, false>(a, begin, end, groups, counter, s);
    // Walks of one length from two wavefronts per SIMD on issue ahead of each
    // other (a call, without -> with): 4096 walks of N = 64 81.6 -> 77.2 us,
    // of N = 120 214 -> 200.  64 walks 30.7 -> 30.95; of mixed lengths, where
    // the shorter walks' steps crowd out those of the longer ones that
    // finish last, 8192 of N in 48..120 199 -> 216 and 4096 of N in 129..256
    // 492 -> 519.
    if (groups == 0 && a.ns == nullptr && end - begin >= ahead_from)
        return launch_wave_t<NWMAX, WPG, false, true>(a, begin, end, 0, counter, s);
    return launch_wave_t<NWMAX, WPG, false, false>(a, begin, end, groups, counter, s);
}

template <int GL, int NL, int WAVES, bool TRACE>
hipError_t launch_group_t(const TabuLaunchArgs &a, int64_t begin, int64_t end, int groups,
                          uint32_t *counter, hipStream_t s) {
    constexpr int G = 64 / GL;
    const int64_t need = (end - begin + G * WAVES - 1) / (G * WAVES);
    if (groups > 0) {
        hipError_t e = launch_fill_u32(counter, 0u, 1, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((tabu_kernel_group<GL, NL, WAVES, true, TRACE>),
                           dim3((unsigned)std::min<int64_t>(groups, need)), dim3(64 * WAVES), 0, s,
                           a, begin, end, counter);
    } else {
        return launch_in_ranges(begin, end, G * WAVES, 64 * WAVES,
                                [&](int64_t b, int64_t e, unsigned grid) {
            hipLaunchKernelGGL((tabu_kernel_group<GL, NL, WAVES, false, TRACE>), dim3(grid),
                               dim3(64 * WAVES), 0, s, a, b, e, counter);
        });
    }
    return hipGetLastError();
}

template <int GL, int NL, int WAVES>
hipError_t launch_group(const TabuLaunchArgs &a, int64_t begin, int64_t end, int groups,
                        uint32_t *counter, hipStream_t s) {
    if (end <= begin) return hipSuccess;
    if constexpr (WAVES > 2) {
        return hipErrorInvalidValue;  // several walks per wavefront: 64- or 128-lane workgroups
    } else {
        return a.trace != nullptr
                   ? launch_group_t<GL, NL, WAVES, true>(a, begin, end, groups, counter, s)
                   : launch_group_t<GL, NL, WAVES, false>(a, begin, end, groups, counter, s);
    }
}

template <int WAVES>
hipError_t launch_group2(const TabuLaunchArgs &a, int first, int64_t begin, int64_t end, int groups,
                         int64_t pairs_to, uint32_t *counter, hipStream_t s) {
    const GroupForm f = group2_form(first, end - begin, pairs_to);
    if (f.lanes == 32) return launch_group<32, 1, WAVES>(a, begin, end, groups, counter, s);
    if (f.neighbours == 1) return launch_group<16, 1, WAVES>(a, begin, end, groups, counter, s);
    return launch_group<16, 2, WAVES>(a, begin, end, groups, counter, s);
}

// One launch per launch group, group g on streams[g] with the queue head of
// its first class (32 words apart).
template <int WPG>
hipError_t launch_tabu_wpg(const TabuLaunchArgs &a, const WalkLaunch &l, const hipStream_t *st) {
    const int64_t *ce = a.class_end;
    const WalkGroups wg = tabu_launch_groups(ce, l.lanes);
    hipError_t e = hipSuccess;
    for (int g = 0; g < wg.n && e == hipSuccess; ++g) {
        const int f = wg.first[g], kind = wg.kind[g];
        const int64_t begin = f ? ce[f - 1] : 0, end = ce[wg.last[g]];
        uint32_t *q = a.counter + 32 * f;
        if (kind == kKindGroup2)
            e = launch_group2<WPG>(a, f, begin, end, l.groups, l.pairs_to, q, st[g]);
        else if (kind == kKindGroup4)
            e = launch_group<16, 1, WPG>(a, begin, end, l.groups, q, st[g]);
        else if (kClassMaxN[f] <= 64)
            e = launch_wave<1, WPG>(a, begin, end, l.groups, l.ahead_from, q, st[g]);
        else if (kClassMaxN[f] <= 128)
            e = launch_wave<2, WPG>(a, begin, end, l.groups, l.ahead_from, q, st[g]);
        else
            e = launch_wave<4, WPG>(a, begin, end, l.groups, l.ahead_from, q, st[g]);
    }
    return e;
}

}  // namespace

hipError_t launch_tabu(const TabuLaunchArgs &a, const WalkLaunch &l, const hipStream_t *streams) {
    if (a.W <= 0) return hipSuccess;
    // every launch range lies inside the processing order [0, W)
    int64_t prev = 0;
    for (int c = 0; c < kWalkClasses; ++c) {
        if (a.class_end[c] < prev || a.class_end[c] > a.W) return hipErrorInvalidValue;
        prev = a.class_end[c];
    }
    if (prev != a.W) return hipErrorInvalidValue;
    switch (l.waves_per_group) {
    case 1: return launch_tabu_wpg<1>(a, l, streams);
    case 2: return launch_tabu_wpg<2>(a, l, streams);
    case 4: return launch_tabu_wpg<4>(a, l, streams);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t grid = (count + 255) / 256;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)grid), dim3(256), 0, s, p, v, count);
    return hipGetLastError();
}

}  // namespace liblabs
