// Memetic kernels of liblabs for gfx950 and their launchers.
//
//   memetic_init_kernel    random populations (Alg. 1, first two lines)
//   memetic_advance_kernel memetic generations (Alg. 1 / Alg. 3), several
//                          children of a replica in flight, population
//                          resident in LDS
//   memetic_step_kernel    the same one generation after another: launches of
//                          one generation, small populations
//   gather_best_kernel     best sequences and energies to caller buffers
#include <algorithm>

#include "labs_device.hpp"
#include "labs_internal.h"

namespace liblabs {

namespace {

constexpr int kMaxK = 128;


// ---------------------------------------------------------------------------
// Memetic replicas.
// ---------------------------------------------------------------------------
// Random populations, one workgroup per replica: member m = lane + 64 h
// (K <= 128) is the bits 128 q .. 128 q + 127 of the draws (pop, m, q, INIT);
// each of WAVES wavefronts makes the draws and takes every WAVES-th lag of
// every member's energy, a member per lane (init_waves).
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void memetic_init_kernel(MemeticLaunchArgs a) {
    __shared__ int part[WAVES][kMaxK];
    const int s = blockIdx.x;
    if (s >= a.n_slots) return;
    const MemeticSlot sl = a.slots[s];
    if (sl.state < 0) return;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int N = __builtin_amdgcn_readfirstlane(sl.n), K = a.K;
    const int64_t base = (int64_t)sl.state * K;
    const int words = (N + 31) >> 5;
    uint32_t wd[2][2 * kStateWords];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int q = 0; q < kStateWords / 2; ++q) {
            Draw4 d = {0u, 0u, 0u, 0u};
            if (128 * q < N && 64 * h < K)
                d = philox10(sl.pop_id, (uint32_t)(lane + 64 * h), (uint32_t)q, kTagInit, sl.k0,
                             sl.k1);
            const uint32_t dw[4] = {d.w0, d.w1, d.w2, d.w3};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int b = N - 32 * (4 * q + i);  // bits of the word inside the sequence
                wd[h][4 * q + i] = dw[i] & (b >= 32 ? ~0u : b <= 0 ? 0u : (1u << b) - 1u);
            }
        }
        part[wave][lane + 64 * h] =
            64 * h < K ? lane_energy<WAVES>(words, wd[h], N, N, wave) : 0;
    }
    __syncthreads();
    if (wave != 0) return;
    int e[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int m = lane + 64 * h;
        e[h] = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) e[h] += part[w][m];
        if (m < K) {
#pragma unroll
            for (int w = 0; w < kStateWords; ++w)
                a.st.pop[(base + m) * kStateWords + w] =
                    (uint64_t)wd[h][2 * w] | ((uint64_t)wd[h][2 * w + 1] << 32);
            a.st.popE[base + m] = e[h];
        } else {
            e[h] = INT_MAX;
        }
    }
    // bestSeq: the lowest-index member of minimum energy.
    const int mn = wave_min(min(e[0], e[1]));
    const uint64_t t0 = ballot(e[0] == mn), t1 = ballot(e[1] == mn);
    const int h = t0 ? 0 : 1;
    const int src = t0 ? __builtin_ctzll(t0) : __builtin_ctzll(t1);
#pragma unroll
    for (int w = 0; w < kStateWords; ++w) {
        const uint32_t lo = h == 0 ? wd[0][2 * w] : wd[1][2 * w];
        const uint32_t hi = h == 0 ? wd[0][2 * w + 1] : wd[1][2 * w + 1];
        a.st.best[(int64_t)sl.state * kStateWords + w] =  // uniform values, every lane
            ((uint64_t)readlane_u(hi, src) << 32) | readlane_u(lo, src);
    }
    a.st.bestE[sl.state] = mn;
    a.st.gen[sl.state] = 0;
    a.st.hit[sl.state] = -1;
}

// The draws of child b of generation g: (pop, g, 2b, GEN), (pop, g, 2b + 1,
// GEN), word 0 of (pop, walk generation, 0, LEN) and the mutation mask, bit i
// of which flips when word i % 4 of (pop, g, 64 b + i / 4, MUT) is below thr.
// Lanes 0, 1 and 2 take the first three counters and, for N <= 128, lane
// 32 + q mutation draw q, so one call of the generator serves them all;
// longer sequences take a second one.  Lanes 3 .. 2 + kLookback take the
// second GEN draw of the children 1 .. kLookback before this one, whose word
// 2 names the member that child replaces; `back` is how many generations
// before this child's that one is (0: the same).
constexpr int kLookback = 28;
template <int NW>
struct ChildDraws {
    Draw4 a, b;
    uint32_t len;
    typename MaskOf<NW>::type flips;
    uint32_t w2;  // per lane: word 2 of the lane's draw
    int back;     // per lane, lanes 3 .. 2 + kLookback
};
template <int NW>
__device__ __forceinline__ ChildDraws<NW> child_draws(const MemeticSlot &sl, uint32_t g,
                                                      uint32_t walk_gen, int b, int B,
                                                      uint32_t magic, int N, uint32_t thr) {
    static_assert(NW <= 2 || NW == 4, "N <= 128 or N <= 256");
    const int lane = lane_id();
    const bool mut = lane >= 32;
    const int dist = lane - 2;  // of an earlier child
    ChildDraws<NW> r;
    // ceil((dist - b) / B): t / B by a product, exact for t < 40 and B <= 8
    r.back = dist > 0 ? (int)(((uint32_t)(dist - b + B - 1) * magic) >> 16) : 0;
    const uint32_t slot = dist > 0 ? 2u * (uint32_t)(b - dist + r.back * B) + 1u
                                   : 2u * (uint32_t)b + (uint32_t)lane;
    const Draw4 d = philox10(sl.pop_id, mut ? g : lane == 2 ? walk_gen : g - (uint32_t)r.back,
                             mut ? 64u * (uint32_t)b + (uint32_t)(lane - 32) : lane == 2 ? 0u : slot,
                             mut ? kTagMut : lane == 2 ? kTagLen : kTagGen, sl.k0, sl.k1);
    r.a = {readlane_u(d.w0, 0), readlane_u(d.w1, 0), readlane_u(d.w2, 0), readlane_u(d.w3, 0)};
    r.b = {readlane_u(d.w0, 1), readlane_u(d.w1, 1), readlane_u(d.w2, 1), readlane_u(d.w3, 1)};
    r.len = readlane_u(d.w0, 2);
    r.w2 = d.w2;
    // bit q of word k: word k of mutation draw q is below thr
    uint64_t hit[4];
    if constexpr (NW <= 2) {
        hit[0] = ballot(d.w0 < thr) >> 32;
        hit[1] = ballot(d.w1 < thr) >> 32;
        hit[2] = ballot(d.w2 < thr) >> 32;
        hit[3] = ballot(d.w3 < thr) >> 32;
    } else {
        const Draw4 e = philox10(sl.pop_id, g, 64u * (uint32_t)b + (uint32_t)lane, kTagMut, sl.k0,
                                 sl.k1);
        hit[0] = ballot(e.w0 < thr);
        hit[1] = ballot(e.w1 < thr);
        hit[2] = ballot(e.w2 < thr);
        hit[3] = ballot(e.w3 < thr);
    }
    // lane i of word h: position i + 64 h, draw (i + 64 h) / 4, word i % 4
    const uint64_t mine = lane & 1 ? (lane & 2 ? hit[3] : hit[1]) : (lane & 2 ? hit[2] : hit[0]);
    uint64_t f[4] = {0ull, 0ull, 0ull, 0ull};
#pragma unroll
    for (int h = 0; h < NW; ++h)
        f[h] = ballot(lane + 64 * h < N && ((mine >> ((lane >> 2) + 16 * h)) & 1ull));
    r.flips = make_mask<NW>(f[0], f[1], f[2], f[3]);
    return r;
}

// The members a child draws, and the child before its walk: ref(m) looks a
// member up, energy(m, ref(m)) and member(m, ref(m)) read it.
struct Parents {
    bool comb;
    int m0, m1, m2, m3;
};
__device__ __forceinline__ Parents parents(const Draw4 &da, const Draw4 &db, uint32_t p_comb,
                                           int K) {
    return {da.w0 < p_comb, (int)below(da.w1, (uint32_t)K), (int)below(da.w2, (uint32_t)K),
            (int)below(da.w3, (uint32_t)K), (int)below(db.w0, (uint32_t)K)};
}
template <int NW, typename Ref, typename Energy, typename Member>
__device__ __forceinline__ typename MaskOf<NW>::type breed(const Parents &p,
                                                           const ChildDraws<NW> &cd, int N,
                                                           Ref ref, Energy energy, Member member) {
    using Mask = typename MaskOf<NW>::type;
    const int r0 = ref(p.m0);
    Mask child;
    if (p.comb) {
        // selectParents: two binary tournaments; Combine: one-point crossover
        const int r1 = ref(p.m1), r2 = ref(p.m2), r3 = ref(p.m3);
        const bool first = energy(p.m0, r0) <= energy(p.m1, r1);
        const bool third = energy(p.m2, r2) <= energy(p.m3, r3);
        const int cut = 1 + (int)below(cd.b.w1, (uint32_t)(N - 1));
        const Mask A = first ? member(p.m0, r0) : member(p.m1, r1);
        const Mask B = third ? member(p.m2, r2) : member(p.m3, r3);
        const Mask lowm = m_low(A, cut);
        child = m_or(m_and(A, lowm), m_and(B, m_not(lowm)));
    } else {
        child = member(p.m0, r0);
    }
    return m_xor(child, cd.flips);  // Mutate
}

// A child's walk of N <= 64 NW (NW = 4: N > 128) on one wavefront, with the
// fewest neighbours per lane that hold it.
template <int NW>
__device__ __forceinline__ WalkResult<NW> child_walk(int N, const typename MaskOf<NW>::type &child,
                                                     const MemeticLaunchArgs &a,
                                                     const MemeticSlot &sl, uint32_t gen,
                                                     uint32_t len, uint8_t *lds) {
    const Schedule sch = make_schedule(a.rule, N, len);
    if (NW == 4 && __builtin_amdgcn_readfirstlane(N) <= 192) {
        const auto r = tabu_walk<NW == 4 ? 3 : NW>(N, child, sch, a.rule.aspiration, sl.k0, sl.k1,
                                                   sl.pop_id, gen, lds, nullptr);
        return {r.best, r.best_e, r.final_e};
    }
    return tabu_walk<NW>(N, child, sch, a.rule.aspiration, sl.k0, sl.k1, sl.pop_id, gen, lds,
                         nullptr);
}

// One workgroup per replica, its children on the workgroup's wavefronts.
//
// The children of a replica (B = a.children per generation, numbered from the
// launch's first) take effect one after another, but a child needs nothing
// of an earlier one unless that one replaces a member it draws (of K, at most
// four drawn, one replaced), and the draws of both are known beforehand.  So
// wavefronts claim children in order, a child starts once the earlier
// children that replace its members are finished, takes such a member from
// the ring where finished children wait, and these are merged in order by
// whichever wavefront finishes next: with K = 100 eight wavefronts keep six
// children going, twelve eight.  The results are those of one child after
// another.
//
//   claimed   next child to start; a wavefront claims, walks, posts, claims
//   merged    children below it are in the population, in order
//   done[i]   child number + 1 once its result stands in ring slot i: a slot
//             is read only by the kLookback children after its own, and the
//             child that takes it next starts after these are merged
//   built[i]  child number + 1 once it has read the population: a generation
//             is merged only when all its B children have, since they are
//             made from the population before it
//   busy      held by the wavefront that merges; nobody waits for it, a
//             wavefront that leaves it looks again
//
// Every wait ends: a child waits only for earlier generations (their results
// and, kLookback children back, their merging; B <= 8 keeps its own
// generation's out of that), children are claimed in order, a claimed child
// that does not wait walks and is posted, and the last of a generation to be
// posted finds all of them built and merges them if nobody else does.
// Children past a reached target are dropped.
//
// A generation is one walk, a serial chain that leaves most of a SIMD idle:
// 64 generations of 256 replicas at N = 120 took 2452 us on one wavefront per
// replica, 37.5 us a generation, and take 460 to 480 us with twelve; 16
// generations of eight children 899 us with a barrier after each generation, 635
// here.
constexpr int kRing = 64;
static_assert(kRing >= 2 * (kLookback + 1) && 2 + kLookback < 32 && kMaxChildren <= kLookback,
              "a slot outlives its readers, its draws have a lane, no wait inside a generation");

template <int NW>
struct __attribute__((aligned(16))) ReplicaLds {
    uint64_t pop[kMaxK][NW];
    uint64_t res[kRing][NW];
    uint64_t best[NW];
    int popE[kMaxK];
    int resE[kRing], resSlot[kRing];
    uint32_t done[kRing], built[kRing];
    uint32_t claimed, merged, busy, stopped;
    int bestE;
    uint32_t total;  // children of this launch
    int64_t g0;      // generations done before it
};

// The launch's arguments and a slot, read again where they are used (scalar
// loads, cached) so that they take no registers during the walks: kept there,
// they spilled into the step loop.
typedef const __attribute__((address_space(4))) MemeticLaunchArgs ConstArgs;
typedef const __attribute__((address_space(4))) MemeticSlot ConstSlot;
__device__ __forceinline__ const MemeticLaunchArgs &fresh_args() {
    ConstArgs *p = (ConstArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const MemeticLaunchArgs *)p;
}
__device__ __forceinline__ const MemeticSlot &fresh_slot(const MemeticLaunchArgs &a) {
    ConstSlot *p = (ConstSlot *)(uintptr_t)(a.slots + blockIdx.x);
    return *(const MemeticSlot *)p;
}

// A replica's population and best between its state (index st) and LDS, and its
// progress.
template <int NW>
__device__ __forceinline__ void load_population(uint64_t (*pop)[NW], int *popE, uint64_t *best,
                                                const MemeticStateDev s, int st, int K) {
    const int64_t base = (int64_t)st * K;
    for (int i = (int)threadIdx.x; i < K; i += (int)blockDim.x) {
#pragma unroll
        for (int w = 0; w < NW; ++w) pop[i][w] = s.pop[(base + i) * kStateWords + w];
        popE[i] = s.popE[base + i];
    }
    if (threadIdx.x < NW) best[threadIdx.x] = s.best[(int64_t)st * kStateWords + threadIdx.x];
}
template <int NW>
__device__ __forceinline__ void store_population(const uint64_t (*pop)[NW], const int *popE,
                                                 const uint64_t *best, const MemeticStateDev s,
                                                 int st, int K) {
    const int64_t base = (int64_t)st * K;
    for (int i = (int)threadIdx.x; i < K; i += (int)blockDim.x) {
#pragma unroll
        for (int w = 0; w < NW; ++w) s.pop[(base + i) * kStateWords + w] = pop[i][w];
        s.popE[base + i] = popE[i];
    }
    if (threadIdx.x < NW) s.best[(int64_t)st * kStateWords + threadIdx.x] = best[threadIdx.x];
}
// One lane: `hit` as it was before the launch, `reached` if the replica's best
// has reached its target.
__device__ __forceinline__ void store_progress(const MemeticLaunchArgs &a, int st, int best_e,
                                               int64_t gen, int64_t hit, bool reached) {
    if (reached && hit < 0) hit = gen;
    a.st.bestE[st] = best_e;
    a.st.gen[st] = gen;
    a.st.hit[st] = hit;
    if (hit >= 0 && a.any_hit != nullptr) atomicOr(a.any_hit, 1u);
}

template <typename T>
__device__ __forceinline__ T lds_get(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_put(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t lds_get_u(const uint32_t *p) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_get(p));
}

// Child c is posted and, at the first of a generation, all B are built.
template <int NW>
__device__ __forceinline__ bool mergeable(const ReplicaLds<NW> &L, uint32_t c, uint32_t B) {
    if (lds_get_u(&L.done[c % kRing]) != c + 1u) return false;
    if (B == 1u || c % B != 0u) return true;
    const uint32_t i = c + min((uint32_t)lane_id(), B - 1u);
    return ballot(lds_get(&L.built[i % kRing]) == i + 1u) == ~0ull;
}

// Merges what is posted, in order, unless another wavefront is at it.
template <int NW>
__device__ __forceinline__ void merge_children(ReplicaLds<NW> &L, uint32_t B, bool targeted,
                                               int target) {
    for (;;) {
        uint32_t held = 1u;
        if (lane_id() == 0)
            held = __hip_atomic_exchange(&L.busy, 1u, __ATOMIC_SEQ_CST,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__builtin_amdgcn_readfirstlane((int)held) != 0) return;
        uint32_t c = lds_get_u(&L.merged);
        bool stop = lds_get_u(&L.stopped) != 0u;
        while (!stop && mergeable<NW>(L, c, B)) {
            const int r = (int)(c % kRing);
            const int slot = __builtin_amdgcn_readfirstlane(L.resSlot[r]);
            const int e = __builtin_amdgcn_readfirstlane(L.resE[r]);
            const auto m = load_mask<NW>(L.res[r]);
            store_mask<NW>(L.pop[slot], m);  // uniform values, every lane
            L.popE[slot] = e;
            int be = __builtin_amdgcn_readfirstlane(L.bestE);
            if (e < be) {
                be = e;
                store_mask<NW>(L.best, m);
                L.bestE = e;
            }
            ++c;
            if (targeted && be <= target && c % B == 0u) {
                stop = true;
                lds_put(&L.stopped, 1u);
            }
        }
        lds_put(&L.merged, c);
        lds_put(&L.busy, 0u);
        if (stop || !mergeable<NW>(L, c, B)) return;
    }
}

template <int NW>
__global__ __launch_bounds__(64 * kMaxMemeticWaves)
__attribute__((amdgpu_waves_per_eu(NW == 4 ? 5 : 7))) void memetic_advance_kernel(
    MemeticLaunchArgs args) {
    using Mask = typename MaskOf<NW>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn_lds[];
    ReplicaLds<NW> &L = *(ReplicaLds<NW> *)dyn_lds;
    if ((int)blockIdx.x >= args.n_slots) return;
    if (args.stop != nullptr && *args.stop != 0u) return;  // one value for the whole grid
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint8_t *lds = dyn_lds + sizeof(ReplicaLds<NW>) + wave * WalkLds<NW>::BYTES;
    {
        const MemeticLaunchArgs &a = fresh_args();
        const MemeticSlot &sl = fresh_slot(a);
        if (sl.state < 0 || (1 << memetic_class(sl.n)) != NW) return;
        const int st = sl.state;
        // every read is out before the first is waited for
        const int64_t g0 = a.st.gen[st], hit0 = a.st.hit[st];
        const int bestE0 = a.st.bestE[st];
        load_population<NW>(L.pop, L.popE, L.best, a.st, st, a.K);
        const int64_t left = min(sl.gen_limit - g0, (int64_t)a.gens);
        if (left <= 0) {
            if (threadIdx.x == 0 && hit0 >= 0 && a.any_hit != nullptr) atomicOr(a.any_hit, 1u);
            return;
        }
        for (int i = (int)threadIdx.x; i < kRing; i += (int)blockDim.x) L.done[i] = L.built[i] = 0u;
        if (threadIdx.x == 0) {
            L.claimed = L.merged = L.busy = 0u;
            L.stopped = sl.target >= 0 && bestE0 <= sl.target ? 1u : 0u;
            L.bestE = bestE0;
            L.total = (uint32_t)left * (uint32_t)a.children;
            L.g0 = g0;
        }
        __syncthreads();
    }

    for (;;) {
        const MemeticLaunchArgs &a = fresh_args();
        const MemeticSlot &sl = fresh_slot(a);
        const int N = sl.n, K = a.K, B = a.children;
        const uint32_t thr = a.mut_rule == 0 ? (uint32_t)(0x100000000ull / (uint64_t)N) : a.p_mut;
        const uint32_t magic = 65536u / (uint32_t)B + 1u;
        uint32_t idx = 0u;
        if (lane == 0)
            idx = __hip_atomic_fetch_add(&L.claimed, 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
        idx = (uint32_t)__builtin_amdgcn_readfirstlane((int)idx);
        if (idx >= lds_get_u(&L.total) || lds_get_u(&L.stopped) != 0u) break;
        const uint32_t gi = idx / (uint32_t)B;
        const int b = (int)(idx - gi * (uint32_t)B);
        const int64_t g = (int64_t)uniform64((uint64_t)L.g0) + (int64_t)gi;
        const uint32_t wgen = (uint32_t)(g * B + b);
        const ChildDraws<NW> cd = child_draws<NW>(sl, (uint32_t)g, wgen, b, B, magic, N, thr);
        const Parents pr = parents(cd.a, cd.b, a.p_comb, K);
        // wait for the earlier children that replace a member drawn here, and
        // for the merging of those out of reach
        const int rep = (int)below(cd.w2, (uint32_t)K);
        const int dist = lane - 2;
        const bool near = dist > 0 && dist <= kLookback && dist <= (int)idx && cd.back > 0;
        const bool clash =
            near && (rep == pr.m0 || (pr.comb && (rep == pr.m1 || rep == pr.m2 || rep == pr.m3)));
        const uint32_t from = idx - (uint32_t)dist;  // the lane's earlier child
        while (((int)lds_get_u(&L.merged) < (int)idx - kLookback ||
                ballot(clash && lds_get(&L.done[from % kRing]) != from + 1u) != 0ull) &&
               lds_get_u(&L.stopped) == 0u)
            __builtin_amdgcn_s_sleep(4);
        if (lds_get_u(&L.stopped) != 0u) break;
        // member m: the ring slot of its nearest replacement, or -1
        const auto replaced = [&](int m) {
            const uint64_t at = ballot(near && rep == m);
            return at ? (int)((idx + 2u - (uint32_t)__builtin_ctzll(at)) % kRing) : -1;
        };
        const Mask child = breed<NW>(
            pr, cd, N, replaced, [&](int m, int r) { return r < 0 ? L.popE[m] : L.resE[r]; },
            [&](int m, int r) { return load_mask<NW>(r < 0 ? L.pop[m] : L.res[r]); });
        const int replaces = (int)below(cd.b.w2, (uint32_t)K);
        if (B > 1) lds_put(&L.built[idx % kRing], idx + 1u);
        const WalkResult<NW> r = child_walk<NW>(N, child, a, sl, wgen, cd.len, lds);
        const MemeticLaunchArgs &a2 = fresh_args();
        const int target = fresh_slot(a2).target;
        const int slot = (int)(idx % kRing);
        store_mask<NW>(L.res[slot], r.best);  // uniform values, every lane
        L.resE[slot] = r.best_e;
        L.resSlot[slot] = replaces;
        lds_put(&L.done[slot], idx + 1u);
        merge_children<NW>(L, (uint32_t)a2.children, target >= 0, target);
    }
    __syncthreads();

    const MemeticLaunchArgs &a = fresh_args();
    const int st = fresh_slot(a).state;
    store_population<NW>(L.pop, L.popE, L.best, a.st, st, a.K);
    if (threadIdx.x == 0)
        store_progress(a, st, L.bestE, L.g0 + (int64_t)(L.merged / (uint32_t)a.children), a.st.hit[st],
                       L.stopped != 0u);
}

// A replica's generations one after another: its children (B = a.children) on
// the workgroup's wavefronts, each waited for before the next generation.  For
// launches of one generation (PLAIN, GRAPH, chunk = 1) and populations too
// small for children in flight, whose claims, ring and flags in LDS cost up to
// a microsecond a launch: 48 launches of one generation of 3-step walks at
// N = 12 on 16 replicas took 433 us with them and take 361 without; of four
// such children, 447 and 374.
constexpr int kMaxStepWaves = kMaxChildren;
template <int NW>
struct __attribute__((aligned(16))) StepLds {
    uint64_t pop[kMaxK][NW];
    uint64_t res[kMaxChildren][NW];
    uint64_t best[NW];
    int popE[kMaxK];
    int resE[kMaxChildren], resSlot[kMaxChildren];
};
template <int NW>
__global__ __launch_bounds__(64 * kMaxStepWaves)
__attribute__((amdgpu_waves_per_eu(NW == 4 ? 5 : 7))) void memetic_step_kernel(
    MemeticLaunchArgs args) {
    using Mask = typename MaskOf<NW>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn_lds[];
    StepLds<NW> &L = *(StepLds<NW> *)dyn_lds;
    if (args.stop != nullptr && *args.stop != 0u) return;  // one value for the whole grid
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint8_t *lds = dyn_lds + sizeof(StepLds<NW>) + wave * WalkLds<NW>::BYTES;
    // wave-uniform, and the same on every wavefront
    int64_t g, hit;
    uint32_t left;
    int be;
    {
        const MemeticLaunchArgs &a = fresh_args();
        const MemeticSlot &sl = fresh_slot(a);
        if (sl.state < 0 || (1 << memetic_class(sl.n)) != NW) return;
        // every read is out before the first is waited for
        const int64_t g0 = a.st.gen[sl.state], hit0 = a.st.hit[sl.state];
        const int bestE0 = a.st.bestE[sl.state];
        load_population<NW>(L.pop, L.popE, L.best, a.st, sl.state, a.K);
        g = (int64_t)uniform64((uint64_t)g0);
        hit = (int64_t)uniform64((uint64_t)hit0);
        be = __builtin_amdgcn_readfirstlane(bestE0);
        const int64_t n = min(sl.gen_limit - g, (int64_t)a.gens);
        if (n <= 0) {
            if (threadIdx.x == 0 && hit >= 0 && a.any_hit != nullptr) atomicOr(a.any_hit, 1u);
            return;
        }
        left = (uint32_t)n;
        __syncthreads();
    }
    bool reached;
    for (;; ++g, --left) {
        const int target = fresh_slot(fresh_args()).target;
        reached = target >= 0 && be <= target;
        if (reached || left == 0u) break;
        const int B = fresh_args().children;
        for (int b = wave; b < B; b += (int)(blockDim.x >> 6)) {
            const MemeticLaunchArgs &a = fresh_args();
            const MemeticSlot &sl = fresh_slot(a);
            const int N = sl.n, K = a.K;
            const uint32_t thr =
                a.mut_rule == 0 ? (uint32_t)(0x100000000ull / (uint64_t)N) : a.p_mut;
            const uint32_t wgen = (uint32_t)(g * B + b);
            const ChildDraws<NW> cd = child_draws<NW>(sl, (uint32_t)g, wgen, b, B,
                                                      65536u / (uint32_t)B + 1u, N, thr);
            const Mask child = breed<NW>(
                parents(cd.a, cd.b, a.p_comb, K), cd, N, [](int) { return 0; },
                [&](int m, int) { return L.popE[m]; },
                [&](int m, int) { return load_mask<NW>(L.pop[m]); });
            const int replaces = (int)below(cd.b.w2, (uint32_t)K);
            const WalkResult<NW> r = child_walk<NW>(N, child, a, sl, wgen, cd.len, lds);
            store_mask<NW>(L.res[b], r.best);  // uniform values, every lane
            L.resE[b] = r.best_e;
            L.resSlot[b] = replaces;
        }
        __syncthreads();
        for (int b = 0; b < B; ++b) {  // Alg. 1's merge, in order
            const int slot = __builtin_amdgcn_readfirstlane(L.resSlot[b]);
            const int e = __builtin_amdgcn_readfirstlane(L.resE[b]);
            const bool better = e < be;
            if (better) be = e;
            if (wave == 0) {
                const Mask m = load_mask<NW>(L.res[b]);
                store_mask<NW>(L.pop[slot], m);
                L.popE[slot] = e;
                if (better) store_mask<NW>(L.best, m);
            }
        }
        __syncthreads();
    }
    const MemeticLaunchArgs &a = fresh_args();
    const int st = fresh_slot(a).state;
    store_population<NW>(L.pop, L.popE, L.best, a.st, st, a.K);
    if (threadIdx.x == 0) store_progress(a, st, be, g, hit, reached);
}

// The stop latch of a chunk boundary (see launch_memetic_latch).
__global__ void memetic_latch_kernel(const uint32_t *any_hit, uint32_t *stop,
                                     const volatile uint32_t *cancel, uint32_t epoch,
                                     int stop_all) {
    const bool hit = stop_all != 0 && *any_hit != 0u;
    const bool cancelled = cancel != nullptr && *cancel != epoch;
    if (hit || cancelled) *stop = 1u;
}

__global__ void gather_best_kernel(MemeticStateDev st, const int32_t *__restrict__ state_idx,
                                   const int32_t *__restrict__ ns, int32_t n_uniform,
                                   int32_t count, int8_t *__restrict__ best_seq,
                                   int32_t out_stride, int32_t *__restrict__ best_e,
                                   int64_t *__restrict__ hit_gen,
                                   int64_t *__restrict__ gens_done) {
    const int i = blockIdx.x;
    if (i >= count) return;
    const int lane = lane_id();
    const int s = state_idx ? state_idx[i] : i;
    const int N = ns ? ns[i] : n_uniform;
    const M256 b = load_mask<4>(st.best + (int64_t)s * kStateWords);
    int8_t *out = best_seq + (int64_t)i * out_stride;
    for (int k = lane; k < out_stride; k += 64)
        out[k] = k < N ? (m_bit(b, k) ? (int8_t)-1 : (int8_t)1) : (int8_t)0;
    best_e[i] = st.bestE[s];  // uniform values, every lane
    if (hit_gen) hit_gen[i] = st.hit[s];
    if (gens_done) gens_done[i] = st.gen[s];
}

}  // namespace

hipError_t launch_memetic_init(const MemeticLaunchArgs &a, hipStream_t s) {
    if (a.n_slots <= 0) return hipSuccess;
    const dim3 grid((unsigned)a.n_slots);
    if (init_waves(a.n_slots, a.classes, a.cus) == 4)
        hipLaunchKernelGGL(memetic_init_kernel<4>, grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(memetic_init_kernel<1>, grid, dim3(64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_memetic_latch(const uint32_t *any_hit, uint32_t *stop,
                                const volatile uint32_t *cancel, uint32_t epoch, int stop_all,
                                hipStream_t s) {
    hipLaunchKernelGGL(memetic_latch_kernel, dim3(1), dim3(1), 0, s, any_hit, stop, cancel, epoch,
                       stop_all);
    return hipGetLastError();
}

namespace {

template <int NW>
hipError_t launch_memetic_nw(const MemeticLaunchArgs &a, hipStream_t s) {
    static_assert(sizeof(ReplicaLds<NW>) + kMaxMemeticWaves * WalkLds<NW>::BYTES <= 65536,
                  "dynamic LDS within the default limit");
    const int w = memetic_waves(NW, a.n_slots, a.K, a.children, a.gens, a.cus);
    if (w == 1 || a.gens == 1) {
        // one generation's children: at most kMaxChildren wavefronts
        static_assert(sizeof(StepLds<NW>) + kMaxStepWaves * WalkLds<NW>::BYTES <= 65536,
                      "dynamic LDS within the default limit");
        hipLaunchKernelGGL(memetic_step_kernel<NW>, dim3((unsigned)a.n_slots), dim3(64 * w),
                           sizeof(StepLds<NW>) + (size_t)w * WalkLds<NW>::BYTES, s, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(memetic_advance_kernel<NW>, dim3((unsigned)a.n_slots), dim3(64 * w),
                       sizeof(ReplicaLds<NW>) + (size_t)w * WalkLds<NW>::BYTES, s, a);
    return hipGetLastError();
}

// Kernels of one memetic length class c (mask words 1 << c) on stream s.
hipError_t launch_memetic_class(const MemeticLaunchArgs &a, int c, hipStream_t s) {
    return c == 0 ? launch_memetic_nw<1>(a, s)
                  : c == 1 ? launch_memetic_nw<2>(a, s) : launch_memetic_nw<4>(a, s);
}

}  // namespace

hipError_t launch_memetic_advance(const MemeticLaunchArgs &a, hipStream_t s,
                                  const SideStreams *sides) {
    if (a.n_slots <= 0) return hipSuccess;
    // the widest class present runs on s, each further one on a side stream
    int present[3], n = 0;
    for (int c = 2; c >= 0; --c)
        if (a.classes & (1 << c)) present[n++] = c;
    const int n_sides = sides != nullptr ? std::min(n - 1, kSideStreams) : 0;
    hipError_t e = hipSuccess;
    if (n_sides > 0) {
        e = hipEventRecord(sides->fork, s);
        for (int i = 0; i < n_sides && e == hipSuccess; ++i)
            e = hipStreamWaitEvent(sides->s[i], sides->fork, 0);
        if (e != hipSuccess) return e;
    }
    for (int i = 0; i < n && e == hipSuccess; ++i)
        e = launch_memetic_class(a, present[i], i > 0 && i <= n_sides ? sides->s[i - 1] : s);
    for (int i = 0; i < n_sides && e == hipSuccess; ++i) {
        e = hipEventRecord(sides->join[i], sides->s[i]);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, sides->join[i], 0);
    }
    return e;
}

hipError_t launch_gather_best(const MemeticStateDev &st, const int32_t *state_idx,
                              const int32_t *ns, int32_t n_uniform, int32_t count,
                              int8_t *best_seq, int32_t out_stride, int32_t *best_e,
                              int64_t *hit_gen, int64_t *gens_done, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_best_kernel, dim3((unsigned)count), dim3(64), 0, s, st, state_idx,
                       ns, n_uniform, count, best_seq, out_stride, best_e, hit_gen, gens_done);
    return hipGetLastError();
}

}  // namespace liblabs
