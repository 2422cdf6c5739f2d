// Internal interface between the C ABI (labs_api.cpp, labs_memetic.cpp,
// labs_server.cpp) and the kernels (labs_walk.hip, labs_memetic_kernels.hip,
// labs_brute.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/liblabs.h"

namespace liblabs {

struct RuleParams {
    int32_t steps_rule, steps_a, tenure_rule;
    int32_t lo_num, lo_den, lo_add, hi_num, hi_den, hi_add;
    int32_t aspiration;
    int32_t slo_num, slo_den, shi_num, shi_den;  // LABS_STEPS_RANGE bounds
};

// Length classes of stand-alone walks, longest first: runs of the processing
// order that one launch may cover.  The last two (N <= 32, N <= 16) are also
// the walks that fit a 32- or 16-lane group of a wavefront that runs several
// walks.
constexpr int kWalkClasses = 8;
constexpr int kClassMaxN[kWalkClasses] = {256, 193, 128, 97, 64, 49, 32, 16};
inline int walk_class(int n) {
    int c = 0;
    while (c + 1 < kWalkClasses && n <= kClassMaxN[c + 1]) ++c;
    return c;
}

struct TabuLaunchArgs {
    const int8_t *starts;     // [W][start_stride] or null
    int32_t start_stride;
    const int32_t *ns;        // device [W] or null
    int32_t n_uniform;
    const int32_t *order;     // device [W] walk ids in processing order, or null
    int64_t W;
    int64_t class_end[kWalkClasses];  // processing-order positions [class_end[c-1],
                                      // class_end[c]) hold the walks of class c
    uint32_t k0, k1;
    RuleParams rule;
    int8_t *best_seq;
    int32_t out_stride;
    int32_t *best_e;
    int32_t *final_e;
    int16_t *trace;
    int32_t trace_stride;
    uint32_t *counter;        // device, 32 words per class: persistent queue heads
};

// Streams besides the caller's one that a batch may fork onto.
constexpr int kSideStreams = kWalkClasses - 1;

// Kernel forms of a launch group.
enum WalkKind : int {
    kKindWave = 0,    // one walk per wavefront
    kKindSplit = 1,   // walks of 64 < N <= 128 apart from the shorter ones (no launch asks for it)
    kKindGroup2 = 2,  // walks of N <= 32, two or four per wavefront (group2_form)
    kKindGroup4 = 4,  // walks of N <= 16, four per wavefront (16 lanes, one neighbour each)
};

// Launch groups of a batch: runs of consecutive length classes (hence of
// consecutive positions of the processing order).  The classes of N > 128,
// when present, form one group and those of N <= 128 another -- or, with
// `split` (which no launch asks for), classes 2..3 (64 < N <= 128) and the
// shorter classes one each.
// With several walks per wavefront (`lanes` = 32 or 16 lanes per walk) the
// walks of N <= 32 leave the one-walk-per-wavefront group: with 32 lanes both
// short classes form one group; with 16, N <= 16 and 16 < N <= 32 one each.
struct WalkGroups {
    int n;
    int first[kWalkClasses], last[kWalkClasses], kind[kWalkClasses];
};
inline WalkGroups walk_launch_groups(const int64_t *class_end, bool split, int lanes = 64) {
    WalkGroups g;
    g.n = 0;
    auto present = [&](int c) { return class_end[c] > (c ? class_end[c - 1] : 0); };
    auto add = [&](int f, int z, int kind) {
        g.first[g.n] = f;
        g.last[g.n] = z;
        g.kind[g.n] = kind;
        ++g.n;
    };
    auto range = [&](int lo, int hi, int kind) {
        int f = -1, z = -1;
        for (int c = lo; c <= hi; ++c)
            if (present(c)) {
                if (f < 0) f = c;
                z = c;
            }
        if (f >= 0) add(f, z, kind);
    };
    const int short_end = lanes < 64 ? 5 : kWalkClasses - 1;
    range(0, 1, kKindWave);
    if (split) {
        if (present(2) || present(3)) add(2, 3, kKindSplit);
        range(4, short_end, kKindWave);
    } else {
        range(2, short_end, kKindWave);
    }
    if (lanes == 32) {
        range(6, 7, kKindGroup2);
    } else if (lanes == 16) {
        range(6, 6, kKindGroup2);
        range(7, 7, kKindGroup4);
    }
    return g;
}

// The launch groups of a walk batch: those above, with neighbouring
// one-walk-per-wavefront groups in one launch (one kernel takes every length:
// a walk's tables are 15 bytes per position, so the longest walk's scratch
// leaves room for all the wavefronts the registers do: six per SIMD, where a
// launch of N <= 64 alone has eight).
inline WalkGroups tabu_launch_groups(const int64_t *class_end, int lanes) {
    const WalkGroups all = walk_launch_groups(class_end, false, lanes);
    WalkGroups g;
    g.n = 0;
    for (int i = 0; i < all.n; ++i) {
        if (g.n > 0 && all.kind[i] == kKindWave && g.kind[g.n - 1] == kKindWave) {
            g.last[g.n - 1] = all.last[i];
            continue;
        }
        g.first[g.n] = all.first[i];
        g.last[g.n] = all.last[i];
        g.kind[g.n] = all.kind[i];
        ++g.n;
    }
    return g;
}

// Lanes per walk and neighbours per lane of the walks of a kKindGroup2 group
// that begins with length class `first` (one walk of N <= 32 on 16 or 32
// lanes).  N <= 16 alone fills 16 lanes.  Longer walks take 32 lanes up to
// `pairs_to` walks, where a step costs its chain of dependent instructions
// (which the second neighbour lengthens), and 16 lanes beyond, where it costs
// the instructions issued.  A call of W walks of N = 32 and 128 steps, 16
// lanes against 32 (MI355X, us): W = 64 64 and 53, 1024 66 and 56, 4096 67 and
// 61, 6144 74 and 70, 8192 75 and 80, 16384 100 and 118; as a persistent grid
// 1024 72 and 67, 2048 79 and 73, 3072 83 and 84, 8192 103 and 128.
struct GroupForm {
    int lanes, neighbours;
};
inline GroupForm group2_form(int first, int64_t walks, int64_t pairs_to) {
    if (kClassMaxN[first] <= 16) return {16, 1};
    if (walks <= pairs_to) return {32, 1};
    return {16, 2};
}

// How labs_tabu_batch launches its walks.
struct WalkLaunch {
    int waves_per_group;  // wavefronts per workgroup
    int lanes;            // walks of N <= 32: 64 (one per wavefront), 32 or 16 (walk_launch_groups)
    int groups;           // persistent grid (0: none)
    int64_t ahead_from;   // walks of two wavefronts per SIMD
    int64_t pairs_to;     // group2_form
};

// Words of a sequence mask in the memetic state (N <= 256).
constexpr int kStateWords = 4;

// Device layout of a memetic replica's state (structure of arrays).
struct MemeticStateDev {
    uint64_t *pop;    // [S][K][kStateWords] member masks (bit i: s_i = -1)
    int32_t *popE;    // [S][K]
    uint64_t *best;   // [S][kStateWords]
    int32_t *bestE;   // [S]
    int64_t *gen;     // [S] generations done
    int64_t *hit;     // [S] hit generation or -1
};

struct MemeticSlot {
    int32_t n;
    uint32_t pop_id;
    uint32_t k0, k1;
    int64_t gen_limit;
    int32_t target;
    int32_t state;    // index into MemeticStateDev arrays; < 0 means idle
};

constexpr int kMaxChildren = 8;  // children per generation (batched variant)

// Length classes of memetic replicas: mask words 1, 2 or 4.
__host__ __device__ inline int memetic_class(int n) { return n <= 64 ? 0 : n <= 128 ? 1 : 2; }

// Side streams a launch may fork onto (fork recorded on the caller's stream,
// side i joined back through join[i]).
struct SideStreams {
    hipStream_t s[kSideStreams];
    hipEvent_t join[kSideStreams];
    hipEvent_t fork;
};

// Wavefronts per replica of a launch, for `words` mask words (1 << memetic_class).
//
// What the device has to spare: twelve up to one replica per compute unit,
// eight up to eight replicas per compute unit (N <= 128) or two (N > 128,
// where a wavefront holds more of the LDS and registers), four beyond.  32
// generations of K = 100 (MI355X, us) on 1, 4, 8 and 12 wavefronts: N = 120
// 1352, 456, 318 and 294 at 256 replicas, 1390, 544, 426 and 424 at 512, 1615,
// 946 and 909 (8) at 2048, 3975, 2853 and 3002 (8) at 8192; N = 200 3075, 1017,
// 716 and 663 at 256, 3209, 1246, 956 and 1237 at 512, 3261, 1492 and 1602 (8)
// at 1024; N = 33 352, 131, 107 and 91 at 256, 887, 769 and 788 (8) at 8192.
//
// What the replica has children for, once two replicas per compute unit leave
// no slots over: those of one generation, and the more members the more of the
// next that wait for none of these.  Wavefronts beyond that hold slots other
// replicas could run in (and up to there draw ahead while they wait: K = 8 at 16
// replicas takes 390 us on 3 wavefronts and 361 on 12).  16 generations (us) on 1, 2, 3,
// 4 and 8 wavefronts, N = 64: K = 2 420, 395, 430, 560 and 817 at 2048
// replicas, 536, 622, 703, 831 and 1459 at 4096; K = 8 427, 339, 342, 403 and
// 559 at 2048, 557, 516, 542, 588 and 939 at 4096; K = 32 422, 303, 291, 309
// and 358 at 2048, 552, 468, 450, 445 and 575 at 4096.  4 generations of 4
// children, K = 2: 422, 297, 289, 272 and 338 at 2048.  N = 200: K = 6 1765,
// 1500, 1471, 1516 and 2472 at 1024 replicas, 2169, 1838, 2390, 2574 and 4523 at
// 2048.
// And no more than the launch has children.
constexpr int kMaxMemeticWaves = 12;
inline int memetic_waves(int words, int64_t replicas, int K, int children, int gens, int cus) {
    const int64_t per_cu = (replicas + cus - 1) / cus;
    const int device = per_cu <= 1 ? kMaxMemeticWaves : per_cu <= (words == 4 ? 2 : 8) ? 8 : 4;
    int useful = (per_cu <= (words == 4 ? 4 : 8) ? 2 : 1) + K / 8;
    if (children > 1) useful = children + K / 8;
    const int64_t all = (int64_t)gens * children;
    const int w = device < useful || per_cu <= 2 ? device : useful;
    return (int)(w < all ? w : all);
}

// Wavefronts per replica of the random populations: four share the lags of
// the members' energies, but each makes all the draws, so one does once the
// replicas fill the device, for N > 128 (where the lags weigh more) later.
// K = 100 (MI355X, a run of no generations, us), one and four: N = 12 38.9 and
// 38.5 at 256 replicas, 45.6 and 45.8 at 1024, 49.1 and 50.7 at 2048, 98.9 and
// 113.9 at 16384; N = 128 45.1 and 40.1, 52.4 and 50.5, 59.2 and 57.8, 158.8
// and 163.8; N = 256 58.2 and 43.9, 66.3 and 61.0, 80.8 and 78.3, 303.9 and
// 314.4, and 113.5 and 111.6 at 4096.
inline int init_waves(int64_t replicas, int classes, int cus) {
    return replicas <= (int64_t)((classes & 4) ? 16 : 4) * cus ? 4 : 1;
}

struct MemeticLaunchArgs {
    const MemeticSlot *slots;
    int32_t n_slots;
    int32_t K;
    uint32_t p_comb;
    int32_t mut_rule;
    uint32_t p_mut;
    RuleParams rule;
    int32_t gens;            // generations per launch
    int32_t classes;         // bit c set: some slot is of memetic_class c
    int32_t children;        // children per generation (1: Alg. 1)
    int32_t cus;             // compute units of the device
    MemeticStateDev st;
    uint32_t *any_hit;       // set to 1 when a replica reaches its target
    const uint32_t *stop;    // nonzero: the launch does nothing (null: never)
};

// Fixed device scratch of the allocation-free tabu batch: queue heads, then
// per-walk lengths and the processing order for at most kNoAllocMaxWalks
// walks of per-walk lengths (a batch of one length needs the heads only).
constexpr int64_t kNoAllocMaxWalks = LABS_NOALLOC_MAX_WALKS;
constexpr size_t kNoAllocHeadBytes = 1024;
constexpr size_t kNoAllocScratchBytes =
    kNoAllocHeadBytes + 2 * (size_t)kNoAllocMaxWalks * sizeof(int32_t);
static_assert(kNoAllocScratchBytes == LABS_NOALLOC_SCRATCH_BYTES, "scratch size as declared");
constexpr int kMaxDevices = 64;
// Device address of that scratch on `device`, which the caller has made
// current; looked up once per device (hipGetSymbolAddress) and kept.
hipError_t noalloc_scratch_address(int device, void **ptr);
// Longest-first processing order of W walks from their device lengths.
hipError_t launch_order_by_length(const int32_t *ns, int64_t W, int32_t *order, hipStream_t s);

hipError_t launch_energy(const int8_t *seqs, const int32_t *ns, int32_t n_uniform,
                         int32_t stride, int64_t count, int32_t *out, hipStream_t s);

// Exhaustive minimum over the 2^(n-1) codes with s_0 = +1.  `waves`
// wavefronts each write (min E, count, smallest code attaining it) to
// part_e/part_count/part_code; a second kernel reduces them into out_e,
// out_count (over all 2^n sequences) and out_code.
struct BruteParts {
    int32_t *part_e;
    int64_t *part_count;
    uint64_t *part_code;
    int32_t *out_e;
    int64_t *out_count;
    uint64_t *out_code;
};
int64_t brute_waves(int n);
hipError_t launch_bruteforce(int n, const BruteParts &p, hipStream_t s);
// The same by branch and bound, from kSearchMinN on (a call: n = 23 69 us by
// enumeration; n = 24 82 us, by search 72; n = 25 138 and 72): `walk_e` holds
// the energies that `walks` walks reached, whose least bounds the search from
// above; `queue` takes search_queue_bytes(), `bound` one word.
constexpr int kSearchMinN = 24;
int64_t search_waves();
size_t search_queue_bytes();
hipError_t launch_search(int n, const BruteParts &p, const int32_t *walk_e, int32_t walks,
                         uint32_t *queue, int32_t *bound, hipStream_t s);
// The same over the skew-symmetric sequences of odd length n (Sec. II.C):
// out_code receives the free-spin pattern (bit i set <=> s_i = -1, i <= c).
int64_t skew_brute_waves(int n);
hipError_t launch_skew_bruteforce(int n, const BruteParts &p, hipStream_t s);

// Launch group g (tabu_launch_groups(a.class_end, l.lanes)) runs on
// streams[g]; a.counter must point at 32 * kWalkClasses writable uint32 (the
// queue head of a group at 32 * its first class).
hipError_t launch_tabu(const TabuLaunchArgs &a, const WalkLaunch &l, const hipStream_t *streams);

hipError_t launch_memetic_init(const MemeticLaunchArgs &a, hipStream_t s);
// At a chunk boundary: *stop becomes (and stays) 1 when stop_all is set and
// *any_hit is, or when *cancel (host memory mapped for the device) no
// longer holds `epoch`.  One thread; capturable.
hipError_t launch_memetic_latch(const uint32_t *any_hit, uint32_t *stop,
                                const volatile uint32_t *cancel, uint32_t epoch, int stop_all,
                                hipStream_t s);
// Advances every slot by a.gens generations.  With several length classes
// present and `sides` given, the widest class runs on s and the others on
// side streams forked from and joined back into s, concurrently; the
// sequence of calls is capturable into a graph.
hipError_t launch_memetic_advance(const MemeticLaunchArgs &a, hipStream_t s,
                                  const SideStreams *sides = nullptr);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t count, hipStream_t s);
hipError_t launch_skew_deviation(const int8_t *seqs, const int32_t *ns, int32_t n_uniform,
                                 int32_t stride, int64_t count, int32_t *out, hipStream_t s);
hipError_t launch_gather_best(const MemeticStateDev &st, const int32_t *state_idx,
                              const int32_t *ns, int32_t n_uniform, int32_t count,
                              int8_t *best_seq, int32_t out_stride, int32_t *best_e,
                              int64_t *hit_gen, int64_t *gens_done, hipStream_t s);

}  // namespace liblabs
