// Internal interface between the host runtime (gv_api.cpp) and the gfx950
// kernels (gv_kernels.hip).  Not part of the C boundary.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gv {

constexpr int kWave = 64;
constexpr int kBlock = 256;  // 4 waves per workgroup
// Row traffic policies (gv_config.coherence).
constexpr int kPlain = 0;        // cached loads and stores
constexpr int kAgent = 1;        // device-scope loads and stores
constexpr int kAtomicAgent = 2;  // device-scope loads, updates as device-scope fp32 atomic adds
constexpr int kMixed = 3;        // as kAtomicAgent for rows flagged warm, plain device-scope store otherwise

constexpr uint32_t kSmallestTile = 16, kLargestTile = 8192;  // samples per workgroup of the tiled kernel

// samples whose gathers a wave of the tiled kernel has in flight together (V floats of a row per lane, K negatives).
// Four of short rows fit the registers, but twice the workgroups with two each keep the same number in flight and wait
// less between a gather and its use (2.2*10^6 samples, d = 128, K = 1: 2.29 ms with four in tiles of 8192, 1.73 with two
// in tiles of 4096; 2^24: 9.80 and 9.67 ms in tiles of 8192).
__host__ __device__ constexpr bool short_rows(int V, int K) { return V * (K + 1) <= 4; }
__host__ __device__ constexpr int tiled_batch(int V, int K) { return V * (K + 1) <= 12 ? 2 : 1; }

// Deterministic mode, pools trained by k_train_flow: on the device.
struct FlowState {
    unsigned long long batches;  // levels of the parts before this one
    uint32_t deepest;            // levels of this part
    uint32_t next_chunk;         // the samples that the next wave takes
    uint32_t first_bad;          // the first sample of the pool that names an id that is no node; UINT32_MAX: none
    uint32_t stalled;            // set where a wave gave up (see k_train_flow)
    uint32_t started;            // workgroups that have begun
    uint32_t chained;            // times 64 namings of a hub are done
    unsigned long long slots[64];  // rows named often: namings << 32 | place of the first
};

// How long a wave of k_train_flow waits for a turn: until nothing of the pool has got on for 2^22 looks at the turns, half a
// second or more.  What has got on is read every 2^16 looks: samples taken (next_chunk) and namings of the hubs done (chained),
// of which one moves before 10^4 links of a chain are done one after the other, 50 ms at most.  The whole wait may be
// longer by any factor: waves run ahead of the hubs' samples, whose chain can be most of a part, 2^20 links of 0.5 us and more.
struct FlowPatience {
    static constexpr uint32_t kLooks = 1u << 16, kIdle = 64;
    uint32_t looks = 0, idle = 0, before = 0;
    // after a look in vain; progress(): what has got on so far
    template <class Progress>
    __host__ __device__ bool ends(Progress &&progress) {
        if (++looks % kLooks != 0u) return false;
        const uint32_t now = progress();
        idle = now == before ? idle + 1u : 0u;
        before = now;
        return idle >= kIdle;
    }
};

// Everything a training launch needs; passed by value as the kernel argument.
struct TrainArgs {
    float *vertex;            // |V| x d, row-major
    float *context;           // |V| x d, row-major
    const uint4 *alias;       // alias table: per bucket {threshold, alias node, hot rank of the bucket's node | hot rank
                              // of the alias << 16, the bucket's node}; the whole graph's table (bucket = node), or
                              // the table of one partition of the nodes (orthogonal blocks)
    uint32_t alias_n;         // buckets in that table
    const uint32_t *pairs;    // count x (u, v)
    const uint32_t *level_starts; // deterministic mode, narrow levels: first record of every level, levels + 1 entries
    uint32_t levels;          // deterministic mode: number of narrow levels, or 0: the records are one level
    const uint32_t *order;    // null, or per sample its index in the pool it was redistributed from: sample i then has
                              // global position first_g + order[i] (its negatives and learning rate) instead of
                              // first_g + i
    const uint16_t *rank;     // per node: its place among the nodes by falling degree (ties by id), 0xFFFF
                              // from place 65535 on ("hot rank")
    const uint32_t *ranked;   // bit i set: node i has a hot rank below 0xFFFF (small enough to stay in cache,
                              // so the rank table is only read for the few nodes that are in it); null when
                              // so many nodes are ranked that the detour does not pay
    uint32_t warm_ranks;      // rows of hot rank below this are warm: their updates must not be lost
                              // (see gv_build_alias)
    uint32_t exchange_every;  // tiled schedule: see AsyncPlan
    uint32_t *records;        // tiled schedule: scratch of count x (K + 3) words, written and read by the launch
                              // (u, v, the K negatives, warm flags of the negatives); deterministic mode: the
                              // samples of the launch in the order of their levels (u, v, the K negatives, place)
    uint32_t *error_flag;     // two words: [0] set to 1 when a sample names a node id >= n (sample skipped), [1] set
                              // to 1 when the tiled kernel meets a row that holds NaN (training has diverged)
    double *loss_slots;       // null, or kLossSlots sums: every wave adds the losses its samples saw before their
                              // steps to slot (workgroup number mod kLossSlots)
    uint64_t first_g;         // global position of pairs[0] (deterministic mode: of the sample of place 0)
    uint64_t total;           // T of the learning-rate schedule
    uint64_t seed;            // Philox key of the negative stream
    uint32_t count;           // samples in this launch
    uint32_t unit, blocks;    // asynchronous launches: see AsyncPlan
    uint32_t report_divergence; // pool order: nonzero: a score that is NaN sets error_flag[1]
    uint32_t n;               // |V|
    uint32_t dim;             // d: row length in floats
    float lr0, lr_min_ratio, neg_weight;
};

// k_train_flow takes these beside (see there, and launch_flow_prepare).  They are no part of TrainArgs, which every launch of
// asynchronous training carries by value.
struct FlowArgs : TrainArgs {
    FlowState *flow;
    const uint32_t *keys, *places, *sorted, *namings;
    uint64_t *turns;              // per row, vertex rows first: low word the place whose turn it is, high word levels so far
};

constexpr uint32_t kLossSlots = 64;

// Shape of an asynchronous launch.
struct AsyncPool {
    uint64_t count;           // samples
    uint32_t n, dim, num_neg;
    uint32_t coherence;
    bool tiled;               // the tiled schedule applies
    bool may_skip_tiles;      // ... and a pool that gains nothing from tiles may be walked in pool order (GV_SCHEDULE_AUTO)
    bool part_of_pool;        // one block of a partitioned graph
    uint32_t warm_ranks;
    double hottest_share;     // share of these samples that name the hottest context row
    uint32_t force_tile = 0;  // tests: the tile, under the policy asked for, whatever the rules say
};
struct AsyncPlan {
    bool tiled;               // k_train_tiled, otherwise k_train_hogwild
    uint32_t coherence;
    uint32_t unit;            // samples of a tile, or samples a wave takes at a time
    uint32_t blocks;          // workgroups
    uint32_t exchange_every;  // samples after which a held row trades its change with memory (tiles only)
};
AsyncPlan async_plan(const AsyncPool &pool);  // gv_plan.cpp

// The launches take their shape from a.unit, a.blocks and a.exchange_every; all return the HIP error of the launch.
hipError_t launch_train_hogwild(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                                hipStream_t stream);
// Tiled stationary-row training (see k_train_tiled).
hipError_t launch_train_tiled(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                              hipStream_t stream);
// Deterministic mode: a.count records of one level, or of a.levels consecutive narrow ones; the caller guarantees
// that no two samples of a level share a vertex row or a context row (negatives included).
hipError_t launch_train_levels(const TrainArgs &a, uint32_t dim, uint32_t num_neg, hipStream_t stream);
constexpr uint32_t kNarrowLevel = 48;  // samples: three rounds of the one workgroup (see k_train_levels)
// records[i] = sample order[i] of the pool, as launch_train_levels takes it.
hipError_t launch_level_records(const uint32_t *pairs, const uint32_t *negatives, const uint32_t *order, uint32_t count,
                                uint32_t num_neg, uint32_t *records, hipStream_t stream);
// Deterministic mode, a pool whose samples wait for each other on the device (see k_train_flow): the ids of the whole pool
// are checked (fresh: the state is cleared first), then each part of it is prepared (which sets a.keys, a.places and a.turns; scratch of
// flow_scratch_words(), turns of 2 n) and trained.  Part: a.pairs, a.count, a.first_g.
uint64_t flow_scratch_words(uint32_t count, uint32_t num_neg);
// The check also writes the rows that some samples name (as launch_flow_prepare does: u, n + v, n + every negative) to
// `named`, which may be host memory: eight runs of 512 samples at equal distances, the one at place t being sample
// flow_look(t, count); count >= kFlowRuns * kFlowRun, or the whole pool and places up to its length.
constexpr uint32_t kFlowRun = 512, kFlowRuns = 8;
__host__ __device__ inline uint32_t flow_looked_at(uint64_t count) {
    return count < kFlowRun * kFlowRuns ? (uint32_t)count : kFlowRun * kFlowRuns;
}
__host__ __device__ inline uint64_t flow_look(uint32_t t, uint64_t count) {
    return count < kFlowRun * kFlowRuns ? t : t / kFlowRun * (count / kFlowRuns) + t % kFlowRun;
}
hipError_t launch_flow_check(const TrainArgs &pool, uint64_t count, uint32_t num_neg, FlowState *state, bool fresh, uint32_t *named,
                             hipStream_t stream);
hipError_t launch_flow_prepare(FlowArgs &a, uint32_t num_neg, uint32_t *scratch, uint64_t *turns, hipStream_t stream);
hipError_t launch_train_flow(FlowArgs a, uint32_t dim, uint32_t num_neg, hipStream_t stream);
hipError_t launch_train_flow_tracked(FlowArgs a, uint32_t dim, uint32_t num_neg, hipStream_t stream);
// The same three launches with kernels that also sum the running loss into a.loss_slots (which must be set for
// these and null for the ones above).
hipError_t launch_train_hogwild_tracked(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                                        hipStream_t stream);
hipError_t launch_train_tiled_tracked(const TrainArgs &a, uint32_t dim, uint32_t num_neg, uint32_t coherence,
                                      hipStream_t stream);
hipError_t launch_train_levels_tracked(const TrainArgs &a, uint32_t dim, uint32_t num_neg, hipStream_t stream);
// out[i*K + k] = negative k of positive sample first_g + i.
hipError_t launch_draw_negatives(const uint4 *alias, uint32_t n, uint64_t seed, uint64_t first_g, uint64_t count,
                                 uint32_t num_neg, uint32_t *out, hipStream_t stream);
// The same with one alias table per partition of the nodes: sample i draws from the table of the partition of its
// context node v[i]; tables[] holds the tables one after the other, partition j owning buckets offsets[j] ..
// offsets[j + 1] - 1.
hipError_t launch_draw_negatives_partitioned(const uint4 *tables, const uint64_t *offsets, const uint8_t *part,
                                             const uint32_t *v, uint64_t seed, uint64_t first_g, uint64_t count,
                                             uint32_t num_neg, uint32_t *out, hipStream_t stream);
// vertex ~ U(-0.5/d, 0.5/d) from Philox stream 1 (context is cleared by the caller).
hipError_t launch_init_vertex(float *vertex, uint64_t rows, uint32_t dim, uint64_t seed, hipStream_t stream);

// Sum of the per-sample losses of a.pairs[0 .. a.count), samples a.first_g on (a.seed = evaluation seed), in *blocks partial
// sums (at most
// kEvalBlocks).
constexpr uint32_t kEvalBlocks = 2048;
hipError_t launch_eval_loss(TrainArgs a, uint32_t dim, uint32_t num_neg, double *partial, uint32_t *blocks, hipStream_t stream);
// waves: that come to work where there are pairs enough.
constexpr uint32_t kWavesOnHostPairs = 2048, kWavesOnDevicePairs = 8192;
hipError_t launch_cosine(const float *vertex, uint32_t n, uint32_t dim, const uint32_t *first, const uint32_t *second,
                         uint32_t count, uint32_t waves, float *out, uint32_t *error_flag, hipStream_t stream);

// The sum of twice[0 .. kRankBlocks) is 2 (pairs of a positive above a negative) + (pairs of equal score) of scores[0 ..
// num_pos) against the num_neg scores behind them, num_pos + num_neg <= 2^31; not_finite[0 .. kRankBlocks) holds a nonzero where
// a score is no number (cleared by the caller).  The negatives are sorted first, and overwritten.  scratch:
// rank_scratch_words(num_neg) words at a multiple of 16 bytes.
constexpr uint32_t kRankBlocks = 256;
uint64_t rank_scratch_words(uint32_t num_neg);
hipError_t launch_rank_sort(uint32_t *negatives, uint32_t num_neg, uint32_t *scratch, unsigned long long *not_finite, hipStream_t stream);
hipError_t launch_rank_sum(const uint32_t *scores, uint32_t num_pos, uint32_t num_neg, unsigned long long *twice,
                           unsigned long long *not_finite, hipStream_t stream);

// One pool of walk samples written on the device (see k_augment).
struct AugmentArgs {
    const uint64_t *offsets;  // CSR row starts, n + 1 entries
    const uint32_t *adj;      // neighbours, both directions of every edge (unless steps is given)
    const uint4 *steps;       // null, or per adjacency entry {neighbour, its degree, its first half-edge (64 bits)}
    const uint4 *weighted_steps; // null, or, of a weighted graph, the same for both outcomes of an entry's alias draw
    const uint32_t *guide;    // null, or owners of the half-edges j << guide_shift, see launch_departure_guide
    uint32_t guide_shift;
    const uint2 *node_table;  // weighted graph: alias table of the departure nodes {threshold, alias node}; else null
    const uint2 *nbr_table;   // weighted graph: per adjacency entry {threshold, alias entry of the same row}; else null
    uint2 *pairs;             // output, count x (u, v)
    uint64_t half_edges;      // offsets[n]
    uint64_t seed, first_walk, walks, count, per_walk;
    uint32_t n, length, window, pseudo_shuffle;
};
// steps[e] = {adj[e], degree and first half-edge of that node}.
hipError_t launch_pack_steps(const uint64_t *offsets, const uint32_t *adj, uint64_t half_edges, uint4 *steps, hipStream_t stream);
// steps[2e], steps[2e + 1]: see k_pack_weighted_steps; fewer than 2^32 half-edges.
hipError_t launch_pack_weighted_steps(const uint64_t *offsets, const uint32_t *adj, const uint2 *nbr_table, uint32_t n,
                                      uint4 *steps, hipStream_t stream);
// owners[j] = node that half-edge j << guide_shift(half_edges) belongs to, (half_edges >> shift) + 2 entries, at most
// kGuideEntries; the owner of half-edge e lies between owners[e >> shift] and owners[(e >> shift) + 1].
constexpr uint32_t kGuideEntries = 65536 + 2;
uint32_t guide_shift(uint64_t half_edges);
hipError_t launch_departure_guide(const uint64_t *offsets, uint32_t n, uint64_t half_edges, uint32_t *owners, hipStream_t stream);
// walk length at most 64
hipError_t launch_augment(const AugmentArgs &a, hipStream_t stream);

bool supported_shape(uint32_t dim, uint32_t num_neg);
int floats_per_lane(uint32_t dim);
// samples whose rows one wave of the tiled kernel gathers together (2, or 1 where rows are long)
uint32_t samples_per_batch(uint32_t dim, uint32_t num_neg);

}  // namespace gv
