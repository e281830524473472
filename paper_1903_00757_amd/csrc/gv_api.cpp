// Host runtime behind the C boundary declared in include/gvhot.h: context,
// alias-table builder, pinned double-buffered pool ring with asynchronous
// host-to-device copies, launch sequencing, levels of deterministic mode.
#include "gvhot.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <exception>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "gv_host.hpp"
#include "gv_internal.hpp"

namespace {

thread_local std::string g_create_error;

enum SlotState { kFree = 0, kFilling = 1, kQueued = 2, kTraining = 3 };

struct PoolSlot {
    uint32_t *host = nullptr;    // pinned, pool_capacity samples
    uint32_t *dev = nullptr;     // device twin
    hipEvent_t copied = nullptr; // host-to-device copy finished (copy stream)
    hipEvent_t trained = nullptr;// training launch that read `dev` finished (compute stream)
    uint64_t count = 0;
    SlotState state = kFree;
};

// Pairs that gv_link_prediction_auc ranks on the host: a sort of one or two thousand there is over before the launches of the
// device's sort are (a call of one pair against one 26 us, of 1000 against 1000 40, with the sort on the device 80; of 2048 against
// 2048 the host takes 155).
constexpr uint64_t kHostRanked = 4096;
constexpr uint64_t kStageWords = 16384, kDeterministicPart = 1u << 20;  // see train_deterministic
// Deterministic pools of more samples than this wait for each other on the device (train_flow) instead of being sorted into
// levels on the host: call and gv_sync, d = 128, K = 1, 10000 samples on 200000 nodes 116 instead of 144 us, 5000 on 5000 nodes 106
// instead of 133, 5000 on 200000 nodes 99 instead of 104, and fewer are levelled before the preparation's dozen launches are
// done.  Not where levels are narrow: a level of a few samples costs 0.8 to 1 us in one workgroup, a link of a chain 0.5 to 1.1, and
// 1.5 to 2.3 from wave to wave.  That is so where the graph's hottest row is named by more than one sample in 24, and in pools that put
// samples of a row close together whatever the graph, such as walks in their own order: those are known by the levels of the samples
// that launch_flow_check looks at (narrow_levels), fewer than 16 samples a level on average.  Both lines were drawn with links of
// 0.9 us (K = 1) to 1.8 (K = 5, d = 256); as things are, levels -> waiting on the device, ms, a pass alone:
// by the hottest row's share, 50000 pairs drawn by degree on 10^4 nodes: K = 1, d = 128: 2 % 2.95 -> 0.91, 4.2 % 3.87 -> 2.00, 8 % 4.74 ->
// 4.23, 12 % 5.93 -> 7.06; K = 5, d = 128: 4.2 % 8.5 -> 4.3, 8 % 10.3 -> 8.0, 12 % 12.3 -> 12.2, 20 % 16.2 -> 21.8; d = 256: 8 % 11.3 -> 9.7, 12 %
// 13.6 -> 14.4 (so the first line lies on the safe side, by a factor of two);
// by samples a level, 30000 pairs on graphs without hubs: K = 1, d = 128: 16.6 2.3 -> 4.3, 27 2.0 -> 2.6, 41 2.1 -> 1.7, 60 1.5 -> 1.2; K = 3:
// 18 3.6 -> 4.4, 27 3.3 -> 3.3; K = 5: 13.5 6.0 -> 8.0, 18 5.4 -> 5.8, 27 5.0 -> 4.0; d = 256: 18 5.6 -> 6.5, 27 5.3 -> 4.5;
// the same of 60000 samples of walks in their own order on graphs with hubs, with the longer links: K = 1: 3.6 12.6 -> 31.4, 8.9 6.7 ->
// 12.1, 15.5 5.1 -> 5.9, 17.4 4.9 -> 4.7, 30 4.3 -> 3.0; K = 5: 2.9 27 -> 60, 12 11.4 -> 10.3, 27 9.7 -> 4.8 (so where hubs make the levels the
// second line lies about right, and graphs of some hundred equal nodes lie on the wrong side of it up to 20 to 40 samples a level).
// The same samples in the producer's shuffled order have 40 to 200 a level.
constexpr uint64_t kFlowFrom = 4096;
constexpr double kFlowShare = 1.0 / 24.0;
constexpr uint32_t kFlowWidth = 16, kMostRows = 5 + 2;  // of a sample: num_neg <= 5

// The pairs of gv_eval_loss and gv_link_prediction_auc are read by the kernels from pinned memory, piece by piece, while the
// next piece is copied there: the host copies 77 GB/s and the kernels read 50, where a copy to the device from the caller's
// pageable arrays takes 78 us for 2 MB and 131 for 4 (25 to 58 for 64 KB to 128 KB), before the first kernel starts.  Evaluation
// loss of 2^18 samples 158 -> 138 us, of 10^4 34 -> 26, link prediction of two pairs 35 -> 26; of 10^4, with the shorter launches
// of its sort, 126 -> 79.  A piece has enough pairs to fill the chip; the fifth waits for the first.  The loss of more than 3*2^17
// samples takes pieces of 2^18, two of which fit: 2^20 samples, copied to the device / in pieces of 2^17 / of 2^18, us, d = 32, K = 1
// 365 / 420 / 338, d = 128, K = 1 491 / 466 / 428, d = 512, K = 5 2357 / 2330 / 2273; 300000 of them 186 / 161 / 178 at d = 128,
// for nothing runs beside the copy of the first piece.  (Copies of the pieces on the copy
// stream, waited for by the host, 180 us for 2^18 samples; workgroups of the kernel that copy for the others, 142 to 159.)
constexpr uint64_t kPiecePairs = 1u << 17;
constexpr int kPieces = 4;

// In pinned memory: what the host waits for at the end of a call, copied there on the compute stream, so that one wait for
// that stream is all (a blocking copy of a few bytes takes 20 us on top of it), and short pools of deterministic mode.
struct HostResults {
    uint32_t flag[4];                                             // three words used: see gv_ctx.error_flag
    uint32_t stage[kStageWords];                                  // deterministic mode
    gv::FlowState flow;                                           // deterministic mode, see train_flow
    double loss_slots[gv::kLossSlots];
    uint32_t pieces[kPieces * 2 * kPiecePairs];                   // gv_eval_loss, gv_link_prediction_auc: see kPiecePairs
    union {                                                       // written by the kernels
        double partial[kPieces][gv::kEvalBlocks];                 // gv_eval_loss
        unsigned long long sums[2 * gv::kRankBlocks];             // gv_link_prediction_auc
        float scores[kHostRanked];                                // gv_link_prediction_auc of few pairs
    };
};

struct TimedSpan {
    hipEvent_t start, stop;
    int kind;  // 0 training launch, 1 host-to-device copy
};

}  // namespace

// Scratch of the entry point that must not allocate (gv_train_device_pool_static): the per-sample records
// of the tiled kernel, in a device array that is part of the loaded code object.  Every GPU holds its own
// copy at its own address; the name below is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) uint32_t scratch[GV_STATIC_SCRATCH_WORDS];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
uint32_t *g_scratch_address[kMaxDevices];  // device address of `scratch` on each GPU, looked up once per GPU
}  // namespace

struct gv_ctx {
    gv_config cfg{};
    uint32_t n = 0;
    std::vector<uint32_t> degree;
    std::vector<double> wdegree;          // weighted graph: sum of the edge weights of every node (else empty)
    uint2 *dev_node_table = nullptr;      // weighted graph: alias table of the departure nodes {threshold, alias}
    uint2 *dev_nbr_table = nullptr;       // weighted graph: one alias table per adjacency row {threshold, alias in row}
    float *vertex = nullptr;
    float *context = nullptr;
    uint4 *alias = nullptr;
    bool alias_ready = false;
    uint16_t *dev_rank = nullptr;         // device, per node: hot rank (see gv::TrainArgs)
    uint32_t *dev_ranked = nullptr;       // device, bitmap of the nodes that have a hot rank
    uint32_t warm_ranks = 0;              // number of warm rows
    uint32_t force_tile = 0;              // see gv_test_force_tile
    double hottest_share = 0.0;           // share of the samples that name the hottest context row
    // orthogonal blocks (cfg.partitions > 0): partition of every node, and one alias table per partition
    std::vector<uint32_t> part;           // host, per node
    std::vector<uint64_t> part_offsets;   // host, partitions + 1: partition j owns table buckets [j] .. [j + 1] - 1
    std::vector<uint32_t> part_members, part_thresh, part_alias;  // host copies of the concatenated tables
    uint4 *dev_part_tables = nullptr;     // device, n buckets
    uint64_t *dev_part_offsets = nullptr; // device
    uint8_t *dev_part = nullptr;          // device, per node
    uint64_t *dev_offsets = nullptr;      // device CSR of the graph (gv_set_adjacency), for the device producer
    uint32_t *dev_adj = nullptr;
    uint4 *dev_steps = nullptr;           // the adjacency as the producer reads it (then dev_adj is null), see prepare_walks
    uint32_t *dev_guide = nullptr;        // where the producer's search for a departure starts
    uint64_t half_edges = 0;
    uint32_t *error_flag = nullptr;       // device: two words of training (see gv::TrainArgs), then one of evaluation
    HostResults *results = nullptr;       // pinned
    double *dev_loss = nullptr;           // device, cfg.track_loss: gv::kLossSlots running sums of the training loss
    uint32_t *negatives = nullptr;        // device scratch, deterministic mode / gv_draw_negatives
    uint64_t negatives_capacity = 0;      // in uint32 elements
    uint32_t *records = nullptr;          // device scratch of the tiled kernel: K + 3 words per sample of a launch
    uint64_t records_capacity = 0;        // in uint32 elements
    uint32_t *static_records = nullptr;   // this GPU's copy of the `scratch` array (GV_STATIC_SCRATCH_WORDS words)
    void *eval_scratch = nullptr;         // device scratch of gv_eval_loss / gv_cosine / gv_auc, grown on demand
    uint64_t eval_capacity = 0;           // in bytes
    hipEvent_t piece_read[kPieces] = {};  // the kernel that reads a piece of an evaluation's pairs has ended
    hipStream_t compute = nullptr;
    hipStream_t copy = nullptr;
    std::vector<PoolSlot> slot;           // ring of cfg.pool_slots pinned slots, each with a device twin
    std::vector<int> queue;               // FIFO of queued slot indices (front = oldest)
    int next_slot = 0;                    // slots are handed out in ring order
    uint64_t next_g = 0;
    gv_stats stats{};
    std::vector<TimedSpan> spans;         // recorded, not yet folded into stats
    std::vector<hipEvent_t> spare_events;
    uint64_t *flow_turns = nullptr;       // device, deterministic mode: see train_flow; 2 n words, then the state
    gv::FlowState *flow_state = nullptr;
    hipEvent_t flow_checked = nullptr;
    bool flow_pending = false;            // its state counts batches that are not in stats yet
    bool flow_fresh = false;              // its state is not cleared yet
    bool flow_stalled = false;            // a wave of it gave up: to be reported
    uint64_t flow_counted = 0;            // batches of the state that are
    std::unique_ptr<uint64_t[]> flow_rows;  // see narrow_levels
    uint32_t force_way = 0;               // see gv_test_force_way
    std::vector<uint32_t> level_vertex, level_context;  // deterministic mode: see train_deterministic
    uint32_t level_base = 0;
    std::string error;
};

namespace {

int fail(gv_ctx *ctx, int code, const char *fmt, ...) noexcept {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    try {
        if (ctx) ctx->error = buf; else g_create_error = buf;
    } catch (...) {  // no memory even for the text: the code alone is returned
    }
    return code;
}

// Every entry point runs its body through this: an exception of the C++ runtime (a container that
// cannot grow, a thread that cannot start) becomes an error code instead of crossing the C boundary.
template <class Body>
int guarded(gv_ctx *ctx, Body &&body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc &) {
        return fail(ctx, GV_ENOMEM, "out of host memory");
    } catch (const std::exception &e) {
        return fail(ctx, GV_EHIP, "host runtime error: %s", e.what());
    } catch (...) {
        return fail(ctx, GV_EHIP, "unknown host runtime error");
    }
}

#define GV_HIP(ctx, expr)                                                                          \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) {                                                                    \
            (void)hipGetLastError(); /* or the next launch would return it as its own */           \
            return fail(ctx, e_ == hipErrorOutOfMemory ? GV_ENOMEM : GV_EHIP, "%s: %s", #expr,     \
                        hipGetErrorString(e_));                                                    \
        }                                                                                          \
    } while (0)

int bind_device(gv_ctx *ctx) {
    GV_HIP(ctx, hipSetDevice(ctx->cfg.device));
    return GV_OK;
}

hipEvent_t take_event(gv_ctx *ctx) {
    if (!ctx->spare_events.empty()) {
        hipEvent_t e = ctx->spare_events.back();
        ctx->spare_events.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Fold finished event pairs into the statistics (called with the device idle).
void fold_spans(gv_ctx *ctx) {
    for (const TimedSpan &s : ctx->spans) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, s.start, s.stop) == hipSuccess) {
            if (s.kind == 0) {
                ctx->stats.train_kernel_ms += ms;
                ctx->stats.timed_launches += 1;
            } else {
                ctx->stats.h2d_ms += ms;
            }
        }
        ctx->spare_events.push_back(s.start);
        ctx->spare_events.push_back(s.stop);
    }
    ctx->spans.clear();
}

// The state of deterministic pools as copied to the host: batches go into the statistics, a wave that gave up is noted.
void fold_flow(gv_ctx *ctx) {
    const gv::FlowState &flow = ctx->results->flow;
    const uint64_t counted = flow.batches + flow.deepest;
    ctx->stats.batches += counted - ctx->flow_counted;
    ctx->flow_counted = counted;
    ctx->flow_pending = false;
    if (flow.stalled) {
        ctx->flow_stalled = true;
        ctx->flow_fresh = true;  // the next pool starts from a cleared state
        ctx->flow_counted = 0;
    }
}

// *evaluation_ids (may be null): set where the report is that the evaluation just queued names ids that are no nodes.
int sync_all(gv_ctx *ctx, bool *evaluation_ids = nullptr) {
    HostResults &r = *ctx->results;
    if (ctx->dev_loss)
        GV_HIP(ctx, hipMemcpyAsync(r.loss_slots, ctx->dev_loss, sizeof r.loss_slots, hipMemcpyDeviceToHost, ctx->compute));
    GV_HIP(ctx, hipMemcpyAsync(r.flag, ctx->error_flag, sizeof r.flag, hipMemcpyDeviceToHost, ctx->compute));
    if (ctx->flow_pending)
        GV_HIP(ctx, hipMemcpyAsync(&r.flow, ctx->flow_state, sizeof r.flow, hipMemcpyDeviceToHost, ctx->compute));
    GV_HIP(ctx, hipStreamSynchronize(ctx->copy));
    GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
    fold_spans(ctx);
    for (PoolSlot &s : ctx->slot)
        if (s.state == kTraining) s.state = kFree;
    if (ctx->dev_loss) {
        double total = 0.0;
        for (double x : r.loss_slots) total += x;
        ctx->stats.train_loss_sum = total;
    }
    if (ctx->flow_pending) fold_flow(ctx);
    const bool stalled = ctx->flow_stalled;
    const uint32_t flag[3] = {r.flag[0], r.flag[1], r.flag[2]};
    if (stalled || flag[0] || flag[1] || flag[2]) {  // the gravest is reported, and none of them again
        GV_HIP(ctx, hipMemset(ctx->error_flag, 0, sizeof r.flag));
        ctx->flow_stalled = false;
        if (stalled)
            return fail(ctx, GV_ESTATE, "a deterministic pool was not trained to its end: a sample waited for one that never came "
                        "(device memory overwritten?)");
        if (flag[0])
            return fail(ctx, GV_EINVAL, "a trained pool named a node id >= n (%u); those samples were skipped", ctx->n);
        if (flag[1])
            return fail(ctx, GV_ESTATE, "training has diverged: an embedding row holds NaN (asynchronous mode on a graph "
                        "where one node takes part in a large share of all samples? see GV_MODE_HOGWILD)");
        if (evaluation_ids) *evaluation_ids = true;
        return fail(ctx, GV_EINVAL, "a pair to evaluate names a node id >= n (%u)", ctx->n);
    }
    return GV_OK;
}

// The adjacency on the device, in whichever form it is there, and the walk tables of a weighted graph.
void free_adjacency(gv_ctx *ctx) {
    if (ctx->dev_offsets) (void)hipFree(ctx->dev_offsets);
    if (ctx->dev_adj) (void)hipFree(ctx->dev_adj);
    if (ctx->dev_steps) (void)hipFree(ctx->dev_steps);
    if (ctx->dev_guide) (void)hipFree(ctx->dev_guide);
    if (ctx->dev_node_table) (void)hipFree(ctx->dev_node_table);
    if (ctx->dev_nbr_table) (void)hipFree(ctx->dev_nbr_table);
    ctx->dev_offsets = nullptr;
    ctx->dev_adj = nullptr;
    ctx->dev_steps = nullptr;
    ctx->dev_guide = nullptr;
    ctx->dev_node_table = nullptr;
    ctx->dev_nbr_table = nullptr;
    ctx->half_edges = 0;
}

void free_matrices(gv_ctx *ctx) {
    if (ctx->flow_turns) (void)hipFree(ctx->flow_turns);
    ctx->flow_turns = nullptr;
    ctx->flow_state = nullptr;
    ctx->flow_pending = false;
    ctx->flow_counted = 0;
    if (ctx->vertex) (void)hipFree(ctx->vertex);
    if (ctx->context) (void)hipFree(ctx->context);
    if (ctx->alias) (void)hipFree(ctx->alias);
    if (ctx->dev_rank) (void)hipFree(ctx->dev_rank);
    if (ctx->dev_ranked) (void)hipFree(ctx->dev_ranked);
    ctx->dev_ranked = nullptr;
    free_adjacency(ctx);
    if (ctx->dev_part_tables) (void)hipFree(ctx->dev_part_tables);
    if (ctx->dev_part_offsets) (void)hipFree(ctx->dev_part_offsets);
    if (ctx->dev_part) (void)hipFree(ctx->dev_part);
    ctx->dev_part_tables = nullptr;
    ctx->dev_part_offsets = nullptr;
    ctx->dev_part = nullptr;
    ctx->vertex = ctx->context = nullptr;
    ctx->alias = nullptr;
    ctx->dev_rank = nullptr;
    ctx->alias_ready = false;
}

// Takes over the degrees of a new graph: allocates the matrices (cleared) and the per-node tables.
int adopt_degrees(gv_ctx *ctx, uint32_t n, std::vector<uint32_t> &&deg) {
    int rc = sync_all(ctx);
    if (rc != GV_OK && rc != GV_EINVAL && rc != GV_ESTATE) return rc;  // reports about pools already trained do not stop this call
    free_matrices(ctx);
    ctx->n = 0;
    const size_t bytes = (size_t)n * ctx->cfg.dim * sizeof(float);
    GV_HIP(ctx, hipMalloc((void **)&ctx->vertex, bytes));
    GV_HIP(ctx, hipMalloc((void **)&ctx->context, bytes));
    GV_HIP(ctx, hipMalloc((void **)&ctx->alias, (size_t)n * sizeof(uint4)));
    GV_HIP(ctx, hipMalloc((void **)&ctx->dev_rank, (size_t)n * sizeof(uint16_t)));  // filled by gv_build_alias
    GV_HIP(ctx, hipMalloc((void **)&ctx->dev_ranked, ((size_t)n + 31) / 32 * sizeof(uint32_t)));
    GV_HIP(ctx, hipMemsetAsync(ctx->vertex, 0, bytes, ctx->compute));
    GV_HIP(ctx, hipMemsetAsync(ctx->context, 0, bytes, ctx->compute));
    GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
    ctx->degree = std::move(deg);
    ctx->wdegree.clear();
    ctx->part.clear();
    ctx->n = n;
    ctx->level_vertex.clear();
    ctx->level_context.clear();
    return GV_OK;
}

// What the device producer reads, from the adjacency just uploaded: the guide of its departures, and the adjacency
// with degree and first half-edge of every neighbour beside it, 16 bytes an entry (32 on a weighted graph, for both
// outcomes of the alias draw), which leaves a walk one dependent load a step instead of two or three (k_pack_steps,
// k_pack_weighted_steps).  Not where that takes the walk out of an L2 cache (4 MiB a die) that holds the plain arrays
// (3.1*10^5 entries, pools of 10^7 pairs: 28 us plain, 36 us packed), and up to 4 GiB and an eighth of the memory that is
// left (the scratch of training comes later); larger adjacencies, and one that finds no memory for it, are walked as
// they are.
int prepare_walks(gv_ctx *ctx) {
    const bool weighted = ctx->dev_nbr_table != nullptr;
    const uint64_t bytes = ctx->half_edges * (weighted ? 2 : 1) * sizeof(uint4);
    // departures of a weighted graph come from its alias table; among 16 nodes the search is as short without a guide
    if (!weighted && ctx->n > 16) {
        if (hipMalloc((void **)&ctx->dev_guide, gv::kGuideEntries * sizeof(uint32_t)) != hipSuccess) {
            (void)hipGetLastError();  // not an error: the search starts from all nodes
            ctx->dev_guide = nullptr;
        } else {
            GV_HIP(ctx, gv::launch_departure_guide(ctx->dev_offsets, ctx->n, ctx->half_edges, ctx->dev_guide, ctx->compute));
        }
    }
    const uint64_t plain = ctx->half_edges * (sizeof(uint32_t) + (weighted ? sizeof(uint2) : 0)) + (uint64_t)ctx->n * sizeof(uint64_t);
    constexpr uint64_t kCached = 3ull << 20;
    size_t left = 0, total = 0;
    if (hipMemGetInfo(&left, &total) != hipSuccess) {
        (void)hipGetLastError();
        left = 0;
    }
    if (bytes <= 1ull << 32 && bytes <= left / 8 && (bytes <= kCached || plain > kCached)) {
        if (hipMalloc((void **)&ctx->dev_steps, bytes) != hipSuccess) {
            (void)hipGetLastError();  // not an error: the walk does without
            ctx->dev_steps = nullptr;
        } else if (weighted) {
            GV_HIP(ctx, gv::launch_pack_weighted_steps(ctx->dev_offsets, ctx->dev_adj, ctx->dev_nbr_table, ctx->n, ctx->dev_steps,
                                                       ctx->compute));
        } else {
            GV_HIP(ctx, gv::launch_pack_steps(ctx->dev_offsets, ctx->dev_adj, ctx->half_edges, ctx->dev_steps, ctx->compute));
        }
    }
    GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
    if (ctx->dev_steps) {
        (void)hipFree(ctx->dev_adj);
        if (weighted) (void)hipFree(ctx->dev_nbr_table);
        ctx->dev_adj = nullptr;
        ctx->dev_nbr_table = nullptr;
    }
    return GV_OK;
}

int need_graph(gv_ctx *ctx) {
    if (!ctx) return GV_EINVAL;
    if (ctx->n == 0) return fail(ctx, GV_ESTATE, "no graph: call gv_set_graph or gv_set_degrees first");
    return bind_device(ctx);
}

int need_trainable(gv_ctx *ctx) {
    int rc = need_graph(ctx);
    if (rc) return rc;
    if (!ctx->alias_ready) return fail(ctx, GV_ESTATE, "no alias table: call gv_build_alias first");
    return GV_OK;
}

int ensure_negatives(gv_ctx *ctx, uint64_t elements) {
    if (elements <= ctx->negatives_capacity) return GV_OK;
    if (ctx->negatives) {
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        (void)hipFree(ctx->negatives);
        ctx->negatives = nullptr;
        ctx->negatives_capacity = 0;
    }
    GV_HIP(ctx, hipMalloc((void **)&ctx->negatives, elements * sizeof(uint32_t)));
    ctx->negatives_capacity = elements;
    return GV_OK;
}

int ensure_records(gv_ctx *ctx, uint64_t elements) {
    if (elements <= ctx->records_capacity) return GV_OK;
    if (ctx->records) {
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        (void)hipFree(ctx->records);
        ctx->records = nullptr;
        ctx->records_capacity = 0;
    }
    GV_HIP(ctx, hipMalloc((void **)&ctx->records, elements * sizeof(uint32_t)));
    ctx->records_capacity = elements;
    return GV_OK;
}

gv::TrainArgs train_args(gv_ctx *ctx, const uint32_t *dev_pairs, uint64_t first_g, uint32_t count) {
    gv::TrainArgs a{};
    a.vertex = ctx->vertex;
    a.context = ctx->context;
    a.alias = ctx->alias;
    a.alias_n = ctx->n;
    a.pairs = dev_pairs;
    a.order = nullptr;
    a.rank = ctx->dev_rank;
    a.ranked = ctx->n > 20u * 0xFFFFu ? ctx->dev_ranked : nullptr;  // under 5 % of the nodes ranked
    a.warm_ranks = ctx->warm_ranks;
    a.error_flag = ctx->error_flag;
    a.loss_slots = ctx->dev_loss;
    a.first_g = first_g;
    a.total = ctx->cfg.total_samples;
    a.seed = ctx->cfg.seed;
    a.count = count;
    a.n = ctx->n;
    a.dim = ctx->cfg.dim;
    a.lr0 = ctx->cfg.lr0;
    a.lr_min_ratio = ctx->cfg.lr_min_ratio;
    a.neg_weight = ctx->cfg.neg_weight;
    return a;
}

int begin_span(gv_ctx *ctx, int kind, hipStream_t stream, TimedSpan *span) {
    span->kind = kind;
    span->start = take_event(ctx);
    span->stop = take_event(ctx);
    if (!span->start || !span->stop) return fail(ctx, GV_EHIP, "hipEventCreate failed");
    GV_HIP(ctx, hipEventRecord(span->start, stream));
    return GV_OK;
}

int end_span(gv_ctx *ctx, hipStream_t stream, const TimedSpan &span) {
    GV_HIP(ctx, hipEventRecord(span.stop, stream));
    ctx->spans.push_back(span);
    if (ctx->spans.size() >= 8192) {  // bound the number of live events: all of them must have completed
        GV_HIP(ctx, hipStreamSynchronize(ctx->copy));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        fold_spans(ctx);
    }
    return GV_OK;
}

// Asynchronous training of `count` samples at dev_pairs: one launch of the tiled
// stationary-row kernel, or of the plain pool-order kernel.
// `fixed_records`: null, or the static scratch of the entry point that must not allocate: then nothing is
// allocated on the way (no scratch growth, no events: the launch is not timed).
// `block`: null, or the part of a redistributed pool that one orthogonal block covers: its samples' pool indices
// and the context partition whose alias table its negatives come from.
struct BlockOfPool {
    const uint32_t *dev_order;
    uint32_t partition;
};
int train_hogwild(gv_ctx *ctx, const uint32_t *dev_pairs, uint64_t count, uint32_t *fixed_records = nullptr,
                  const BlockOfPool *block = nullptr) {
    // GV_SCHEDULE_AUTO: the tiled schedule exists for rows that many samples of a tile share.  A graph
    // without a single warm row has none, and there the sort, the records and the rank reads are pure
    // cost: such a graph is trained in pool order (with the mixed policy all of its rows are cold, i.e.
    // updated with device-scope stores).
    const bool wants_tiled = ctx->cfg.schedule == GV_SCHEDULE_TILED ||
                             (ctx->cfg.schedule == GV_SCHEDULE_AUTO && ctx->warm_ranks > 0);
    const bool tiled = wants_tiled && ctx->n <= 0x80000000u;
    uint32_t coherence = ctx->cfg.coherence;
    if (!tiled && ctx->cfg.schedule == GV_SCHEDULE_AUTO && coherence == GV_COHERENCE_MIXED && ctx->warm_ranks == 0)
        coherence = GV_COHERENCE_AGENT;
    const gv::AsyncPlan plan = gv::async_plan(gv::AsyncPool{count, ctx->n, ctx->cfg.dim, ctx->cfg.num_neg, coherence, tiled,
                                                            ctx->cfg.schedule == GV_SCHEDULE_AUTO, block != nullptr,
                                                            ctx->warm_ranks,
                                                            ctx->hottest_share * (block ? ctx->cfg.partitions : 1u),
                                                            ctx->force_tile});
    if (tiled && fixed_records) {
        const uint64_t words = count * (ctx->cfg.num_neg + 3);
        if (words > GV_STATIC_SCRATCH_WORDS)
            return fail(ctx, GV_EINVAL, "pool of %llu samples needs %llu words of scratch, the static scratch holds %llu "
                        "(at most %llu samples at K = %u)", (unsigned long long)count, (unsigned long long)words,
                        (unsigned long long)GV_STATIC_SCRATCH_WORDS,
                        (unsigned long long)(GV_STATIC_SCRATCH_WORDS / (ctx->cfg.num_neg + 3)), ctx->cfg.num_neg);
    } else if (plan.tiled) {  // before the timed span: an allocation must not count as kernel time
        int rc = ensure_records(ctx, count * (ctx->cfg.num_neg + 3));
        if (rc) return rc;
    }
    TimedSpan span{};
    const bool timed = ctx->cfg.profile != 0 && !fixed_records;
    if (timed) {
        int rc = begin_span(ctx, 0, ctx->compute, &span);
        if (rc) return rc;
    }
    gv::TrainArgs a = train_args(ctx, dev_pairs, ctx->next_g, (uint32_t)count);
    if (block) {
        a.order = block->dev_order;
        a.alias = ctx->dev_part_tables + ctx->part_offsets[block->partition];
        a.alias_n = (uint32_t)(ctx->part_offsets[block->partition + 1] - ctx->part_offsets[block->partition]);
    }
    a.unit = plan.unit;
    a.blocks = plan.blocks;
    a.exchange_every = plan.exchange_every;
    a.report_divergence = tiled ? 1u : 0u;
    if (plan.tiled) {
        a.records = fixed_records ? fixed_records : ctx->records;
        GV_HIP(ctx, (a.loss_slots ? gv::launch_train_tiled_tracked : gv::launch_train_tiled)(
                        a, ctx->cfg.dim, ctx->cfg.num_neg, plan.coherence, ctx->compute));
    } else {
        GV_HIP(ctx, (a.loss_slots ? gv::launch_train_hogwild_tracked : gv::launch_train_hogwild)(
                        a, ctx->cfg.dim, ctx->cfg.num_neg, plan.coherence, ctx->compute));
    }
    ctx->stats.train_launches += 1;
    ctx->stats.tiled_launches += plan.tiled ? 1 : 0;
    if (ctx->dev_loss) ctx->stats.train_loss_samples += count;
    if (timed) return end_span(ctx, ctx->compute, span);
    return GV_OK;
}

// The kernels of an evaluation, and the check of a deterministic pool, use pinned memory of the context that the next call
// writes: whatever ends a call early, they have ended when it returns.
struct PinnedInUse {
    gv_ctx *ctx;
    bool ended = false;  // waited for already
    ~PinnedInUse() {
        if (ended) return;
        (void)hipStreamSynchronize(ctx->copy);
        (void)hipStreamSynchronize(ctx->compute);
    }
};

// What train_flow needs on the device beside the pool: 6 words for every row that a sample of a part names, and 4 words a
// node.  GV_ENOMEM where that does not fit (or the nodes' would take more than an eighth of the memory that is left): then
// nothing is held for it, and the scratch of levels stays, for every pool asks anew.
int ensure_flow(gv_ctx *ctx, uint64_t count) {
    const uint64_t words = gv::flow_scratch_words((uint32_t)std::min(count, kDeterministicPart), ctx->cfg.num_neg);
    if (ctx->flow_turns && words <= ctx->records_capacity) return GV_OK;
    size_t left = 0, total = 0;
    GV_HIP(ctx, hipMemGetInfo(&left, &total));
    const size_t bytes = (size_t)ctx->n * 2 * sizeof(uint64_t);
    if (!ctx->flow_turns && bytes > left / 8) return GV_ENOMEM;
    if (words > ctx->records_capacity) {
        if ((words - ctx->records_capacity) * sizeof(uint32_t) > left) return GV_ENOMEM;
        if (words * sizeof(uint32_t) > left) {  // in the place of the old scratch only
            int rc = ensure_records(ctx, words);
            if (rc) return rc;
        } else {
            uint32_t *records = nullptr;
            GV_HIP(ctx, hipMalloc((void **)&records, words * sizeof(uint32_t)));
            std::swap(records, ctx->records);
            ctx->records_capacity = words;
            if (records) {
                const hipError_t e = hipStreamSynchronize(ctx->compute);
                (void)hipFree(records);
                GV_HIP(ctx, e);
            }
        }
    }
    if (!ctx->flow_turns) {
        if (!ctx->flow_checked) GV_HIP(ctx, hipEventCreateWithFlags(&ctx->flow_checked, hipEventDisableTiming));
        uint64_t *turns = nullptr;
        GV_HIP(ctx, hipMalloc((void **)&turns, bytes + sizeof(gv::FlowState)));
        ctx->flow_turns = turns;
        ctx->flow_state = (gv::FlowState *)((char *)turns + bytes);
        ctx->flow_fresh = true;
    }
    return GV_OK;
}

// The levels (see train_deterministic) of the first `per_run` samples of every run, one run after the other, counted as far as
// `enough`; named[kFlowRuns][kFlowRun][num_neg + 2].  The rows met so far stand in a table of `slots` entries, row + 1 << 32 |
// level, a power of two and, with fewer rows, twice their number.
uint32_t levels_of(const uint32_t *named, uint32_t per_run, uint32_t num_neg, uint32_t enough, uint64_t *table, uint32_t slots) {
    const uint32_t rows = num_neg + 2;
    const int shift = 32 - __builtin_ctz(slots);
    memset(table, 0, slots * sizeof *table);
    uint32_t deepest = 0;
    for (uint32_t r = 0; r < gv::kFlowRuns; ++r) {
        for (uint32_t i = 0; i < per_run && deepest < enough; ++i) {
            const uint32_t *const row = named + ((size_t)r * gv::kFlowRun + i) * rows;
            uint64_t *entry[kMostRows];
            uint32_t level = 0;
            for (uint32_t j = 0; j < rows; ++j) {
                const uint64_t key = (uint64_t)row[j] + 1u << 32;  // the rows are less than 2^32 - 1
                uint32_t slot = (row[j] * 0x9E3779B1u) >> shift;
                while (table[slot] != 0 && (table[slot] ^ key) >> 32 != 0) slot = (slot + 1u) & (slots - 1u);
                if (table[slot] == 0) table[slot] = key;
                entry[j] = table + slot;
                level = std::max(level, (uint32_t)table[slot]);
            }
            ++level;
            for (uint32_t j = 0; j < rows; ++j) *entry[j] = (*entry[j] >> 32 << 32) | level;
            deepest = std::max(deepest, level);
        }
    }
    return deepest;
}

// Whether the samples that launch_flow_check looked at have levels of fewer than kFlowWidth samples on average.  For most pools
// an eighth of those samples tells, the heads of the runs (5 us of the host at K = 1, 25 at K = 5, while the device prepares the
// pool; all of them take 100 and 200).  Of walks in their own order, where a sample often names the vertex of the one before,
// the heads have to do half as well again: (i, j) comes after (i, j - 1) and (i - 1, j), and such chains are longer than a head.
bool narrow_levels(gv_ctx *ctx, const uint32_t *named, uint32_t num_neg) {
    constexpr uint32_t kSlots = 1u << 16, kFew = gv::kFlowRun / 8;
    static_assert(2 * gv::kFlowRuns * gv::kFlowRun * kMostRows < kSlots, "room");
    if (!ctx->flow_rows) ctx->flow_rows.reset(new (std::nothrow) uint64_t[kSlots]);
    if (!ctx->flow_rows) return false;  // the results are the same either way
    uint32_t same = 0;  // samples of the heads that name the vertex of the sample before
    for (uint32_t r = 0; r < gv::kFlowRuns; ++r)
        for (uint32_t i = 1; i < kFew; ++i) {
            const uint32_t *const row = named + ((size_t)r * gv::kFlowRun + i) * (num_neg + 2);
            same += row[0] == *(row - (num_neg + 2));
        }
    const uint32_t wide = gv::kFlowRuns * kFew / kFlowWidth, few_levels = (same * 4 > gv::kFlowRuns * kFew ? wide * 2 / 3 : wide) + 1;
    if (levels_of(named, kFew, num_neg, few_levels, ctx->flow_rows.get(), kSlots / 8) < few_levels) return false;
    constexpr uint32_t kLevels = gv::kFlowRuns * gv::kFlowRun / kFlowWidth + 1;
    return levels_of(named, gv::kFlowRun, num_neg, kLevels, ctx->flow_rows.get(), kSlots) == kLevels;
}

// Deterministic training of a pool that is not short: every sample waits on the device for the earlier samples that name
// one of its rows (k_train_flow).  The namings of the rows are sorted there, and the host waits only for the check of the
// ids.  *narrow: set, and nothing trained, where the levels are narrow (see kFlowFrom).
int train_flow(gv_ctx *ctx, const uint32_t *dev_pairs, uint64_t count, bool *narrow) {
    const uint32_t K = ctx->cfg.num_neg;
    const uint64_t part = std::min(count, kDeterministicPart);
    int rc = GV_OK;
    PinnedInUse in_use{ctx};
    uint32_t *const named = ctx->results->pieces;  // no evaluation runs meanwhile
    static_assert(sizeof ctx->results->pieces >= gv::kFlowRuns * gv::kFlowRun * kMostRows * sizeof(uint32_t), "room");
    GV_HIP(ctx, gv::launch_flow_check(train_args(ctx, dev_pairs, ctx->next_g, 0), count, K, ctx->flow_state, ctx->flow_fresh, named,
                                      ctx->compute));
    ctx->flow_fresh = false;
    gv::FlowState &flow = ctx->results->flow;
    GV_HIP(ctx, hipMemcpyAsync(&flow, ctx->flow_state, sizeof flow, hipMemcpyDeviceToHost, ctx->compute));
    GV_HIP(ctx, hipEventRecord(ctx->flow_checked, ctx->compute));
    for (uint64_t first = 0; first < count; first += part) {
        const uint64_t here = std::min(part, count - first);
        gv::FlowArgs a{};
        (gv::TrainArgs &)a = train_args(ctx, dev_pairs + 2 * first, ctx->next_g + first, (uint32_t)here);
        a.flow = ctx->flow_state;
        GV_HIP(ctx, gv::launch_flow_prepare(a, K, ctx->records, ctx->flow_turns, ctx->compute));
        if (first == 0) {  // the whole pool is looked at before any of it is trained
            GV_HIP(ctx, hipEventSynchronize(ctx->flow_checked));
            in_use.ended = true;
            if (flow.first_bad != UINT32_MAX)
                return fail(ctx, GV_EINVAL, "sample %llu names node id >= n (%u)", (unsigned long long)flow.first_bad, ctx->n);
            *narrow = !ctx->force_way && narrow_levels(ctx, named, K);
            if (*narrow) return GV_OK;
        }
        TimedSpan span{};
        const bool timed = ctx->cfg.profile != 0;
        if (timed) {
            rc = begin_span(ctx, 0, ctx->compute, &span);
            if (rc) return rc;
        }
        GV_HIP(ctx, (ctx->dev_loss ? gv::launch_train_flow_tracked : gv::launch_train_flow)(a, ctx->cfg.dim, K, ctx->compute));
        ctx->flow_pending = true;
        ctx->stats.train_launches += 1;
        if (ctx->dev_loss) ctx->stats.train_loss_samples += here;
        if (timed) {
            rc = end_span(ctx, ctx->compute, span);
            if (rc) return rc;
        }
    }
    return GV_OK;
}

// Deterministic training: draw the pool's negatives on the device, bring them and the pairs to the host, and sort
// the samples into levels: a sample's level is one more than the highest level of the earlier samples that name
// one of its rows (vertex[u], context[v] or a negative's).  Samples of one level commute exactly (Def. 1, Sec. 3.2) and
// samples that share a row stay in pool order, so training level after level gives the sequential result up to fp32
// rounding inside a sample.  The number of levels is close to the number of samples that name the hottest row, however
// far apart they stand in the pool: 1051 for 2*10^5 samples on 10^4 nodes, where maximal runs of consecutive samples
// without a shared row number 32046 (6 samples each, one launch each: 112 ms; levels: 5 ms).
//
// A pool is taken in parts of at most kDeterministicPart samples, one after the other, which bounds what the host and the
// device hold of it beside the pairs.  Pools whose arrays fit the pinned stage use that: copies to and from pageable
// memory wait for each other (30 samples, K = 1: 56 us a call from pageable arrays, 28 staged).
int train_deterministic(gv_ctx *ctx, const uint32_t *dev_pairs, const uint32_t *host_pairs, uint64_t count) {
    const uint32_t K = ctx->cfg.num_neg;
    const uint64_t part = std::min(count, kDeterministicPart);
    // device scratch: the draws, then the order of the samples and the starts of the levels (at most one per sample)
    int rc = ensure_negatives(ctx, part * K + 2 * part + 1);
    if (rc) return rc;
    rc = ensure_records(ctx, part * (K + 3));
    if (rc) return rc;
    uint32_t *const dev_order = ctx->negatives + part * K, *const dev_starts = dev_order + part;
    // the same on the host, the level of every sample, and the pairs if they are on the device only
    const uint64_t words = part * K + 3 * part + 1 + (host_pairs ? 0 : 2 * count);
    const bool staged = words <= kStageWords;
    std::unique_ptr<uint32_t[]> arrays(staged ? nullptr : new uint32_t[words]);
    uint32_t *const neg = staged ? ctx->results->stage : arrays.get(), *const order = neg + part * K, *const starts = order + part,
                    *const level = starts + part + 1, *const pairs_copy = level + part;
    // Whatever ends the call early leaves rows with levels of samples that were not trained, and copies in flight to the
    // arrays above: the next call starts from cleared rows, and the arrays outlive the copies.
    struct Levelling {
        gv_ctx *ctx;
        bool complete;
        ~Levelling() {
            if (complete) return;
            (void)hipStreamSynchronize(ctx->compute);
            ctx->level_vertex.clear();
            ctx->level_context.clear();
        }
    } levelling{ctx, false};
    // level_vertex / level_context: per row, ctx->level_base + the lowest level that the next sample naming it may
    // have; an entry of an earlier part is at most level_base
    if (ctx->level_vertex.size() != ctx->n || ctx->level_context.size() != ctx->n) {
        ctx->level_vertex.assign(ctx->n, 0);
        ctx->level_context.assign(ctx->n, 0);
        ctx->level_base = 0;
    }
    uint32_t *const row_u = ctx->level_vertex.data(), *const row_c = ctx->level_context.data();
    const uint32_t *const pairs = host_pairs ? host_pairs : pairs_copy;
    const auto launch = ctx->dev_loss ? gv::launch_train_levels_tracked : gv::launch_train_levels;

    for (uint64_t first = 0; first < count; first += part) {
        const uint64_t here = std::min(part, count - first);
        const uint32_t *const part_pairs = dev_pairs + 2 * first;
        GV_HIP(ctx, gv::launch_draw_negatives(ctx->alias, ctx->n, ctx->cfg.seed, ctx->next_g + first, here, K, ctx->negatives,
                                              ctx->compute));
        if (first == 0 && !host_pairs)
            GV_HIP(ctx, hipMemcpyAsync(pairs_copy, dev_pairs, count * 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->compute));
        GV_HIP(ctx, hipMemcpyAsync(neg, ctx->negatives, here * K * sizeof(uint32_t), hipMemcpyDeviceToHost, ctx->compute));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        if (first == 0) {  // the whole pool is looked at before any of it is trained
            uint32_t largest = 0;
            for (uint64_t i = 0; i < 2 * count; ++i) largest = std::max(largest, pairs[i]);
            if (largest >= ctx->n) {
                uint64_t i = 0;
                while (pairs[i] < ctx->n) ++i;
                return fail(ctx, GV_EINVAL, "sample %llu names node id >= n (%u)", (unsigned long long)(i / 2), ctx->n);
            }
        }
        if (ctx->level_base > UINT32_MAX - here) {
            std::fill(ctx->level_vertex.begin(), ctx->level_vertex.end(), 0u);
            std::fill(ctx->level_context.begin(), ctx->level_context.end(), 0u);
            ctx->level_base = 0;
        }
        const uint32_t base = ctx->level_base;
        uint32_t levels = 0;
        starts[0] = 0;
        for (uint64_t i = 0; i < here; ++i) {  // starts[l + 1]: samples of level l
            const uint32_t u = pairs[2 * (first + i)], v = pairs[2 * (first + i) + 1];
            uint32_t at = std::max(std::max(base, row_u[u]), row_c[v]);
            for (uint32_t k = 0; k < K; ++k) at = std::max(at, row_c[neg[i * K + k]]);
            level[i] = at - base;
            if (level[i] == levels) starts[++levels] = 0;
            starts[level[i] + 1] += 1;
            row_u[u] = row_c[v] = at + 1;
            for (uint32_t k = 0; k < K; ++k) row_c[neg[i * K + k]] = at + 1;
        }
        ctx->level_base = base + levels;
        for (uint32_t l = 0; l < levels; ++l) starts[l + 1] += starts[l];
        for (uint64_t i = 0; i < here; ++i) order[starts[level[i]]++] = (uint32_t)i;  // leaves starts[l] at the end of level l
        memmove(starts + 1, starts, levels * sizeof(uint32_t));
        starts[0] = 0;
        if (here == part) {
            GV_HIP(ctx, hipMemcpyAsync(dev_order, order, (part + levels + 1) * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
        } else {  // the last part of several
            GV_HIP(ctx, hipMemcpyAsync(dev_order, order, here * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
            GV_HIP(ctx, hipMemcpyAsync(dev_starts, starts, (levels + 1) * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
        }
        GV_HIP(ctx, gv::launch_level_records(part_pairs, ctx->negatives, dev_order, (uint32_t)here, K, ctx->records, ctx->compute));
        // the arrays go out of scope; the stage stays, and is written again only behind the wait above
        if (!staged) GV_HIP(ctx, hipStreamSynchronize(ctx->compute));

        TimedSpan span{};
        const bool timed = ctx->cfg.profile != 0;
        if (timed) {
            rc = begin_span(ctx, 0, ctx->compute, &span);
            if (rc) return rc;
        }
        auto narrow = [&](uint32_t l) { return starts[l + 1] - starts[l] <= gv::kNarrowLevel; };
        gv::TrainArgs a = train_args(ctx, part_pairs, ctx->next_g + first, 0);
        for (uint32_t l = 0; l < levels;) {
            uint32_t end = l + 1;
            while (narrow(l) && end < levels && narrow(end)) ++end;
            a.count = starts[end] - starts[l];
            // a run of narrow levels reads its records by their place among all of them, a wide level from its first
            a.levels = narrow(l) ? end - l : 0u;
            a.level_starts = dev_starts + l;
            a.records = ctx->records + (narrow(l) ? 0 : (size_t)starts[l] * (K + 3));
            GV_HIP(ctx, launch(a, ctx->cfg.dim, K, ctx->compute));
            ctx->stats.train_launches += 1;
            l = end;
        }
        ctx->stats.batches += levels;
        if (ctx->dev_loss) ctx->stats.train_loss_samples += here;
        if (timed) {
            rc = end_span(ctx, ctx->compute, span);
            if (rc) return rc;
        }
    }
    levelling.complete = true;
    return GV_OK;
}

int train_any(gv_ctx *ctx, const uint32_t *dev_pairs, const uint32_t *host_pairs, uint64_t count) {
    if (count == 0) return GV_OK;
    int rc = GV_OK;
    if (ctx->cfg.mode != GV_MODE_DETERMINISTIC) {
        rc = train_hogwild(ctx, dev_pairs, count);
    } else {
        const bool flows = ctx->force_way ? ctx->force_way == 1 : count > kFlowFrom && ctx->hottest_share <= kFlowShare;
        const int room = flows && ctx->n <= 0x80000000u ? ensure_flow(ctx, count) : GV_ENOMEM;
        if (room != GV_OK && room != GV_ENOMEM) return room;
        bool narrow = false;
        if (room == GV_OK) rc = train_flow(ctx, dev_pairs, count, &narrow);
        if (room != GV_OK || narrow) rc = train_deterministic(ctx, dev_pairs, host_pairs, count);
    }
    if (rc) return rc;
    ctx->next_g += count;
    ctx->stats.samples_trained = ctx->next_g;
    ctx->stats.pools_trained += 1;
    return GV_OK;
}

// Wait until a slot no longer feeds a running launch, then mark it free.
int release_slot(gv_ctx *ctx, PoolSlot &s) {
    if (s.state == kTraining) {
        GV_HIP(ctx, hipEventSynchronize(s.trained));
        s.state = kFree;
    }
    return GV_OK;
}

// Next slot of the ring that is not being filled and not waiting to be trained (ring order =
// oldest first, so a slot still feeding a launch is the one whose launch ends soonest).
int pick_free_slot(gv_ctx *ctx, int *index) {
    const int slots = (int)ctx->slot.size();
    for (int t = 0; t < slots; ++t) {
        const int i = (ctx->next_slot + t) % slots;
        PoolSlot &s = ctx->slot[i];
        if (s.state == kFree || s.state == kTraining) {
            int rc = release_slot(ctx, s);
            if (rc) return rc;
            *index = i;
            ctx->next_slot = (i + 1) % slots;
            return GV_OK;
        }
    }
    return fail(ctx, GV_ESTATE, "all %d pool slots are filling or queued: train a pool first", slots);
}

// The pieces of an evaluation's pairs.  No kernel that reads one waits for one before it, except that a piece's memory is used
// again.
struct Pieces {
    gv_ctx *ctx;
    const uint64_t size;   // pairs of a piece
    const uint64_t slots;
    const bool again;      // some piece's memory is used twice
    uint64_t number = 0;
    Pieces(gv_ctx *c, uint64_t count, uint64_t size_)
        : ctx(c), size(size_), slots(kPieces * kPiecePairs / size_), again(count > (slots - 1) * size_) {}
    // body(first, pairs, slot, memory) for every piece of `count` pairs, in order: it may write `memory` and launches what
    // reads it on `stream`
    template <class Body>
    int take(uint64_t count, hipStream_t stream, Body &&body) {
        for (uint64_t first = 0; first < count; first += size, ++number) {
            const int slot = (int)(number % slots);
            if (again && !ctx->piece_read[slot]) GV_HIP(ctx, hipEventCreateWithFlags(&ctx->piece_read[slot], hipEventDisableTiming));
            if (number >= slots) GV_HIP(ctx, hipEventSynchronize(ctx->piece_read[slot]));
            int rc = body(first, std::min(size, count - first), slot, ctx->results->pieces + slot * 2 * size);
            if (rc) return rc;
            if (again) GV_HIP(ctx, hipEventRecord(ctx->piece_read[slot], stream));
        }
        return GV_OK;
    }
};

// Device scratch shared by the evaluation calls: grown when a call needs more, kept otherwise.
int ensure_eval_scratch(gv_ctx *ctx, uint64_t bytes) {
    if (bytes <= ctx->eval_capacity) return GV_OK;
    if (ctx->eval_scratch) {
        (void)hipFree(ctx->eval_scratch);
        ctx->eval_scratch = nullptr;
        ctx->eval_capacity = 0;
    }
    GV_HIP(ctx, hipMalloc(&ctx->eval_scratch, bytes));
    ctx->eval_capacity = bytes;
    return GV_OK;
}

// Area under the ROC curve of `pos` against `neg` as the rank statistic
// (sum of the positives' ranks - P (P + 1) / 2) / (P N), equal scores sharing their mean rank.
double rank_auc(const float *pos, uint64_t num_pos, const float *neg, uint64_t num_neg) {
    std::vector<std::pair<float, uint8_t>> all;
    all.reserve(num_pos + num_neg);
    for (uint64_t i = 0; i < num_pos; ++i) all.emplace_back(pos[i], (uint8_t)1);
    for (uint64_t i = 0; i < num_neg; ++i) all.emplace_back(neg[i], (uint8_t)0);
    std::sort(all.begin(), all.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    double positive_ranks = 0.0;
    for (size_t lo = 0; lo < all.size();) {
        size_t hi = lo;
        uint64_t positives = 0;
        while (hi < all.size() && all[hi].first == all[lo].first) positives += all[hi++].second;
        positive_ranks += (double)positives * (0.5 * ((double)(lo + 1) + (double)hi));  // ranks lo+1 .. hi share their mean
        lo = hi;
    }
    const double P = (double)num_pos, N = (double)num_neg;
    return (positive_ranks - P * (P + 1.0) / 2.0) / (P * N);
}

}  // namespace

extern "C" {

const char *gv_last_error(const gv_ctx *ctx) { return ctx ? ctx->error.c_str() : g_create_error.c_str(); }

int gv_create(const gv_config *cfg, gv_ctx **out) {
    if (out) *out = nullptr;
    if (!cfg || !out) return fail(nullptr, GV_EINVAL, "null argument");
    return guarded(nullptr, [&]() -> int {
        if (!gv::supported_shape(cfg->dim, cfg->num_neg))
            return fail(nullptr, GV_EINVAL, "unsupported shape: dim %u (a multiple of 32 in 32..512), num_neg %u (1..5)",
                        cfg->dim, cfg->num_neg);
        if (cfg->total_samples == 0) return fail(nullptr, GV_EINVAL, "total_samples must be > 0");
        if (cfg->pool_capacity == 0 || cfg->pool_capacity > (1ull << 31))
            return fail(nullptr, GV_EINVAL, "pool_capacity must be in 1..2^31 samples");
        if (cfg->partitions == 1 || cfg->partitions > GV_MAX_PARTITIONS)
            return fail(nullptr, GV_EINVAL, "partitions must be 0 (none) or in 2..%d", GV_MAX_PARTITIONS);
        if (cfg->pool_slots == 1 || cfg->pool_slots > GV_MAX_POOL_SLOTS)
            return fail(nullptr, GV_EINVAL, "pool_slots must be 0 (= 2) or in 2..%d", GV_MAX_POOL_SLOTS);
        if (cfg->mode > GV_MODE_DETERMINISTIC || cfg->coherence > GV_COHERENCE_MIXED ||
            cfg->schedule > GV_SCHEDULE_AUTO)
            return fail(nullptr, GV_EINVAL, "bad mode / coherence / schedule field");
        const bool default_weight = cfg->neg_weight == GV_NEG_WEIGHT_DEFAULT;
        if (!(cfg->lr0 >= 0.0f) || !(cfg->lr_min_ratio >= 0.0f) || !(default_weight || cfg->neg_weight >= 0.0f) ||
            !isfinite(cfg->lr0) || !isfinite(cfg->neg_weight))
            return fail(nullptr, GV_EINVAL,
                        "lr0, lr_min_ratio and neg_weight must be finite and >= 0 (neg_weight may be GV_NEG_WEIGHT_DEFAULT)");
        int devices = 0;
        if (hipGetDeviceCount(&devices) != hipSuccess || devices <= 0)
            return fail(nullptr, GV_EHIP, "no HIP device available");
        if (cfg->device < 0 || cfg->device >= devices)
            return fail(nullptr, GV_EINVAL, "device %d out of range (%d present)", cfg->device, devices);
        gv_ctx *ctx = new (std::nothrow) gv_ctx;
        if (!ctx) return fail(nullptr, GV_ENOMEM, "out of host memory");
        ctx->cfg = *cfg;
        // Sec. 4.3: one negative whose gradient is scaled by 5, to match the gradient scale of 5 negatives
        if (default_weight) ctx->cfg.neg_weight = 5.0f / (float)cfg->num_neg;
        if (ctx->cfg.pool_slots == 0) ctx->cfg.pool_slots = 2;
        auto bail = [&](int code) {
            g_create_error = ctx->error;
            gv_destroy(ctx);
            return code;
        };
#define GV_TRY(expr)                                                                                       \
    do {                                                                                                   \
        hipError_t e_ = (expr);                                                                            \
        if (e_ != hipSuccess) {                                                                            \
            (void)hipGetLastError();                                                                       \
            fail(ctx, e_ == hipErrorOutOfMemory ? GV_ENOMEM : GV_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
            return bail(e_ == hipErrorOutOfMemory ? GV_ENOMEM : GV_EHIP);                                  \
        }                                                                                                  \
    } while (0)
        try {
            ctx->slot.resize(ctx->cfg.pool_slots);
            ctx->queue.reserve(ctx->cfg.pool_slots);
        } catch (...) {
            fail(ctx, GV_ENOMEM, "out of host memory");
            return bail(GV_ENOMEM);
        }
        GV_TRY(hipSetDevice(cfg->device));
        if (cfg->device < kMaxDevices) {  // once per GPU, with that GPU current: where its copy of `scratch` lies
            std::lock_guard<std::mutex> lock(g_scratch_mutex);
            if (!g_scratch_address[cfg->device]) {
                void *address = nullptr;
                GV_TRY(hipGetSymbolAddress(&address, HIP_SYMBOL(scratch)));
                g_scratch_address[cfg->device] = (uint32_t *)address;
            }
            ctx->static_records = g_scratch_address[cfg->device];
        }
        GV_TRY(hipStreamCreateWithFlags(&ctx->compute, hipStreamNonBlocking));
        GV_TRY(hipStreamCreateWithFlags(&ctx->copy, hipStreamNonBlocking));
        GV_TRY(hipHostMalloc((void **)&ctx->results, sizeof(HostResults), hipHostMallocDefault));
        GV_TRY(hipMalloc((void **)&ctx->error_flag, 4 * sizeof(uint32_t)));
        GV_TRY(hipMemset(ctx->error_flag, 0, 4 * sizeof(uint32_t)));
        if (cfg->track_loss) {
            GV_TRY(hipMalloc((void **)&ctx->dev_loss, gv::kLossSlots * sizeof(double)));
            GV_TRY(hipMemset(ctx->dev_loss, 0, gv::kLossSlots * sizeof(double)));
        }
        const size_t pool_bytes = (size_t)cfg->pool_capacity * 2 * sizeof(uint32_t);
        for (PoolSlot &s : ctx->slot) {
            GV_TRY(hipHostMalloc((void **)&s.host, pool_bytes, hipHostMallocDefault));
            GV_TRY(hipMalloc((void **)&s.dev, pool_bytes));
            GV_TRY(hipEventCreateWithFlags(&s.copied, hipEventDisableTiming));
            GV_TRY(hipEventCreateWithFlags(&s.trained, hipEventDisableTiming));
        }
#undef GV_TRY
        *out = ctx;
        return GV_OK;
    });
}

void gv_destroy(gv_ctx *ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->cfg.device);
    if (ctx->copy) (void)hipStreamSynchronize(ctx->copy);
    if (ctx->compute) (void)hipStreamSynchronize(ctx->compute);
    try {
        fold_spans(ctx);
    } catch (...) {
    }
    for (const TimedSpan &s : ctx->spans) {  // left over only if folding failed
        (void)hipEventDestroy(s.start);
        (void)hipEventDestroy(s.stop);
    }
    for (hipEvent_t e : ctx->spare_events) (void)hipEventDestroy(e);
    for (PoolSlot &s : ctx->slot) {
        if (s.host) (void)hipHostFree(s.host);
        if (s.dev) (void)hipFree(s.dev);
        if (s.copied) (void)hipEventDestroy(s.copied);
        if (s.trained) (void)hipEventDestroy(s.trained);
    }
    free_matrices(ctx);
    if (ctx->negatives) (void)hipFree(ctx->negatives);
    if (ctx->records) (void)hipFree(ctx->records);
    if (ctx->eval_scratch) (void)hipFree(ctx->eval_scratch);
    if (ctx->error_flag) (void)hipFree(ctx->error_flag);
    if (ctx->results) (void)hipHostFree(ctx->results);
    if (ctx->dev_loss) (void)hipFree(ctx->dev_loss);
    if (ctx->flow_checked) (void)hipEventDestroy(ctx->flow_checked);
    for (hipEvent_t e : ctx->piece_read)
        if (e) (void)hipEventDestroy(e);
    if (ctx->copy) (void)hipStreamDestroy(ctx->copy);
    if (ctx->compute) (void)hipStreamDestroy(ctx->compute);
    delete ctx;
}

int gv_set_graph(gv_ctx *ctx, uint32_t n, uint64_t m, const uint32_t *host_src, const uint32_t *host_dst) {
    if (!ctx) return GV_EINVAL;
    return guarded(ctx, [&]() -> int {
        if (n == 0 || (m > 0 && (!host_src || !host_dst)))
            return fail(ctx, GV_EINVAL, "empty graph or null edge arrays");
        int rc = bind_device(ctx);
        if (rc) return rc;
        std::vector<uint32_t> deg(n, 0u);
        for (uint64_t i = 0; i < m; ++i) {
            const uint32_t a = host_src[i], b = host_dst[i];
            if (a >= n || b >= n)
                return fail(ctx, GV_EINVAL, "edge %llu names node id >= n (%u)", (unsigned long long)i, n);
            if (deg[a] == UINT32_MAX || deg[b] == UINT32_MAX) return fail(ctx, GV_EINVAL, "degree overflow");
            ++deg[a];
            ++deg[b];
        }
        return adopt_degrees(ctx, n, std::move(deg));
    });
}

int gv_set_degrees(gv_ctx *ctx, uint32_t n, const uint32_t *host_deg) {
    if (!ctx) return GV_EINVAL;
    return guarded(ctx, [&]() -> int {
        if (n == 0 || !host_deg) return fail(ctx, GV_EINVAL, "empty graph or null degree array");
        int rc = bind_device(ctx);
        if (rc) return rc;
        return adopt_degrees(ctx, n, std::vector<uint32_t>(host_deg, host_deg + n));
    });
}

int gv_set_weighted_graph(gv_ctx *ctx, uint32_t n, const uint64_t *host_offsets, const uint32_t *host_adj,
                          const float *host_weights) {
    if (!ctx) return GV_EINVAL;
    return guarded(ctx, [&]() -> int {
        if (n == 0 || !host_offsets || !host_adj || !host_weights) return fail(ctx, GV_EINVAL, "empty graph or null arrays");
        int rc = bind_device(ctx);
        if (rc) return rc;
        if (host_offsets[0] != 0) return fail(ctx, GV_EINVAL, "offsets[0] must be 0");
        std::vector<uint32_t> counts(n);
        for (uint32_t i = 0; i < n; ++i) {
            if (host_offsets[i + 1] < host_offsets[i] || host_offsets[i + 1] - host_offsets[i] > 0xFFFFFFFFull)
                return fail(ctx, GV_EINVAL, "offsets must ascend (row %u)", i);
            counts[i] = (uint32_t)(host_offsets[i + 1] - host_offsets[i]);
        }
        const uint64_t half_edges = host_offsets[n];
        if (half_edges == 0) return fail(ctx, GV_EINVAL, "graph without edges");
        for (uint64_t e = 0; e < half_edges; ++e) {
            if (host_adj[e] >= n) return fail(ctx, GV_EINVAL, "adjacency entry %llu names node id >= n", (unsigned long long)e);
            if (!(host_weights[e] >= 0.0f) || !isfinite(host_weights[e]))
                return fail(ctx, GV_EINVAL, "weight %llu is negative or not finite", (unsigned long long)e);
        }
        std::vector<double> wdeg(n);
        std::vector<uint32_t> node_thresh(n), node_alias(n), nbr_thresh(half_edges), nbr_alias(half_edges);
        rc = gv_build_walk_tables(n, host_offsets, host_weights, wdeg.data(), node_thresh.data(), node_alias.data(),
                                  nbr_thresh.data(), nbr_alias.data());
        if (rc == GV_ENOMEM) return fail(ctx, GV_ENOMEM, "out of host memory");
        if (rc) return fail(ctx, GV_EINVAL, "a node has edges but no weight, or the graph has no weight at all");
        rc = adopt_degrees(ctx, n, std::move(counts));
        if (rc) return rc;
        std::vector<uint2> node_table(n), nbr_table(half_edges);
        for (uint32_t i = 0; i < n; ++i) node_table[i] = make_uint2(node_thresh[i], node_alias[i]);
        for (uint64_t e = 0; e < half_edges; ++e) nbr_table[e] = make_uint2(nbr_thresh[e], nbr_alias[e]);
        auto upload = [&]() -> int {
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_offsets, ((size_t)n + 1) * sizeof(uint64_t)));
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_adj, (size_t)half_edges * sizeof(uint32_t)));
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_node_table, (size_t)n * sizeof(uint2)));
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_nbr_table, (size_t)half_edges * sizeof(uint2)));
            GV_HIP(ctx, hipMemcpy(ctx->dev_offsets, host_offsets, ((size_t)n + 1) * sizeof(uint64_t), hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_adj, host_adj, (size_t)half_edges * sizeof(uint32_t), hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_node_table, node_table.data(), (size_t)n * sizeof(uint2), hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_nbr_table, nbr_table.data(), (size_t)half_edges * sizeof(uint2), hipMemcpyHostToDevice));
            ctx->half_edges = half_edges;
            return prepare_walks(ctx);
        };
        rc = upload();
        if (rc) {
            free_adjacency(ctx);  // a part of it would be taken for the walk tables of the next adjacency
            return rc;
        }
        ctx->wdegree = std::move(wdeg);
        return GV_OK;
    });
}

int gv_build_alias(gv_ctx *ctx, double power) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (power != 0.75 && power != 1.0 && power != 0.0)
            return fail(ctx, GV_EINVAL, "power must be 0.75, 1.0 or 0.0");
        const uint32_t n = ctx->n;
        // the degree of a node, or on a weighted graph the sum of the weights of its edges
        const bool weighted = ctx->wdegree.size() == n;
        auto degree_of = [&](uint32_t node) { return weighted ? ctx->wdegree[node] : (double)ctx->degree[node]; };
        auto weight = [&](uint32_t node) {
            const double d = degree_of(node);
            if (power == 0.75) {
                const double root = sqrt(d);
                return root * sqrt(root);
            }
            return power == 1.0 ? d : 1.0;
        };
        std::vector<double> q(n);
        double degree_sum = 0.0;
        for (uint32_t i = 0; i < n; ++i) {
            degree_sum += degree_of(i);
            q[i] = weight(i);
        }
        std::vector<uint32_t> thresh(n), alias(n);
        double sum = 0.0;
        if (!gv::vose_table(q.data(), n, thresh.data(), alias.data(), &sum))
            return fail(ctx, GV_EINVAL, "all weights are zero (graph without edges)");
        // Hot ranks: the 65535 nodes of highest degree in falling order (ties by id); the rest share
        // the value 0xFFFF.  The tiled kernel keeps the row of lowest rank of a sample in registers.
        // A row is warm when, with kInFlight samples being processed at once (the order of magnitude of
        // a full launch: 2048 waves at a time, each with the samples of one batch), the expected number
        // of other in-flight samples naming the same row (as a walk endpoint, share deg/sum(deg),
        // or as one of the K negatives, share q/sum(q) each) exceeds kWarmThreshold: the mixed policy then updates it with
        // atomic adds.  Colder rows are updated with plain device-scope stores, which can drop an
        // update only when two of the few samples naming such a row are in flight together.  The
        // share grows with the degree, so the warm rows are the first warm_ranks of the ranking.
        // Under the orthogonal-block schedule the samples in flight all come from one block, where a
        // row's share is `partitions` times its share of the pool.
        const uint32_t B = ctx->cfg.partitions;
        const double kInFlight = 2048.0 * gv::samples_per_batch(ctx->cfg.dim, ctx->cfg.num_neg) * (B > 0 ? (double)B : 1.0);
        const double kWarmThreshold = 0.05;
        const uint32_t kRanked = 0xFFFFu;
        auto hotter = [&](uint32_t x, uint32_t y) {
            const double dx = degree_of(x), dy = degree_of(y);
            return dx != dy ? dx > dy : x < y;
        };
        std::vector<uint32_t> order(n);
        for (uint32_t i = 0; i < n; ++i) order[i] = i;
        const uint32_t ranked = n < kRanked ? n : kRanked;
        if (B > 0)
            std::sort(order.begin(), order.end(), hotter);  // the partition needs the whole order
        else
            std::partial_sort(order.begin(), order.begin() + ranked, order.end(), hotter);
        std::vector<uint16_t> rank(n, (uint16_t)kRanked);
        std::vector<uint32_t> ranked_bits(((size_t)n + 31) / 32, 0u);
        uint32_t warm_ranks = 0;
        double hottest_share = 0.0;
        for (uint32_t r = 0; r < ranked; ++r) {
            const uint32_t i = order[r];
            rank[i] = (uint16_t)r;
            ranked_bits[i >> 5] |= 1u << (i & 31u);
            const double share = (degree_sum > 0.0 ? degree_of(i) / degree_sum : 0.0) + (double)ctx->cfg.num_neg * q[i] / sum;
            if (share * kInFlight > kWarmThreshold) warm_ranks = r + 1;
            hottest_share = std::max(hottest_share, share);
        }
        std::vector<uint4> table(n);
        for (uint32_t i = 0; i < n; ++i)  // ranks of both candidates and the bucket's node save the kernel gathers
            table[i] = make_uint4(thresh[i], alias[i], (uint32_t)rank[i] | (uint32_t)rank[alias[i]] << 16, i);

        // Orthogonal blocks (Sec. 3.2, Alg. 3): degree-guided partition (Sec. 4.3: nodes by falling degree dealt
        // back and forth over the partitions) and one alias table per partition, over its nodes in increasing id.
        std::vector<uint32_t> part, members, part_thresh, part_alias;
        std::vector<uint64_t> part_offsets;
        std::vector<uint4> part_tables;
        std::vector<uint8_t> part_bytes;
        if (B > 0) {
            part.resize(n);
            for (uint32_t r = 0; r < n; ++r) {
                const uint32_t round = r / B, k = r % B;
                part[order[r]] = round % 2 == 0 ? k : B - 1 - k;
            }
            part_offsets.assign(B + 1, 0);
            for (uint32_t i = 0; i < n; ++i) part_offsets[part[i] + 1] += 1;
            for (uint32_t j = 0; j < B; ++j) part_offsets[j + 1] += part_offsets[j];
            members.resize(n);
            std::vector<uint64_t> fill(part_offsets.begin(), part_offsets.end() - 1);
            for (uint32_t i = 0; i < n; ++i) members[fill[part[i]]++] = i;
            part_thresh.resize(n);
            part_alias.resize(n);
            part_tables.resize(n);
            for (uint32_t j = 0; j < B; ++j) {
                const uint64_t lo = part_offsets[j], size = part_offsets[j + 1] - lo;
                std::vector<double> qj(size);
                for (uint64_t l = 0; l < size; ++l) qj[l] = weight(members[lo + l]);
                std::vector<uint32_t> tj(size), aj(size);
                if (size == 0 || !gv::vose_table(qj.data(), size, tj.data(), aj.data(), nullptr))
                    return fail(ctx, GV_EINVAL, "partition %u of %u has no node with a positive weight", j, B);
                for (uint64_t l = 0; l < size; ++l) {
                    const uint32_t self = members[lo + l], other = members[lo + aj[l]];
                    part_thresh[lo + l] = tj[l];
                    part_alias[lo + l] = other;
                    part_tables[lo + l] = make_uint4(tj[l], other, (uint32_t)rank[self] | (uint32_t)rank[other] << 16, self);
                }
            }
            part_bytes.resize(n);
            for (uint32_t i = 0; i < n; ++i) part_bytes[i] = (uint8_t)part[i];
        }
        order.clear();
        order.shrink_to_fit();

        rc = sync_all(ctx);
        if (rc != GV_OK && rc != GV_EINVAL && rc != GV_ESTATE) return rc;  // reports about pools already trained do not stop this call
        GV_HIP(ctx, hipMemcpy(ctx->alias, table.data(), (size_t)n * sizeof(uint4), hipMemcpyHostToDevice));
        GV_HIP(ctx, hipMemcpy(ctx->dev_rank, rank.data(), (size_t)n * sizeof(uint16_t), hipMemcpyHostToDevice));
        GV_HIP(ctx, hipMemcpy(ctx->dev_ranked, ranked_bits.data(), ranked_bits.size() * sizeof(uint32_t),
                              hipMemcpyHostToDevice));
        if (B > 0) {
            if (!ctx->dev_part_tables) {
                GV_HIP(ctx, hipMalloc((void **)&ctx->dev_part_tables, (size_t)n * sizeof(uint4)));
                GV_HIP(ctx, hipMalloc((void **)&ctx->dev_part_offsets, ((size_t)B + 1) * sizeof(uint64_t)));
                GV_HIP(ctx, hipMalloc((void **)&ctx->dev_part, (size_t)n));
            }
            GV_HIP(ctx, hipMemcpy(ctx->dev_part_tables, part_tables.data(), (size_t)n * sizeof(uint4), hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_part_offsets, part_offsets.data(), ((size_t)B + 1) * sizeof(uint64_t),
                                  hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_part, part_bytes.data(), (size_t)n, hipMemcpyHostToDevice));
            ctx->part = std::move(part);
            ctx->part_offsets = std::move(part_offsets);
            ctx->part_members = std::move(members);
            ctx->part_thresh = std::move(part_thresh);
            ctx->part_alias = std::move(part_alias);
        }
        ctx->warm_ranks = warm_ranks;
        ctx->hottest_share = hottest_share;
        ctx->stats.warm_rows = warm_ranks;
        ctx->alias_ready = true;
        return GV_OK;
    });
}

int gv_get_alias(gv_ctx *ctx, uint32_t *host_thresh, uint32_t *host_alias) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (!host_thresh || !host_alias) return fail(ctx, GV_EINVAL, "null output");
        std::vector<uint4> table(ctx->n);
        GV_HIP(ctx, hipMemcpy(table.data(), ctx->alias, (size_t)ctx->n * sizeof(uint4), hipMemcpyDeviceToHost));
        for (uint32_t i = 0; i < ctx->n; ++i) {
            host_thresh[i] = table[i].x;
            host_alias[i] = table[i].y;
        }
        return GV_OK;
    });
}

int gv_init_embeddings(gv_ctx *ctx, uint64_t seed) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        rc = sync_all(ctx);
        if (rc != GV_OK && rc != GV_EINVAL && rc != GV_ESTATE) return rc;  // reports about pools already trained do not stop this call
        GV_HIP(ctx, gv::launch_init_vertex(ctx->vertex, ctx->n, ctx->cfg.dim, seed, ctx->compute));
        GV_HIP(ctx, hipMemsetAsync(ctx->context, 0, (size_t)ctx->n * ctx->cfg.dim * sizeof(float), ctx->compute));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        return GV_OK;
    });
}

static int matrix_window(gv_ctx *ctx, int which, uint64_t row0, uint64_t rows, float **base) {
    if (which != GV_VERTEX && which != GV_CONTEXT) return fail(ctx, GV_EINVAL, "which must be GV_VERTEX or GV_CONTEXT");
    if (row0 > ctx->n || rows > ctx->n - row0)
        return fail(ctx, GV_EINVAL, "rows [%llu, %llu) outside the matrix (%u rows)", (unsigned long long)row0,
                    (unsigned long long)(row0 + rows), ctx->n);
    *base = (which == GV_VERTEX ? ctx->vertex : ctx->context) + row0 * ctx->cfg.dim;
    return GV_OK;
}

int gv_set_embeddings(gv_ctx *ctx, int which, const float *host_rows, uint64_t row0, uint64_t rows) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        float *base = nullptr;
        rc = matrix_window(ctx, which, row0, rows, &base);
        if (rc) return rc;
        if (rows == 0) return GV_OK;
        if (!host_rows) return fail(ctx, GV_EINVAL, "null input");
        rc = sync_all(ctx);
        if (rc != GV_OK && rc != GV_EINVAL && rc != GV_ESTATE) return rc;  // reports about pools already trained do not stop this call
        GV_HIP(ctx, hipMemcpy(base, host_rows, rows * ctx->cfg.dim * sizeof(float), hipMemcpyHostToDevice));
        return GV_OK;
    });
}

int gv_read_embeddings(gv_ctx *ctx, int which, float *host_rows, uint64_t row0, uint64_t rows) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        float *base = nullptr;
        rc = matrix_window(ctx, which, row0, rows, &base);
        if (rc) return rc;
        if (rows == 0) return GV_OK;
        if (!host_rows) return fail(ctx, GV_EINVAL, "null output");
        rc = sync_all(ctx);
        if (rc) return rc;
        GV_HIP(ctx, hipMemcpy(host_rows, base, rows * ctx->cfg.dim * sizeof(float), hipMemcpyDeviceToHost));
        return GV_OK;
    });
}

int gv_device_embeddings(gv_ctx *ctx, int which, float **dev_rows) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (!dev_rows) return fail(ctx, GV_EINVAL, "null output");
        return matrix_window(ctx, which, 0, 0, dev_rows);
    });
}

int gv_acquire_pool_slot(gv_ctx *ctx, uint32_t **host_pairs) {
    if (!ctx || !host_pairs) return ctx ? fail(ctx, GV_EINVAL, "null output") : GV_EINVAL;
    return guarded(ctx, [&]() -> int {
        int rc = bind_device(ctx);
        if (rc) return rc;
        int i = -1;
        rc = pick_free_slot(ctx, &i);
        if (rc) return rc;
        ctx->slot[i].state = kFilling;
        *host_pairs = ctx->slot[i].host;
        return GV_OK;
    });
}

int gv_push_pool(gv_ctx *ctx, const uint32_t *host_pairs, uint64_t count) {
    return guarded(ctx, [&]() -> int {
        if (!ctx) return GV_EINVAL;
        int i = -1;  // the acquired slot this push refers to, if any
        for (size_t t = 0; t < ctx->slot.size(); ++t)
            if (ctx->slot[t].state == kFilling && ctx->slot[t].host == host_pairs) i = (int)t;
        // a push that fails gives an acquired slot back: it would otherwise stay out of the ring for good
        auto give_back = [&](int rc) -> int {
            if (i >= 0) ctx->slot[i].state = kFree;
            return rc;
        };
        int rc = need_trainable(ctx);
        if (rc) return give_back(rc);
        if (count > ctx->cfg.pool_capacity)
            return give_back(fail(ctx, GV_EINVAL, "pool of %llu samples exceeds pool_capacity %llu",
                                  (unsigned long long)count, (unsigned long long)ctx->cfg.pool_capacity));
        if (count > 0 && !host_pairs) return fail(ctx, GV_EINVAL, "null pool");
        if (i < 0) {
            rc = pick_free_slot(ctx, &i);
            if (rc) return rc;
            memcpy(ctx->slot[i].host, host_pairs, count * 2 * sizeof(uint32_t));
            ctx->slot[i].state = kFilling;
        }
        PoolSlot &s = ctx->slot[i];
        s.count = count;
        auto hip_step = [&](hipError_t e, const char *what) -> int {
            if (e == hipSuccess) return GV_OK;
            return give_back(fail(ctx, e == hipErrorOutOfMemory ? GV_ENOMEM : GV_EHIP, "%s: %s", what, hipGetErrorString(e)));
        };
        TimedSpan span{};
        const bool timed = ctx->cfg.profile != 0 && count > 0;
        if (timed) {
            rc = begin_span(ctx, 1, ctx->copy, &span);
            if (rc) return give_back(rc);
        }
        if (count > 0) {
            rc = hip_step(hipMemcpyAsync(s.dev, s.host, count * 2 * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->copy),
                          "hipMemcpyAsync of the pool");
            if (rc) return rc;
        }
        if (timed) {
            rc = end_span(ctx, ctx->copy, span);
            if (rc) return give_back(rc);
        }
        rc = hip_step(hipEventRecord(s.copied, ctx->copy), "hipEventRecord");
        if (rc) return rc;
        ctx->stats.h2d_bytes += count * 2 * sizeof(uint32_t);
        s.state = kQueued;
        ctx->queue.push_back(i);
        return GV_OK;
    });
}

int gv_train_pool(gv_ctx *ctx) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (ctx->queue.empty()) return fail(ctx, GV_ESTATE, "no pool queued: call gv_push_pool first");
        const int i = ctx->queue.front();
        ctx->queue.erase(ctx->queue.begin());
        PoolSlot &s = ctx->slot[i];
        // Whatever goes wrong from here on, the slot returns to the ring only after the copy into its
        // device twin and every launch that may read it have ended.
        auto drop_slot = [&](int rc) -> int {
            (void)hipStreamSynchronize(ctx->copy);
            (void)hipStreamSynchronize(ctx->compute);
            s.state = kFree;
            return rc;
        };
        hipError_t e = hipStreamWaitEvent(ctx->compute, s.copied, 0);
        if (e != hipSuccess) return drop_slot(fail(ctx, GV_EHIP, "hipStreamWaitEvent: %s", hipGetErrorString(e)));
        rc = train_any(ctx, s.dev, s.host, s.count);
        if (rc) return drop_slot(rc);
        e = hipEventRecord(s.trained, ctx->compute);
        if (e != hipSuccess) return drop_slot(fail(ctx, GV_EHIP, "hipEventRecord: %s", hipGetErrorString(e)));
        s.state = kTraining;
        return GV_OK;
    });
}

int gv_train_device_pool(gv_ctx *ctx, const uint32_t *dev_pairs, uint64_t count) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (count > (1ull << 31)) return fail(ctx, GV_EINVAL, "at most 2^31 samples per call");
        if (count > 0 && !dev_pairs) return fail(ctx, GV_EINVAL, "null pool");
        return train_any(ctx, dev_pairs, nullptr, count);
    });
}

int gv_train_device_pool_static(gv_ctx *ctx, const uint32_t *dev_pairs, uint64_t count) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (ctx->cfg.mode != GV_MODE_HOGWILD)
            return fail(ctx, GV_ESTATE, "gv_train_device_pool_static trains asynchronously only (GV_MODE_HOGWILD)");
        if (!ctx->static_records) return fail(ctx, GV_ESTATE, "no static scratch on device %d", ctx->cfg.device);
        if (count > (1ull << 31)) return fail(ctx, GV_EINVAL, "at most 2^31 samples per call");
        if (count == 0) return GV_OK;
        if (!dev_pairs) return fail(ctx, GV_EINVAL, "null pool");
        rc = train_hogwild(ctx, dev_pairs, count, ctx->static_records);
        if (rc) return rc;
        ctx->next_g += count;
        ctx->stats.samples_trained = ctx->next_g;
        ctx->stats.pools_trained += 1;
        return GV_OK;
    });
}

int gv_get_partitions(gv_ctx *ctx, uint32_t *host_part, uint64_t *host_offsets, uint32_t *host_members,
                      uint32_t *host_thresh, uint32_t *host_alias) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (ctx->cfg.partitions == 0 || ctx->part.size() != ctx->n)
            return fail(ctx, GV_ESTATE, "the context was created without partitions");
        if (!host_part || !host_offsets || !host_members || !host_thresh || !host_alias)
            return fail(ctx, GV_EINVAL, "null output");
        std::copy(ctx->part.begin(), ctx->part.end(), host_part);
        std::copy(ctx->part_offsets.begin(), ctx->part_offsets.end(), host_offsets);
        std::copy(ctx->part_members.begin(), ctx->part_members.end(), host_members);
        std::copy(ctx->part_thresh.begin(), ctx->part_thresh.end(), host_thresh);
        std::copy(ctx->part_alias.begin(), ctx->part_alias.end(), host_alias);
        return GV_OK;
    });
}

int gv_train_device_blocks(gv_ctx *ctx, const uint32_t *dev_pairs, const uint32_t *dev_order,
                           const uint64_t *host_block_offsets, uint64_t count) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        const uint32_t B = ctx->cfg.partitions;
        if (B == 0 || ctx->part.size() != ctx->n) return fail(ctx, GV_ESTATE, "the context was created without partitions");
        if (ctx->cfg.mode != GV_MODE_HOGWILD)
            return fail(ctx, GV_ESTATE, "orthogonal blocks are trained asynchronously only (GV_MODE_HOGWILD)");
        if (count > (1ull << 32)) return fail(ctx, GV_EINVAL, "at most 2^32 samples per call");
        if (!host_block_offsets) return fail(ctx, GV_EINVAL, "null block offsets");
        const uint64_t blocks = (uint64_t)B * B;
        if (host_block_offsets[0] != 0 || host_block_offsets[blocks] != count)
            return fail(ctx, GV_EINVAL, "block offsets must run from 0 to count");
        for (uint64_t b = 0; b < blocks; ++b)
            if (host_block_offsets[b] > host_block_offsets[b + 1] ||
                host_block_offsets[b + 1] - host_block_offsets[b] > (1ull << 31))
                return fail(ctx, GV_EINVAL, "block offsets must ascend, at most 2^31 samples per block");
        if (count == 0) return GV_OK;
        if (!dev_pairs || !dev_order) return fail(ctx, GV_EINVAL, "null pool");
        // sub-episode o = b / B trains the blocks (i, (i + o) mod B), i = b mod B, one launch each, in order
        for (uint64_t b = 0; b < blocks; ++b) {
            const uint64_t lo = host_block_offsets[b], size = host_block_offsets[b + 1] - lo;
            if (size == 0) continue;
            const uint32_t o = (uint32_t)(b / B), i = (uint32_t)(b % B);
            const BlockOfPool block{dev_order + lo, (i + o) % B};
            rc = train_hogwild(ctx, dev_pairs + 2 * lo, size, nullptr, &block);
            if (rc) return rc;
        }
        ctx->next_g += count;
        ctx->stats.samples_trained = ctx->next_g;
        ctx->stats.pools_trained += 1;
        return GV_OK;
    });
}

int gv_draw_negatives_partitioned(gv_ctx *ctx, uint64_t first_g, uint64_t count, const uint32_t *host_v,
                                  uint32_t *host_out) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (ctx->cfg.partitions == 0 || ctx->part.size() != ctx->n)
            return fail(ctx, GV_ESTATE, "the context was created without partitions");
        if (count == 0) return GV_OK;
        if (!host_v || !host_out) return fail(ctx, GV_EINVAL, "null argument");
        if (count > (1ull << 31)) return fail(ctx, GV_EINVAL, "at most 2^31 samples per call");
        for (uint64_t i = 0; i < count; ++i)
            if (host_v[i] >= ctx->n) return fail(ctx, GV_EINVAL, "sample %llu names node id >= n", (unsigned long long)i);
        const uint32_t K = ctx->cfg.num_neg;
        rc = sync_all(ctx);
        if (rc) return rc;
        rc = ensure_negatives(ctx, count * K);
        if (rc) return rc;
        rc = ensure_eval_scratch(ctx, count * sizeof(uint32_t));
        if (rc) return rc;
        uint32_t *dev_v = (uint32_t *)ctx->eval_scratch;
        GV_HIP(ctx, hipMemcpyAsync(dev_v, host_v, count * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
        GV_HIP(ctx, gv::launch_draw_negatives_partitioned(ctx->dev_part_tables, ctx->dev_part_offsets, ctx->dev_part, dev_v,
                                                          ctx->cfg.seed, first_g, count, K, ctx->negatives, ctx->compute));
        GV_HIP(ctx, hipMemcpyAsync(host_out, ctx->negatives, count * K * sizeof(uint32_t), hipMemcpyDeviceToHost,
                                   ctx->compute));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        return GV_OK;
    });
}

int gv_set_adjacency(gv_ctx *ctx, const uint64_t *host_offsets, const uint32_t *host_adj) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (!host_offsets || !host_adj) return fail(ctx, GV_EINVAL, "null adjacency");
        const uint32_t n = ctx->n;
        if (host_offsets[0] != 0) return fail(ctx, GV_EINVAL, "offsets[0] must be 0");
        for (uint32_t i = 0; i < n; ++i)
            if (host_offsets[i + 1] - host_offsets[i] != (uint64_t)ctx->degree[i])
                return fail(ctx, GV_EINVAL, "row %u of the adjacency has %llu entries, the graph gives node %u degree %u",
                            i, (unsigned long long)(host_offsets[i + 1] - host_offsets[i]), i, ctx->degree[i]);
        const uint64_t half_edges = host_offsets[n];
        if (half_edges == 0) return fail(ctx, GV_EINVAL, "graph without edges");
        for (uint64_t e = 0; e < half_edges; ++e)
            if (host_adj[e] >= n)
                return fail(ctx, GV_EINVAL, "adjacency entry %llu names node id >= n", (unsigned long long)e);
        rc = sync_all(ctx);
        if (rc != GV_OK && rc != GV_EINVAL && rc != GV_ESTATE) return rc;  // reports about pools already trained do not stop this call
        if (ctx->wdegree.size() == n)
            return fail(ctx, GV_ESTATE, "the graph is weighted: gv_set_weighted_graph has uploaded its adjacency already");
        free_adjacency(ctx);
        auto upload = [&]() -> int {
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_offsets, ((size_t)n + 1) * sizeof(uint64_t)));
            GV_HIP(ctx, hipMalloc((void **)&ctx->dev_adj, (size_t)half_edges * sizeof(uint32_t)));
            GV_HIP(ctx, hipMemcpy(ctx->dev_offsets, host_offsets, ((size_t)n + 1) * sizeof(uint64_t), hipMemcpyHostToDevice));
            GV_HIP(ctx, hipMemcpy(ctx->dev_adj, host_adj, (size_t)half_edges * sizeof(uint32_t), hipMemcpyHostToDevice));
            ctx->half_edges = half_edges;
            return prepare_walks(ctx);
        };
        rc = upload();
        if (rc) free_adjacency(ctx);
        return rc;
    });
}

int gv_augment_device(gv_ctx *ctx, uint64_t seed, uint32_t walk_length, uint32_t window, uint64_t first_walk,
                      uint64_t count, uint32_t shuffle, uint32_t *dev_pairs, uint64_t *walks_used) {
    if (walks_used) *walks_used = 0;
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (!ctx->dev_offsets) return fail(ctx, GV_ESTATE, "no adjacency: call gv_set_adjacency first");
        if (walk_length == 0 || walk_length > 64 || window == 0 || window > GV_MAX_WINDOW || shuffle > GV_SHUFFLE_PSEUDO)
            return fail(ctx, GV_EINVAL, "walk_length must be in 1..64, window in 1..GV_MAX_WINDOW, shuffle GV_SHUFFLE_*");
        if (count == 0) return GV_OK;
        if (!dev_pairs) return fail(ctx, GV_EINVAL, "null output");
        gv::AugmentArgs a{};
        a.offsets = ctx->dev_offsets;
        a.adj = ctx->dev_adj;
        const bool weighted = ctx->dev_node_table != nullptr;
        a.steps = weighted ? nullptr : ctx->dev_steps;
        a.weighted_steps = weighted ? ctx->dev_steps : nullptr;
        a.guide = ctx->dev_guide;
        a.guide_shift = gv::guide_shift(ctx->half_edges);
        a.pairs = (uint2 *)dev_pairs;
        a.half_edges = ctx->half_edges;
        a.seed = seed;
        a.first_walk = first_walk;
        a.count = count;
        a.per_walk = 0;  // pairs (i, j), i < j <= min(i + window, walk_length)
        for (uint32_t d = 1; d <= window && d <= walk_length; ++d) a.per_walk += walk_length + 1 - d;
        a.walks = (count + a.per_walk - 1) / a.per_walk;
        a.n = ctx->n;
        a.length = walk_length;
        a.window = window;
        a.pseudo_shuffle = shuffle == GV_SHUFFLE_PSEUDO ? 1u : 0u;
        a.node_table = ctx->dev_node_table;
        a.nbr_table = ctx->dev_nbr_table;
        if (walks_used) *walks_used = a.walks;
        GV_HIP(ctx, gv::launch_augment(a, ctx->compute));
        return GV_OK;
    });
}

int gv_draw_negatives(gv_ctx *ctx, uint64_t first_g, uint64_t count, uint32_t *host_out) {
    return guarded(ctx, [&]() -> int {
        int rc = need_trainable(ctx);
        if (rc) return rc;
        if (count == 0) return GV_OK;
        if (!host_out) return fail(ctx, GV_EINVAL, "null output");
        if (count > (1ull << 32)) return fail(ctx, GV_EINVAL, "at most 2^32 samples per call");
        const uint32_t K = ctx->cfg.num_neg;
        rc = ensure_negatives(ctx, count * K);
        if (rc) return rc;
        GV_HIP(ctx, gv::launch_draw_negatives(ctx->alias, ctx->n, ctx->cfg.seed, first_g, count, K, ctx->negatives,
                                              ctx->compute));
        GV_HIP(ctx, hipMemcpyAsync(host_out, ctx->negatives, count * K * sizeof(uint32_t), hipMemcpyDeviceToHost,
                                   ctx->compute));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        return GV_OK;
    });
}

int gv_eval_loss(gv_ctx *ctx, const uint32_t *host_pairs, uint64_t count, uint64_t eval_seed, double *mean_loss) {
    return guarded(ctx, [&]() -> int {
        if (int rc = need_trainable(ctx)) return rc;
        if (!mean_loss || (count > 0 && !host_pairs)) return fail(ctx, GV_EINVAL, "null argument");
        if (count == 0 || count > (1ull << 32) - 1) return fail(ctx, GV_EINVAL, "count must be in 1 .. 2^32-1");
        // everything below is ordered behind the training on the compute stream; what that has to report is read at
        // the end, together with the result
        HostResults &r = *ctx->results;
        double total = 0.0;
        uint32_t blocks[kPieces] = {};
        auto take_in = [&](int slot) {
            for (uint32_t b = 0; b < blocks[slot]; ++b) total += r.partial[slot][b];
            blocks[slot] = 0;
        };
        PinnedInUse in_use{ctx};
        Pieces pieces(ctx, count, count > 3 * kPiecePairs ? 2 * kPiecePairs : kPiecePairs);
        int rc = pieces.take(count, ctx->compute, [&](uint64_t first, uint64_t here, int slot, uint32_t *pairs) -> int {
            take_in(slot);
            memcpy(pairs, host_pairs + 2 * first, here * 2 * sizeof(uint32_t));
            gv::TrainArgs a = train_args(ctx, pairs, first, (uint32_t)here);
            a.seed = eval_seed;
            a.error_flag = ctx->error_flag + 2;
            GV_HIP(ctx, gv::launch_eval_loss(a, ctx->cfg.dim, ctx->cfg.num_neg, r.partial[slot], &blocks[slot], ctx->compute));
            return GV_OK;
        });
        if (rc) return rc;
        bool bad_ids = false;  // then the result covers the other pairs
        rc = sync_all(ctx, &bad_ids);
        in_use.ended = rc != GV_EHIP;
        if (rc && !bad_ids) return rc;
        for (int slot = 0; slot < kPieces; ++slot) take_in(slot);
        *mean_loss = total / (double)count;
        return rc;
    });
}

// cosines of `count` node pairs into host_out, through the evaluation scratch
static int cosine_scores(gv_ctx *ctx, const uint32_t *host_first, const uint32_t *host_second, uint64_t count,
                         float *host_out) {
    int rc = ensure_eval_scratch(ctx, count * (2 * sizeof(uint32_t) + sizeof(float)));
    if (rc) return rc;
    uint32_t *dev_ids = (uint32_t *)ctx->eval_scratch;
    float *dev_out = (float *)(dev_ids + 2 * count);
    GV_HIP(ctx, hipMemcpyAsync(dev_ids, host_first, count * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
    GV_HIP(ctx, hipMemcpyAsync(dev_ids + count, host_second, count * sizeof(uint32_t), hipMemcpyHostToDevice, ctx->compute));
    GV_HIP(ctx, gv::launch_cosine(ctx->vertex, ctx->n, ctx->cfg.dim, dev_ids, dev_ids + count, (uint32_t)count,
                                  gv::kWavesOnDevicePairs, dev_out, ctx->error_flag + 2, ctx->compute));
    GV_HIP(ctx, hipMemcpyAsync(host_out, dev_out, count * sizeof(float), hipMemcpyDeviceToHost, ctx->compute));
    GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
    return GV_OK;
}

int gv_cosine(gv_ctx *ctx, const uint32_t *host_first, const uint32_t *host_second, uint64_t count, float *host_out) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (count == 0) return GV_OK;
        if (!host_first || !host_second || !host_out) return fail(ctx, GV_EINVAL, "null argument");
        if (count > (1ull << 32) - 1) return fail(ctx, GV_EINVAL, "at most 2^32-1 pairs per call");
        rc = sync_all(ctx);
        if (rc) return rc;
        rc = cosine_scores(ctx, host_first, host_second, count, host_out);
        if (rc) return rc;
        return sync_all(ctx);
    });
}

int gv_auc(const float *host_pos, uint64_t num_pos, const float *host_neg, uint64_t num_neg, double *auc) {
    if (!auc) return GV_EINVAL;
    *auc = 0.0;
    if (num_pos == 0 || num_neg == 0 || !host_pos || !host_neg) return GV_EINVAL;
    return guarded(nullptr, [&]() -> int {
        for (uint64_t i = 0; i < num_pos; ++i)
            if (!isfinite(host_pos[i])) return fail(nullptr, GV_EINVAL, "positive score %llu is not finite", (unsigned long long)i);
        for (uint64_t i = 0; i < num_neg; ++i)
            if (!isfinite(host_neg[i])) return fail(nullptr, GV_EINVAL, "negative score %llu is not finite", (unsigned long long)i);
        *auc = rank_auc(host_pos, num_pos, host_neg, num_neg);
        return GV_OK;
    });
}

int gv_link_prediction_auc(gv_ctx *ctx, const uint32_t *host_edge_first, const uint32_t *host_edge_second,
                           uint64_t num_edges, const uint32_t *host_other_first, const uint32_t *host_other_second,
                           uint64_t num_others, double *auc) {
    return guarded(ctx, [&]() -> int {
        int rc = need_graph(ctx);
        if (rc) return rc;
        if (!auc || !host_edge_first || !host_edge_second || !host_other_first || !host_other_second)
            return fail(ctx, GV_EINVAL, "null argument");
        if (num_edges == 0 || num_others == 0 || num_edges + num_others > (1ull << 31))
            return fail(ctx, GV_EINVAL, "both pair sets must be non-empty and hold at most 2^31 pairs together");
        const uint64_t count = num_edges + num_others;
        auto rank_on_host = [&](const float *scores) -> int {
            for (uint64_t i = 0; i < count; ++i)
                if (!isfinite(scores[i])) return fail(ctx, GV_EINVAL, "an embedding row is not finite");
            *auc = rank_auc(scores, num_edges, scores + num_edges, num_others);
            return GV_OK;
        };
        // scratch: the sort's, then the scores; those of few pairs go to pinned memory
        const bool few = count <= kHostRanked;
        const uint64_t sorting = few ? 0 : (gv::rank_scratch_words((uint32_t)num_others) + 3u) & ~3ull;
        rc = few ? GV_OK : ensure_eval_scratch(ctx, (sorting + count) * sizeof(uint32_t));
        if (rc == GV_ENOMEM) {  // the cosines of one set after the other may take less
            rc = sync_all(ctx);
            if (rc) return rc;
            std::vector<float> scores(count);
            rc = cosine_scores(ctx, host_edge_first, host_edge_second, num_edges, scores.data());
            if (rc) return rc;
            rc = cosine_scores(ctx, host_other_first, host_other_second, num_others, scores.data() + num_edges);
            if (rc) return rc;
            rc = sync_all(ctx);  // ids >= n
            return rc ? rc : rank_on_host(scores.data());
        }
        if (rc) return rc;
        HostResults &r = *ctx->results;
        uint32_t *dev_sorting = (uint32_t *)ctx->eval_scratch;
        float *const scores = few ? r.scores : (float *)(dev_sorting + sorting);
        // Many edges are scored on another stream while the others are sorted, which is latency of short launches (500000 pairs
        // 278 -> 258 us, 2*10^6 903 -> 820; two streams cost more than they hide up to 200000: 165 and 165, 40000 101 and 129).
        // It has nothing to wait for but the training before, and the host waits for that.
        hipStream_t const beside = count > 1u << 18 ? ctx->copy : ctx->compute;
        if (beside != ctx->compute) GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        PinnedInUse in_use{ctx};
        Pieces pieces(ctx, count + kPiecePairs, kPiecePairs);
        auto score = [&](const uint32_t *host_first, const uint32_t *host_second, uint64_t pairs, float *to, hipStream_t on) {
            return pieces.take(pairs, on, [&](uint64_t first, uint64_t here, int, uint32_t *firsts) -> int {
                uint32_t *const seconds = firsts + here;
                memcpy(firsts, host_first + first, here * sizeof(uint32_t));
                memcpy(seconds, host_second + first, here * sizeof(uint32_t));
                GV_HIP(ctx, gv::launch_cosine(ctx->vertex, ctx->n, ctx->cfg.dim, firsts, seconds, (uint32_t)here,
                                              gv::kWavesOnHostPairs, to + first, ctx->error_flag + 2, on));
                return GV_OK;
            });
        };
        rc = score(host_other_first, host_other_second, num_others, scores + num_edges, ctx->compute);
        if (rc) return rc;
        if (!few) {
            std::fill_n(r.sums + gv::kRankBlocks, gv::kRankBlocks, 0ull);  // in use by no kernel: every call waits for its own
            GV_HIP(ctx, gv::launch_rank_sort((uint32_t *)scores + num_edges, (uint32_t)num_others, dev_sorting, r.sums + gv::kRankBlocks,
                                             ctx->compute));
        }
        rc = score(host_edge_first, host_edge_second, num_edges, scores, beside);
        if (rc) return rc;
        if (!few) {
            if (beside != ctx->compute) GV_HIP(ctx, hipStreamSynchronize(beside));
            GV_HIP(ctx, gv::launch_rank_sum((uint32_t *)scores, (uint32_t)num_edges, (uint32_t)num_others, r.sums, r.sums + gv::kRankBlocks,
                                            ctx->compute));
        }
        rc = sync_all(ctx);  // also reports ids >= n, and what training before had to report
        in_use.ended = rc != GV_EHIP;
        if (rc) return rc;
        if (few) return rank_on_host(r.scores);
        unsigned long long twice = 0, not_finite = 0;
        for (uint32_t b = 0; b < gv::kRankBlocks; ++b) {
            twice += r.sums[b];
            not_finite |= r.sums[gv::kRankBlocks + b];
        }
        if (not_finite) return fail(ctx, GV_EINVAL, "an embedding row is not finite");
        *auc = 0.5 * (double)twice / ((double)num_edges * (double)num_others);
        return GV_OK;
    });
}

int gv_sync(gv_ctx *ctx) {
    if (!ctx) return GV_EINVAL;
    return guarded(ctx, [&]() -> int {
        int rc = bind_device(ctx);
        if (rc) return rc;
        return sync_all(ctx);
    });
}

int gv_get_stats(gv_ctx *ctx, gv_stats *out) {
    if (!ctx || !out) return ctx ? fail(ctx, GV_EINVAL, "null output") : GV_EINVAL;
    const int rc = guarded(ctx, [&]() -> int {
        if (!ctx->flow_pending) return GV_OK;
        int rc = bind_device(ctx);
        if (rc) return rc;
        GV_HIP(ctx, hipMemcpyAsync(&ctx->results->flow, ctx->flow_state, sizeof(gv::FlowState), hipMemcpyDeviceToHost, ctx->compute));
        GV_HIP(ctx, hipStreamSynchronize(ctx->compute));
        fold_flow(ctx);  // what it has to report is left to the next synchronising call
        return GV_OK;
    });
    *out = ctx->stats;
    return rc;
}

int gv_set_position(gv_ctx *ctx, uint64_t next_g) {
    if (!ctx) return GV_EINVAL;
    ctx->next_g = next_g;
    ctx->stats.samples_trained = next_g;
    return GV_OK;
}

// Not part of the boundary: lets a test run the kernels of long pools on short ones.  Launches that the schedule walks in
// tiles take tiles of `samples` under the context's own policy; 0: as async_plan decides.  GV_EINVAL for a size that the
// policy and the row length have no kernel for.
int gv_test_force_tile(gv_ctx *ctx, uint32_t samples) {
    if (!ctx) return GV_EINVAL;
    const bool smaller = ctx->cfg.coherence == GV_COHERENCE_ATOMIC_AGENT ||
                         (ctx->cfg.coherence == GV_COHERENCE_MIXED &&
                          gv::short_rows(gv::floats_per_lane(ctx->cfg.dim), (int)ctx->cfg.num_neg));
    const bool size = samples >= gv::kSmallestTile && samples <= gv::kLargestTile && !(samples & (samples - 1u));
    if (samples != 0 && !(size && (smaller || samples == gv::kLargestTile)))
        return fail(ctx, GV_EINVAL, "no kernel with tiles of %u samples", samples);
    ctx->force_tile = samples;
    return GV_OK;
}

// Not part of the boundary: lets a test take either way of deterministic pools.  1: they wait on the device, whatever their
// length and rows (where that finds memory); 2: they are sorted into levels; 0: as kFlowFrom tells.
int gv_test_force_way(gv_ctx *ctx, uint32_t way) {
    if (!ctx) return GV_EINVAL;
    if (way > 2) return fail(ctx, GV_EINVAL, "no way %u", way);
    ctx->force_way = way;
    return GV_OK;
}

}  // extern "C"
