// The runtime behind the C boundary (gv_api.cpp) on a device made of host memory, so that what it does when memory
// runs out, and the arguments it hands to the kernels, can be checked without a GPU.  The HIP calls that it makes are
// defined here (they take precedence over the runtime's), and so are the launches: each of them reads and writes what
// its kernel would, so that AddressSanitizer sees an array that is too short, and checks what its kernel relies on.
// One argument: the name of the check.  Exit code 0 = it passed.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <set>
#include <new>
#include <vector>

#include "gv_internal.hpp"
#include "gvhot.h"

extern "C" int gv_test_force_tile(gv_ctx *ctx, uint32_t samples);
extern "C" int gv_test_force_way(gv_ctx *ctx, uint32_t way);

#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            exit(1);                                                                 \
        }                                                                            \
    } while (0)

// ---------------------------------------------------------------------------------------------------- memory
namespace {
long host_allocations_left = -1;    // this many more, then one fails; negative: no limit
long device_allocations_left = -1;  // the same of hipMalloc
uint64_t device_allocations = 0, device_frees = 0;
long launches_left = -1;            // of kernels that use pinned memory, the same
std::set<hipStream_t> using_pinned; // streams with such kernels that nothing has waited for
uint32_t row_without_end = UINT32_MAX;  // node whose cosines are not finite
size_t device_largest = SIZE_MAX;   // bytes that a hipMalloc may ask for
size_t device_free = SIZE_MAX;      // bytes that hipMemGetInfo says are left
}  // namespace

void *operator new(size_t size) {
    if (host_allocations_left == 0) {
        host_allocations_left = -1;
        throw std::bad_alloc();
    }
    if (host_allocations_left > 0) --host_allocations_left;
    void *p = malloc(size);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new[](size_t size) { return operator new(size); }
void *operator new(size_t size, const std::nothrow_t &) noexcept { return malloc(size); }
void *operator new[](size_t size, const std::nothrow_t &) noexcept {
    try {
        return operator new(size);
    } catch (const std::bad_alloc &) {
        return nullptr;
    }
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
void operator delete[](void *p) noexcept { free(p); }
void operator delete[](void *p, size_t) noexcept { free(p); }

extern "C" {
static hipError_t last_error = hipSuccess;
hipError_t hipMalloc(void **p, size_t size) {
    if (device_allocations_left == 0) {
        device_allocations_left = -1;
        *p = nullptr;
        return last_error = hipErrorOutOfMemory;
    }
    if (device_allocations_left > 0) --device_allocations_left;
    *p = size <= device_largest ? malloc(size) : nullptr;
    device_allocations += *p != nullptr;
    return *p ? hipSuccess : last_error = hipErrorOutOfMemory;
}
hipError_t hipMemGetInfo(size_t *left, size_t *total) {
    *left = device_free;
    *total = SIZE_MAX;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    device_frees += 1;
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t size, unsigned) {
    *p = malloc(size);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipMemcpy(void *to, const void *from, size_t size, hipMemcpyKind) {
    memcpy(to, from, size);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t size, hipMemcpyKind kind, hipStream_t) {
    return hipMemcpy(to, from, size, kind);
}
hipError_t hipMemset(void *p, int value, size_t size) {
    memset(p, value, size);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int value, size_t size, hipStream_t) { return hipMemset(p, value, size); }
static int handle;  // events: everything is done in the order of the calls
static char stream_names[1024];
static int streams = 0;
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)&stream_names[streams++ % 1024];
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    using_pinned.erase(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)&handle;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.0f;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *count) {
    *count = 1;
    return hipSuccess;
}
hipError_t hipGetLastError() {  // what a launch after a failed allocation would return for its own
    const hipError_t error = last_error;
    last_error = hipSuccess;
    return error;
}
const char *hipGetErrorString(hipError_t) { return "as told"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static std::vector<uint32_t> scratch(GV_STATIC_SCRATCH_WORDS);
    *p = scratch.data();
    return hipSuccess;
}
}  // extern "C"

// ---------------------------------------------------------------------------------------------------- launches
namespace {
struct Trained {  // of deterministic mode, in the order of training
    uint32_t level;
    std::vector<uint32_t> rows;  // u, then n + every context row
    uint64_t place;
};
std::vector<Trained> trained;
uint32_t levels_trained = 0;
uint64_t flowed = 0;  // samples trained by launch_train_flow
bool stall_next = false;  // the next launch_train_flow gives up
int training_reports = -1;  // word of the error flag that asynchronous training sets, if any
bool tiled_launched = false;
uint32_t launched_unit = 0;
bool ranked_on_device = false;
bool walked_weighted = false, walked_packed = false;  // by the device producer
uint64_t touched = 0;  // of the arrays that a kernel would read

uint32_t draw(uint64_t g, uint32_t k, uint32_t n) { return (uint32_t)((g * 0x9E3779B97F4A7C15ull + k * 0xD1B54A32D192ED03ull) >> 40) % n; }

template <class T>
void read_all(const T *array, uint64_t count) {
    const unsigned char *bytes = (const unsigned char *)array;
    for (uint64_t i = 0; i < count * sizeof(T); ++i) touched += bytes[i];
}
}  // namespace

namespace gv {
hipError_t launch_train_hogwild(const TrainArgs &a, uint32_t, uint32_t, uint32_t, hipStream_t) {
    launched_unit = a.unit;
    if (training_reports >= 0) a.error_flag[training_reports] = 1u;
    return hipGetLastError();
}
hipError_t launch_train_tiled(const TrainArgs &a, uint32_t, uint32_t, uint32_t, hipStream_t) {
    tiled_launched = true;
    launched_unit = a.unit;
    if (training_reports >= 0) a.error_flag[training_reports] = 1u;
    return hipGetLastError();
}
hipError_t launch_train_hogwild_tracked(const TrainArgs &, uint32_t, uint32_t, uint32_t, hipStream_t) { return hipGetLastError(); }
hipError_t launch_train_tiled_tracked(const TrainArgs &, uint32_t, uint32_t, uint32_t, hipStream_t) { return hipGetLastError(); }
hipError_t launch_train_levels(const TrainArgs &a, uint32_t, uint32_t num_neg, hipStream_t) {
    const long left = host_allocations_left;  // what this function allocates is not the library's
    host_allocations_left = -1;
    const uint32_t levels = a.levels ? a.levels : 1u;
    for (uint32_t l = 0; l < levels; ++l) {
        const uint32_t begin = a.levels ? a.level_starts[l] : 0u, end = a.levels ? a.level_starts[l + 1] : a.count;
        CHECK(begin < end);
        for (uint32_t i = begin; i < end; ++i) {
            const uint32_t *record = a.records + (size_t)i * (num_neg + 3);
            Trained t{levels_trained, {record[0]}, a.first_g + record[num_neg + 2]};
            for (uint32_t k = 0; k <= num_neg; ++k) t.rows.push_back(a.n + record[1 + k]);
            trained.push_back(t);
        }
        ++levels_trained;
    }
    host_allocations_left = left;
    return hipGetLastError();
}
hipError_t launch_train_levels_tracked(const TrainArgs &a, uint32_t dim, uint32_t num_neg, hipStream_t s) {
    return launch_train_levels(a, dim, num_neg, s);
}
static_assert(sizeof(TrainArgs) == 176, "carried by every launch of asynchronous training: arguments of one kernel go into a struct of their own");
bool launches(hipStream_t stream) {
    if (launches_left == 0) {
        launches_left = -1;
        return false;
    }
    if (launches_left > 0) --launches_left;
    const long left = host_allocations_left;
    host_allocations_left = -1;
    using_pinned.insert(stream);
    host_allocations_left = left;
    return true;
}
uint64_t flow_scratch_words(uint32_t count, uint32_t num_neg) { return 6ull * count * (num_neg + 2); }
hipError_t launch_flow_check(const TrainArgs &pool, uint64_t count, uint32_t num_neg, FlowState *state, bool fresh, uint32_t *named,
                             hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    const uint32_t *const pairs = pool.pairs, n = pool.n;
    for (uint32_t t = 0; t < flow_looked_at(count); ++t) {
        const uint64_t i = flow_look(t, count);
        CHECK(i < count && (t == 0 || i > flow_look(t - 1, count)));
        *named++ = pairs[2 * i] < n ? pairs[2 * i] : 0u;
        *named++ = n + (pairs[2 * i + 1] < n ? pairs[2 * i + 1] : 0u);
        for (uint32_t k = 0; k < num_neg; ++k) *named++ = n + draw(pool.first_g + i, k, n);
    }
    if (fresh) state->batches = state->deepest = state->stalled = 0;
    state->first_bad = UINT32_MAX;
    for (uint64_t i = count; i-- > 0;)
        if (pairs[2 * i] >= n || pairs[2 * i + 1] >= n) state->first_bad = (uint32_t)i;
    return hipGetLastError();
}
hipError_t launch_flow_prepare(FlowArgs &a, uint32_t num_neg, uint32_t *scratch, uint64_t *turns, hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    a.flow->batches += a.flow->deepest;
    a.flow->deepest = 0;
    memset(scratch, 0, flow_scratch_words(a.count, num_neg) * sizeof *scratch);
    memset(turns, 0, 2 * (size_t)a.n * sizeof *turns);
    for (uint64_t i = 0; i < a.count; ++i) {
        uint32_t *key = scratch + i * (num_neg + 2);
        key[0] = a.pairs[2 * i];
        key[1] = a.n + a.pairs[2 * i + 1];
        for (uint32_t k = 0; k < num_neg; ++k) key[2 + k] = a.n + draw(a.first_g + i, k, a.n);
    }
    a.keys = scratch;
    return hipGetLastError();
}
hipError_t launch_train_flow(FlowArgs a, uint32_t, uint32_t num_neg, hipStream_t) {
    const long left = host_allocations_left;
    host_allocations_left = -1;
    CHECK(a.flow->first_bad == UINT32_MAX);
    for (uint64_t i = 0; i < a.count; ++i) {  // one after the other
        const uint32_t *key = a.keys + i * (num_neg + 2);
        trained.push_back(Trained{levels_trained++, std::vector<uint32_t>(key, key + num_neg + 2), a.first_g + i});
    }
    a.flow->deepest = a.count;
    if (stall_next) a.flow->stalled = 1;
    stall_next = false;
    flowed += a.count;
    host_allocations_left = left;
    return hipGetLastError();
}
hipError_t launch_train_flow_tracked(FlowArgs a, uint32_t dim, uint32_t num_neg, hipStream_t s) {
    return launch_train_flow(a, dim, num_neg, s);
}
hipError_t launch_level_records(const uint32_t *pairs, const uint32_t *negatives, const uint32_t *order, uint32_t count,
                                uint32_t num_neg, uint32_t *records, hipStream_t) {
    for (uint32_t i = 0; i < count; ++i) {
        uint32_t *record = records + (size_t)i * (num_neg + 3);
        record[0] = pairs[2 * (size_t)order[i]];
        record[1] = pairs[2 * (size_t)order[i] + 1];
        for (uint32_t k = 0; k < num_neg; ++k) record[2 + k] = negatives[(size_t)order[i] * num_neg + k];
        record[2 + num_neg] = order[i];
    }
    return hipGetLastError();
}
hipError_t launch_draw_negatives(const uint4 *, uint32_t n, uint64_t, uint64_t first_g, uint64_t count, uint32_t num_neg,
                                 uint32_t *out, hipStream_t) {
    for (uint64_t i = 0; i < count; ++i)
        for (uint32_t k = 0; k < num_neg; ++k) out[i * num_neg + k] = draw(first_g + i, k, n);
    return hipGetLastError();
}
hipError_t launch_draw_negatives_partitioned(const uint4 *, const uint64_t *, const uint8_t *, const uint32_t *, uint64_t,
                                             uint64_t, uint64_t, uint32_t, uint32_t *, hipStream_t) {
    return hipGetLastError();
}
hipError_t launch_init_vertex(float *, uint64_t, uint32_t, uint64_t, hipStream_t) { return hipGetLastError(); }
hipError_t launch_eval_loss(TrainArgs a, uint32_t, uint32_t, double *partial, uint32_t *blocks, hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    *blocks = 1;
    partial[0] = 0.0;
    for (uint32_t i = 0; i < a.count; ++i) {
        if (a.pairs[2 * i] < a.n && a.pairs[2 * i + 1] < a.n) partial[0] += 0.5;
        else *a.error_flag = 1u;
    }
    return hipGetLastError();
}
hipError_t launch_cosine(const float *, uint32_t n, uint32_t, const uint32_t *first, const uint32_t *second, uint32_t count, uint32_t,
                         float *out, uint32_t *error_flag, hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    for (uint32_t i = 0; i < count; ++i) {
        out[i] = first[i] == row_without_end || second[i] == row_without_end ? INFINITY : (float)first[i] - (float)second[i];
        if (first[i] >= n || second[i] >= n) *error_flag = 1u;
    }
    return hipGetLastError();
}
uint64_t rank_scratch_words(uint32_t num_neg) { return num_neg + num_neg / 2; }
hipError_t launch_rank_sort(uint32_t *negatives, uint32_t num_neg, uint32_t *, unsigned long long *not_finite, hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    ranked_on_device = true;
    for (uint32_t b = 0; b < kRankBlocks; ++b) CHECK(not_finite[b] == 0);  // the caller clears them
    for (uint32_t j = 0; j < num_neg; ++j)
        if (((const float *)negatives)[j] == INFINITY) not_finite[j % kRankBlocks] = 1ull;
    return hipGetLastError();
}
hipError_t launch_rank_sum(const uint32_t *scores, uint32_t num_pos, uint32_t num_neg, unsigned long long *twice,
                           unsigned long long *not_finite, hipStream_t stream) {
    if (!launches(stream)) return hipErrorUnknown;
    memset(twice, 0, kRankBlocks * sizeof *twice);
    const float *positive = (const float *)scores, *negative = positive + num_pos;
    for (uint32_t i = 0; i < num_pos; ++i)
        if (positive[i] == INFINITY) not_finite[i % kRankBlocks] = 1ull;
    for (uint32_t i = 0; i < num_pos; ++i)
        for (uint32_t j = 0; j < num_neg; ++j) twice[0] += positive[i] > negative[j] ? 2u : positive[i] == negative[j] ? 1u : 0u;
    return hipGetLastError();
}
hipError_t launch_pack_steps(const uint64_t *offsets, const uint32_t *adj, uint64_t half_edges, uint4 *steps, hipStream_t) {
    for (uint64_t e = 0; e < half_edges; ++e) {
        const uint64_t begin = offsets[adj[e]];
        steps[e] = make_uint4(adj[e], (uint32_t)(offsets[adj[e] + 1] - begin), (uint32_t)begin, (uint32_t)(begin >> 32));
    }
    return hipGetLastError();
}
hipError_t launch_pack_weighted_steps(const uint64_t *offsets, const uint32_t *adj, const uint2 *nbr_table, uint32_t n,
                                      uint4 *steps, hipStream_t) {
    for (uint64_t e = 0; e < offsets[n]; ++e) {
        steps[2 * e] = make_uint4(nbr_table[e].x, adj[e], 0u, 0u);
        steps[2 * e + 1] = make_uint4(0u, 0u, 0u, 0u);
    }
    return hipGetLastError();
}
uint32_t guide_shift(uint64_t) { return 0; }
hipError_t launch_departure_guide(const uint64_t *, uint32_t, uint64_t, uint32_t *owners, hipStream_t) {
    memset(owners, 0, kGuideEntries * sizeof *owners);
    return hipGetLastError();
}
hipError_t launch_augment(const AugmentArgs &a, hipStream_t) {
    walked_weighted = a.node_table != nullptr;
    walked_packed = a.steps || a.weighted_steps;
    read_all(a.offsets, (uint64_t)a.n + 1);
    CHECK(!(a.steps && a.weighted_steps));
    if (a.node_table) {
        read_all(a.node_table, a.n);
        CHECK(!a.steps && !a.guide && (a.weighted_steps || a.nbr_table));
    } else {
        CHECK(!a.weighted_steps && !a.nbr_table);
        if (a.guide) read_all(a.guide, kGuideEntries);
    }
    if (a.weighted_steps) read_all(a.weighted_steps, 2 * a.half_edges);
    if (a.steps) read_all(a.steps, a.half_edges);
    if (!a.steps && !a.weighted_steps) read_all(a.adj, a.half_edges);
    if (a.nbr_table) read_all(a.nbr_table, a.half_edges);
    return hipGetLastError();
}
}  // namespace gv

// ---------------------------------------------------------------------------------------------------- checks
namespace {
gv_config configuration(uint32_t mode, uint32_t num_neg, uint32_t schedule) {
    gv_config cfg{};
    cfg.dim = 32;
    cfg.num_neg = num_neg;
    cfg.lr0 = 0.025f;
    cfg.neg_weight = GV_NEG_WEIGHT_DEFAULT;
    cfg.mode = mode;
    cfg.total_samples = 1000000;
    cfg.pool_capacity = 8;
    cfg.coherence = GV_COHERENCE_MIXED;
    cfg.schedule = schedule;
    return cfg;
}
gv_ctx *context(uint32_t mode, uint32_t num_neg, uint32_t schedule = GV_SCHEDULE_AUTO) {
    const gv_config cfg = configuration(mode, num_neg, schedule);
    gv_ctx *ctx = nullptr;
    CHECK(gv_create(&cfg, &ctx) == GV_OK);
    return ctx;
}

std::vector<uint32_t> random_pool(uint32_t n, uint32_t count, uint32_t seed) {
    std::vector<uint32_t> pool(2 * (size_t)count);
    for (size_t i = 0; i < pool.size(); ++i) pool[i] = draw(i + 1, seed, n);
    return pool;
}

// `count` samples from position g were trained in conflict-free levels that keep the order of samples sharing a row.
void check_levels(const std::vector<uint32_t> &pool, uint64_t g, uint32_t n, uint32_t num_neg) {
    const uint64_t count = pool.size() / 2;
    CHECK(trained.size() == count);
    std::vector<bool> seen(count, false);
    std::map<uint32_t, const Trained *> last;
    for (const Trained &t : trained) {
        const uint64_t i = t.place - g;
        CHECK(i < count && !seen[i]);
        seen[i] = true;
        CHECK(t.rows[0] == pool[2 * i] && t.rows[1] == n + pool[2 * i + 1]);
        for (uint32_t k = 0; k < num_neg; ++k) CHECK(t.rows[2 + k] == n + draw(t.place, k, n));
        for (uint32_t row : t.rows) {
            const Trained *before = last.count(row) ? last[row] : nullptr;
            CHECK(!before || before == &t || (before->level < t.level && before->place < t.place));
            last[row] = &t;
        }
    }
    trained.clear();
}

// Deterministic mode: a call that runs out of host memory, wherever it does, reports it and leaves nothing behind.
void levels_after_failed_allocations(uint32_t count, int at_least) {
    const uint32_t n = 200, K = 2;
    const std::vector<uint32_t> degrees(n, 3), first = random_pool(n, count, 1), second = random_pool(n, count, 2);
    int failures = 0;
    for (long at = 0;; ++at) {
        gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        host_allocations_left = at;
        const int rc = gv_train_device_pool(ctx, first.data(), count);
        const bool done = host_allocations_left >= 0;  // nothing was left to fail
        host_allocations_left = -1;
        CHECK(rc == GV_OK || rc == GV_ENOMEM);
        uint64_t g = 0;
        if (rc == GV_OK) {
            check_levels(first, 0, n, K);
            g = count;
        }
        failures += rc != GV_OK;
        CHECK(trained.empty());
        CHECK(gv_train_device_pool(ctx, second.data(), count) == GV_OK);
        check_levels(second, g, n, K);
        CHECK(gv_train_device_pool(ctx, first.data(), count) == GV_OK);
        check_levels(first, g + count, n, K);
        gv_destroy(ctx);
        if (done) break;
    }
    CHECK(failures >= at_least);
}
void levels_after_failed_allocations() {
    levels_after_failed_allocations(300, 2);   // through the pinned stage: the levels of either matrix
    levels_after_failed_allocations(4000, 3);  // through arrays of its own
}

// A pool of more than one part is trained in order, with no more scratch than one part has, and a bad id at its end is
// found before any of it is trained.
void pools_in_parts() {
    const uint32_t n = 100000, K = 2, part = 1u << 20;
    const std::vector<uint32_t> degrees(n, 3);
    gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
    CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
    device_largest = (size_t)part * (K + 3) * sizeof(uint32_t);
    uint64_t g = 0;
    for (uint32_t count : {part + 12345u, 1000u, part, part + 1u}) {
        std::vector<uint32_t> pool = random_pool(n, count, count);
        pool[2 * count - 1] = n;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_EINVAL && trained.empty());
        pool[2 * count - 1] = 0;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK);
        check_levels(pool, g, n, K);
        g += count;
    }
    device_largest = SIZE_MAX;
    gv_destroy(ctx);
}

// Pools that are not short wait for each other on the device where that finds memory, and are levelled on the host where
// it does not, or where the hottest row is named by many; a bad id is found before any sample is trained; the batches of
// either way are counted.
void flowing_pools() {
    const uint32_t n = 2000, K = 2, count = 5000;
    const std::vector<uint32_t> degrees(n, 3), pool = random_pool(n, count, 1);
    std::vector<uint32_t> bad = pool;
    bad[2 * 4321 + 1] = n;
    uint64_t levelled = 0;
    for (long at = 0;; ++at) {
        gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        device_allocations_left = at;
        flowed = 0;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK);
        const bool done = device_allocations_left >= 0;
        device_allocations_left = -1;
        CHECK(flowed == (done ? count : 0));  // a node's or a sample's words do not fit: levels
        levelled += flowed == 0;
        check_levels(pool, 0, n, K);
        CHECK(gv_train_device_pool(ctx, bad.data(), count) == GV_EINVAL && trained.empty());
        CHECK(strstr(gv_last_error(ctx), "sample 4321 names node id >= n"));
        flowed = 0;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && flowed == count);
        check_levels(pool, count, n, K);
        gv_stats stats;
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.batches >= count && stats.samples_trained == 2 * count);
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && gv_sync(ctx) == GV_OK);
        const uint64_t before = stats.batches;
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.batches == before + count);
        trained.clear();
        // a graph anew
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && gv_sync(ctx) == GV_OK);
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.batches == before + 2 * count);
        trained.clear();
        gv_destroy(ctx);
        if (done) break;
    }
    CHECK(levelled == 2);
    // shorter, on a hub, and where the nodes' words would take more than an eighth of the memory that is left
    std::vector<uint32_t> star(n, 1);
    star[7] = n;
    for (int which = 0; which < 3; ++which) {
        gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
        CHECK(gv_set_degrees(ctx, n, which == 1 ? star.data() : degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        device_free = which == 2 ? 8 * 16 * n - 1 : SIZE_MAX;
        flowed = 0;
        CHECK(gv_train_device_pool(ctx, pool.data(), which == 0 ? 4096 : count) == GV_OK && flowed == 0);
        device_free = SIZE_MAX;
        trained.clear();
        gv_destroy(ctx);
    }
}

// Pools whose levels are narrow are levelled, whatever the degrees of the graph: walks in their own order, and a row that one
// sample in ten names; the same walks shuffled, a row that one sample in forty names, and a long pool of random pairs are not.
void narrow_pools() {
    const uint32_t n = 20000, K = 1, count = 30000, length = 40, window = 5;
    const std::vector<uint32_t> degrees(n, 3);
    std::vector<uint32_t> walks;
    for (uint32_t w = 0; walks.size() < 2 * count; ++w) {
        uint32_t walk[length];
        for (uint32_t i = 0; i < length; ++i) walk[i] = draw(w * 64ull + i, 3, 40) < 36 ? draw(w * 64ull + i, 5, n) : draw(w * 64ull + i, 7, 50);
        for (uint32_t i = 0; i < length; ++i)
            for (uint32_t j = i + 1; j < std::min(i + window + 1, length); ++j) walks.insert(walks.end(), {walk[i], walk[j]});
    }
    walks.resize(2 * count);
    std::vector<uint32_t> shuffled;
    for (uint32_t b = 0; b < window; ++b)
        for (uint32_t i = b; i < count; i += window) shuffled.insert(shuffled.end(), {walks[2 * i], walks[2 * i + 1]});
    auto planted = [&](uint32_t one_in) {
        std::vector<uint32_t> pool = random_pool(n, count, 9);
        for (uint32_t i = 0; i < count; ++i)
            if (draw(i, 11, one_in) == 0) pool[2 * i] = 7;
        return pool;
    };
    const std::vector<uint32_t> tenth = planted(10), fortieth = planted(40), random = random_pool(n, 9 * count, 2);
    struct Pool {
        const std::vector<uint32_t> &pairs;
        bool flows;
    };
    gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
    CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
    uint64_t g = 0;
    for (const Pool &p : {Pool{walks, false}, Pool{shuffled, true}, Pool{tenth, false}, Pool{fortieth, true}, Pool{random, true}}) {
        for (uint32_t way : {0u, 1u, 2u}) {
            flowed = 0;
            CHECK(gv_test_force_way(ctx, way) == GV_OK);
            CHECK(gv_train_device_pool(ctx, p.pairs.data(), p.pairs.size() / 2) == GV_OK);
            CHECK(flowed == ((way ? way == 1 : p.flows) ? p.pairs.size() / 2 : 0));
            check_levels(p.pairs, g, n, K);
            g += p.pairs.size() / 2;
        }
    }
    gv_destroy(ctx);
    // without host memory for the look at the first pool, that one waits on the device
    ctx = context(GV_MODE_DETERMINISTIC, K);
    CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
    flowed = 0;
    host_allocations_left = 0;
    CHECK(gv_train_device_pool(ctx, walks.data(), count) == GV_OK && flowed == count && host_allocations_left == -1);
    check_levels(walks, 0, n, K);
    CHECK(gv_train_device_pool(ctx, walks.data(), count) == GV_OK && flowed == count);
    check_levels(walks, count, n, K);
    gv_destroy(ctx);
}

// A pool that was not trained to its end is reported once, by the next call that synchronises, not by gv_get_stats; it hides
// no other report for longer than that, does not stop calls that begin anew, and the batches of pools behind it are counted.
void pools_that_give_up() {
    const uint32_t n = 2000, K = 2, count = 5000;
    const std::vector<uint32_t> degrees(n, 3), pool = random_pool(n, count, 1);
    std::vector<uint32_t> bad(pool.begin(), pool.begin() + 20);
    bad[3] = n;
    gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
    CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
    double loss = 0.0;
    gv_stats stats;
    for (int which = 0; which < 4; ++which) {
        stall_next = true;
        memset(&stats, 0xFF, sizeof stats);
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK);
        const uint64_t trained_so_far = (uint64_t)(3 * which + 1) * count;
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.samples_trained == trained_so_far && stats.batches == trained_so_far);
        if (which == 0) CHECK(gv_sync(ctx) == GV_ESTATE && strstr(gv_last_error(ctx), "not trained to its end"));
        if (which == 1) CHECK(gv_eval_loss(ctx, bad.data(), 10, 7, &loss) == GV_ESTATE && strstr(gv_last_error(ctx), "not trained to its end"));
        if (which == 2) CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        if (which == 3) CHECK(gv_init_embeddings(ctx, 5) == GV_OK);
        CHECK(gv_eval_loss(ctx, pool.data(), 10, 7, &loss) == GV_OK && gv_sync(ctx) == GV_OK);
        for (int again = 0; again < 2; ++again) {
            CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK);
            if (again == which % 2) CHECK(gv_sync(ctx) == GV_OK);
        }
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.batches == trained_so_far + 2 * count && gv_sync(ctx) == GV_OK);
        trained.clear();
    }
    gv_destroy(ctx);
}

// A wave that waits for a turn gives up where nothing of the pool gets on, and there within a bounded number of looks; not for as
// long as the chain that it waits for gets on, however long that is: here 2^20 links of 10 us, which are counted 64 at a time,
// while the wave looks every 130 ns, and the samples taken stand still.
void patience_of_waiting() {
    constexpr double kLook = 0.13, kLink = 10.0;  // us
    constexpr uint64_t kLinks = 1u << 20;
    gv::FlowPatience patience;
    uint64_t look = 0;
    for (; (double)look * kLook < (double)kLinks * kLink; ++look) {
        const uint64_t links = (uint64_t)((double)look * kLook / kLink);
        CHECK(!patience.ends([&] { return 4711u + (uint32_t)(links / 64u); }));
    }
    uint32_t in_vain = 0;
    while (!patience.ends([&] { return 4711u + (uint32_t)(kLinks / 64u); })) CHECK(++in_vain < 1u << 23);
    CHECK(in_vain >= 1u << 21);
    // nothing from the first look on
    gv::FlowPatience fresh;
    in_vain = 0;
    while (!fresh.ends([] { return 0u; })) CHECK(++in_vain < 1u << 23);
    CHECK(in_vain >= (1u << 22) - 1);
}

// Where the words of a sample do not fit, in whole or beside what is there, a second pool of the same size changes nothing on the
// device, and nothing is held for the way that was refused; where they fit in the place of the old ones, they take it.
void refused_scratch() {
    const uint32_t n = 2000, K = 2, count = 5000;
    const std::vector<uint32_t> degrees(n, 3), pool = random_pool(n, count, 1);
    const size_t levels = (size_t)count * (K + 3) * sizeof(uint32_t), waiting = 6 * (size_t)count * (K + 2) * sizeof(uint32_t);
    for (int which = 0; which < 3; ++which) {
        gv_ctx *ctx = context(GV_MODE_DETERMINISTIC, K);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        flowed = 0;
        if (which == 0) device_largest = waiting - 1;
        else device_free = waiting - levels - 1;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && flowed == 0);
        const uint64_t allocations = device_allocations, frees = device_frees;
        CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && flowed == 0);
        CHECK(device_allocations == allocations && device_frees == frees);
        if (which == 2) {
            device_free = waiting - levels;
            CHECK(gv_train_device_pool(ctx, pool.data(), count) == GV_OK && flowed == count);
            CHECK(device_allocations == allocations + 2 && device_frees == frees + 1);
        }
        device_largest = device_free = SIZE_MAX;
        trained.clear();
        gv_destroy(ctx);
    }
}

// A launch that fails, wherever it stands in an evaluation or a deterministic pool, leaves no kernel behind that uses the pinned
// memory of the context, and the next call is whole.
void early_ends() {
    const uint32_t n = 2000, count = 300000;
    const std::vector<uint32_t> degrees(n, 3), pool = random_pool(n, count, 1), other = random_pool(n, 20, 2);
    for (uint32_t mode : {GV_MODE_HOGWILD, GV_MODE_DETERMINISTIC}) {
        gv_ctx *ctx = context(mode, 1);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        for (uint32_t pairs : {1000u, count})
            for (int which = 0; which < (mode == GV_MODE_DETERMINISTIC ? 3 : 2); ++which) {
                double got = -1.0, whole = -1.0;
                auto call = [&](double *result) -> int {
                    if (which == 0) return gv_eval_loss(ctx, pool.data(), pairs, 7, result);
                    if (which == 1)
                        return gv_link_prediction_auc(ctx, pool.data(), pool.data() + pairs, pairs, other.data(), other.data() + 20, 20,
                                                      result);
                    *result = whole;
                    return gv_train_device_pool(ctx, pool.data(), 5000);
                };
                CHECK(call(&whole) == GV_OK && gv_sync(ctx) == GV_OK && using_pinned.empty());
                int failures = 0;
                for (long at = 0;; ++at) {
                    launches_left = at;
                    const int rc = call(&got);
                    const bool done = launches_left >= 0;
                    launches_left = -1;
                    if (done) break;
                    CHECK(rc == GV_EHIP && using_pinned.empty());
                    CHECK(call(&got) == GV_OK && got == whole && gv_sync(ctx) == GV_OK);
                    ++failures;
                }
                CHECK(failures >= (which == 0 && pairs == 1000 ? 1 : 2));
                trained.clear();
            }
        gv_destroy(ctx);
    }
}

// A graph of a ring with chords: every node has its two neighbours and the nodes two steps away.
struct Ring {
    static constexpr uint32_t n = 50;
    std::vector<uint64_t> offsets;
    std::vector<uint32_t> degrees, adj;
    std::vector<float> weights;
    Ring() : degrees(n, 4) {
        for (uint32_t i = 0; i <= n; ++i) offsets.push_back(4ull * i);
        for (uint32_t i = 0; i < n; ++i)
            for (uint32_t step : {1u, 2u, n - 1u, n - 2u}) {
                adj.push_back((i + step) % n);
                weights.push_back(1.0f + (float)(step % 3u));
            }
    }
};

// A weighted graph that runs out of device memory, wherever it does, leaves nothing that a later graph without weights
// would be walked by; the device producer reads the tables of the graph that was taken last, whole.
void walks_after_failed_allocations() {
    const Ring ring;
    std::vector<uint32_t> pairs(2 * 1000);
    uint64_t walks = 0;
    auto walk = [&](gv_ctx *ctx) {
        return gv_augment_device(ctx, 1, 5, 2, 0, 1000, GV_SHUFFLE_NONE, pairs.data(), &walks);
    };
    int refused = 0, taken = 0;
    for (long at = 0;; ++at) {
        gv_ctx *ctx = context(GV_MODE_HOGWILD, 1);
        device_allocations_left = at;
        const int rc = gv_set_weighted_graph(ctx, ring.n, ring.offsets.data(), ring.adj.data(), ring.weights.data());
        const bool done = device_allocations_left >= 0;
        device_allocations_left = -1;
        CHECK(rc == GV_OK || rc == GV_ENOMEM);
        refused += rc != GV_OK;
        if (rc == GV_OK) {
            CHECK(walk(ctx) == GV_OK && walked_weighted);
        } else {
            CHECK(walk(ctx) == GV_ESTATE);
            const int next = gv_set_adjacency(ctx, ring.offsets.data(), ring.adj.data());
            CHECK(next == GV_OK || next == GV_ESTATE);  // no graph yet, or one that knows its degrees
            taken += next == GV_OK;
            if (next == GV_OK) CHECK(walk(ctx) == GV_OK && !walked_weighted);
            CHECK(gv_set_weighted_graph(ctx, ring.n, ring.offsets.data(), ring.adj.data(), ring.weights.data()) == GV_OK);
            CHECK(walk(ctx) == GV_OK && walked_weighted);
        }
        CHECK(gv_set_degrees(ctx, ring.n, ring.degrees.data()) == GV_OK && walk(ctx) == GV_ESTATE);
        CHECK(gv_set_adjacency(ctx, ring.offsets.data(), ring.adj.data()) == GV_OK && walk(ctx) == GV_OK && !walked_weighted);
        gv_destroy(ctx);
        if (done) break;
    }
    CHECK(refused == 9 && taken >= 4);  // for want of the matrices and node tables (5) and the adjacency with its tables (4)
    // the same of a graph without weights: all but the adjacency itself can be done without
    refused = 0;
    for (long at = 0;; ++at) {
        gv_ctx *ctx = context(GV_MODE_HOGWILD, 1);
        CHECK(gv_set_degrees(ctx, ring.n, ring.degrees.data()) == GV_OK);
        device_allocations_left = at;
        const int rc = gv_set_adjacency(ctx, ring.offsets.data(), ring.adj.data());
        const bool done = device_allocations_left >= 0;
        device_allocations_left = -1;
        CHECK(rc == GV_OK || rc == GV_ENOMEM);
        refused += rc != GV_OK;
        CHECK(walk(ctx) == (rc == GV_OK ? GV_OK : GV_ESTATE));
        CHECK(gv_set_adjacency(ctx, ring.offsets.data(), ring.adj.data()) == GV_OK && walk(ctx) == GV_OK && !walked_weighted);
        gv_destroy(ctx);
        if (done) break;
    }
    CHECK(refused == 2);
}

// What training has to report comes first, whatever the evaluation call that waits for it was given, and the call's own
// bad ids are reported by the next call that names them.
void reports_of_evaluation() {
    const std::vector<uint32_t> degrees(10, 3), good = {0, 1, 2, 3}, bad = {0, 1, 2, 10}, other = {4, 5};
    gv_ctx *ctx = context(GV_MODE_HOGWILD, 1);
    CHECK(gv_set_degrees(ctx, 10, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
    double result = 0.0;
    auto loss = [&](const std::vector<uint32_t> &pairs) {
        result = -1.0;
        return gv_eval_loss(ctx, pairs.data(), 2, 1, &result);
    };
    auto auc = [&](const std::vector<uint32_t> &pairs) {
        result = -1.0;
        return gv_link_prediction_auc(ctx, pairs.data(), pairs.data() + 2, 2, other.data(), other.data() + 1, 1, &result);
    };
    for (int word : {0, 1}) {
        const int code = word == 0 ? GV_EINVAL : GV_ESTATE;
        auto train = [&] {
            training_reports = word;
            CHECK(gv_train_device_pool(ctx, good.data(), 2) == GV_OK);
        };
        train();
        CHECK(loss(bad) == code && result == -1.0);
        CHECK(loss(bad) == GV_EINVAL && result == 0.25);  // of the pairs whose ids are nodes
        CHECK(loss(good) == GV_OK && result == 0.5);
        train();
        CHECK(loss(good) == code && result == -1.0 && loss(good) == GV_OK);
        train();
        CHECK(auc(bad) == code && auc(bad) == GV_EINVAL && result == -1.0 && auc(good) == GV_OK);
        train();
        CHECK(auc(good) == code && auc(good) == GV_OK && gv_sync(ctx) == GV_OK);
        float scores[2];
        train();
        CHECK(gv_cosine(ctx, bad.data(), bad.data() + 2, 2, scores) == code);
        CHECK(gv_cosine(ctx, bad.data(), bad.data() + 2, 2, scores) == GV_EINVAL && gv_sync(ctx) == GV_OK);
    }
    gv_destroy(ctx);
}

// Every kind of pool against the plan that it is meant to get, and what the launches rely on for pools of all sizes.
void plans_of_pools() {
    using gv::AsyncPlan;
    using gv::AsyncPool;
    constexpr uint32_t agent = gv::kAgent, atomic = gv::kAtomicAgent, mixed = gv::kMixed;
    struct Expected {
        const char *what;
        AsyncPool pool;  // samples, n, dim, K, policy, tiled schedule, may skip tiles, block, warm rows, hottest share
        AsyncPlan plan;  // tiles, policy, samples to a tile or wave, workgroups, exchange every
    };
    const Expected all[] = {
        {"a pool that fills the chip", {1 << 24, 1000000, 128, 1, mixed, true, true, false, 15000, 0.011}, {true, mixed, 8192, 2048, 4}},
        {"long rows", {1 << 22, 1000000, 512, 5, mixed, true, true, false, 8000, 0.011}, {true, mixed, 8192, 512, 2}},
        {"rows of 64 floats", {1 << 24, 1000000, 64, 1, mixed, true, true, false, 15000, 0.011}, {true, mixed, 4096, 4096, 4}},
        {"too few tiles of 8192 to fill the chip", {3000000, 1000000, 128, 1, mixed, true, true, false, 15000, 0.011}, {true, mixed, 4096, 733, 4}},
        {"short enough for atomic adds, hubs", {1 << 20, 1000000, 64, 2, mixed, true, true, false, 15000, 0.011}, {true, atomic, 1024, 1024, 4}},
        {"the same, few hubs", {1000003, 200003, 96, 3, mixed, true, true, false, 30000, 0.01}, {false, atomic, 16, 256, 0}},
        {"a few thousand samples", {4096, 100000, 128, 1, mixed, true, true, false, 20000, 0.005}, {false, atomic, 4, 256, 0}},
        {"a small graph, all rows warm", {2000000, 10000, 128, 1, mixed, true, true, false, 10000, 0.006}, {false, atomic, 16, 156, 0}},
        {"short pool, hubs", {65536, 100000, 64, 1, mixed, true, true, false, 20000, 0.035}, {true, atomic, 64, 390, 4}},
        {"shorter pool, hubs", {8192, 100000, 64, 1, mixed, true, true, false, 20000, 0.035}, {true, atomic, 16, 390, 4}},
        {"short pool, hubs, fewer nodes", {65536, 30000, 64, 2, mixed, true, true, false, 20000, 0.03}, {true, atomic, 64, 256, 4}},
        {"tiles asked for", {4099, 300000, 128, 1, mixed, true, false, false, 60000, 0.0001}, {true, atomic, 16, 257, 4}},
        {"tiles and stores asked for", {100000, 100000, 128, 1, agent, true, false, false, 20000, 0.01}, {true, agent, 8192, 13, 4}},
        {"tiles and atomic adds asked for", {1 << 24, 1000000, 128, 1, atomic, true, false, false, 15000, 0.011}, {true, atomic, 8192, 2048, 4}},
        {"one of 8 x 8 blocks, hubs", {1 << 21, 1000000, 128, 1, mixed, true, true, true, 65535, 0.145}, {true, mixed, 8192, 256, 2}},
        {"one of 2 x 2 blocks, hubs", {1 << 25, 1000000, 128, 1, mixed, true, true, true, 65535, 0.036}, {true, mixed, 8192, 4096, 2}},
        {"one of 8 x 8 blocks, few hubs", {1 << 21, 1000000, 64, 1, mixed, true, true, true, 65535, 0.028}, {true, mixed, 8192, 256, 4}},
        {"one of 2 x 2 blocks, few hubs", {1 << 25, 1000000, 64, 1, mixed, true, true, true, 65535, 0.007}, {true, mixed, 8192, 4096, 4}},
        {"a block with long rows", {1 << 18, 1000000, 256, 1, mixed, true, true, true, 65535, 0.007}, {true, mixed, 8192, 32, 2}},
        {"no warm row", {1 << 22, 4000000, 128, 1, agent, false, true, false, 0, 0.0}, {false, agent, 64, 2048, 0}},
        {"pool order and atomic adds asked for", {1 << 24, 1000000, 128, 1, atomic, false, false, false, 15000, 0.011}, {false, atomic, 64, 2048, 0}},
    };
    for (const Expected &e : all) {
        const AsyncPlan got = gv::async_plan(e.pool), &want = e.plan;
        const bool same = got.tiled == want.tiled && got.coherence == want.coherence && got.unit == want.unit &&
                          got.blocks == want.blocks && got.exchange_every == want.exchange_every;
        if (!same)
            fprintf(stderr, "%s: {%d, %u, %u, %u, %u}\n", e.what, got.tiled, got.coherence, got.unit, got.blocks, got.exchange_every);
        CHECK(same);
    }
    for (uint32_t n : {2u, 100u, 10000u, 65535u, 65536u, 300000u, 1000000u, 66000000u, 0x80000000u})
        for (uint32_t dim : {32u, 64u, 128u, 160u, 512u})
            for (uint32_t K : {1u, 2u, 5u})
                for (uint64_t count : {1ull, 15ull, 4096ull, 100003ull, 1000000ull, 3000000ull, 1ull << 24, 1ull << 31})
                    for (uint32_t policy : {(uint32_t)gv::kPlain, agent, atomic, mixed})
                        for (int flags = 0; flags < 8; ++flags)
                            for (double share : {0.0, 0.01, 1.0}) {
                                const bool tiled = flags & 1, skip = flags & 2, block = flags & 4;
                                const AsyncPlan p = gv::async_plan(AsyncPool{count, n, dim, K, policy, tiled, skip, block,
                                                                            std::min(n, 65535u) / 2u, share});
                                CHECK(p.blocks >= 1 && p.blocks <= (count + p.unit - 1) / p.unit);
                                CHECK(tiled || !p.tiled);                       // pool order is never left
                                CHECK(p.tiled || !tiled || (skip && policy == mixed));  // tiles only where they may be
                                CHECK(p.coherence == policy || p.coherence == atomic);  // no update is lost that was kept
                                if (p.tiled) {
                                    CHECK(p.unit >= gv::kSmallestTile && p.unit <= gv::kLargestTile && !(p.unit & (p.unit - 1)));
                                    CHECK(p.unit == gv::kLargestTile || p.coherence == atomic ||  // the instantiations there are
                                          (p.coherence == mixed && gv::short_rows(gv::floats_per_lane(dim), (int)K)));
                                    CHECK(p.exchange_every == 2 || p.exchange_every == 4);
                                } else {
                                    CHECK(p.unit >= 1 && p.unit <= 64);
                                    CHECK(policy != agent || p.coherence == agent);
                                }
                            }
}

// gv_stats.tiled_launches counts the launches of the tiled kernel, whatever the schedule of the graph.
void counted_launches() {
    const uint32_t n = 20000;
    std::vector<uint32_t> degrees(n, 3), pool = random_pool(n, 400000, 3);
    degrees[7] = 3000;  // a few percent of the samples name it
    struct Expected {
        uint32_t schedule, hub;
        uint64_t count;
        bool tiled;
    };
    for (const Expected &e : {Expected{GV_SCHEDULE_AUTO, 3000, 400000, true}, Expected{GV_SCHEDULE_AUTO, 3, 400000, false},
                              Expected{GV_SCHEDULE_AUTO, 3000, 100, false}, Expected{GV_SCHEDULE_TILED, 3, 100, true},
                              Expected{GV_SCHEDULE_POOL_ORDER, 3000, 400000, false}}) {
        degrees[7] = e.hub;
        gv_ctx *ctx = context(GV_MODE_HOGWILD, 1, e.schedule);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        training_reports = -1;
        tiled_launched = false;
        CHECK(gv_train_device_pool(ctx, pool.data(), e.count) == GV_OK);
        gv_stats stats;
        CHECK(gv_get_stats(ctx, &stats) == GV_OK && stats.train_launches == 1);
        CHECK(tiled_launched == e.tiled && stats.tiled_launches == (e.tiled ? 1u : 0u));
        gv_destroy(ctx);
    }
    // the tests' own choice of the tile: sizes that there are kernels for, where the schedule walks in tiles at all
    for (uint32_t schedule : {GV_SCHEDULE_TILED, GV_SCHEDULE_POOL_ORDER}) {
        gv_ctx *ctx = context(GV_MODE_HOGWILD, 1, schedule);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK && gv_build_alias(ctx, 0.75) == GV_OK);
        for (uint32_t bad : {1u, 8u, 4095u, 16384u}) CHECK(gv_test_force_tile(ctx, bad) == GV_EINVAL);
        for (uint32_t tile : {16u, 4096u, 8192u}) {
            CHECK(gv_test_force_tile(ctx, tile) == GV_OK && gv_train_device_pool(ctx, pool.data(), 100) == GV_OK);
            CHECK(launched_unit == (schedule == GV_SCHEDULE_TILED ? tile : 64u));
        }
        CHECK(gv_test_force_tile(ctx, 0) == GV_OK && gv_train_device_pool(ctx, pool.data(), 100000) == GV_OK);
        CHECK(launched_unit == 64u);
        gv_destroy(ctx);
    }
}

// The packed adjacency takes no more than an eighth of the device memory that is left.
void packed_walks_leave_room() {
    const Ring ring;
    std::vector<uint32_t> pairs(2 * 1000);
    uint64_t walks = 0;
    for (bool weighted : {false, true}) {
        const size_t packed = ring.adj.size() * (weighted ? 32 : 16);
        for (size_t left : {8 * packed, 8 * packed - 8}) {
            gv_ctx *ctx = context(GV_MODE_HOGWILD, 1);
            device_free = left;
            if (weighted) {
                CHECK(gv_set_weighted_graph(ctx, ring.n, ring.offsets.data(), ring.adj.data(), ring.weights.data()) == GV_OK);
            } else {
                CHECK(gv_set_degrees(ctx, ring.n, ring.degrees.data()) == GV_OK);
                CHECK(gv_set_adjacency(ctx, ring.offsets.data(), ring.adj.data()) == GV_OK);
            }
            device_free = SIZE_MAX;
            CHECK(gv_augment_device(ctx, 1, 5, 2, 0, 1000, GV_SHUFFLE_NONE, pairs.data(), &walks) == GV_OK);
            CHECK(walked_weighted == weighted && walked_packed == (left == 8 * packed));
            gv_destroy(ctx);
        }
    }
}

// A context that was refused for want of memory, wherever it ran out, does not spoil the next one.
void contexts_after_failed_allocations() {
    const std::vector<uint32_t> degrees(10, 3);
    for (long at = 0;; ++at) {
        gv_config cfg = configuration(GV_MODE_HOGWILD, 1, GV_SCHEDULE_AUTO);
        cfg.track_loss = 1;
        gv_ctx *ctx = nullptr;
        device_allocations_left = at;
        const int rc = gv_create(&cfg, &ctx);
        const bool done = device_allocations_left >= 0;
        device_allocations_left = -1;
        CHECK(rc == (done ? GV_OK : GV_ENOMEM) && (ctx != nullptr) == done);
        if (!ctx) ctx = context(GV_MODE_HOGWILD, 1);
        CHECK(gv_set_degrees(ctx, 10, degrees.data()) == GV_OK && gv_init_embeddings(ctx, 1) == GV_OK);
        gv_destroy(ctx);
        if (done) break;
    }
}

// Link prediction ranks few pairs on the host, more on the device, and more on the host where the device has no memory
// left for it: the same result all ways.
void ranking_where_it_can_be_done() {
    const uint32_t n = 100;
    const std::vector<uint32_t> degrees(n, 3);
    struct Expected {
        uint32_t edges, others;
        size_t largest;
        bool on_device;
    };
    for (const Expected &e : {Expected{1, 1, SIZE_MAX, false}, Expected{2048, 2048, SIZE_MAX, false},
                              Expected{2049, 2048, SIZE_MAX, true}, Expected{3000, 4000, SIZE_MAX, true},
                              Expected{3000, 4000, 51999, false}, Expected{3000, 4000, 52000, true},
                              Expected{4000, 3000, 46000, true}, Expected{100, 4000, 40400, true}, Expected{4000, 4000, 48000, false}}) {
        gv_ctx *ctx = context(GV_MODE_HOGWILD, 1);
        CHECK(gv_set_degrees(ctx, n, degrees.data()) == GV_OK);
        const std::vector<uint32_t> edges = random_pool(n, e.edges, 5), others = random_pool(n, e.others, 6);
        std::vector<uint32_t> ends[4];
        for (uint32_t i = 0; i < e.edges; ++i) ends[0].push_back(edges[2 * i]), ends[1].push_back(edges[2 * i + 1]);
        for (uint32_t i = 0; i < e.others; ++i) ends[2].push_back(others[2 * i]), ends[3].push_back(others[2 * i + 1]);
        double wins = 0.0, got = -1.0;
        for (uint32_t i = 0; i < e.edges; ++i)
            for (uint32_t j = 0; j < e.others; ++j) {
                const float a = (float)ends[0][i] - (float)ends[1][i], b = (float)ends[2][j] - (float)ends[3][j];
                wins += a > b ? 1.0 : a == b ? 0.5 : 0.0;
            }
        ranked_on_device = false;
        device_largest = e.largest;
        const int rc = gv_link_prediction_auc(ctx, ends[0].data(), ends[1].data(), e.edges, ends[2].data(), ends[3].data(),
                                              e.others, &got);
        device_largest = SIZE_MAX;
        CHECK(rc == GV_OK && got == wins / ((double)e.edges * e.others) && ranked_on_device == e.on_device);
        // a row that is not finite among the edges, among the others: refused, and the next call is not
        for (int set : {1, 3}) {
            const uint32_t node = ends[set].back();
            row_without_end = ends[set].back() = n - 1;
            for (std::vector<uint32_t> &all : ends) std::replace(all.begin(), &all == &ends[set] ? all.end() - 1 : all.end(), n - 1, n - 2);
            auto auc = [&] {
                return gv_link_prediction_auc(ctx, ends[0].data(), ends[1].data(), e.edges, ends[2].data(), ends[3].data(), e.others, &got);
            };
            CHECK(auc() == GV_EINVAL && auc() == GV_EINVAL);
            ends[set].back() = std::min(node, n - 2);
            CHECK(auc() == GV_OK);
        }
        row_without_end = UINT32_MAX;
        gv_ctx *full = context(GV_MODE_HOGWILD, 1);
        float scores[1];
        CHECK(gv_set_degrees(full, n, degrees.data()) == GV_OK);
        // not even for the cosines of the larger set; few pairs need none
        device_largest = std::min<size_t>(12 * std::max(e.edges, e.others), 4 * (e.edges + e.others + ((gv::rank_scratch_words(e.others) + 3) & ~3ull))) - 1;
        const bool few = e.edges + e.others <= 4096;
        const uint64_t allocations = device_allocations;
        CHECK(gv_link_prediction_auc(full, ends[0].data(), ends[1].data(), e.edges, ends[2].data(), ends[3].data(), e.others,
                                     &got) == (few ? GV_OK : GV_ENOMEM));
        CHECK(!few || device_allocations == allocations);
        device_largest = SIZE_MAX;
        CHECK(gv_cosine(full, ends[0].data(), ends[1].data(), 1, &scores[0]) == GV_OK);  // the failure is not reported again
        gv_destroy(full);
        gv_destroy(ctx);
    }
}
}  // namespace

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> checks = {
        {"contexts after failed allocations", contexts_after_failed_allocations},
        {"levels after failed allocations", levels_after_failed_allocations},
        {"flowing pools", flowing_pools},
        {"narrow pools", narrow_pools},
        {"patience of waiting", patience_of_waiting},
        {"pools that give up", pools_that_give_up},
        {"refused scratch", refused_scratch},
        {"early ends", early_ends},
        {"pools in parts", pools_in_parts},
        {"walks after failed allocations", walks_after_failed_allocations},
        {"packed walks leave room", packed_walks_leave_room},
        {"reports of evaluation", reports_of_evaluation},
        {"plans of pools", plans_of_pools},
        {"counted launches", counted_launches},
        {"ranking where it can be done", ranking_where_it_can_be_done},
    };
    if (argc != 2 || !checks.count(argv[1])) return 2;
    checks.at(argv[1])();
    printf("host device driver: all checks passed\n");
    return 0;
}
