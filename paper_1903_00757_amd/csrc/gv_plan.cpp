// Launch shapes of asynchronous training: which kernel, how many samples to a workgroup or a wave, how many workgroups.
// Host code without a call to the device.
#include <math.h>

#include <algorithm>

#include "gv_internal.hpp"

namespace gv {

// the smallest V in {1, 2, 4, 8} with 64 V >= dim: floats of a row that a lane holds
int floats_per_lane(uint32_t dim) { return dim <= 64 ? 1 : (dim <= 128 ? 2 : (dim <= 256 ? 4 : 8)); }

uint32_t samples_per_batch(uint32_t dim, uint32_t num_neg) { return (uint32_t)tiled_batch(floats_per_lane(dim), (int)num_neg); }

bool supported_shape(uint32_t dim, uint32_t num_neg) {
    return dim >= 32 && dim <= 512 && dim % 32 == 0 && num_neg >= 1 && num_neg <= 5;
}

// Shape of an asynchronous launch.
//
// A pool that fills the chip with tiles of 8192 is bound by the rows that it moves (2^24 samples, d = 128, K = 1, a
// million nodes: 9.7 ms, 5.3 TB/s; tiles of 4096 and 2048 9.9 and 10.4 ms, since fewer samples of a tile share their
// hottest row).  A shorter one is bound by the walk of one wave over its quarter of a tile, 1.8 ms for any pool of up
// to 10^6 samples at d = 128, K = 1.  Smaller tiles spread it over the chip, but then more samples are in flight and
// the mixed policy's stores to cold rows lose more updates; so where it is short enough for that to be the faster
// way, all its rows are updated with atomic adds, which lose none.  They move 1.1 TB/s of rows, which about 1000 waves
// in pool order reach; more of them only put more samples in flight.  Rows that a percent of the samples name are
// what pool order is slow at: then tiles small enough for 1024 workgroups combine their updates.  (4096 samples,
// d = 128, K = 1: 1.82 -> 0.02 ms; 10^6 samples, d = 96, K = 3: 3.5 -> 1.7 ms; 10^6 samples, d = 64, K = 2, a million
// nodes: 2.0 -> 1.0 ms with tiles of 1024, 1.45 in pool order.  2.2*10^6 samples at d = 128, K = 1: 1.7 ms with the mixed
// policy, 2.8 with atomic adds.)  Whole runs in pools of 8192 to 500000 samples, learning rate 0.025 to 0, on six graphs of
// 10^4 to 3*10^5 nodes: rows end 1.1 to 9 times closer to the sequential ones than after tiles of 8192, the final loss
// +0.02 to +0.40 % from the sequential one (tiles of 8192: -0.36 to +0.49 %).  The same holds for any pool of a graph
// whose rows are all warm, where the mixed policy is atomic adds with the bookkeeping of the store policies (2*10^6 samples
// on 10^4 nodes: 7.7 -> 2.9 ms); since 65535 rows are ranked, that is a graph of up to 65535 nodes.
AsyncPlan async_plan(const AsyncPool &p) {
    constexpr uint32_t kWaves = kBlock / kWave;
    auto pieces = [&](uint32_t size) { return (uint32_t)((p.count + size - 1) / size); };
    // Every sample in flight works on values that miss the updates of the others (Def. 1, Sec. 3.2: the order of
    // updates stops mattering only while concurrent samples rarely share rows), and a small graph gains nothing from
    // thousands of waves: n / 32 of them, and at least 256.
    constexpr uint32_t kFullGrid = 2048;  // workgroups that fill the chip
    const uint32_t by_rows = std::max(p.n / 32u / kWaves, 64u), limit = std::min(by_rows, kFullGrid);
    const bool shorts = short_rows(floats_per_lane(p.dim), (int)p.num_neg);
    const uint32_t batch = samples_per_batch(p.dim, p.num_neg);
    // A held row trades with memory every four samples, or every two where rows are so long that an exchange is a
    // small part of a sample's traffic: the shorter interval halves how far the run's scores lag behind the other
    // holders of the row (measured on d = 512, K = 5: distance to the sequential trajectory after 4 pools
    // -0.33 % -> -0.10 % in loss at 3 % more time).
    // The samples of a block of a partitioned graph name its rows `partitions` times as often as those of a pool, and with
    // an interval of four its hottest rows run away once some 300 of the samples in flight name one of them: a million
    // nodes, exponent 2.1, pools of 2^24 in 4 x 4 blocks (600 such samples) and 8 x 8 (300): every long run diverged, 2 x 2
    // (590 of a share half as large): ends 0.5 % higher in loss than with two.  Where at most 128 do, four is as good as
    // two to the fourth digit of the loss, and faster (exponent 2.5: 2 x 2, 115 samples, 2.42 against 2.33*10^9 samples/s;
    // 8 x 8, 57 samples, 5.9 against 5.5*10^8; 200000 nodes in 2 x 2, 49 samples: 1.10*10^9 against 0.98); at 190 it
    // ends 0.2 % higher.
    auto exchange_every = [&](uint32_t blocks) {
        if (!shorts) return 2u;
        const double in_flight = (double)std::min(blocks, kFullGrid) * kWaves * batch;
        return p.part_of_pool && in_flight * p.hottest_share > 128.0 ? 2u : 4u;
    };
    auto tiled = [&](uint32_t coherence, uint32_t tile) {
        // one workgroup per tile, started by the hardware in tile order as earlier ones end, unless the graph is so
        // small that a fixed number of workgroups has to stride over the tiles (n / 8 samples in flight where rows are
        // short, else n / 16 or n / 32)
        const uint32_t most = std::min(shorts ? 2u * by_rows : by_rows, kFullGrid);
        const uint32_t blocks = most == kFullGrid ? pieces(tile) : std::min(pieces(tile), most);
        return AsyncPlan{true, coherence, tile, blocks, exchange_every(blocks)};
    };
    auto pool_order = [&](uint32_t coherence, uint32_t chunk, uint32_t blocks) {
        return AsyncPlan{false, coherence, chunk, std::min((pieces(chunk) + kWaves - 1) / kWaves, blocks), 0u};
    };
    if (!p.tiled) return pool_order(p.coherence, kWave, limit);
    if (p.force_tile) return tiled(p.coherence, p.force_tile);
    const AsyncPlan full = tiled(p.coherence, kLargestTile);
    // One block of a partitioned graph keeps tiles of 8192: it names its rows `partitions` times as often as a pool
    // does, and more samples in flight show in the loss (10^4 nodes, 8 x 8 blocks: +2.3 %).
    if (p.part_of_pool || p.coherence == kAgent) return full;

    // Microseconds.  A sample of a wave that walks a tile takes 0.2 + 0.33 K + 0.18 V (measured, d = 64 .. 512, K = 1
    // .. 5, one wave per SIMD), a little less in pool order; one row takes 16 million additions a second, of
    // which tiles combine four into one.
    const double V = floats_per_lane(p.dim), K = p.num_neg, sample_us = 0.2 + 0.33 * K + 0.18 * V;
    auto walk_us = [&](const AsyncPlan &t) {
        return (double)((pieces(t.unit) + t.blocks - 1) / t.blocks) * std::max(t.unit / kWaves, 1u) * sample_us;
    };
    const double add_us = (double)p.count * (K + 2.0) * p.dim * sizeof(float) / 1.1e6;
    const double hot_us = (double)p.count * p.hottest_share * 0.06;
    const double full_us = p.warm_ranks >= p.n ? HUGE_VAL : walk_us(full);

    uint32_t tile = kSmallestTile;
    while (tile < kLargestTile && (uint64_t)tile * 2048u <= p.count) tile *= 2;  // 1024 .. 2047 tiles
    // n / 32 samples in flight (at least 256 workgroups): the hottest rows set the pace, and four times as many took as
    // long and left training further behind (10^5 nodes, exponent 2.1, d = 64, K = 1, whole runs from a learning rate of
    // 0.025, final loss against the sequential one: pools of 500000, 65536 and 8192 samples +1.5, +0.9 and +0.3 % at n / 8,
    // +0.4, +0.3 and +0.2 % at n / 32; 490 -> 500, 96 -> 98 and 16 -> 20 us a pool).
    AsyncPlan small = tiled(kAtomicAgent, tile);
    if (tile < kLargestTile) small.blocks = std::min(small.blocks, std::max(p.n / 32u / (kWaves * batch), 256u));
    const double small_us = std::max({add_us, 0.25 * hot_us, walk_us(small)});

    // in pool order a wave has one sample in flight instead of a batch: n / 16 waves are half of what tiles have
    const uint32_t waves = std::min(std::max(p.n / 16u, 256u), 1024u);
    uint32_t chunk = 4;  // as few samples to a wave as keep the waves busy, up to 16
    while (chunk < 16u && pieces(chunk) > waves) chunk *= 2;
    const AsyncPlan short_pool = pool_order(kAtomicAgent, chunk, waves / kWaves);
    const double short_us = std::max({add_us + 0.5 * hot_us, hot_us, (double)p.count / (short_pool.blocks * kWaves) * sample_us});

    if (p.coherence == kMixed && p.may_skip_tiles && short_us < 1.25 * small_us && short_us < full_us) return short_pool;
    if (p.coherence == kAtomicAgent || small_us < full_us) return small;
    // Short rows take tiles of 4096 with the mixed policy as long as that puts no more samples in flight than four to a
    // wave of an 8192-sample tile would: where these are too few to fill the chip, and up to d = 64 always (2^24
    // samples, d = 64, K = 1: 6.6 -> 5.9 ms).
    if (p.coherence == kMixed && shorts && (V == 1.0 || pieces(kLargestTile) < 640u)) return tiled(kMixed, kLargestTile / 2u);
    return full;
}

}  // namespace gv
