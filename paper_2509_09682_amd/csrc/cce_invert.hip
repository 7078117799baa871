// dE of per-position negatives through an inverted index (item -> the (position, slot) pairs that sampled it).
//
// Alg. 2 updates the classifier gradient with one indexed row add per (position, candidate) pair.  With N*K pairs
// spread over a large table that is N*K*d floating-point atomics, and this chip retires scattered fp32 atomics at about
// 1.3 TB/s of payload against 7 TB/s for plain stores.  The same sum can be taken item by item: count the pairs of
// every item, turn the counts into offsets, file each pair under its item (a counting sort with integer atomics on a
// V-word table), then let one lane group per item recompute its few scores against hidden states that sit in L2 and
// add the finished row to dE once, without atomics.  Table rows are read once and written once; no score is stored.
// The correct items (power-law hot rows) are not part of the index: the aggregated scatter adds them.
#include <algorithm>

#include "cce_device.hpp"
#include "cce_kernels.hpp"
#include "cce_scatter.hpp"

namespace cce {
namespace {

constexpr int kThreads = 256;

// One thread per (position, slot) pair of a valid position whose negative takes part.
__device__ __forceinline__ bool pair_live(const InvertArgs &a, int64_t pair, int32_t &id)
{
    const int64_t i = pair / a.K;
    if (a.mask && a.mask[i] == 0) return false;
    id = a.smp.kind ? sample1(a.smp, (uint64_t)i, (uint32_t)(pair - i * a.K) + 1u) : a.neg[pair];
    const int32_t ti = a.tgt[i];
    if (a.validate && (ti < 0 || (int64_t)ti >= a.V || id < 0 || (int64_t)id >= a.V)) return false;  // flagged elsewhere
    return !(a.collide && id == ti);
}

// ---- exclusive scan of an int array in two launches: block-local scan + block totals, then every block adds the
//      totals of the blocks in front of it (read directly: n/4096 values at most)
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;
constexpr int kScanChunk = kScanThreads * kScanItems;

__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t *lds, int32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    __syncthreads();  // lds may still be read from a previous call
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t run = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            const int32_t c = lds[w];
            lds[w] = run;
            run += c;
        }
        lds[kScanThreads / 64] = run;
    }
    __syncthreads();
    total = lds[kScanThreads / 64];
    return incl - v + lds[wave];
}

__global__ __launch_bounds__(kScanThreads) void scan_local_kernel(int32_t *data, int64_t n, int32_t *block_sums)
{
    __shared__ int32_t lds[kScanThreads / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    int32_t v[kScanItems], sum = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        v[t] = (base + t < n) ? data[base + t] : 0;
        sum += v[t];
    }
    int32_t total;
    int32_t run = block_exclusive_scan(sum, lds, total);
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        if (base + t < n) data[base + t] = run;
        run += v[t];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void scan_add_kernel(int32_t *data, int64_t n, const int32_t *block_sums)
{
    __shared__ int32_t lds[kScanThreads / 64 + 1];
    int32_t part = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kScanThreads) part += block_sums[b];
    int32_t total;
    (void)block_exclusive_scan(part, lds, total);
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t)
        if (base + t < n) data[base + t] += total;
}

hipError_t launch_scan(int32_t *data, int64_t n, int32_t *block_sums, hipStream_t stream)
{
    const unsigned blocks = (unsigned)((n + kScanChunk - 1) / kScanChunk);
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(scan_local_kernel, dim3(blocks), dim3(kScanThreads), 0, stream, data, n, block_sums);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scan_add_kernel, dim3(blocks), dim3(kScanThreads), 0, stream, data, n, block_sums);
    return hipGetLastError();
}

// ---- fallback index build for huge catalogues: integer atomics on the V-word table (scattered atomics are slow:
//      about 27 G/s for the count, 10 G/s for the returning ones of the fill)
__global__ __launch_bounds__(kThreads) void count_kernel(InvertArgs a)
{
    const int64_t pair = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (pair >= a.N * a.K) return;
    int32_t id;
    if (pair_live(a, pair, id)) atomicAdd(a.cursor + id, 1);
}

// File every live pair under its item.  Afterwards cursor[v] is the END of item v's segment; it starts where the
// segment of v-1 ends.
__global__ __launch_bounds__(kThreads) void fill_kernel(InvertArgs a)
{
    const int64_t pair = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (pair >= a.N * a.K) return;
    int32_t id;
    if (pair_live(a, pair, id)) {
        const int32_t slot = atomicAdd(a.cursor + id, 1);
        static_cast<int32_t *>(a.pairs)[slot] = (int32_t)(pair / a.K);  // only the position is needed downstream
    }
}

// ---- index build by two-level counting sort without global atomics.
//  Level 1 partitions the pairs into buckets of 2^bucket_shift consecutive item ids: every block histograms its chunk of
//  pairs in LDS, the (bucket, block) counts are scanned bucket-major, and the block scatters (id, position) into its
//  reserved ranges.  Level 2 gives each bucket to one block, which counting-sorts it by id inside LDS and writes the
//  positions item by item together with the end offset of every item.
constexpr int kMaxBucketShift = 11;
constexpr int kMaxBucketIds = 1 << kMaxBucketShift;  // LDS histogram of level 2: 8 KiB
// Ids per bucket (a power of two): 256 to 512 buckets up to a million items, so that level 2 has blocks for the
// chip and a bucket of a small catalogue does not outgrow a slice (25,600 positions, K = 256, d = 128: with 2048 ids per
// bucket always, 20,000 items, every bucket beyond an eighth of the budget: 41.8 ms a step; 50,000 items, 25 blocks in
// level 2: 1.37 ms; with this rule 0.76 and 0.66 ms; 1 M items: 489 buckets, 3 % faster than 977).
int bucket_shift(int64_t V)
{
    int s = 0;
    while (s < kMaxBucketShift && (V >> s) >= 512) ++s;
    return s;
}
constexpr int kMaxBuckets = 2048;               // LDS histogram of level 1: 8 KiB
constexpr int kChunkPairs = 8192;               // pairs per chunk in level 1; a block takes chunks blockIdx.x, + gridDim.x, ...
// Chunks are smaller, 2048 pairs at least, where there would be fewer than 256 of them: the passes over few pairs wait for the chain
// of a block's batches (60,000 pairs: counting 8.7 -> 4.5 us, filing 18 -> 11).
constexpr int kMinChunkPairs = 2048, kFewChunks = 256;
constexpr int kMaxPartBlocks = 4096;            // blocks of level 1: bounds the (bucket, block) histogram at 32 MiB
// The index is built and used up in SLICES of the item-id range, so that its memory is bounded by a pair budget B instead
// of growing with N * K: every slice is a run of consecutive buckets that holds at most B pairs, gets filed into the same
// B-entry arrays, and is consumed by the item pass before the next one is filed.  Every table row is still read and
// written once; a further slice costs one more reading of the ids (4 bytes per pair) and four launches.
//   B = max(2^22, N K / 8) pairs, 2^23 for 2^22 where pairs are narrow (below);  slices = 1 if N K <= B, else
//   ceil(N K / (7/8 B)): the pairs of the ordinary buckets are cut at the quantiles j / slices of their running count, so a
//   slice holds at most N K / slices + (one bucket) <= 7/8 B + 1/8 B pairs, PROVIDED no bucket holds more than B / 8 pairs.
//   Buckets beyond that (consecutive ids drawing more than half a million pairs, a million narrow ones, an eighth of everything:
//   a popularity law far more skewed than any workload here) stay out of the index: their pairs are added to dE one by one with
//   atomics (hot_bucket_kernel).
constexpr int64_t kMinPairBudget = int64_t(1) << 22;
// A pair on its way to its item: the id and the position, 8 bytes, and the position alone once it is filed, 4.  Up to 2^16
// positions both fit half of that, because the bucket is known where an entry is read: the id's offset in it (kMaxBucketShift
// bits at most) and 16 bits of position.  The same memory then holds twice the pairs, and every index pass moves half the bytes.
// 25,600 positions, K = 256, 1 M items: one slice instead of two, filing 62 + 30 -> 82 us, sort 2 x 27 -> 39, step 887 -> 853; drawn by
// popularity: filing 111 + 113 -> 141, step 1476 -> 1257.
constexpr int64_t kNarrowPositions = int64_t(1) << 16;
static_assert(kMaxBucketShift <= 16, "an id's offset in its bucket and 16 bits of position fit a word");
struct WidePair {
    using Entry = int2;
    using Pos = int32_t;
    static __device__ __forceinline__ Entry make(int32_t k, int32_t pos) { return make_int2(k, pos); }
    static __device__ __forceinline__ int32_t item(Entry e) { return e.x; }
    static __device__ __forceinline__ Pos pos(Entry e) { return e.y; }
};
struct NarrowPair {
    using Entry = uint32_t;
    using Pos = uint16_t;
    static __device__ __forceinline__ Entry make(int32_t k, int32_t pos) { return (uint32_t)k << 16 | (uint32_t)pos; }
    static __device__ __forceinline__ int32_t item(Entry e) { return (int32_t)(e >> 16); }
    static __device__ __forceinline__ Pos pos(Entry e) { return (Pos)(e & 0xffffu); }
};
constexpr int kMaxSlices = 32;
constexpr int kSliceHot = -1;                   // slice_of[] of a bucket that stays out of the index

// The pairs of a block's chunk, kPairBatch per thread at a time: all mask bytes are requested first, then ids and
// targets of the valid positions only (entries of padded positions are never read), so a thread waits for two round
// trips per batch instead of three per pair.  Fewer than 2^31 pairs on this path: 32-bit pair arithmetic.
constexpr int kPairBatch = 8;
static_assert(kMinChunkPairs % (kThreads * kPairBatch) == 0, "whole batches per chunk");

// Stored and drawn ids have loops of their own, chosen once per launch (for_live_pairs): with the generator in the same loop,
// stored ids waited behind its branches (part_count_kernel 26 -> 17 us, the filing passes 63 + 37 -> 61 + 30 us on the
// per-position workload).
template <typename F>
__device__ __forceinline__ void for_stored_pairs(const InvertArgs &a, int64_t chunk, F &&visit)
{
    const uint32_t p0 = (uint32_t)chunk * (uint32_t)a.chunk_pairs, total = (uint32_t)(a.N * a.K), K = (uint32_t)a.K;
    for (int u0 = threadIdx.x; u0 < a.chunk_pairs; u0 += kThreads * kPairBatch) {
        uint32_t pos[kPairBatch];
        bool live[kPairBatch];
        int32_t id[kPairBatch], ti[kPairBatch];
#pragma unroll
        for (int j = 0; j < kPairBatch; ++j) {
            const uint32_t pair = p0 + u0 + j * kThreads;
            pos[j] = pair / K;
            live[j] = pair < total && (a.mask == nullptr || a.mask[pos[j]] != 0);
        }
#pragma unroll
        for (int j = 0; j < kPairBatch; ++j) {
            id[j] = ti[j] = 0;
            if (live[j]) {
                id[j] = a.neg[p0 + u0 + j * kThreads];
                ti[j] = a.tgt[pos[j]];
            }
        }
#pragma unroll
        for (int j = 0; j < kPairBatch; ++j) {
            if (a.validate && (ti[j] < 0 || (int64_t)ti[j] >= a.V || id[j] < 0 || (int64_t)id[j] >= a.V)) live[j] = false;  // flagged elsewhere
            if (a.collide && id[j] == ti[j]) live[j] = false;
            if (live[j]) visit(id[j], (int32_t)pos[j]);
        }
    }
}

// Sampled negatives are drawn again instead of being read, in groups of four draws (a generator call yields two or four), two
// groups per thread at a time (one draw a thread, eight at a time, each with a generator call of its own: the index of 2.4 M
// uniform draws from 20,000 items 84 us, so 68).  Draw 0 of a position is its correct item: K / 4 + 1 groups a position, chunk_pairs / 4 to a chunk.
constexpr int kDrawGroups = 2;
__host__ __device__ inline int64_t draw_groups(int64_t K) { return K / 4 + 1; }
template <typename F>
__device__ __forceinline__ void for_drawn_pairs(const InvertArgs &a, int64_t chunk, F &&visit)
{
    const uint32_t per = (uint32_t)draw_groups(a.K), total = (uint32_t)a.N * per, g0 = (uint32_t)chunk * (uint32_t)(a.chunk_pairs / 4);
    for (int u0 = threadIdx.x; u0 < a.chunk_pairs / 4; u0 += kThreads * kDrawGroups) {
        uint32_t pos[kDrawGroups], q[kDrawGroups];
        bool live[kDrawGroups];
        int32_t ti[kDrawGroups], id[kDrawGroups][4];
        Draws d[kDrawGroups];
#pragma unroll
        for (int j = 0; j < kDrawGroups; ++j) {
            const uint32_t grp = g0 + u0 + j * kThreads;
            pos[j] = grp / per;
            q[j] = grp - pos[j] * per;
            live[j] = grp < total && (a.mask == nullptr || a.mask[pos[j]] != 0);
        }
#pragma unroll
        for (int j = 0; j < kDrawGroups; ++j) {
            d[j] = Draws{};
            ti[j] = 0;
            if (live[j]) {
                ti[j] = a.tgt[pos[j]];
                draw4(a.smp, pos[j], q[j], d[j]);
            }
        }
        resolve4(a.smp, d, id);
#pragma unroll
        for (int j = 0; j < kDrawGroups; ++j) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint32_t draw = 4 * q[j] + t;
                bool on = live[j] && draw >= 1 && draw <= (uint32_t)a.K;
                if (a.validate && (ti[j] < 0 || (int64_t)ti[j] >= a.V || id[j][t] < 0 || (int64_t)id[j][t] >= a.V)) on = false;  // flagged elsewhere
                if (a.collide && id[j][t] == ti[j]) on = false;
                if (on) visit(id[j][t], (int32_t)pos[j]);
            }
        }
    }
}

template <typename F>
__device__ __forceinline__ void for_live_pairs(const InvertArgs &a, int64_t chunk, F &&visit)
{
    if (a.smp.kind) for_drawn_pairs(a, chunk, visit);
    else for_stored_pairs(a, chunk, visit);
}

// The alias table with both words of an entry side by side.
__global__ __launch_bounds__(kThreads) void pack_alias_kernel(Sampler s, uint2 *out)
{
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c < s.V) out[c] = make_uint2(s.thresh[c], (uint32_t)s.alias[c]);
}

__global__ __launch_bounds__(kThreads) void part_count_kernel(InvertArgs a)
{
    __shared__ int32_t hist[kMaxBuckets];
    for (int b = threadIdx.x; b < a.n_buckets; b += kThreads) hist[b] = 0;
    __syncthreads();
    for (int64_t chunk = blockIdx.x; chunk < a.n_chunks; chunk += gridDim.x)
        for_live_pairs(a, chunk, [&](int32_t id, int32_t) { atomicAdd(&hist[id >> a.bucket_shift], 1); });
    __syncthreads();
    for (int b = threadIdx.x; b < a.n_buckets; b += kThreads) a.part_hist[(int64_t)b * gridDim.x + blockIdx.x] = hist[b];
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.part_total = 0;  // last entry of the scanned array: receives the grand total
}

// Cuts the buckets into slices (see above) from the scanned (bucket, block) counts: slice_of[b], the start of every
// bucket inside its slice's arrays, and the cleared work-list counters of the slices.  One block.
__global__ __launch_bounds__(kScanThreads) void plan_slices_kernel(InvertArgs a)
{
    __shared__ int32_t lds[kScanThreads / 64 + 1];
    __shared__ int32_t base[kMaxSlices], lo[kMaxSlices], hi[kMaxSlices], any_hot;
    constexpr int PER = kMaxBuckets / kScanThreads;
    const int64_t nb = a.n_part_blocks;
    int32_t cnt[PER], cum[PER], sum = 0;
    bool hot[PER];
    for (int j = threadIdx.x; j < kMaxSlices; j += kScanThreads) {
        base[j] = lo[j] = 0x7fffffff;
        hi[j] = -1;
        a.slice_hot[j] = 0;
    }
    if (threadIdx.x == 0) any_hot = 0;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int b = threadIdx.x * PER + t;
        cnt[t] = 0;
        if (b < a.n_buckets) {
            const int32_t s0 = a.part_hist[(int64_t)b * nb];
            const int32_t s1 = (b + 1 < a.n_buckets) ? a.part_hist[(int64_t)(b + 1) * nb] : a.part_total[0];
            cnt[t] = s1 - s0;
        }
        hot[t] = a.n_slices > 1 && (int64_t)cnt[t] > a.budget / 8;
        cum[t] = sum;                  // running count of the ordinary buckets in front of this one, within the thread
        if (!hot[t]) sum += cnt[t];
    }
    int32_t total;
    const int32_t before = block_exclusive_scan(sum, lds, total);
    const int32_t per_slice = (total + a.n_slices - 1) / a.n_slices > 0 ? (total + a.n_slices - 1) / a.n_slices : 1;
    int32_t sl[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        cum[t] += before;
        sl[t] = hot[t] ? kSliceHot : min(cum[t] / per_slice, a.n_slices - 1);
        const int b = threadIdx.x * PER + t;
        if (b < a.n_buckets && !hot[t]) {
            atomicMin(&base[sl[t]], cum[t]);
            atomicMin(&lo[sl[t]], b);
            atomicMax(&hi[sl[t]], b);
        }
        if (b < a.n_buckets && hot[t]) any_hot = 1;
    }
    __syncthreads();
    // buckets [slice_lo, slice_hi] of a slice (an empty slice has hi < lo), and whether any bucket stays out of the index
    for (int j = threadIdx.x; j < kMaxSlices; j += kScanThreads) {
        a.slice_hot[kMaxSlices + j] = lo[j];
        a.slice_hot[2 * kMaxSlices + j] = hi[j];
    }
    if (threadIdx.x == 0) a.slice_hot[3 * kMaxSlices] = any_hot;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int b = threadIdx.x * PER + t;
        if (b < a.n_buckets) {
            a.slice_of[b] = sl[t];
            a.bucket_start[b] = hot[t] ? 0 : cum[t] - base[sl[t]];
        }
    }
}

// D_SC != 0: the first sc_blocks blocks scatter the gradient rows of the correct items (hidden size D_SC) instead;
// nothing in this launch or the next reads or writes dE, and their latency hides under the filing of the pairs.
template <typename P, int D_SC>
__global__ __launch_bounds__(kThreads) void part_scatter_kernel(InvertArgs a, TileArgs sc, int64_t sc_blocks)
{
    // Narrow pairs of one chunk a block are put in order of their buckets in LDS first and leave as runs: written one by one, 64
    // lines an instruction, the launch waited for its stores.  (Wide ones would take 64 KB of staging, two blocks a CU.)
    // 6.5 M pairs in 489 buckets: 82 -> 53 us, drawn by popularity 141 -> 90.
    constexpr bool kStaged = sizeof(typename P::Entry) == 4;
    // 40 KB, four blocks a CU.
    __shared__ __align__(16) int32_t cur[kMaxBuckets];
    __shared__ typename P::Entry stage[kStaged ? kChunkPairs : 1];
    static_assert(kThreads == kPosChunk && kMaxBuckets * 4 >= kPosChunk * 8, "the scatter role sorts 256 keys in this array");
    if (D_SC != 0 && (int64_t)blockIdx.x < sc_blocks) {
        pos_scatter_block<(D_SC != 0 ? D_SC : 64)>(sc, (int64_t)blockIdx.x, reinterpret_cast<uint64_t *>(cur), pos_parts(sc.N));
        return;
    }
    // Buckets of this slice: the block's cursor starts at the block's scanned offset inside the bucket, moved to where
    // the bucket starts in the slice's arrays.  Buckets of other slices get a negative cursor and are skipped.
    const int64_t blk = (int64_t)blockIdx.x - (D_SC != 0 ? sc_blocks : 0);
    const int64_t nb = a.n_part_blocks;
    if (kStaged && a.n_chunks <= nb) {
        // where each bucket's run starts in the block's chunk: the block's scanned counts of one bucket and the next block's
        // are apart by what this block brings
        constexpr int PER = kMaxBuckets / kThreads;
        const int per = (a.n_buckets + kThreads - 1) / kThreads;  // consecutive buckets a thread
        int32_t n[PER], sl[PER], sum = 0;
#pragma unroll
        for (int t = 0; t < PER; ++t) {  // all loads before the first use
            n[t] = 0;
            sl[t] = -2;
            if (t < per) {
                const int b = min((int)threadIdx.x * per + t, a.n_buckets - 1);
                const int32_t *h = a.part_hist + (int64_t)b * nb + blk;
                n[t] = h[1] - h[0];
                sl[t] = a.slice_of[b];
            }
        }
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            if (t >= per || (int)threadIdx.x * per + t >= a.n_buckets || sl[t] != a.slice) n[t] = -1;
            else sum += n[t];
        }
        int32_t incl = sum, *wave_sums = reinterpret_cast<int32_t *>(stage);
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        if (lane == 63) wave_sums[wave] = incl;
        __syncthreads();
        int32_t run = incl - sum;
        for (int w = 0; w < wave; ++w) run += wave_sums[w];
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int b = threadIdx.x * per + t;
            if (t < per && b < a.n_buckets) cur[b] = n[t] < 0 ? ~run : run;  // other slices' buckets: negative, skipped
            if (n[t] > 0) run += n[t];
        }
        __syncthreads();
        for_live_pairs(a, blk, [&](int32_t id, int32_t pos) {
            int32_t *c = &cur[id >> a.bucket_shift];
            if (*c >= 0) stage[atomicAdd(c, 1)] = P::make(id & ((1 << a.bucket_shift) - 1), pos);
        });
        __syncthreads();
        // sixteen lanes a bucket, kRuns buckets at a time; a run starts where the one before it ended
        constexpr int kRuns = 8, kStep = kThreads / 16;
        typename P::Entry *out = static_cast<typename P::Entry *>(a.tmp);
        for (int b0 = threadIdx.x / 16; b0 < a.n_buckets; b0 += kRuns * kStep) {
            int32_t begin[kRuns], end[kRuns], to[kRuns];
#pragma unroll
            for (int t = 0; t < kRuns; ++t) {
                const int b = min(b0 + t * kStep, a.n_buckets - 1);
                const int32_t before = b ? cur[b - 1] : 0;
                begin[t] = before < 0 ? ~before : before;
                end[t] = b0 + t * kStep < a.n_buckets ? cur[b] : -1;
                to[t] = a.part_hist[(int64_t)b * nb + blk] - a.part_hist[(int64_t)b * nb] + a.bucket_start[b];
            }
#pragma unroll
            for (int t = 0; t < kRuns; ++t)
                for (int32_t k = begin[t] + threadIdx.x % 16; k < end[t]; k += 16) out[to[t] + k - begin[t]] = stage[k];
        }
        return;
    }
    for (int b = threadIdx.x; b < a.n_buckets; b += kThreads)
        cur[b] = (a.slice_of[b] == a.slice) ? a.part_hist[(int64_t)b * nb + blk] - a.part_hist[(int64_t)b * nb] + a.bucket_start[b] : -1;
    __syncthreads();
    for (int64_t chunk = blk; chunk < a.n_chunks; chunk += nb)
        for_live_pairs(a, chunk, [&](int32_t id, int32_t pos) {
            int32_t *c = &cur[id >> a.bucket_shift];
            if (*c >= 0)  // cursors only grow: the sign never changes
                static_cast<typename P::Entry *>(a.tmp)[atomicAdd(c, 1)] = P::make(id & ((1 << a.bucket_shift) - 1), pos);
        });
}

// Pairs of the buckets that stay out of the index (more than an eighth of the budget): each is
// scored and added to dE on its own, one thread per pair, d atomics.  A correctness path for extreme skew, not a fast one.
template <typename T>
__global__ __launch_bounds__(kThreads) void hot_bucket_kernel(InvertArgs a)
{
    __shared__ int8_t is_hot[kMaxBuckets];
    if (a.slice_hot[3 * kMaxSlices] == 0) return;  // no such bucket (block-uniform)
    for (int b = threadIdx.x; b < a.n_buckets; b += kThreads) is_hot[b] = a.slice_of[b] == kSliceHot;
    __syncthreads();
    const T *Hp = static_cast<const T *>(a.H), *Ep = static_cast<const T *>(a.E);
    for (int64_t chunk = blockIdx.x; chunk < a.n_chunks; chunk += gridDim.x)
        for_live_pairs(a, chunk, [&](int32_t id, int32_t pos) {
            if (!is_hot[id >> a.bucket_shift]) return;
            const T *h = Hp + (int64_t)pos * a.d, *e = Ep + (int64_t)id * a.d;
            float o = 0.f;
            for (int t = 0; t < a.d; ++t) o = fmaf(load1(h + t), load1(e + t), o);
            const float G = (a.g ? a.g[pos] : 1.f) * fast_exp(o - a.lse_in[pos]);
            float *row = a.dE + (int64_t)id * a.d;
            for (int t = 0; t < a.d; ++t) unsafeAtomicAdd(row + t, G * load1(h + t));
        });
}

// Level 2 reads a bucket's entries BATCH a thread at a time.  A hot item owns most entries of its bucket, and 64 lanes adding to
// one LDS word take 64 turns: in a crowded bucket a wavefront counts the entries that hold the same id as its first lane by
// ballots over the batch, and one lane adds them at once.  The block of the most crowded bucket is what the launch waits for
// (6.5 M pairs drawn with p ~ rank^-0.9 from 1 M items, a slice: one add for every 64 entries 157 us, for 512, the next entries on
// their way meanwhile, 75 us).
template <typename P, int BATCH>
struct CrowdedBucket {
    const typename P::Entry *tmp;
    int32_t rb, re;
    int32_t k[BATCH];  // id's offset in the bucket, -1 past its end
    typename P::Entry t[BATCH], t_next[BATCH];

    __device__ __forceinline__ void fetch(int32_t e0, typename P::Entry (&to)[BATCH]) const
    {
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int32_t e = e0 + j * kScanThreads + (int32_t)threadIdx.x;
            to[j] = typename P::Entry{};
            if (e < re) to[j] = tmp[e];
        }
    }
    // visit(lead, the lanes that hold it): every batch of the bucket, the next one on its way meanwhile
    template <typename F>
    __device__ __forceinline__ void walk(F &&visit)
    {
        fetch(rb, t);
        for (int32_t e0 = rb; e0 < re; e0 += BATCH * kScanThreads) {
            fetch(e0 + BATCH * kScanThreads, t_next);
#pragma unroll
            for (int j = 0; j < BATCH; ++j) k[j] = (e0 + j * kScanThreads + (int32_t)threadIdx.x < re) ? P::item(t[j]) : -1;
            visit(__builtin_amdgcn_readfirstlane(k[0]));
#pragma unroll
            for (int j = 0; j < BATCH; ++j) t[j] = t_next[j];
        }
    }
    __device__ __forceinline__ void count(int32_t *hist)
    {
        walk([&](int32_t lead) {
            int32_t same = 0;
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                same += (int32_t)__popcll(__ballot(k[j] == lead));
                if (k[j] >= 0 && k[j] != lead) atomicAdd(&hist[k[j]], 1);
            }
            if ((threadIdx.x & 63) == 0 && lead >= 0) atomicAdd(&hist[lead], same);
        });
    }
    __device__ __forceinline__ void file(int32_t *hist, typename P::Pos *pairs)
    {
        const int lane = threadIdx.x & 63;
        walk([&](int32_t lead) {
            int32_t before[BATCH], same = 0;
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {  // ranks among the entries of the first lane's id
                const uint64_t m = __ballot(k[j] == lead);
                before[j] = same + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
                same += (int32_t)__popcll(m);
            }
            int32_t base = 0;
            if (lane == 0 && lead >= 0) base = atomicAdd(&hist[lead], same);
            base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                if (k[j] < 0) continue;
                const int32_t slot = k[j] == lead ? base + before[j] : atomicAdd(&hist[k[j]], 1);
                pairs[rb + slot] = P::pos(t[j]);
            }
        });
    }
};

template <typename P>
__global__ __launch_bounds__(kScanThreads) void bucket_sort_kernel(InvertArgs a)
{
    __shared__ int32_t hist[kMaxBucketIds];
    const int ids = 1 << a.bucket_shift;
    __shared__ int32_t lds[kScanThreads / 64 + 1];
    const int b = blockIdx.x;
    if (a.slice_of[b] != a.slice) return;  // block-uniform
    const int64_t n_blocks1 = a.n_part_blocks;
    // the bucket's range in tmp: it starts where the slice plan put it and holds as many pairs as the scanned (bucket,
    // block 0) entries of this bucket and the next are apart
    const int32_t s0 = a.part_hist[(int64_t)b * n_blocks1];
    const int32_t s1 = (b + 1 < a.n_buckets) ? a.part_hist[(int64_t)(b + 1) * n_blocks1] : a.part_total[0];
    const int32_t rb = a.bucket_start[b];
    const int32_t re = rb + (s1 - s0);
    const int64_t id0 = (int64_t)b << a.bucket_shift;
    const typename P::Entry *tmp = static_cast<const typename P::Entry *>(a.tmp);
    typename P::Pos *pairs = static_cast<typename P::Pos *>(a.pairs);
    for (int k = threadIdx.x; k < kMaxBucketIds; k += kScanThreads) hist[k] = 0;
    __syncthreads();
    // Block-uniform; ordinary buckets take the plain loops, crowded ones of a few batches an entry a thread at a time (3748
    // items, 60,000 pairs: eight 7.2 us, one 4.7).
    constexpr int kSortBatch = 8;
    const bool crowded = re - rb > 16 * ids, batches = re - rb > 2 * kSortBatch * kScanThreads;
    CrowdedBucket<P, kSortBatch> many;
    CrowdedBucket<P, 1> few;
    many.tmp = few.tmp = tmp;
    many.rb = few.rb = rb;
    many.re = few.re = re;
    if (!crowded)
        for (int32_t e = rb + (int32_t)threadIdx.x; e < re; e += kScanThreads) atomicAdd(&hist[P::item(tmp[e])], 1);
    else if (batches) many.count(hist);
    else few.count(hist);
    __syncthreads();
    // exclusive scan over the counts: consecutive ids per thread
    int32_t v[kMaxBucketIds / kScanThreads], sum = 0;
#pragma unroll
    for (int t = 0; t < kMaxBucketIds / kScanThreads; ++t) {
        v[t] = hist[threadIdx.x * (kMaxBucketIds / kScanThreads) + t];
        sum += v[t];
    }
    int32_t total;
    int32_t run = block_exclusive_scan(sum, lds, total);
#pragma unroll
    for (int t = 0; t < kMaxBucketIds / kScanThreads; ++t) {
        const int k = threadIdx.x * (kMaxBucketIds / kScanThreads) + t;
        hist[k] = run;  // start of the item's segment inside the bucket; advanced below while filing
        run += v[t];
        if (k < ids && id0 + k < a.V) a.cursor[id0 + k] = rb + run;  // END of the item's segment
    }
    __syncthreads();
    if (!crowded)
        for (int32_t e = rb + (int32_t)threadIdx.x; e < re; e += kScanThreads) {
            const typename P::Entry t = tmp[e];
            const int32_t slot = atomicAdd(&hist[P::item(t)], 1);
            pairs[rb + slot] = P::pos(t);
        }
    else if (batches) many.file(hist, pairs);
    else few.file(hist, pairs);
}

// Rows of a table below 4 GiB by 32-bit offsets; a load beyond its end brings zeros.
struct RowBuffer {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ RowBuffer(const void *base, uint32_t bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00027000)) {}
    __device__ __forceinline__ void load(uint32_t off, RawChunk<uint16_t> &to) const
    {
        const u32x4_nt v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
        to.v = make_uint4(v.x, v.y, v.z, v.w);
    }
    __device__ __forceinline__ void load(uint32_t off, RawChunk<float> &to) const
    {
        const u32x4_nt v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
        const u32x4_nt w = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 16, 0);
        to.a = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
        to.b = make_float4(__uint_as_float(w.x), __uint_as_float(w.y), __uint_as_float(w.z), __uint_as_float(w.w));
    }
};

// Walks the positions filed in pairs[r, r_end) for the item whose row e the lane group holds, four at a time:
// recomputes each score against the hidden state (L2-resident), forms g exp(o - lse) and adds G h to acc.
// The lanes of a group enter together; groups of a wavefront leave when their own segment ends.  What bounds the walk is a mix
// of vector issue (60 %) and waiting for rows, so both were cut: past the end of a segment its last position is walked again with
// weight 0 (nothing to clear, no lane masks), rows are addressed by 32-bit offsets where positions have 16 bits, and the next
// four positions are on their way before the rows at hand are used.
// 25,600 positions, K = 256, 1 M items: item pass 470 -> 460 us; drawn by popularity 568 -> 543, crowded items 93 -> 82.  Six
// wavefronts a SIMD for five: 471 (the hidden states, 6.5 MB, share 4 MB of L2 with what is streamed).
template <typename T, typename P, int LPR>
__device__ __forceinline__ void walk_segment(const InvertArgs &a, const RawChunk<T> &e_raw, int32_t r, int32_t r_end, bool col_ok,
                                             int c, float (&acc)[8])
{
    // Four rows in flight: segments are short (6.5 pairs on average on the per-position workload) and the lane groups of a
    // wavefront go in step, so that a batch of eight was half empty (item pass 480 -> 465 us).
    constexpr int U = 4;
    constexpr bool kNarrow = sizeof(typename P::Pos) == 2;
    const char *lse_base = reinterpret_cast<const char *>(a.lse_in), *g_base = a.g ? reinterpret_cast<const char *>(a.g) : lse_base;
    const uint32_t row_bytes = (uint32_t)a.d * (uint32_t)sizeof(T), col_bytes = (uint32_t)c * 8u * (uint32_t)sizeof(T);
    // narrow: 2^16 rows of at most 512 elements, 2^27 bytes; a lane beyond the row reads beyond the buffer, that is zeros
    const RowBuffer rows(a.H, kNarrow ? (uint32_t)a.N * row_bytes : 0u);
    const uint32_t col_off = col_ok ? col_bytes : 0x80000000u;
    uint32_t pos[U];
    RawChunk<T> raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) raw[u].clear();
    auto positions = [&](int32_t at) {  // at most 2^28 pairs a slice
#pragma unroll
        for (int u = 0; u < U; ++u)
            pos[u] = (uint32_t)stream_load(reinterpret_cast<const typename P::Pos *>(
                static_cast<const char *>(a.pairs) + (uint32_t)max(min(at + u, r_end - 1), 0) * (uint32_t)sizeof(typename P::Pos)));
    };
    // The fences keep the loads where they stand: the compiler moves the two calls into one at the head of the loop otherwise,
    // where nothing runs ahead of the rows.
    positions(r);
    asm volatile("" ::: "memory");
    float e[8];
    e_raw.widen(e);
    while (r < r_end) {
        float lse[U], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t at = kNarrow ? (size_t)(pos[u] * 4u) : (size_t)pos[u] * 4;
            lse[u] = *reinterpret_cast<const float *>(lse_base + at);
            g[u] = *reinterpret_cast<const float *>(g_base + at);
        }
        if (kNarrow) {
#pragma unroll
            for (int u = 0; u < U; ++u) rows.load(__umul24(pos[u], row_bytes) + col_off, raw[u]);
        } else if (col_ok) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                raw[u].load(reinterpret_cast<const T *>(static_cast<const char *>(a.H) + (uint64_t)pos[u] * row_bytes + col_bytes));
        }
        const int32_t left = r_end - r;
        r += U;
        positions(r);  // whatever is left: a load in a branch of its own would make the rows wait for it
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float h[8];
            raw[u].widen(h);
            float part = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) part = fmaf(h[t], e[t], part);
            part = group_sum<LPR>(part);  // the lanes of a group share the item
            const float G = (u < left ? (a.g ? g[u] : 1.f) : 0.f) * fast_exp(part - lse[u]);
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = fmaf(G, h[t], acc[t]);
        }
    }
}

// An item sampled by more than kHotPairs positions (popularity-weighted negatives: the head of the law collects
// percents of all pairs) would keep one lane group walking for milliseconds.  Its segment is cut into chunks of
// kHotChunk instead, filed in a work list, and hot_item_kernel spreads the chunks over the chip, one block each, and
// adds their partial rows with atomics (d atomics per chunk).
constexpr int kHotPairs = 256;
constexpr int kHotChunk = 1024;
constexpr int kItemBlocks = 16384;  // grid of the item pass over a slice

// One group of LPR lanes per item: e_v stays in registers, the positions that sampled it are walked four at a time.
template <typename T, typename P, int LPR>
__global__ __launch_bounds__(kThreads) void item_dE_kernel(InvertArgs a)
{
    constexpr int GPW = 64 / LPR;  // items per wavefront
    constexpr int IPB = (kThreads / 64) * GPW;  // items per block and trip
    const int lane = threadIdx.x & 63;
    const int c = lane % LPR;
    const bool col_ok = c * 8 < a.d;
    // items of this launch: the whole table, or the buckets of the slice at hand (a fixed grid strides over them)
    int64_t v_lo = 0, v_hi = a.V;
    if (a.slice_of) {
        v_lo = (int64_t)a.slice_hot[kMaxSlices + a.slice] << a.bucket_shift;
        v_hi = min(a.V, ((int64_t)a.slice_hot[2 * kMaxSlices + a.slice] + 1) << a.bucket_shift);
    }
    // cursor[v] is the end of item v's segment; it starts where the one before it ends, the first item of a bucket
    // where the bucket starts in the slice's arrays (without slices: one running array over all items).  The segments of the next
    // trip are looked up before the walk of this one; every load is issued whatever the others bring.
    const int32_t *slice_of = a.slice_of ? a.slice_of : a.cursor, *start_of = a.slice_of ? a.bucket_start : a.cursor;
    const int shift = a.slice_of ? a.bucket_shift : 0;
    struct Segment {
        int32_t slice, start, before, end;
    };
    auto look_up = [&](int64_t v) {
        const int64_t w = v < v_hi ? v : v_hi - 1;  // (an empty slice has v_hi <= v_lo and takes no trip: any item)
        const int64_t x = w > 0 ? w : 0;
        return Segment{slice_of[x >> shift], start_of[x >> shift], a.cursor[x > 0 ? x - 1 : 0], a.cursor[x]};
    };
    const int64_t step = (int64_t)gridDim.x * IPB, own = (threadIdx.x >> 6) * GPW + lane / LPR;
    Segment next = look_up(v_lo + (int64_t)blockIdx.x * IPB + own);
    for (int64_t v0 = v_lo + (int64_t)blockIdx.x * IPB; v0 < v_hi; v0 += step) {
    const int64_t v = v0 + own;
    const Segment at = next;
    next = look_up(v + step);
    const bool first = a.slice_of ? (v & ((1 << a.bucket_shift) - 1)) == 0 : v == 0;
    int32_t r = first ? (a.slice_of ? at.start : 0) : at.before, r_end = at.end;
    if (v >= v_hi || (a.slice_of && at.slice != a.slice)) r = r_end = 0;
    if (!__any(r < r_end)) continue;
    if (r_end - r > kHotPairs) {  // hot item: file its chunks and leave it to hot_item_kernel
        const int32_t n_chunks = (r_end - r + kHotChunk - 1) / kHotChunk;
        int32_t slot = 0;
        if (c == 0) slot = atomicAdd(a.hot_count, n_chunks);
        slot = __shfl(slot, lane - c, 64);
        for (int32_t k = c; k < n_chunks; k += LPR) {
            const int32_t b = r + k * kHotChunk;
            if (slot + k < a.hot_capacity) a.hot_list[slot + k] = make_int4((int32_t)v, b, min(b + kHotChunk, r_end), 0);
        }
        r = r_end = 0;
    }
    RawChunk<T> e;
    e.clear();
    float acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = 0.f;
    // the item row and the dE row it will be added to are requested together, before the walk over the positions
    const bool mine = r < r_end && col_ok;
    float4 *row = reinterpret_cast<float4 *>(a.dE + (mine ? v : 0) * (int64_t)a.d + c * 8);
    float4 dx = make_float4(0.f, 0.f, 0.f, 0.f), dy = dx;
    if (mine) {  // used once each: they must not push the hidden states out of L2
        e.load_stream(static_cast<const T *>(a.E) + v * (int64_t)a.d + c * 8);
        dx = stream_load(row);
        dy = stream_load(row + 1);
    }
    walk_segment<T, P, LPR>(a, e, r, r_end, col_ok, c, acc);
    // the row belongs to this lane group alone: plain read-modify-write
    if (mine) {
        dx.x += acc[0]; dx.y += acc[1]; dx.z += acc[2]; dx.w += acc[3];
        dy.x += acc[4]; dy.y += acc[5]; dy.z += acc[6]; dy.w += acc[7];
        stream_store(row, dx);
        stream_store(row + 1, dy);
    }
    }  // item groups of this block
}

// The chunks item_dE_kernel filed: one block per chunk, a fixed grid strides over the list.  Every lane group walks a
// consecutive share; the wavefronts' sums meet in LDS, so that an atomic instruction covers 64 consecutive floats of the
// row.  What bounds the pass is the hottest item: its chunks add to one row, one instruction after the other (25 ns
// each).  With 256 pairs a chunk, a lane group per chunk and eight strided floats per lane (eight instructions) a third
// of the item's time was spent there: 6.5 M pairs drawn with p ~ rank^-0.9 from 1 M items, d = 128: 348 us before.
constexpr int kHotBlocks = 2048;
template <typename T, typename P, int LPR>
__global__ __launch_bounds__(kThreads) void hot_item_kernel(InvertArgs a)
{
    constexpr int GPW = 64 / LPR, WAVES = kThreads / 64;
    __shared__ float part[WAVES][LPR * 8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane % LPR, grp = lane / LPR;
    const bool col_ok = c * 8 < a.d;
    const int32_t n = min(*a.hot_count, a.hot_capacity);
    for (int32_t ent = (int32_t)blockIdx.x; ent < n; ent += (int32_t)gridDim.x) {  // uniform over the block
        const int4 h = a.hot_list[ent];
        RawChunk<T> e;
        e.clear();
        float acc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = 0.f;
        if (col_ok) e.load(static_cast<const T *>(a.E) + h.x * (int64_t)a.d + c * 8);
        const int32_t share = (h.z - h.y + WAVES * GPW - 1) / (WAVES * GPW), r = h.y + (wave * GPW + grp) * share;
        walk_segment<T, P, LPR>(a, e, r, min(r + share, h.z), col_ok, c, acc);
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] += __shfl_xor(acc[t], off, 64);
        }
        if (grp == 0) {
#pragma unroll
            for (int t = 0; t < 8; ++t) part[wave][c * 8 + t] = acc[t];
        }
        __syncthreads();
        for (int col = threadIdx.x; col < a.d; col += kThreads) {
            float sum = part[0][col];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) sum += part[w][col];
            unsafeAtomicAdd(a.dE + h.x * (int64_t)a.d + col, sum);
        }
        __syncthreads();
    }
}

template <typename T, typename P, int LPR>
hipError_t launch_item_dE(const InvertArgs &a, hipStream_t stream)
{
    constexpr int items_per_block = (kThreads / 64) * (64 / LPR);
    ProfScope prof(PROF_ITEM_DE, stream);
    if (!a.slice_of) {  // the sliced index build has cleared the work-list counters on its way (plan_slices_kernel)
        const hipError_t e = launch_fill_zero(a.hot_count, 1, stream);
        if (e != hipSuccess) return e;
    }
    // unsliced: one trip per block; sliced: the slice's item range is only known on the device, a grid of at most
    // kItemBlocks strides over it
    int64_t item_blocks = (a.V + items_per_block - 1) / items_per_block;
    if (a.slice_of && item_blocks > kItemBlocks) item_blocks = kItemBlocks;
    hipLaunchKernelGGL((item_dE_kernel<T, P, LPR>), dim3((unsigned)item_blocks), dim3(kThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((hot_item_kernel<T, P, LPR>), dim3(kHotBlocks), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
}

template <typename T, typename P>
hipError_t launch_item_dE_by_width(const InvertArgs &a, hipStream_t stream)
{
    const int chunks = (a.d + 7) / 8;
    if (chunks <= 2) return launch_item_dE<T, P, 2>(a, stream);
    if (chunks <= 4) return launch_item_dE<T, P, 4>(a, stream);
    if (chunks <= 8) return launch_item_dE<T, P, 8>(a, stream);
    if (chunks <= 16) return launch_item_dE<T, P, 16>(a, stream);
    if (chunks <= 32) return launch_item_dE<T, P, 32>(a, stream);
    return launch_item_dE<T, P, 64>(a, stream);
}

// One thread per four consecutive draws of a position.  (Arguments in this order: what it reads of them is 64 bytes; the
// output behind the sampler lay beyond: 2.20 us, so 2.07.)
__global__ __launch_bounds__(kThreads) void sample_kernel(int32_t *out, int64_t n_pos, int32_t K, Sampler smp)
{
    const int64_t quads = ((int64_t)K + 4) / 4;  // draws 0..K cover K/4 + 1 groups of four
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= n_pos * quads) return;
    const int64_t i = t / quads;
    const uint32_t q4 = (uint32_t)(t - i * quads);
    int32_t id[4];
    sample4(smp, (uint64_t)i, q4, id);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int64_t j = 4 * (int64_t)q4 + w;  // draw number; slot j - 1
        if (j >= 1 && j <= K) out[i * K + (j - 1)] = id[w];
    }
}

}  // namespace

hipError_t launch_sample(const Sampler &smp, int64_t n_pos, int32_t K, int32_t *out, hipStream_t stream)
{
    const int64_t threads = n_pos * (((int64_t)K + 4) / 4);
    if (n_pos <= 0 || K <= 0) return hipSuccess;
    hipLaunchKernelGGL(sample_kernel, dim3((unsigned)((threads + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, out, n_pos, K, smp);
    return hipGetLastError();
}

hipError_t launch_pack_alias(const Sampler &smp, hipStream_t stream)
{
    hipLaunchKernelGGL(pack_alias_kernel, dim3((unsigned)(((int64_t)smp.V + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, smp,
                       const_cast<uint2 *>(smp.packed));
    return hipGetLastError();
}

bool invert_narrow(int64_t N, int64_t V) { return N <= kNarrowPositions && invert_partitioned(V); }
int64_t invert_pair_budget(int64_t N, int64_t K, int64_t V)
{
    const int64_t least = kMinPairBudget * (invert_narrow(N, V) ? 2 : 1), eighth = (N * K + 7) / 8;
    return eighth > least ? eighth : least;
}
int invert_slices(int64_t N, int64_t K, int64_t V)
{
    const int64_t pairs = N * K, B = invert_pair_budget(N, K, V), room = B - B / 8;
    return pairs <= B ? 1 : (int)((pairs + room - 1) / room);
}
int64_t invert_index_pairs(int64_t N, int64_t K, int64_t V)   // entries of the arrays the index is filed into
{
    const int64_t pairs = N * K, B = invert_pair_budget(N, K, V);
    return pairs < B ? pairs : B;
}
// (with the narrow budget also where pairs are wide: a workspace made for many positions serves fewer)
size_t invert_hot_capacity(int64_t N, int64_t K)
{
    const int64_t pairs = N * K, most = std::max(2 * kMinPairBudget, (pairs + 7) / 8);
    return (size_t)(2 * (std::min(pairs, most) / kHotPairs) + 16);
}
size_t invert_scan_blocks(int64_t n) { return (size_t)((n + kScanChunk - 1) / kScanChunk); }
// Chunks of level 1: pairs a chunk and how many, for `pairs` stored ids or draws (whose groups of four hold the correct item and
// the rest of the last group as well).
int32_t chunk_pairs_of(int64_t pairs)
{
    int32_t c = kChunkPairs;
    while (c > kMinChunkPairs && pairs < (int64_t)c * kFewChunks) c /= 2;
    return c;
}
// Blocks of level 1 at most, stored or drawn; does not fall as N grows.
int64_t invert_part_blocks(int64_t N, int64_t K)
{
    const int64_t pairs = N * draw_groups(K) * 4, few = (pairs + kMinChunkPairs - 1) / kMinChunkPairs;
    const int64_t chunks = std::max(std::min<int64_t>(few, 2 * kFewChunks), (pairs + kChunkPairs - 1) / kChunkPairs);
    return chunks < kMaxPartBlocks ? chunks : kMaxPartBlocks;
}
int64_t invert_buckets(int64_t V) { return (V + (int64_t(1) << bucket_shift(V)) - 1) >> bucket_shift(V); }
bool invert_partitioned(int64_t V) { return invert_buckets(V) <= kMaxBuckets; }
int invert_plan_words() { return 3 * kMaxSlices + 8; }  // work-list counters, first and last bucket of every slice, one flag

namespace {
// Catalogues cut into buckets: count, scan, plan, then slice by slice file, sort and consume.
template <typename P>
hipError_t launch_sliced_dE(bool bf16, InvertArgs a, const TileArgs *scatter, hipStream_t stream)
{
    hipError_t e;
    auto check = [&]() { return (e = hipGetLastError()) == hipSuccess; };
    a.n_buckets = (int32_t)invert_buckets(a.V);
    a.bucket_shift = bucket_shift(a.V);
    const int64_t level1 = a.smp.kind ? a.N * draw_groups(a.K) * 4 : a.N * a.K;
    a.chunk_pairs = chunk_pairs_of(level1);
    a.n_chunks = (level1 + a.chunk_pairs - 1) / a.chunk_pairs;
    a.n_part_blocks = std::min<int64_t>(a.n_chunks, kMaxPartBlocks);  // a chunk each: 13 blocks of 800 with two held up the rest
    a.budget = invert_pair_budget(a.N, a.K, a.V);
    a.n_slices = invert_slices(a.N, a.K, a.V);
    if (a.n_slices > kMaxSlices) return hipErrorInvalidValue;  // cannot happen: at most 11 by construction
    const int64_t n_hist = (int64_t)a.n_buckets * a.n_part_blocks;
    a.part_total = a.part_hist + n_hist;  // one extra word: scanning n_hist + 1 entries leaves the grand total there
    {
        ProfScope prof(PROF_INDEX, stream);
        hipLaunchKernelGGL(part_count_kernel, dim3((unsigned)a.n_part_blocks), dim3(kThreads), 0, stream, a);
        if (!check()) return e;
        if ((e = launch_scan(a.part_hist, n_hist + 1, a.block_sums, stream)) != hipSuccess) return e;
        hipLaunchKernelGGL(plan_slices_kernel, dim3(1), dim3(kScanThreads), 0, stream, a);
        if (!check()) return e;
    }
    for (int32_t j = 0; j < a.n_slices; ++j) {
        if (j > 0 && a.smp.packed && (e = launch_pack_alias(a.smp, stream)) != hipSuccess) return e;  // it lies where the pairs are filed
        a.slice = j;
        a.hot_count = a.slice_hot + j;
        {
            ProfScope prof(PROF_INDEX, stream);
            if (scatter && j == 0) {  // the correct items' rows ride at the head of the first filing launch
                const int64_t sc_blocks = pos_scatter_blocks(scatter->N);
                const dim3 grid((unsigned)(a.n_part_blocks + sc_blocks));
                switch (scatter->d) {
                case 64: hipLaunchKernelGGL((part_scatter_kernel<P, 64>), grid, dim3(kThreads), 0, stream, a, *scatter, sc_blocks); break;
                case 128: hipLaunchKernelGGL((part_scatter_kernel<P, 128>), grid, dim3(kThreads), 0, stream, a, *scatter, sc_blocks); break;
                case 256: hipLaunchKernelGGL((part_scatter_kernel<P, 256>), grid, dim3(kThreads), 0, stream, a, *scatter, sc_blocks); break;
                default: return hipErrorInvalidValue;
                }
            } else {
                hipLaunchKernelGGL((part_scatter_kernel<P, 0>), dim3((unsigned)a.n_part_blocks), dim3(kThreads), 0, stream, a, TileArgs{}, 0);
            }
            if (!check()) return e;
            hipLaunchKernelGGL((bucket_sort_kernel<P>), dim3((unsigned)a.n_buckets), dim3(kScanThreads), 0, stream, a);
            if (!check()) return e;
        }
        e = bf16 ? launch_item_dE_by_width<uint16_t, P>(a, stream) : launch_item_dE_by_width<float, P>(a, stream);
        if (e != hipSuccess) return e;
    }
    if (a.n_slices > 1) {  // buckets too crowded for any slice, if there are any
        ProfScope prof(PROF_ITEM_DE, stream);
        a.smp.packed = nullptr;  // under the pairs of the last slice
        if (bf16) hipLaunchKernelGGL(hot_bucket_kernel<uint16_t>, dim3((unsigned)a.n_part_blocks), dim3(kThreads), 0, stream, a);
        else hipLaunchKernelGGL(hot_bucket_kernel<float>, dim3((unsigned)a.n_part_blocks), dim3(kThreads), 0, stream, a);
        if (!check()) return e;
    }
    return hipSuccess;
}
}  // namespace

hipError_t launch_inverted_dE(bool bf16, const InvertArgs &a_in, const TileArgs *scatter, hipStream_t stream)
{
    InvertArgs a = a_in;
    if (a.N == 0) return hipSuccess;
    if (a.K == 0) return scatter ? launch_pos_scatter(*scatter, stream) : hipSuccess;
    const int64_t pairs = a.N * a.K;
    hipError_t e;
    auto check = [&]() { return (e = hipGetLastError()) == hipSuccess; };
    if (!invert_partitioned(a.V)) {
        // catalogue too large for the LDS bucket histogram (the caller only comes here when all pairs fit the budget):
        // counting sort with integer atomics on the V-word table, one running array over all items
        a.slice_of = nullptr;
        a.bucket_start = nullptr;
        {
            ProfScope prof(PROF_INDEX, stream);
            if (scatter && (e = launch_pos_scatter(*scatter, stream)) != hipSuccess) return e;
            const unsigned pair_blocks = (unsigned)((pairs + kThreads - 1) / kThreads);
            if ((e = launch_fill_zero(a.cursor, (size_t)a.V, stream)) != hipSuccess) return e;
            hipLaunchKernelGGL(count_kernel, dim3(pair_blocks), dim3(kThreads), 0, stream, a);
            if (!check()) return e;
            if ((e = launch_scan(a.cursor, a.V, a.block_sums, stream)) != hipSuccess) return e;
            hipLaunchKernelGGL(fill_kernel, dim3(pair_blocks), dim3(kThreads), 0, stream, a);
            if (!check()) return e;
        }
        return bf16 ? launch_item_dE_by_width<uint16_t, WidePair>(a, stream) : launch_item_dE_by_width<float, WidePair>(a, stream);
    }
    return invert_narrow(a.N, a.V) ? launch_sliced_dE<NarrowPair>(bf16, a, scatter, stream) : launch_sliced_dE<WidePair>(bf16, a, scatter, stream);
}

}  // namespace cce
