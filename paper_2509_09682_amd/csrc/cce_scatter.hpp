// Scatter of the correct items' gradient rows, shared by the matrix-core kernels and the per-position path.
#pragma once
#include "cce_device.hpp"
#include "cce_kernels.hpp"

namespace cce {

// Position row of compacted index x (identity when there is no mask).
__device__ __forceinline__ int64_t pos_row(const TileArgs &a, int64_t x) { return a.idx ? (int64_t)a.idx[x] : x; }

// dE of the correct items: dE[tgt_i] += coef_i * H_i.  Targets follow a power law, so plain atomics would serialise
// on a few hot rows (an atomic on one address completes every ~25 ns).  A block sorts 256 (target, position) pairs in
// LDS; every wavefront then walks up to 64 consecutive sorted pairs with lane = column, sums runs of equal targets in
// registers and issues one row of atomics per run.  These blocks ride at the head of another launch (the dE pass of the
// matrix-core path, the second index pass of the per-position path), so that their latency (sort, dependent gathers)
// hides under that launch's own work.
//
// A block is a chain of latencies: vector-memory operations complete in order, so the rows of a batch wait for the
// atomics of the batch before (a wavefront with four batches of 16 rows: 31 us at d = 256, whatever else runs).  With
// few chunks kPosParts blocks therefore sort the same pairs and take a share each, one batch per wavefront (13 us);
// runs of equal targets are cut more often that way, and the blocks take slots, so many chunks go whole.  Where the
// scatter is a launch of its own, many chunks are of 1024 pairs: longer runs, fewer rows of atomics (largest workload:
// 60 k instead of 78 k).  Launch with the dH scaling at d = 256, us, whole 1024 / shared 256: 1000 positions 45 / 13,
// 3200: 52 / 15, 32,768: 53 / 34, 65,536: 66 / 62, 204,800: 202 / 213.
constexpr int kPosChunk = 256;        // pairs per chunk
constexpr int kPosChunkApart = 1024;  // pairs per chunk of the stand-alone scatter kernels with many positions
constexpr int kPosParts = 4;
constexpr int64_t kPosApartAbove = 65536;  // stand-alone: positions from which chunks are long and whole
// Riding in another launch: positions up to which blocks share a chunk.  dE launch, us, whole / shared: 3200 positions, d = 64:
// 19 / 14; 8000, d = 320: 100 / 52.  Steps above the line, K = 1024, bf16: tiles, d = 64, 10,880 positions 50.1 / 50.2, 12,800
// 55.5 / 55.5, 25,600 63.4 / 66.2; d = 128 72.0 / 72.1, 76.2 / 77.6, 97.9 / 101.9.  The line is that of the tiles; the dense
// kernels and the index passes differ: d = 320, 10,880: 199 / 160, 25,600: 275 / 249, 51,200: 436 / 467; fp32 d = 64, 25,600:
// 148 / 150; buckets of fp32 d = 128, 25,600: 117 / 136; per position, d = 128, K = 128, 25,600: 403 / 395.
constexpr int64_t kPosShareBelow = 8192;
__host__ __device__ inline int pos_parts(int64_t N) { return N <= kPosShareBelow ? kPosParts : 1; }
inline int64_t pos_scatter_blocks(int64_t N) { return (N + kPosChunk - 1) / kPosChunk * pos_parts(N); }

template <int D, int CHUNK = kPosChunk>
__device__ __forceinline__ void pos_scatter_block(const TileArgs &a, int64_t block, uint64_t *keys, int parts)
{
    const int64_t chunk = block / parts;
    const int part = (int)(block % parts), pairs = 64 / parts;  // pairs per wavefront
    constexpr int CPL = D / 64;         // columns per lane
    constexpr int kPosBatch = 16;        // rows in flight per wavefront
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n_pos = a.n_valid_ptr ? (int64_t)*a.n_valid_ptr : a.N;
    const int64_t base = chunk * CHUNK;
    if (base >= n_pos) return;
    const bool sorter = tid < CHUNK;  // blocks of more threads than pairs: the rest only keep the barriers company
    if (sorter) {
        uint64_t key = ~0ull;  // padding sorts last
        if (base + tid < n_pos) {
            const int64_t row = pos_row(a, base + tid);
            if (!a.pos_mask || a.pos_mask[row] != 0) {  // ids of padded positions are never read
                const int32_t ti = a.tgt[row];
                if (!a.validate || (ti >= 0 && (int64_t)ti < a.V)) key = ((uint64_t)(uint32_t)ti << 32) | (uint32_t)row;
            }
        }
        keys[tid] = key;
    }
    __syncthreads();
    for (int k = 2; k <= CHUNK; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int partner = tid ^ j;
            if (sorter && partner > tid) {
                const uint64_t ka = keys[tid], kb = keys[partner];
                const bool up = ((tid & k) == 0);
                if ((ka > kb) == up) {
                    keys[tid] = kb;
                    keys[partner] = ka;
                }
            }
            __syncthreads();
        }
    }

    if (!sorter) return;  // no barrier below this point
    float accv[CPL];
#pragma unroll
    for (int t = 0; t < CPL; ++t) accv[t] = 0.f;
    uint32_t cur = 0xffffffffu;
    auto flush = [&]() {
        if (cur != 0xffffffffu) {
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                unsafeAtomicAdd(a.dE + (int64_t)cur * D + t * 64 + lane, accv[t]);  // an instruction covers 64 consecutive floats
                accv[t] = 0.f;
            }
        }
    };
    // lane l holds pair l of the wavefront's sorted pairs and its coefficient; the walk broadcasts them lane by lane
    const uint64_t my_key = keys[(part * (CHUNK / 64) + wave) * pairs + (lane & (pairs - 1))];
    const uint32_t my_id = (uint32_t)(my_key >> 32), my_row = (uint32_t)my_key;
    const float my_cf = (my_id != 0xffffffffu) ? a.coef[my_row] * ((a.g_separate && a.g) ? a.g[my_row] : 1.f) : 0.f;
    for (int b = 0; b < pairs; b += kPosBatch) {
        uint32_t id[kPosBatch];
        float hv[kPosBatch][CPL];
#pragma unroll
        for (int u = 0; u < kPosBatch; ++u) {
            id[u] = __builtin_amdgcn_readlane(my_id, b + u);
            const uint32_t row = __builtin_amdgcn_readlane(my_row, b + u);
#pragma unroll
            for (int t = 0; t < CPL; ++t) hv[u][t] = 0.f;
            if (id[u] != 0xffffffffu) {
#pragma unroll
                for (int t = 0; t < CPL; ++t) hv[u][t] = load1(a.H + (int64_t)row * D + t * 64 + lane);
            }
        }
#pragma unroll
        for (int u = 0; u < kPosBatch; ++u) {
            if (id[u] != cur) {
                flush();
                cur = id[u];
            }
            const float cf = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_cf), b + u));
#pragma unroll
            for (int t = 0; t < CPL; ++t) accv[t] = fmaf(cf, hv[u][t], accv[t]);
        }
    }
    flush();
}

}  // namespace cce
