// Matrix-core kernels in fp32 precision for shared candidate lists: fp32 inputs of any hidden size, and bf16 inputs of
// the hidden sizes the bf16-weight tiles (cce_tile_body.hpp) do not serve.
//
// The row-gather kernels recompute a dot product per (position, candidate) pair on the vector units and move every
// candidate row once per position.  With one list for many positions both are contractions; here they run on the matrix
// cores without giving up a bit of the arithmetic:
//   scores   bf16 rows: v_mfma_f32_32x32x16_bf16 (products exact, fp32 sums); fp32 rows: v_mfma_f32_16x16x4_f32.
//   weights  stay fp32.  For the second product with bf16 rows a weight is cut into three bf16 pieces (8 + 8 + 8
//            significant bits: the cut is exact), which meet the rows in three matrix instructions.  Three instructions
//            of the bf16 rate are five times as fast as one of the fp32 rate.
// One kernel template serves both directions, as in the bf16-weight family: a stationary operand X (one row per lane
// column, in registers), a streamed operand Y (tiles through LDS), S = Y X^T, W = f(S), acc += Y^T W.
//   position side (DM_FWD / DM_FDH / DM_DH): X = hidden states, Y = candidate rows.
//   candidate side (DM_DE):                  X = candidate rows, Y = hidden states.
// The correct item is never a column: a column that holds it is dropped (collision mask; always in full-catalogue mode)
// and the item enters by its own score, which also is the first reference of the exponentials, so that a sum of
// weights is at least one and no empty maximum exists.
//
// Above a hidden size of 192 (bf16) the accumulators of a whole row do not fit beside the stationary row: DS wavefronts
// share the rows and keep 1/DS of the output columns each.  A score is formed once: a wavefront takes its share of a score
// block (quads of 16 x 16), cuts the weights into pieces and files them in LDS, where the others read them (12,800 positions,
// K = 1024, d = 512: position side 158 -> 95 us, candidate side 254 -> 172).
//
// Bound: the matrix pipe on large problems (fp32, 5120 positions, 9000 items, d = 192: position side 347 us, 102 of 157
// TFLOP/s; bf16, 46,080 positions, K = 1024, d = 320: 166 us a side, 30 % of the pipe's peak counting each of the three
// pieces; with every score formed twice and rows staged in registers 199 and 230 us), the atomics of the candidate side for
// short lists, chains of first loads below about 2000 positions.
// Steps, row-gather kernels against these: 51,200 positions, K = 1024, d = 320, bf16 8.01 / 0.33 ms; 12,800 positions,
// K = 1024, d = 64, fp32 407 / 92 us; 512 positions, K = 128, d = 64, fp32 32 / 25 us.
#pragma once
#include <atomic>
#include <type_traits>

#include "cce_device.hpp"
#include "cce_kernels.hpp"
#include "cce_scatter.hpp"

namespace cce {
namespace {

typedef __bf16 dbf16x8 __attribute__((ext_vector_type(8)));
typedef float df32x16 __attribute__((ext_vector_type(16)));
typedef float df32x4 __attribute__((ext_vector_type(4)));
typedef short ds16x4 __attribute__((ext_vector_type(4)));
typedef ds16x4 __attribute__((address_space(3))) *dlds_v4;
typedef void __attribute__((address_space(3))) *dlds_ptr;
typedef const void __attribute__((address_space(1))) *dglobal_cptr;

// Four rows by sixteen columns of a tile, turned round.  The restrict qualifier gives the read an alias scope of its own;
// without one the compiler guards it with a wait for every load into LDS in flight.
__device__ __forceinline__ ds16x4 read_tr(dlds_v4 __restrict__ p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p); }

typedef uint64_t __attribute__((address_space(3))) *dlds_u64;
__device__ __forceinline__ void write_half(dlds_u64 __restrict__ p, uint2 v) { *p = (uint64_t)v.y << 32 | v.x; }  // (restrict: as above)

__device__ uint4 no_row;  // sixteen bytes of zeros: what a row that takes no part is loaded from

template <int K>
__device__ __forceinline__ void dwait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(K) : "memory"); }

enum { DM_FWD = 0, DM_FDH = 1, DM_DH = 2, DM_DE = 3 };

constexpr int kDenseThreads = 256;
constexpr int kDenseScatter = kPosChunk;
constexpr float kRescaleAbove = 20.f;  // a score this far above the reference moves it (weights stay below e^20)

// KD: hidden size rounded up, in units of 32.
template <typename T, int KD, int MODE>
struct DenseGeo {
    static constexpr bool B16 = sizeof(T) == 2;
    static constexpr int XR = B16 ? 32 : 16;  // stationary rows per wavefront
    static constexpr int DS = MODE == DM_FWD ? 1 : B16 ? (KD <= 6 ? 1 : (KD <= 12 ? 2 : 4)) : (KD <= 10 ? 1 : 2);
    static constexpr int NW = kDenseThreads / 64;
    static constexpr int XPB = NW / DS * XR;  // stationary rows per block
    static constexpr int BY = dense_tile_rows(B16, KD * 32);    // streamed rows per tile
    static constexpr int CPR = KD * 2 * (int)sizeof(T);        // 16-byte chunks of a padded row
    // LDS row pitch in chunks.  Odd: the 128-bit operand reads of 16 consecutive rows fall on 16 different chunk slots.
    // Not 1 or 15 modulo 16 for bf16: the transpose reads (4 rows x 4 chunks at once) then meet at most two to a slot.
    static constexpr int PITCH = CPR + ((B16 && KD % 4 == 0) ? 3 : 1);
    static constexpr int BUF = (BY * PITCH + 63) / 64 * 64;  // chunks per tile buffer, in whole load instructions
    // EX: the DS wavefronts of a group of stationary rows form a quarter (DS = 4) or half (DS = 2) of a score block each, in
    // quads of 16 x 16, and exchange the weights through LDS.
    static constexpr bool EX = B16 && DS > 1;
    static constexpr int NG = DS == 2 ? 2 : 1;  // EX: quads of a wavefront, side by side (16 stationary rows each)
    static constexpr int NX = EX ? NG * KD : 2 * KD;  // 16-byte pieces of stationary rows a lane holds
    static constexpr int EXQ = NW / DS * 3 * 4 * 32;  // EX: chunks of the exchange, (piece, eight streamed rows, stationary row)
    static constexpr int OC = B16 ? 32 : 16;           // output columns per accumulator block
    static constexpr int OB = KD * 32 / OC / DS;       // accumulator blocks per wavefront
    // DIRECT: the streamed rows go straight into LDS, short rows through registers.  A direct load is cheap to wait for and
    // holds no register, but its address takes three times the arithmetic (a chunk of padding after every row).  Position side,
    // us, through registers / direct: 1000 positions, 9000 items, d = 48, bf16 26.8 / 29.7; scoring 2000 positions, 20,000
    // items, d = 128, fp32 109 / 117; 5120 positions, K = 1024, d = 192, fp32 57.1 / 57.4; 3000 positions, 9000 items, d = 256,
    // fp32 358 / 348; 3000 positions, 20,000 items, d = 320, bf16 289 / 265.
    static constexpr bool DIRECT = KD >= 8;
    static constexpr int LPT = DIRECT ? BUF / 64 : (BY * CPR + kDenseThreads - 1) / kDenseThreads;  // load instructions per tile / per thread
    // Tiles requested ahead: two where three buffers leave room for two blocks per compute unit.
    static constexpr int PF = !DIRECT ? 1 : 3 * BUF * 16 + (EX ? EXQ * 16 : 0) + 3072 <= 80 * 1024 ? 2 : 1;
    static constexpr int IDS = PF + 2;                       // tiles whose row numbers (and constants) are at hand
    typedef typename std::conditional<B16, df32x16, df32x4>::type acc_t;
    static constexpr int AQ = B16 ? 4 : 1;  // groups of four consecutive columns in an accumulator block
    static constexpr int EPI = NW * XR * 33 / 4 + 1;  // chunks of the transpose buffers of the candidate side
    static constexpr int KEYS = kDenseScatter / 2;    // chunks of the sort keys of a scatter block
    static constexpr int LDS_TILES = (PF + 1) * BUF > EPI ? (PF + 1) * BUF : EPI;
    static constexpr int LDS = LDS_TILES > KEYS ? LDS_TILES : KEYS;
};

__device__ __forceinline__ dbf16x8 as_b8(uint4 v)
{
    dbf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// A barrier of the block that orders LDS accesses and does not wait for global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Fp32 weights as three bf16 operands whose sum they are, exactly (up to weights below 2^-110).
__device__ __forceinline__ void split3(const float (&v)[4], uint2 (&pl)[3])
{
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[0][i] = __float_as_uint(v[i]);
        const float r = v[i] - __uint_as_float(w[0][i] & 0xffff0000u);
        w[1][i] = __float_as_uint(r);
        w[2][i] = __float_as_uint(r - __uint_as_float(w[1][i] & 0xffff0000u));
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
        pl[p] = make_uint2(__builtin_amdgcn_perm(w[p][1], w[p][0], 0x07060302u), __builtin_amdgcn_perm(w[p][3], w[p][2], 0x07060302u));
}
__device__ __forceinline__ void split3(const float *v, uint4 (&pl)[3])
{
    uint32_t a[8], b[8], c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = __float_as_uint(v[i]);
        const float r = v[i] - __uint_as_float(a[i] & 0xffff0000u);
        b[i] = __float_as_uint(r);
        c[i] = __float_as_uint(r - __uint_as_float(b[i] & 0xffff0000u));
    }
    auto pack = [](const uint32_t (&w)[8]) {  // the upper halves of eight words
        return make_uint4(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u),
                          __builtin_amdgcn_perm(w[5], w[4], 0x07060302u), __builtin_amdgcn_perm(w[7], w[6], 0x07060302u));
    };
    pl[0] = pack(a);
    pl[1] = pack(b);
    pl[2] = pack(c);
}

__device__ __forceinline__ void widen4(const float *p, float (&v)[4])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}
__device__ __forceinline__ void widen4(const uint16_t *p, float (&v)[4])
{
    const uint2 a = *reinterpret_cast<const uint2 *>(p);
    v[0] = bf16_lo(a.x); v[1] = bf16_hi(a.x); v[2] = bf16_lo(a.y); v[3] = bf16_hi(a.y);
}

__device__ __forceinline__ void store_dH4(const DenseArgs &a, int64_t row, int col, const float (&v)[4])
{
    if (a.dH_bf16)
        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(a.dH) + row * a.d + col) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    else
        *reinterpret_cast<float4 *>(static_cast<float *>(a.dH) + row * a.d + col) = make_float4(v[0], v[1], v[2], v[3]);
}

// Positions a launch works on, before compaction and masks: slots [0, n).
__device__ __forceinline__ int64_t dense_slots(const DenseArgs &a) { return a.n_valid_ptr ? (int64_t)*a.n_valid_ptr : a.N; }
// Row of a slot; -1 when the position takes no part.
__device__ __forceinline__ int32_t dense_row(const DenseArgs &a, int64_t x)
{
    if (a.order) {
        const int64_t r = a.order[x];
        return (r >= 0 && r < a.n_rows) ? (int32_t)r : -1;
    }
    if (a.idx) return a.idx[x];
    return (a.mask && a.mask[x] == 0) ? -1 : (int32_t)x;
}

// Target of the position in slot x (row `row`).
__device__ __forceinline__ int32_t dense_tgt(const DenseArgs &a, int64_t x, int32_t row) { return a.tgt_slot ? a.tgt_slot[x] : a.tgt[row]; }

// Bucket a block belongs to: largest b with start[b] <= block (start ascends, start[0] = 0, stride of 3 words).
__device__ __forceinline__ int dense_bucket(const int32_t *start, int n, int32_t block)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[3 * mid] <= block) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// dE of the correct items: as pos_scatter_block (see there), for any hidden size and either type.
template <typename T, int CPL>
__device__ __forceinline__ void dense_scatter_block(const DenseArgs &a, int64_t block, uint64_t *keys)
{
    constexpr int BATCH = CPL <= 4 ? 16 : 8;  // rows in flight per wavefront
    const int parts = pos_parts(a.N), part = (int)(block % parts), pairs = 64 / parts;
    const int64_t chunk = block / parts;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n_pos = dense_slots(a), x = chunk * kDenseScatter + tid;
    if (chunk * kDenseScatter >= n_pos) return;
    uint64_t key = ~0ull;
    if (x < n_pos) {
        const int32_t row = dense_row(a, x);
        if (row >= 0) key = ((uint64_t)(uint32_t)dense_tgt(a, x, row) << 32) | (uint32_t)x;
    }
    keys[tid] = key;
    __syncthreads();
    for (int k = 2; k <= kDenseScatter; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int partner = tid ^ j;
            if (partner > tid) {
                const uint64_t ka = keys[tid], kb = keys[partner];
                if ((ka > kb) == ((tid & k) == 0)) {
                    keys[tid] = kb;
                    keys[partner] = ka;
                }
            }
            __syncthreads();
        }
    }
    const uint64_t mine = keys[(part * (kDenseScatter / 64) + wave) * pairs + (lane & (pairs - 1))];
    const uint32_t my_id = (uint32_t)(mine >> 32), my_x = (uint32_t)mine;
    int32_t my_row = 0;
    float my_cf = 0.f;
    if (my_id != 0xffffffffu) {
        my_row = dense_row(a, my_x);
        my_cf = a.coef[a.by_slot ? (int64_t)my_x : (int64_t)my_row] * ((a.g_separate && a.g) ? a.g[my_row] : 1.f);
    }
    float sum[CPL];
#pragma unroll
    for (int t = 0; t < CPL; ++t) sum[t] = 0.f;
    uint32_t cur = 0xffffffffu;
    auto flush = [&]() {
        if (cur == 0xffffffffu) return;
#pragma unroll
        for (int t = 0; t < CPL; ++t) {
            if (t * 64 + lane < a.d) unsafeAtomicAdd(a.dE + (int64_t)cur * a.d + t * 64 + lane, sum[t]);
            sum[t] = 0.f;
        }
    };
    const T *Hp = static_cast<const T *>(a.H);
    for (int b = 0; b < pairs; b += BATCH) {
        float hv[BATCH][CPL];
        uint32_t id[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            id[u] = __builtin_amdgcn_readlane(my_id, b + u);
            const int32_t row = __builtin_amdgcn_readlane(my_row, b + u);
#pragma unroll
            for (int t = 0; t < CPL; ++t) {
                hv[u][t] = 0.f;
                if (id[u] != 0xffffffffu && t * 64 + lane < a.d) hv[u][t] = load1(Hp + (int64_t)row * a.d + t * 64 + lane);
            }
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (id[u] != cur) {
                flush();
                cur = id[u];
            }
            const float cf = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_cf), b + u));
#pragma unroll
            for (int t = 0; t < CPL; ++t) sum[t] = fmaf(cf, hv[u][t], sum[t]);
        }
    }
    flush();
}

// dH = grad_loss * U of valid positions, zero rows for the others; four columns per thread and turn.  Without U (a dH
// pass of its own went ahead) the zero rows only.
__device__ __forceinline__ void dense_scale_block(const DenseArgs &a, int64_t block)
{
    const int cpr = a.d / 4;
    const int64_t total = a.N * (int64_t)cpr;
#pragma unroll
    for (int j = 0; j < kDenseScaleTurns; ++j) {
        const int64_t e = (block * kDenseScaleTurns + j) * kDenseThreads + threadIdx.x;
        if (e >= total) return;
        const int64_t i = e / cpr;
        const int col = (int)(e % cpr) * 4;
        bool valid = a.pos_mask == nullptr || a.pos_mask[i] != 0;
        if (valid && a.validate) valid = a.tgt[i] >= 0 && (int64_t)a.tgt[i] < a.V;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if (valid) {
            if (!a.U) continue;
            const float g = a.g ? a.g[i] : 1.f;
            widen4(a.U + i * a.d + col, v);
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] *= g;
        }
        store_dH4(a, i, col, v);
    }
}

// What a position's sums become: lse, loss, the correct item's coefficient and what the candidate side needs.
// sn: weights of the negatives relative to exp(ref); op: score of the correct item.
__device__ __forceinline__ float dense_finish(const DenseArgs &a, int64_t x, int32_t row, float ref, float sn, float op, bool files)
{
    const float wp = fast_exp(op - ref), s = sn + wp;
    const float l2 = fast_log(s);
    a.lse[row] = ref + l2;
    a.loss[row] = (ref - op) + l2;
    const float inv = 1.f / s;
    if (files) {
        const int64_t at = a.by_slot ? x : (int64_t)row;
        a.coef[at] = -sn * inv;  // p+ - 1, without the cancellation
        a.ref[at] = ref;
        a.inv[at] = inv;
    }
    return inv;
}

// A column of U: inv * sum + (p+ - 1) E_tgt.  The item's -1 stays exact while p+ is small (it is most of the row then);
// near one the difference comes as ct = -negatives / all, without cancellation.
__device__ __forceinline__ float dense_row_value(float sum, float inv, float pp, float ct, float et)
{
    return fmaf(sum, inv, pp <= 0.5f ? fmaf(pp, et, -et) : ct * et);
}

// min two blocks of four wavefronts per compute unit: 256 registers a lane
template <typename T, int KD, int MODE>
__global__ __launch_bounds__(kDenseThreads, 2) void dense_kernel(DenseArgs a)
{
    typedef DenseGeo<T, KD, MODE> G;
    constexpr bool DE = MODE == DM_DE, B16 = G::B16, EX = G::EX;
    constexpr int NG = G::NG;
    constexpr int BY = G::BY, XR = G::XR, OB = G::OB;
    __shared__ uint4 lds[G::LDS];
    __shared__ __align__(16) int32_t ids[G::IDS][BY];                     // candidate ids / position rows of the tile, -1: no part
    __shared__ float4 cst[DE ? G::IDS : 1][DE ? BY / 4 * 3 : 1];  // candidate side: reference, weight factor, target of a row
    __shared__ uint4 xch[EX ? G::EXQ : 1];                   // EX: weights of the score blocks at hand
    __shared__ float xsum[EX && !DE ? G::NW / G::DS * 2 * 32 : 1];  // EX: a number per stationary row and half of the streamed rows
    __shared__ int32_t xflag[EX && !DE ? 2 : 1];             // EX: a score has outgrown its reference (by parity of the tile)

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lo = lane & (XR - 1), hi = lane / XR;  // column of the stationary operand, share of the reduction index
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    const int sl = wave % G::DS, xg = wave / G::DS;
    const int l16 = lane & 15, h16 = lane >> 4;                               // EX: stationary row of a quad, its four streamed rows
    const int xhalf = sl & 1, xcol = (G::DS == 4 ? sl >> 1 : 0) * 16 + l16;  // EX: streamed half, first stationary row of this lane
    int64_t block = blockIdx.x;
    if (DE) {
        if (block < a.scatter_blocks) {
            dense_scatter_block<T, (KD + 1) / 2>(a, block, reinterpret_cast<uint64_t *>(lds));
            return;
        }
        block -= a.scatter_blocks;
        if (block >= a.tile_blocks) {
            dense_scale_block(a, block - a.tile_blocks);
            return;
        }
    }
    const T *Hp = static_cast<const T *>(a.H), *Ep = static_cast<const T *>(a.E);
    const int32_t *neg = a.neg;

    // ---- what the block works on: stationary rows [x0, x0 + XPB) of nx, streamed rows [y0, y1)
    int64_t pos0 = 0, pos1 = dense_slots(a), split, xb;
    if (a.tab) {  // buckets of positions, each with a list of its own
        const int b = dense_bucket(a.tab + (DE ? 2 : 1), a.n_buckets, (int32_t)(DE ? block : blockIdx.x));
        pos0 = a.tab[3 * b];
        pos1 = a.tab[3 * b + 3];
        neg += (int64_t)b * a.n_cols;
        const int64_t in = (DE ? block : (int64_t)blockIdx.x) - a.tab[3 * b + (DE ? 2 : 1)];
        xb = DE ? in % a.x_blocks : in;
        split = DE ? in / a.x_blocks : (int64_t)blockIdx.y;
    } else {
        xb = DE ? block % a.x_blocks : block;
        split = DE ? block / a.x_blocks : (int64_t)blockIdx.y;
    }
    const int64_t nx = DE ? a.n_cols : pos1 - pos0, ny = DE ? pos1 - pos0 : a.n_cols;
    const int64_t x0 = xb * G::XPB;
    int64_t tiles = (ny + BY - 1) / BY, t0, t1;
    if (DE && a.tab) {
        t0 = split * a.tiles_per_split;
        t1 = t0 + a.tiles_per_split < tiles ? t0 + a.tiles_per_split : tiles;
    } else {
        const int64_t per = (tiles + a.splits - 1) / a.splits;
        t0 = split * per;
        t1 = t0 + per < tiles ? t0 + per : tiles;
    }
    if (x0 >= nx) return;
    if (DE && t0 >= t1) return;  // (the position side still files an empty share)

    // ---- stationary row of this lane
    const int64_t x = x0 + xg * XR + lo;
    int32_t xrow = -1;  // row number in H (position side) or E (candidate side)
    int32_t ti = -1;
    if (x < nx) {
        if (DE) {
            xrow = neg ? neg[x] : (int32_t)x;
            if (a.validate && (xrow < 0 || (int64_t)xrow >= a.V)) xrow = -1;
        } else {
            xrow = dense_row(a, pos0 + x);
            if (xrow >= 0) ti = dense_tgt(a, pos0 + x, xrow);
        }
    }
    const int dch = a.d * (int)sizeof(T) / 16;  // 16-byte chunks of a row
    uint4 xr[G::NX];
    if constexpr (EX) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int32_t row = __shfl(xrow, xcol + 16 * g, 64);
            const uint4 *src = reinterpret_cast<const uint4 *>((DE ? Ep : Hp) + (int64_t)(row < 0 ? 0 : row) * a.d);
#pragma unroll
            for (int k = 0; k < KD; ++k) {
                const int ch = k * 4 + h16;
                xr[g * KD + k] = make_uint4(0, 0, 0, 0);
                if (row >= 0 && ch < dch) xr[g * KD + k] = src[ch];
            }
        }
    } else {
        const uint4 *src = reinterpret_cast<const uint4 *>(DE ? Ep + (int64_t)(xrow < 0 ? 0 : xrow) * a.d : Hp + (int64_t)(xrow < 0 ? 0 : xrow) * a.d);
#pragma unroll
        for (int k = 0; k < G::NX; ++k) {
            const int ch = k * (64 / XR) + hi;
            xr[k] = make_uint4(0, 0, 0, 0);
            if (xrow >= 0 && ch < dch) xr[k] = src[ch];
        }
    }
    float op = 0.f, ref = 0.f;
    auto dot16 = [](uint4 e, uint4 x) {  // 16 bytes of two rows
        const uint32_t ew[4] = {e.x, e.y, e.z, e.w}, xw[4] = {x.x, x.y, x.z, x.w};
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (B16) {
                part = fmaf(bf16_lo(xw[t]), bf16_lo(ew[t]), part);
                part = fmaf(bf16_hi(xw[t]), bf16_hi(ew[t]), part);
            } else {
                part = fmaf(__uint_as_float(xw[t]), __uint_as_float(ew[t]), part);
            }
        }
        return part;
    };
    const bool drop_own = a.drop_own != 0;
    const int32_t x_drop = drop_own ? (DE ? xrow : ti) : -2;  // a column of the other kind with this number takes no part
    float qref[EX ? NG : 1], qsn[EX ? NG : 1];                // EX: reference and sum of the stationary rows of this wavefront's quads
    int32_t qdrop[EX ? NG : 1];
    if constexpr (EX) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            qsn[g] = qref[g] = 0.f;
            qdrop[g] = __shfl(x_drop, xcol + 16 * g, 64);
            if (DE) continue;
            const int32_t own = __shfl(ti, xcol + 16 * g, 64);
            const bool on = __shfl(xrow, xcol + 16 * g, 64) >= 0;
            const uint4 *src = reinterpret_cast<const uint4 *>(Ep + (int64_t)(own < 0 ? 0 : own) * a.d);
#pragma unroll
            for (int k = 0; k < KD; ++k) {
                uint4 e = make_uint4(0, 0, 0, 0);
                if (on && k * 4 + h16 < dch) e = src[k * 4 + h16];
                qref[g] += dot16(e, xr[g * KD + k]);
            }
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) qref[g] += __shfl_xor(qref[g], off, 64);
            if (xhalf == 0 && h16 == 0) xsum[xg * 64 + xcol + 16 * g] = qref[g];
        }
        if (!DE && tid < 2) xflag[tid] = 0;
    } else if (!DE) {  // score of the correct item
        const uint4 *src = reinterpret_cast<const uint4 *>(Ep + (int64_t)(ti < 0 ? 0 : ti) * a.d);
#pragma unroll
        for (int k = 0; k < G::NX; ++k) {
            const int ch = k * (64 / XR) + hi;
            uint4 e = make_uint4(0, 0, 0, 0);
            if (xrow >= 0 && ch < dch) e = src[ch];
            op += dot16(e, xr[k]);
        }
#pragma unroll
        for (int off = XR; off < 64; off <<= 1) op += __shfl_xor(op, off, 64);
        ref = op;
    }
    if (MODE == DM_DH) ref = xrow >= 0 ? a.lse_in[xrow] : 0.f;

    // ---- streaming: rows PF tiles ahead, their numbers one more
    // Lane e of the first wavefront fetches the number of streamed row e, and on the candidate side its constants, in two
    // steps: loads at an address that always exists, whose results nothing looks at until they are filed a tile later (a
    // check in between would wait for the load with the whole block behind it).
    const int ye = tid & (BY - 1);
    struct Raw { uint32_t lo, hi, on; };
    auto y_clamped = [&](int64_t t) -> int64_t {
        const int64_t y = t * BY + ye;
        return y < ny ? y : ny - 1;  // ny > 0
    };
    const char *none = reinterpret_cast<const char *>(&no_row);  // read in the place of a row or an array that is not there
    asm volatile("" : "+s"(none));                              // (its address is looked up once)
    auto word = [&](const void *base, int64_t at) {
        return *(const uint32_t __attribute__((address_space(1))) *)(base ? static_cast<const char *>(base) + at : none);
    };
    auto fetch_id = [&](int64_t t) -> Raw {
        const int64_t y = y_clamped(t), at = pos0 + y;
        Raw r{0u, 0u, 1u};
        if (DE) {
            r.lo = word(a.order ? static_cast<const void *>(a.order) : a.idx, at * (a.order ? 8 : 4));
            r.hi = word(a.order, at * 8 + 4);
            r.on = *(const uint8_t __attribute__((address_space(1))) *)(a.mask ? reinterpret_cast<const char *>(a.mask) + at : none);
        } else {
            r.lo = word(neg, y * 4);
        }
        return r;
    };
    auto id_of = [&](int64_t t, Raw r) -> int32_t {  // -1: takes no part
        const int64_t y = t * BY + ye;
        int32_t id;
        if (DE) {
            id = (a.order || a.idx) ? (int32_t)r.lo : (int32_t)(pos0 + y);
            if (a.order && (r.hi != 0 || (int64_t)r.lo >= a.n_rows)) id = -1;
            if (a.mask && !a.order && !a.idx && r.on == 0) id = -1;
        } else {
            id = neg ? (int32_t)r.lo : (int32_t)y;
            if (a.validate && (uint32_t)id >= (uint32_t)a.V) id = -1;
        }
        return (t < t1 && y < ny) ? id : -1;
    };
    struct Cst { uint32_t ref, g, inv, ti; };
    auto fetch_cst = [&](int64_t t, int32_t row) -> Cst {
        Cst c{0u, 0u, 0u, 0u};
        if (!DE) return c;
        const int64_t slot = pos0 + y_clamped(t), r = row < 0 ? 0 : row, at = a.by_slot ? slot : r;
        c.g = word(a.g, r * 4);
        c.inv = word(a.inv, at * 4);
        c.ti = a.tgt_slot ? word(a.tgt_slot, slot * 4) : word(a.tgt, r * 4);
        c.ref = word(a.ref, at * 4);
        return c;
    };
    auto file = [&](int slot, int32_t id, const Cst &c) {
        if (tid >= BY) return;
        ids[slot][tid] = id;
        if (!DE) return;
        float *f = reinterpret_cast<float *>(cst[DE ? slot : 0]);
        const float g = a.g ? __uint_as_float(c.g) : 1.f;
        const float w = id < 0 ? 0.f : (a.inv ? g * __uint_as_float(c.inv) : g);
        f[tid] = w != 0.f ? __uint_as_float(c.ref) : INFINITY;  // a zero factor keeps exp(-inf) = 0: no 0 * inf
        f[BY + tid] = w;
        f[2 * BY + tid] = __int_as_float(id >= 0 ? (int32_t)c.ti : -1);
    };
    // One load group: the rows of a tile.  DIRECT: the buffer is a row of chunks in the order of its pitch; an instruction
    // fills 64 of them, lane l the l-th.  Rows that take no part, columns beyond d and the chunks between rows come from a
    // chunk of zeros.  The destination is handed over as a bare offset, so that the compiler does not guard every operand read
    // with a wait for all loads in flight (landed() and the barrier behind it see to that).
    const T *Yp = DE ? Hp : Ep;
    const int32_t row_bytes = a.d * (int)sizeof(T);
    uint4 stage[G::DIRECT ? 1 : G::LPT];
    auto issue = [&](int buffer, int slot) {
        if constexpr (!G::DIRECT) {
#pragma unroll
            for (int i = 0; i < G::LPT; ++i) {
                const int c = i * kDenseThreads + tid;
                stage[i] = make_uint4(0, 0, 0, 0);
                if (c < BY * G::CPR) {
                    const int r = c / G::CPR, ch = c % G::CPR;
                    const int32_t id = ids[slot][r];
                    if (id >= 0 && ch < dch) stage[i] = reinterpret_cast<const uint4 *>(Yp + (int64_t)id * a.d)[ch];
                }
            }
            return;
        }
        uint32_t dst = (uint32_t)(uintptr_t)(dlds_ptr)(lds + buffer * G::BUF);
        asm volatile("" : "+s"(dst));
        uint32_t me = (uint32_t)tid;
        asm volatile("" : "+v"(me));  // recomputed at every tile: carried, the chunk numbers would cost a register each
        // the last wavefronts take what does not divide: the first, which also fetches the numbers, has the fewest loads in flight
        constexpr int WHOLE = G::LPT / G::NW, REST = G::LPT % G::NW, MOST = WHOLE + (REST ? 1 : 0);
        auto inst = [&](int i) { return i < WHOLE ? swave + i * G::NW : WHOLE * G::NW + swave - (G::NW - REST); };
        constexpr int AT_ONCE = MOST <= 6 ? MOST : 3;  // row numbers held at a time
#pragma unroll
        for (int i0 = 0; i0 < MOST; i0 += AT_ONCE) {
            int32_t id[AT_ONCE];
            uint32_t ofs[AT_ONCE];
#pragma unroll
            for (int j = 0; j < AT_ONCE; ++j) {
                const uint32_t c = (me & 63) + (uint32_t)(inst(i0 + j) * 64), r = c / G::PITCH, ch = c - r * G::PITCH;
                id[j] = ids[slot][r < BY ? r : BY - 1];
                if ((int)ch >= dch || r >= BY) id[j] = -1;
                ofs[j] = ch * 16;
            }
#pragma unroll
            for (int j = 0; j < AT_ONCE; ++j) {
                const int i = i0 + j;
                if (i >= MOST || (i >= WHOLE && swave < G::NW - REST)) continue;
                const char *src = reinterpret_cast<const char *>(Yp) + ((int64_t)id[j] * row_bytes + ofs[j]);
                if (id[j] < 0) src = none;
                __builtin_amdgcn_global_load_lds((dglobal_cptr)src, (dlds_ptr)(uintptr_t)(dst + (uint32_t)inst(i) * 1024u), 16, 0, 0);
            }
            if (AT_ONCE < MOST) __builtin_amdgcn_sched_barrier(0);
        }
    };
    // DIRECT: waits until at most the youngest PF - 1 load groups are in flight.  A group is requested at every tile, beyond the
    // last one of zeros, so that the counts are the same on every path.
    auto landed = [&](int buffer) {
        if constexpr (!G::DIRECT) {
            uint4 *const buf = lds + buffer * G::BUF;
#pragma unroll
            for (int i = 0; i < G::LPT; ++i) {
                const int c = i * kDenseThreads + tid;
                if (c < BY * G::CPR) buf[(c / G::CPR) * G::PITCH + c % G::CPR] = stage[i];
            }
        } else if constexpr (G::PF == 1) {
            dwait_vm<0>();
        } else {
            if (G::LPT % G::NW != 0 && swave >= G::NW - G::LPT % G::NW) dwait_vm<G::LPT / G::NW + 1>();
            else dwait_vm<G::LPT / G::NW>();
        }
    };
    Raw raw{0u, 0u, 0u};  // number of row ye of the tile after those at hand
    if (swave == 0 && ny > 0) {  // numbers of the first tiles in one round trip, their constants in another
        Raw first[G::PF + 1];
        int32_t id[G::PF + 1];
        Cst c[G::PF + 1];
#pragma unroll
        for (int q = 0; q < G::PF + 1; ++q) first[q] = fetch_id(t0 + q);
        if (DE) raw = fetch_id(t0 + G::PF + 1);
#pragma unroll
        for (int q = 0; q < G::PF + 1; ++q) {
            id[q] = id_of(t0 + q, first[q]);
            c[q] = fetch_cst(t0 + q, id[q]);
        }
#pragma unroll
        for (int q = 0; q < G::PF + 1; ++q) file(q, id[q], c[q]);
    }
    __syncthreads();
    if constexpr (EX && !DE) {
        op = xsum[xg * 64 + lo];
        if (MODE != DM_DH) ref = op;
        if (MODE == DM_DH) {
#pragma unroll
            for (int g = 0; g < NG; ++g) qref[g] = __shfl(ref, xcol + 16 * g, 64);
        }
    }
    // The stationary rows are waited for here: a load that may be in flight at the head of the loop would have the compiler
    // wait for all loads at its first use in every turn (51,200 positions, K = 1024, d = 320, bf16: candidate side 191 us, so
    // 183).  By a wait that the compiler counts in: an empty asm block that takes them tied their registers as well (52 lists of
    // 3171 candidates for 24 positions each, d = 256: candidate side 175 us, so 161).  Rows staged in registers need no such wait.
    if (G::DIRECT) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
#pragma unroll
    for (int q = 0; q < G::PF; ++q) issue(q, q);

    typename G::acc_t acc[MODE == DM_FWD ? 1 : OB];
    if (MODE != DM_FWD) {
#pragma unroll
        for (int b = 0; b < OB; ++b)
#pragma unroll
            for (int i = 0; i < 4 * G::AQ; ++i) acc[b][i] = 0.f;
    }
    float sn = 0.f;
    // fp32 weights of one score block (4 AQ values a lane: streamed rows row_of(i)), then the second product
    constexpr int SUB = BY / XR;  // score blocks per tile
    int slot = 0, at = 0;  // of tile t: entry of ids and cst, buffer
    // Rows staged in registers are asked for before the numbers of a later tile, and not beyond the last one: the next tile waits
    // for them.  Numbers first / rows first, us: steps of 108 positions, K = 182, d = 192, bf16 33.0 / 32.2, d = 128, fp32
    // 26.8 / 25.9; scoring 1302 positions, 299 candidates, d = 48, bf16 11.7 / 11.2; 5000 positions, K = 1024, d = 128, fp32
    // 89.8 / 91.6.  Short fp32 rows keep the numbers first on the candidate side (12,800 positions, K = 1024, d = 64: 89.5 / 91.0).
    // So do rows of 65 to 96 columns on either side, us: step of 657 positions, 25,508 items, d = 96, bf16 113.6 / 118.6; 588
    // positions, 70,369 items, fp32 525 / 535; 2560 positions, K = 2000, bf16 50.9 / 52.9; scoring 8000 positions, 17,000 items
    // 63.1 / 64.9 bf16, 282.0 / 285.6 fp32; 1302 positions, 299 candidates 12.44 / 12.51.
    constexpr bool kRowsFirst = !G::DIRECT && KD != 3 && (!DE || B16 || KD >= 4);
    landed(0);
    for (int64_t t = t0; t < t1; ++t) {
        const uint4 *buf = lds + at * G::BUF;
        lds_barrier();
        // rows of tile t + PF, into the buffer that tile t - 1 has left; position side: numbers of tile t + PF + 1; candidate side:
        // constants of that tile and numbers of the next
        const bool more = t + 1 < t1;
        int32_t id2 = -1;
        Cst c2{0u, 0u, 0u, 0u};
        if (kRowsFirst && more) issue(at == 0 ? G::PF : at - 1, (slot + G::PF) % G::IDS);
        if (swave == 0 && (MODE != DM_FWD || more || KD == 3)) {
            if (DE) {
                id2 = id_of(t + G::PF + 1, raw);
                c2 = fetch_cst(t + G::PF + 1, id2);
            }
            raw = fetch_id(t + G::PF + (DE ? 2 : 1));
        }
        if (!kRowsFirst) issue(at == 0 ? G::PF : at - 1, (slot + G::PF) % G::IDS);
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb) {
            uint4 *const xq = xch + xg * (3 * 4 * 32);
            float v[4 * G::AQ];
            // operands of the second product for half c of the streamed rows, one per block of output columns: rows hi 4 + j / 4
            // and 8 below (j: lane of sixteen; EX, odd hi: the other way round), columns of this lane's half of a block of 32
            uint4 ya[EX ? 2 : 1][OB];
            auto read_operand = [&](int c, int b) {
                const uint16_t *tb = reinterpret_cast<const uint16_t *>(buf) + (c * 16 + hi * 4 + (l16 >> 2)) * (G::PITCH * 8) +
                                     sl * OB * 32 + (h16 & 1) * 16 + (l16 & 3) * 4;
                const int turn = EX ? hi * 8 * (G::PITCH * 8) : 0;
                const ds16x4 r0 = read_tr((dlds_v4)(tb + b * 32 + turn)), r1 = read_tr((dlds_v4)(tb + b * 32 + 8 * (G::PITCH * 8) - turn));
                uint4 y;
                __builtin_memcpy(&y.x, &r0, 8);
                __builtin_memcpy(&y.z, &r1, 8);
                return y;
            };
            auto read_half = [&](int c, uint4 (&y)[OB]) {
#pragma unroll
                for (int b = 0; b < OB; ++b) y[b] = read_operand(c, b);
            };
            if constexpr (EX) {
                // quads of the score block: streamed rows 16 xhalf + 4 h16 + r, stationary rows xcol + 16 g
                df32x4 s[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) s[g] = df32x4{0.f, 0.f, 0.f, 0.f};
                const uint4 *arow = buf + (xhalf * 16 + l16) * G::PITCH + h16;
                // Operands well ahead of their use: left to itself the compiler reads two at a time and waits for each pair.  All
                // of them at once, or two batches in flight where that would spill.
                constexpr int OPS = (!DE && KD == 10) ? 4 : KD, BATCHES = (KD + OPS - 1) / OPS;
                uint4 o[BATCHES > 1 ? 2 : 1][OPS];
                auto read_ops = [&](int n) {
#pragma unroll
                    for (int k = 0; k < OPS; ++k)
                        if (n * OPS + k < KD) o[n & 1][k] = arow[(n * OPS + k) * 4];
                };
                read_ops(0);
#pragma unroll
                for (int n = 0; n < BATCHES; ++n) {
                    if (n + 1 < BATCHES) read_ops(n + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int k = 0; k < OPS; ++k)
#pragma unroll
                        for (int g = 0; g < NG; ++g)
                            if (n * OPS + k < KD)
                                s[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_b8(o[n & 1][k]), as_b8(xr[g * KD + n * OPS + k]), s[g], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                read_half(0, ya[0]);  // the first operands of the second product land under the weights
                __builtin_amdgcn_sched_barrier(0);
                const int e4 = xhalf * 4 + h16;  // four streamed rows
                // weights of a quad.  A chunk of the exchange is what one lane of the second product takes: rows hi 4 .. + 3 of a
                // half and those 8 below, for odd hi the other way round, so that a store instruction meets every bank once
                auto put = [&](int g, const float (&w)[4]) {
                    uint2 pc[3];
                    split3(w, pc);
#pragma unroll
                    for (int p = 0; p < 3; ++p)
                    {
                        write_half((dlds_u64)(reinterpret_cast<uint2 *>(xq + (p * 4 + xhalf * 2 + (h16 & 1)) * 32 + xcol + 16 * g) + ((h16 >> 1) ^ (h16 & 1))), pc[p]);
                        asm volatile("" ::: "memory");  // two stores made into one would lose their alias scope
                    }
                };
                if constexpr (DE) {
                    const float4 *cf = cst[slot];
                    const float4 r4 = cf[e4], w4 = cf[BY / 4 + e4], t4 = cf[BY / 2 + e4];
                    const float rr[4] = {r4.x, r4.y, r4.z, r4.w}, ww[4] = {w4.x, w4.y, w4.z, w4.w}, tt[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        float w[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            w[r] = ww[r] * fast_exp(s[g][r] - rr[r]);
                            if (__float_as_int(tt[r]) == qdrop[g]) w[r] = 0.f;
                        }
                        put(g, w);
                    }
                    lds_barrier();
                } else {
                    const int4 i4 = *reinterpret_cast<const int4 *>(&ids[slot][4 * e4]);
                    const int32_t ii[4] = {i4.x, i4.y, i4.z, i4.w};
                    float top[NG], part[NG];
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (ii[r] < 0 || ii[r] == qdrop[g]) s[g][r] = -INFINITY;
                        top[g] = fmaxf(fmaxf(s[g][0], s[g][1]), fmaxf(s[g][2], s[g][3]));
                    }
                    auto weigh = [&](int g) {
                        float w[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) w[r] = fast_exp(s[g][r] - qref[g]);
                        put(g, w);
                        part[g] = (w[0] + w[1]) + (w[2] + w[3]);
                    };
                    const int par = (int)(t - t0) & 1;
                    if (MODE != DM_DH) {
                        bool high = top[0] > qref[0] + kRescaleAbove;
                        if (NG == 2) high = high || top[NG - 1] > qref[NG - 1] + kRescaleAbove;
                        if (__any(high) && lane == 0) xflag[par] = 1;
                    }
#pragma unroll
                    for (int g = 0; g < NG; ++g) weigh(g);
                    lds_barrier();
                    if (MODE != DM_DH && __builtin_amdgcn_readfirstlane(xflag[par]) != 0) {
                        // rare, and the same decision in every wavefront of the block: the references move up to the largest
                        // score of the tile, the sums are rescaled and the weights formed again
#pragma unroll
                        for (int g = 0; g < NG; ++g) {
                            float m = top[g];
#pragma unroll
                            for (int off = 16; off < 64; off <<= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
                            if (h16 == 0) xsum[(xg * 2 + xhalf) * 32 + xcol + 16 * g] = m;
                        }
                        lds_barrier();
#pragma unroll
                        for (int g = 0; g < NG; ++g) {
                            const float *m = xsum + xg * 64 + xcol + 16 * g;
                            const float to = fmaxf(qref[g], fmaxf(m[0], m[32]));
                            qsn[g] *= fast_exp(qref[g] - to);
                            qref[g] = to;
                            weigh(g);
                        }
                        const float to = fmaxf(ref, fmaxf(xsum[xg * 64 + lo], xsum[xg * 64 + 32 + lo])), sc = fast_exp(ref - to);
                        ref = to;
#pragma unroll
                        for (int b = 0; b < (MODE == DM_FWD ? 0 : OB); ++b)
#pragma unroll
                            for (int i = 0; i < 4 * G::AQ; ++i) acc[b][i] *= sc;
                        lds_barrier();
                        if (tid == 0) xflag[par] = 0;
                    }
#pragma unroll
                    for (int g = 0; g < NG; ++g) qsn[g] += part[g];
                }
            } else {
            typename G::acc_t s;
#pragma unroll
            for (int i = 0; i < 4 * G::AQ; ++i) s[i] = 0.f;
            const uint4 *arow = buf + (sb * XR + lo) * G::PITCH + hi;
#pragma unroll
            for (int k = 0; k < G::NX; ++k) {
                const uint4 o = arow[k * (64 / XR)];
                if constexpr (B16) {
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_b8(o), as_b8(xr[k]), s, 0, 0, 0);
                } else {
                    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(o.x), __uint_as_float(xr[k].x), s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(o.y), __uint_as_float(xr[k].y), s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(o.z), __uint_as_float(xr[k].z), s, 0, 0, 0);
                    s = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(o.w), __uint_as_float(xr[k].w), s, 0, 0, 0);
                }
            }
            // weights: value 4 q + r belongs to streamed row sb XR + 8 q + 4 hi + r (bf16) or sb XR + 4 hi + r (fp32)
            if (DE) {
                const float4 *cf = cst[DE ? slot : 0];
#pragma unroll
                for (int q = 0; q < G::AQ; ++q) {
                    const int e4 = sb * (XR / 4) + 2 * q + hi;
                    const float4 r4 = cf[e4], w4 = cf[BY / 4 + e4], t4 = cf[BY / 2 + e4];
                    const float rr[4] = {r4.x, r4.y, r4.z, r4.w}, ww[4] = {w4.x, w4.y, w4.z, w4.w}, tt[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float w = ww[r] * fast_exp(s[4 * q + r] - rr[r]);
                        v[4 * q + r] = (__float_as_int(tt[r]) == x_drop) ? 0.f : w;
                    }
                }
            } else {
                float top = -INFINITY;
#pragma unroll
                for (int q = 0; q < G::AQ; ++q) {
                    const int4 i4 = *reinterpret_cast<const int4 *>(&ids[slot][sb * XR + 8 * q + 4 * hi]);
                    const int32_t ii[4] = {i4.x, i4.y, i4.z, i4.w};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v[4 * q + r] = (ii[r] < 0 || ii[r] == x_drop) ? -INFINITY : s[4 * q + r];
                        top = fmaxf(top, v[4 * q + r]);
                    }
                }
                if (MODE != DM_DH && __any(top > ref + kRescaleAbove)) {  // rare: move the reference up, rescale the sums
#pragma unroll
                    for (int off = XR; off < 64; off <<= 1) top = fmaxf(top, __shfl_xor(top, off, 64));
                    const float to = fmaxf(ref, top), sc = fast_exp(ref - to);
                    ref = to;
                    sn *= sc;
                    if (MODE != DM_FWD) {
#pragma unroll
                        for (int b = 0; b < OB; ++b)
#pragma unroll
                            for (int i = 0; i < 4 * G::AQ; ++i) acc[b][i] *= sc;
                    }
                }
                float part[G::AQ];
#pragma unroll
                for (int q = 0; q < G::AQ; ++q) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[4 * q + r] = fast_exp(v[4 * q + r] - ref);
                    part[q] = (v[4 * q] + v[4 * q + 1]) + (v[4 * q + 2] + v[4 * q + 3]);
                }
                if constexpr (G::AQ == 4) sn += (part[0] + part[1]) + (part[2] + part[3]);
                else sn += part[0];
            }
            }
            if (MODE == DM_FWD) continue;
            if constexpr (B16) {
                if constexpr (EX) {
                    auto read_weights = [&](int c, uint4 (&pl)[3]) {
#pragma unroll
                        for (int p = 0; p < 3; ++p) pl[p] = xq[(p * 4 + c * 2 + hi) * 32 + lo];
                    };
                    auto product = [&](int c, uint4 w) {
#pragma unroll
                        for (int b = 0; b < OB; ++b)
                            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_b8(ya[c][b]), as_b8(w), acc[b], 0, 0, 0);
                    };
                    uint4 p0[3], p1[3];
                    constexpr bool EARLY = DE || KD != 10;  // registers for all operands at once
                    read_weights(0, p0);
                    if (EARLY) read_half(1, ya[1]);
                    __builtin_amdgcn_sched_barrier(0);
                    product(0, p0[2]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (EARLY) read_weights(1, p1);
                    __builtin_amdgcn_sched_barrier(0);
                    product(0, p0[1]);
                    if (!EARLY) {
                        __builtin_amdgcn_sched_barrier(0);
                        read_weights(1, p1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    product(0, p0[0]);
                    if (!EARLY) {
                        __builtin_amdgcn_sched_barrier(0);
                        read_half(1, ya[0]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    product(EARLY ? 1 : 0, p1[2]);
                    product(EARLY ? 1 : 0, p1[1]);
                    product(EARLY ? 1 : 0, p1[0]);
                } else {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        uint4 pl[3];
                        split3(v + 8 * c, pl);
                        // an operand at a time: all of them at once take 24 registers at d = 192 (12,800 positions, K = 1024:
                        // candidate side 86 us, so 82)
#pragma unroll
                        for (int b = 0; b < OB; ++b) {
                            const uint4 y = read_operand(c, b);
#pragma unroll
                            for (int p = 2; p >= 0; --p)
                                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_b8(y), as_b8(pl[p]), acc[b], 0, 0, 0);
                        }
                    }
                }
            } else {
                const float *tb = reinterpret_cast<const float *>(buf) + (sb * XR + 4 * hi) * (G::PITCH * 4) + sl * OB * 16 + lo;
#pragma unroll
                for (int b = 0; b < OB; ++b) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(tb[r * (G::PITCH * 4) + b * 16], v[r], acc[b], 0, 0, 0);
                }
            }
        }
        if (kRowsFirst && more) landed(at == G::PF ? 0 : at + 1);
        if (swave == 0 && (!kRowsFirst || more)) file((slot + G::PF + 1) % G::IDS, DE ? id2 : id_of(t + G::PF + 1, raw), c2);
        slot = slot == G::IDS - 1 ? 0 : slot + 1;
        at = at == G::PF ? 0 : at + 1;
        if (!kRowsFirst) landed(at);
    }
    if (G::DIRECT) dwait_vm<0>();  // the groups beyond the last tile, before their buffers are used again or given back

    if constexpr (DE) {
        // rows of the candidates: blocks of 32 columns turned round in LDS, so that an atomic instruction covers 32
        // consecutive floats of two rows
        __syncthreads();
        float *tr = reinterpret_cast<float *>(lds) + wave * (XR * 33);
        constexpr int PER = 32 / G::OC;  // accumulator blocks per 32 columns
#pragma unroll
        for (int b0 = 0; b0 < OB; b0 += PER) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int b = 0; b < PER; ++b)
#pragma unroll
                for (int i = 0; i < 4 * G::AQ; ++i) tr[lo * 33 + b * G::OC + (i >> 2) * 8 + hi * 4 + (i & 3)] = acc[b0 + b][i];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int col = (sl * OB + b0) * G::OC + (lane & 31);
#pragma unroll
            for (int i = 0; i < XR / 2; ++i) {
                const int r = 2 * i + (lane >> 5);
                const int32_t id = __shfl(xrow, r, 64);
                const float val = tr[r * 33 + (lane & 31)];
                if (id >= 0 && col < a.d) unsafeAtomicAdd(a.dE + (int64_t)id * a.d + col, val);
            }
        }
        return;
    } else {
        if constexpr (EX) {
            lds_barrier();  // (a rescaling of the last tile may still be reading xsum)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
#pragma unroll
                for (int off = 16; off < 64; off <<= 1) qsn[g] += __shfl_xor(qsn[g], off, 64);
                if (h16 == 0) xsum[(xg * 2 + xhalf) * 32 + xcol + 16 * g] = qsn[g];
            }
            lds_barrier();
            sn = xsum[xg * 64 + lo] + xsum[xg * 64 + 32 + lo];
        } else {
#pragma unroll
            for (int off = XR; off < 64; off <<= 1) sn += __shfl_xor(sn, off, 64);
        }
        const int64_t xs = pos0 + x;  // slot
        if (a.splits > 1) {  // partial results, combined by dense_merge_kernel
            if (x >= nx) return;
            if (hi == 0 && sl == 0) {
                a.part_ms[split * a.N + xs] = make_float2(ref, sn);
                if (split == 0) a.part_o[xs] = op;
            }
            if (MODE != DM_FWD && xrow >= 0) {
#pragma unroll
                for (int b = 0; b < OB; ++b)
#pragma unroll
                    for (int q = 0; q < G::AQ; ++q) {
                        const int col = (sl * OB + b) * G::OC + q * 8 + hi * 4;
                        if (col < a.d)
                            *reinterpret_cast<float4 *>(a.part_U + (split * a.N + xs) * a.d + col) =
                                make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
                    }
            }
            return;
        }
        if (x >= nx) return;
        if (xrow < 0) {
            // padded (only without compaction); the candidate launch writes zero dH rows
            if (MODE != DM_DH && !a.order && hi == 0 && sl == 0) a.loss[xs] = a.lse[xs] = 0.f;
            return;
        }
        float inv = 1.f, ct;
        if (MODE == DM_DH) {
            ct = fast_exp(op - ref) - 1.f;
            if (hi == 0 && sl == 0) a.coef[xrow] = (a.g ? a.g[xrow] : 1.f) * ct;
        } else {
            if (hi == 0 && sl == 0) inv = dense_finish(a, xs, xrow, ref, sn, op, MODE == DM_FDH);
            else inv = 1.f / (sn + fast_exp(op - ref));
            ct = -sn * inv;
        }
        if (MODE == DM_FWD) return;
        const float pp = fast_exp(op - ref) * inv;
        const float g = (MODE == DM_DH || a.direct_dH) ? (a.g ? a.g[xrow] : 1.f) : 1.f;
#pragma unroll
        for (int b = 0; b < OB; ++b)
#pragma unroll
            for (int q = 0; q < G::AQ; ++q) {
                const int col = (sl * OB + b) * G::OC + q * 8 + hi * 4;
                if (col >= a.d) continue;
                float et[4], u[4];
                widen4(Ep + (int64_t)ti * a.d + col, et);
#pragma unroll
                for (int r = 0; r < 4; ++r) u[r] = g * dense_row_value(acc[b][4 * q + r], inv, pp, ct, et[r]);
                if (MODE == DM_DH || a.direct_dH) store_dH4(a, xrow, col, u);
                else *reinterpret_cast<float4 *>(a.U + (int64_t)xrow * a.d + col) = make_float4(u[0], u[1], u[2], u[3]);
            }
    }
}

// Combines the shares of a split position side: one thread per position and four columns, so that a small batch still
// spreads over the chip (1000 positions, d = 512, 32 shares, sixteen threads a position: 48 us, all of it latency).
template <typename T, int MODE>
__global__ __launch_bounds__(256) void dense_merge_kernel(DenseArgs a)
{
    const int cpr = MODE == DM_FWD ? 1 : a.d / 4;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t x = e / cpr;
    const int c = (int)(e % cpr);
    if (x >= dense_slots(a)) return;
    const int32_t row = dense_row(a, x);
    if (row < 0) {
        if (MODE != DM_DH && !a.order && c == 0) a.loss[x] = a.lse[x] = 0.f;
        return;
    }
    float M = -INFINITY, sn = 0.f;
#pragma unroll 4
    for (int k = 0; k < a.splits; ++k) M = fmaxf(M, a.part_ms[k * a.N + x].x);
    float u[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k = 0; k < a.splits; ++k) {
        const float2 ms = a.part_ms[k * a.N + x];
        const float sc = MODE == DM_DH ? 1.f : fast_exp(ms.x - M);
        sn += ms.y * sc;
        if (MODE != DM_FWD) {
            float pv[4];
            widen4(a.part_U + (k * a.N + x) * a.d + c * 4, pv);
#pragma unroll
            for (int r = 0; r < 4; ++r) u[r] = fmaf(pv[r], sc, u[r]);
        }
    }
    const float op = a.part_o[x];
    float inv = 1.f, ct;
    if (MODE == DM_DH) {
        ct = fast_exp(op - M) - 1.f;
        if (c == 0) a.coef[row] = (a.g ? a.g[row] : 1.f) * ct;
    } else {
        if (c == 0) inv = dense_finish(a, x, row, M, sn, op, MODE == DM_FDH);
        else inv = 1.f / (sn + fast_exp(op - M));
        ct = -sn * inv;
    }
    if (MODE == DM_FWD) return;
    const float pp = fast_exp(op - M) * inv;
    const bool to_dH = MODE == DM_DH || a.direct_dH;
    const float g = (to_dH && a.g) ? a.g[row] : 1.f;
    float et[4];
    widen4(static_cast<const T *>(a.E) + (int64_t)dense_tgt(a, x, row) * a.d + c * 4, et);
#pragma unroll
    for (int r = 0; r < 4; ++r) u[r] = g * dense_row_value(u[r], inv, pp, ct, et[r]);
    if (to_dH) store_dH4(a, row, c * 4, u);
    else *reinterpret_cast<float4 *>(a.U + (int64_t)row * a.d + c * 4) = make_float4(u[0], u[1], u[2], u[3]);
}

template <typename T, int KD>
hipError_t launch_dense_kd(int pass, DenseArgs a, hipStream_t stream)
{
    const dim3 threads(kDenseThreads);
    if (pass == DENSE_DE) {
        const int64_t blocks = a.scatter_blocks + a.tile_blocks + a.scale_blocks;
        if (blocks == 0) return hipSuccess;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        ProfScope prof(PROF_DENSE_DE, stream);
        hipLaunchKernelGGL((dense_kernel<T, KD, DM_DE>), dim3((unsigned)blocks), threads, 0, stream, a);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)a.x_blocks, (unsigned)a.splits);
    {
        ProfScope prof(PROF_DENSE_POS, stream);
        if (pass == DENSE_FWD) hipLaunchKernelGGL((dense_kernel<T, KD, DM_FWD>), grid, threads, 0, stream, a);
        else if (pass == DENSE_FDH) hipLaunchKernelGGL((dense_kernel<T, KD, DM_FDH>), grid, threads, 0, stream, a);
        else hipLaunchKernelGGL((dense_kernel<T, KD, DM_DH>), grid, threads, 0, stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.splits == 1) return e;
    ProfScope prof(PROF_DENSE_MERGE, stream);
    const int64_t merged = a.N * (pass == DENSE_FWD ? 1 : a.d / 4);
    const dim3 mgrid((unsigned)((merged + 255) / 256));
    if (pass == DENSE_FWD) hipLaunchKernelGGL((dense_merge_kernel<T, DM_FWD>), mgrid, dim3(256), 0, stream, a);
    else if (pass == DENSE_FDH) hipLaunchKernelGGL((dense_merge_kernel<T, DM_FDH>), mgrid, dim3(256), 0, stream, a);
    else hipLaunchKernelGGL((dense_merge_kernel<T, DM_DH>), mgrid, dim3(256), 0, stream, a);
    return hipGetLastError();
}

// Shape of a pass and the blocks of it that the current device holds at once, asked once per kernel and device.
template <typename T, int KD, int MODE>
DenseShape dense_shape_mode()
{
    typedef DenseGeo<T, KD, MODE> G;
    constexpr int kMaxDevices = 64;
    static std::atomic<int> cache[kMaxDevices];  // 0 = not asked yet
    int per_cu = 0, dev = 0, cus = 0, slots = 512;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
        const int known = cache[dev].load(std::memory_order_relaxed);
        if (known > 0) {
            slots = known;
        } else if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 &&
                   hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, dense_kernel<T, KD, MODE>, kDenseThreads, 0) == hipSuccess && per_cu > 0) {
            slots = per_cu * cus;
            cache[dev].store(slots, std::memory_order_relaxed);
        }
    }
    // matrix instructions of a tile, 32 cycles each, two wavefronts to a SIMD at 2.4 GHz; scoring alone, where a few blocks
    // have the chip to themselves, as measured (64 positions; fp32, d = 32 / 64 / 128 / 256: 0.87, 1.22, 1.87, 3.15 us; bf16,
    // d = 48 / 320: 0.79, 1.56)
    constexpr int insts = G::B16 ? 2 * KD / G::DS + 6 * G::OB : G::BY / 16 * (8 * KD + 4 * G::OB);
    constexpr int alone = G::B16 ? 600 + 96 * KD : 550 + 163 * KD * (G::BY / 16);
    return DenseShape{G::XPB, G::BY, slots, MODE == DM_FWD ? alone : insts * 64 * 10 / 24};
}
template <typename T, int KD>
DenseShape dense_shape_kd(int pass)
{
    if (pass == DENSE_FWD) return dense_shape_mode<T, KD, DM_FWD>();
    if (pass == DENSE_FDH) return dense_shape_mode<T, KD, DM_FDH>();
    if (pass == DENSE_DH) return dense_shape_mode<T, KD, DM_DH>();
    return dense_shape_mode<T, KD, DM_DE>();
}

template <typename T, typename F>
auto dense_by_width(int d, F f)
{
    const int kd = (d + 31) / 32;
    if (kd <= 1) return f(std::integral_constant<int, 1>{});
    if (kd <= 2) return f(std::integral_constant<int, 2>{});
    if (kd <= 3) return f(std::integral_constant<int, 3>{});
    if (kd <= 4) return f(std::integral_constant<int, 4>{});
    if (kd <= 6) return f(std::integral_constant<int, 6>{});
    if (kd <= 8) return f(std::integral_constant<int, 8>{});
    if (kd <= 10) return f(std::integral_constant<int, 10>{});
    return f(std::integral_constant<int, 16>{});
}

}  // namespace
}  // namespace cce
