// LBVH build over the high-poly triangles (the paper's "GPU BVH built on the
// high-poly mesh", Sec. 6.4), after Karras 2012 (binary radix tree over sorted
// Morton codes):
//   1. reduction of the triangle-centroid bounds,
//   2. 30-bit Morton code of each centroid, value = original triangle index,
//   3. stable LSD radix sort of (code, index), 8-bit digits, LDS-ranked with
//      wave64 ballots, so equal codes keep ascending index order (assets of at
//      most 8,192 triangles: 1 to 3 by one workgroup, 10-bit digits),
//   4. hierarchy, boxes and compressed nodes in one pass, bottom-up: a subtree
//      joins the neighbour it shares the longer common prefix with (code,
//      extended by the index on equal codes), so the tree is the radix tree over
//      the codes and every node is met with both child boxes in hand (after
//      Apetrei 2014, with Karras's node numbering).  The same kernel packs the
//      leaves (vertices copied bit-exactly, original index kept) and writes the
//      nodes compressed (32 B each).
// In a batch every asset gets its own tree over its own bounds; sort tiles
// never straddle two assets, and each tile places its keys from its asset's
// per-tile and per-super-tile digit counts (section 3).
#include <algorithm>
#include <utility>

#include "internal.h"

namespace bake {

namespace {

constexpr int kBlock = 256;
constexpr int kSortBlock = 1024;                     // sort workgroups: 16 waves
constexpr int kSortRounds = kSortTile / kSortBlock;  // 4 keys per thread and pass
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kBwdSortGrid = 1024;                   // two workgroups a CU, twice

constexpr float kLeafEps = 1.0f / 16384.0f;  // edge tolerance of the hit rule (traverse.hip)

__device__ __forceinline__ int3 tri_idx(const int32_t* __restrict__ F, int64_t g, int64_t nv,
                                        bool* bad) {
    int32_t a = F[3 * g], b = F[3 * g + 1], c = F[3 * g + 2];
    bool ok = a >= 0 && b >= 0 && c >= 0 && a < nv && b < nv && c < nv;
    *bad = !ok;
    if (!ok) a = b = c = 0;  // degenerate stand-in: never hit, never out of bounds
    return make_int3(a, b, c);
}

__device__ __forceinline__ float3 ldv(const float* __restrict__ V, int32_t i) {
    return make_float3(V[3 * (int64_t)i], V[3 * (int64_t)i + 1], V[3 * (int64_t)i + 2]);
}

__device__ __forceinline__ float3 centroid(const float* __restrict__ V, int3 t) {
    float3 a = ldv(V, t.x), b = ldv(V, t.y), c = ldv(V, t.z);
    const float k = 1.0f / 3.0f;
    return make_float3((a.x + b.x + c.x) * k, (a.y + b.y + c.y) * k, (a.z + b.z + c.z) * k);
}

__device__ __forceinline__ int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---------------------------------------------------------------------------
// 1. centroid bounds: partials per sort tile, which every code tile reduces
// ---------------------------------------------------------------------------

__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ void block_minmax6(float v[6], float* out) {
    __shared__ float red[kBlock / 64][6];
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = wave_min(v[k]);
#pragma unroll
    for (int k = 3; k < 6; ++k) v[k] = wave_max(v[k]);
    if (lane == 0)
        for (int k = 0; k < 6; ++k) red[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            for (int k = 0; k < 3; ++k) v[k] = fminf(v[k], red[w][k]);
            for (int k = 3; k < 6; ++k) v[k] = fmaxf(v[k], red[w][k]);
        }
        for (int k = 0; k < 6; ++k) out[k] = v[k];
    }
}

__global__ __launch_bounds__(kBlock) void bounds_part_kernel(Batch Bt, float* __restrict__ part) {
    // kBoundsSplit workgroups per sort tile, each over its 1/kBoundsSplit of it
    int64_t lt;
    const int sub = (int)(blockIdx.x % kBoundsSplit);
    const AssetDev& As = Bt.A[block_asset(Bt, kGSort, blockIdx.x / kBoundsSplit, &lt)];
    const float* __restrict__ V = As.hi_V;
    const int32_t* __restrict__ F = As.hi_F;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    bool anybad = false, nonfin = false;
    constexpr int64_t kPart = kSortTile / kBoundsSplit;
    const int64_t first = lt * kSortTile + sub * kPart;
    const int64_t end = min((int64_t)As.nhf, first + kPart);
    // kU triangles per thread and trip, their index and vertex loads issued
    // together (one gather latency per trip instead of per triangle)
    constexpr int kU = 4;
    for (int64_t g0 = first + threadIdx.x; g0 < end; g0 += kU * kBlock) {
        int3 t[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            bool bad = false;
            const int64_t g = g0 + (int64_t)u * kBlock;
            t[u] = g < end ? tri_idx(F, g, As.nhv, &bad) : make_int3(0, 0, 0);
            anybad |= bad;
        }
        float3 c[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) c[u] = centroid(V, t[u]);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (g0 + (int64_t)u * kBlock >= end) continue;
            if (!(isfinite(c[u].x) && isfinite(c[u].y) && isfinite(c[u].z))) {
                nonfin = true;
                continue;
            }
            v[0] = fminf(v[0], c[u].x); v[1] = fminf(v[1], c[u].y); v[2] = fminf(v[2], c[u].z);
            v[3] = fmaxf(v[3], c[u].x); v[4] = fmaxf(v[4], c[u].y); v[5] = fmaxf(v[5], c[u].z);
        }
    }
    if (anybad) set_status(Bt, kStHiIndex);
    if (nonfin) set_status(Bt, kStNonFinite);
    block_minmax6(v, part + 6 * (kBoundsSplit * (As.stile + lt) + sub));
}

// ---------------------------------------------------------------------------
// 2. Morton codes (value = asset-local triangle index)
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t spread10(uint32_t x) {
    // 10 bits -> every third bit of 30
    x &= 0x3FFu;
    x = (x | (x << 16)) & 0x030000FFu;
    x = (x | (x << 8)) & 0x0300F00Fu;
    x = (x | (x << 4)) & 0x030C30C3u;
    x = (x | (x << 2)) & 0x09249249u;
    return x;
}

__device__ __forceinline__ uint32_t quant10(float c, float lo, float inv) {
    float q = (c - lo) * inv * 1024.0f;
    q = fminf(fmaxf(q, 0.0f), 1023.0f);  // NaN -> 0
    return (uint32_t)q;
}

__device__ __forceinline__ uint32_t morton(float3 c, const float* bounds) {
    float ex = bounds[3] - bounds[0], ey = bounds[4] - bounds[1], ez = bounds[5] - bounds[2];
    float ix = ex > 0.f ? 1.0f / ex : 0.f, iy = ey > 0.f ? 1.0f / ey : 0.f,
          iz = ez > 0.f ? 1.0f / ez : 0.f;
    uint32_t x = quant10(c.x, bounds[0], ix), y = quant10(c.y, bounds[1], iy),
             z = quant10(c.z, bounds[2], iz);
    return (spread10(x) << 2) | (spread10(y) << 1) | spread10(z);
}

// ---------------------------------------------------------------------------
// 3. stable LSD radix sort, 8-bit digits, per asset
// ---------------------------------------------------------------------------

// Digit offsets without a separate scan.  A pass is two launches: the
// histogram kernel writes each tile's 256 digit counts as a row
// (hist[hbase + 256 lt + digit]) and adds them into its super-tile's row
// (kSuper consecutive tiles of one asset, sup[sbase + 256 (lt / kSuper) +
// digit], integer atomics: the sums do not depend on their order); the
// scatter kernel then finds where its tile's keys of digit d start from
//   start + (the asset's keys with a smaller digit: all super-tile rows)
//         + (earlier tiles' keys of digit d: earlier super-tiles' rows and the
//            rows of the earlier tiles in its own super-tile),
// which is the exclusive scan of the counts in (digit, tile) order.
// The tile of a sort block: its asset's keys [start, start + count) in the
// concatenated arrays, its count row (hbase + 256 lt), its super-tile rows
// (from sbase; an asset's super-tiles start at tile_base / kSuper + asset,
// which keeps assets apart) and its local tile lt.  BWD: the backward's merged
// pairs, whose count lives on the device, with rows sized for the capacity
// 3 res^2.
struct SortTile {
    int64_t start, count, hbase, sbase, lt;
};

// BWD blocks share out the tiles that hold pairs.
template <bool BWD>
__device__ __forceinline__ SortTile sort_tile(const Batch& Bt, int64_t blk) {
    SortTile T;
    int a;
    if (BWD) {
        a = upper_asset(Bt.bt_pf, Bt.n, blk);
        T.lt = blk - Bt.bt_pf[a];
    } else {
        a = block_asset(Bt, kGSort, blk, &T.lt);
    }
    const AssetDev& As = Bt.A[a];
    const int64_t tile_base = BWD ? As.btile : As.stile;
    if (BWD) {
        T.start = 3 * (int64_t)Bt.ray_pf[a];
        T.count = Bt.cnt[(int64_t)a * kCntSlots + kCntPairs];
    } else {
        T.start = As.hf;
        T.count = As.nhf;
    }
    T.hbase = 256 * tile_base;
    T.sbase = 256 * (tile_base / kSuper + a);
    return T;
}

// Tiles of a launch: block b takes b, b + gridDim.x, ...  The backward's are known
// on the device only, and a workspace that no longer holds the saved forward has
// none.
template <bool BWD>
__device__ __forceinline__ int64_t sort_tiles(const Batch& Bt) {
    if (!BWD) return gridDim.x;
    return sealed(Bt) ? Bt.gcnt[kGcBwdTiles] : 0;
}

// The thread's index, formed anew for each tile: what follows from it is not worth
// the registers from one tile to the next (two workgroups a CU leave 64).
template <bool BWD>
__device__ __forceinline__ int tile_thread() {
    int t = threadIdx.x;
    if (BWD) asm volatile("" : "+v"(t));
    return t;
}

// The keys of the backward's first pass lie batch by batch, each batch's at three
// times its first ray.  Draws tile T's together into kout, with their places as
// values, and counts their digits in h.  A batch has some sixty of 192: the
// bucket that holds the tile's first pair comes from the buckets' prefix, the
// batches from there on are summed 1,024 at a time, and a wave copies a batch.
// ONE: an asset by itself of at most 1,024 batches, which this launch sums
// without buckets; its first block writes what pair_table_kernel would.  Returns
// whether the tile has pairs.
template <bool ONE>
__device__ __forceinline__ bool gather_pairs(const Batch& Bt, const SortTile& T, int a, int shift,
                                             const uint32_t* __restrict__ sparse,
                                             const uint32_t* __restrict__ pairs,
                                             const uint32_t* __restrict__ bucket, uint32_t* __restrict__ kout,
                                             uint32_t* __restrict__ vout, uint32_t* __restrict__ bt_pf,
                                             uint32_t* h) {
    __shared__ uint32_t s_at[kSortBlock], s_n[kSortBlock], s_w[kSortWaves];
    const int tid = tile_thread<true>(), lane = tid & 63, wave = tid >> 6;
    const int64_t q0 = Bt.rb_pf[a], nb = Bt.rb_pf[a + 1] - q0, nk = ceil_div(nb, kPairBucket);
    const uint32_t* __restrict__ pre = bucket + pair_bucket(q0, a);
    const uint32_t e0 = (uint32_t)(T.lt * kSortTile);
    uint32_t e1 = ONE ? e0 + 1 : (uint32_t)min((int64_t)e0 + kSortTile, T.count);
    int64_t k = -1;  // the last bucket that starts at or before e0
    uint32_t base = 0;
    if (ONE) {
        k = 0;
    } else {
        const uint32_t zero = pre[0];
        for (int64_t c = 0; c < nk; c += kSortBlock) {
            const int m = __syncthreads_count(c + tid < nk && pre[min(c + tid, nk - 1)] - zero <= e0);
            k += m;
            if (m < kSortBlock) break;
        }
        base = pre[k] - zero;
    }
    for (int64_t b0 = k * kPairBucket; base < e1 && b0 < nb; b0 += kSortBlock) {
        const uint32_t n = b0 + tid < nb ? pairs[q0 + b0 + tid] : 0u;
        uint32_t x = n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        __syncthreads();
        if (lane == 63) s_w[wave] = x;
        __syncthreads();
        uint32_t all = 0;
#pragma unroll 4
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t y = s_w[w];
            if (w < wave) x += y;
            all += y;
        }
        if (ONE) {
            if (T.lt == 0 && tid == 0) {
                const uint32_t nt = (all + kSortTile - 1) / kSortTile;
                Bt.cnt[kCntPairs] = all;
                Bt.gcnt[kGcBwdTiles] = nt;
                bt_pf[0] = 0;
                bt_pf[1] = nt;
            }
            if (e0 >= all) return false;
            e1 = min(e0 + kSortTile, all);
        }
        x += base - n;
        s_at[tid] = x;
        s_n[tid] = n;
        const int j0 = __syncthreads_count(x + n <= e0), j1 = __syncthreads_count(x < e1);
        constexpr int kU = 2;
        for (int j = j0 + wave; j < j1; j += kU * kSortWaves) {
            uint32_t key[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int ju = min(j + u * kSortWaves, kSortBlock - 1);
                const bool on = j + u * kSortWaves < j1 && lane < (int)s_n[ju];
                key[u] = sparse[T.start + (on ? 192 * (b0 + ju) + lane : 0)];
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int ju = j + u * kSortWaves;
                if (ju >= j1) break;
                const uint32_t at = s_at[ju];
                const int m = (int)s_n[ju];
                const int64_t from = T.start + 192 * (b0 + ju);
#pragma unroll 1
                for (int i = lane; i < m; i += 64) {
                    const uint32_t e = at + (uint32_t)i;
                    if (e < e0 || e >= e1) continue;
                    const uint32_t v = i < 64 ? key[u] : sparse[from + i];
                    kout[T.start + e] = v;
                    vout[T.start + e] = (uint32_t)(from + i);
                    atomicAdd(&h[(v >> shift) & 255u], 1u);
                }
            }
        }
        base += all;
        if (ONE) break;
    }
    return true;
}

enum SortKeys : int { kSortBvhKeys = 0, kSortPairs = 1, kSortPairsFirst = 2, kSortPairsOne = 3 };

struct HistArgs {
    Batch B;
    const uint32_t* keys;
    int shift;
    uint32_t *hist, *sup;
    // first pass of the backward: see gather_pairs
    const uint32_t *pairs, *bucket;
    uint32_t *kout, *vout, *bt_pf;
};

// An asset's partial bounds reduced into the first of them, by one workgroup.
__global__ __launch_bounds__(kSortBlock) void bounds_reduce_kernel(Batch Bt, float* __restrict__ part) {
    __shared__ float s_red[kSortWaves][6];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const AssetDev& As = Bt.A[blockIdx.x];
    const int64_t nparts = kBoundsSplit * ceil_div(As.nhf, kSortTile);
    if (nparts == 0) return;
    float* p = part + 6 * kBoundsSplit * As.stile;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll 4
    for (int64_t i = tid; i < nparts; i += kSortBlock)
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = k < 3 ? fminf(v[k], p[6 * i + k]) : fmaxf(v[k], p[6 * i + k]);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) s_red[wave][k] = v[k];
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float x = s_red[lane & (kSortWaves - 1)][k];
        v[k] = k < 3 ? wave_min(x) : wave_max(x);
        if (lane == 0) p[k] = v[k];
    }
}

// Codes of a sort tile, their indices and the first pass's digit counts.  Each
// tile reduces its asset's partial bounds by itself (four per tile of the asset, from
// L2), or takes the one that bounds_reduce_kernel left (ONE), and counts the digits
// that a histogram launch read the keys again for.
template <bool ONE>
__global__ __launch_bounds__(kSortBlock) __attribute__((amdgpu_waves_per_eu(8))) void code_kernel(
    Batch Bt, const float* __restrict__ part, uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ sup) {
    __shared__ uint32_t h[256];
    __shared__ float s_red[kSortWaves][6];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SortTile T = sort_tile<false>(Bt, blockIdx.x);
    int64_t lt;
    const AssetDev& As = Bt.A[block_asset(Bt, kGSort, blockIdx.x, &lt)];
    const float* __restrict__ V = As.hi_V;
    const int32_t* __restrict__ F = As.hi_F;
    const int64_t g0 = lt * kSortTile + tid;
    int3 t[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        bool bad;
        t[r] = tri_idx(F, min(g0 + (int64_t)r * kSortBlock, T.count - 1), As.nhv, &bad);
    }
    const int64_t nparts = ONE ? 1 : kBoundsSplit * ceil_div(T.count, kSortTile);
    const float* p = part + 6 * kBoundsSplit * As.stile;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = tid; i < nparts; i += kSortBlock)
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = k < 3 ? fminf(v[k], p[6 * i + k]) : fmaxf(v[k], p[6 * i + k]);
    float3 c[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) c[r] = centroid(V, t[r]);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) s_red[wave][k] = v[k];
    if (tid < 256) h[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float x = s_red[lane & (kSortWaves - 1)][k];
        v[k] = k < 3 ? wave_min(x) : wave_max(x);
    }
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t g = g0 + (int64_t)r * kSortBlock;
        if (g >= T.count) break;
        const uint32_t key = morton(c[r], v);
        keys[T.start + g] = key;
        vals[T.start + g] = (uint32_t)g;
        atomicAdd(&h[key & 255u], 1u);
    }
    __syncthreads();
    if (tid < 256) {
        const uint32_t n = h[tid];
        hist[T.hbase + 256 * T.lt + tid] = n;
        if (n) atomicAdd(&sup[T.sbase + 256 * (T.lt / kSuper) + tid], n);
    }
}

template <int WHICH>
__global__ __launch_bounds__(kSortBlock) __attribute__((amdgpu_waves_per_eu(8))) void radix_hist_kernel(HistArgs p) {
    constexpr bool BWD = WHICH != kSortBvhKeys;
    __shared__ uint32_t h[256];
    const Batch& Bt = p.B;
    // ONE: a block per tile of the capacity
    const int64_t tiles = WHICH == kSortPairsOne ? (sealed(Bt) ? gridDim.x : 0) : sort_tiles<BWD>(Bt);
    for (int64_t blk = blockIdx.x; blk < tiles; blk += gridDim.x) {
        SortTile T;
        if constexpr (WHICH == kSortPairsOne) {
            T = SortTile{3 * (int64_t)Bt.ray_pf[0], 0, 0, 0, blk};
        } else {
            T = sort_tile<BWD>(Bt, blk);
        }
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        __syncthreads();
        if constexpr (WHICH == kSortPairsFirst) {
            gather_pairs<false>(Bt, T, upper_asset(Bt.bt_pf, Bt.n, blk), p.shift, p.keys, p.pairs, p.bucket, p.kout,
                                p.vout, p.bt_pf, h);
        } else if constexpr (WHICH == kSortPairsOne) {
            if (!gather_pairs<true>(Bt, T, 0, p.shift, p.keys, p.pairs, p.bucket, p.kout, p.vout, p.bt_pf, h)) return;
        } else {
            const int64_t base = T.lt * kSortTile;
            // all rounds' keys are loaded before the first count (one load latency)
            uint32_t k[kSortRounds];
#pragma unroll
            for (int r = 0; r < kSortRounds; ++r) {
                const int64_t i = base + (int64_t)r * kSortBlock + threadIdx.x;
                k[r] = p.keys[T.start + min(i, T.count - 1)];
            }
#pragma unroll
            for (int r = 0; r < kSortRounds; ++r)
                if (base + (int64_t)r * kSortBlock + threadIdx.x < T.count)
                    atomicAdd(&h[(k[r] >> p.shift) & 255u], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            const uint32_t c = h[threadIdx.x];
            p.hist[T.hbase + 256 * T.lt + threadIdx.x] = c;
            if (c) atomicAdd(&p.sup[T.sbase + 256 * (T.lt / kSuper) + threadIdx.x], c);
        }
        if (BWD) __syncthreads();
    }
}

// The wave's valid lanes whose digit is the lane's.
template <int BITS>
__device__ __forceinline__ uint64_t equal_lanes(uint32_t dig, bool valid) {
    uint32_t lo = 0, hi = 0;  // lanes that differ in a bit
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t mine = (uint32_t)((int32_t)(dig << (31 - b)) >> 31);
        const uint64_t m = __ballot(mine != 0);
        lo |= (uint32_t)m ^ mine;
        hi |= (uint32_t)(m >> 32) ^ mine;
    }
    return ~((uint64_t)hi << 32 | lo) & __ballot(valid);
}

// Element r*1024 + tid of the block's tile is ranked among equal digits by
// (earlier rounds, earlier waves, earlier lanes): a stable order.  The tile is
// first placed in LDS in that order (digit runs contiguous), then written out
// with consecutive lanes on consecutive positions of each run.  The tile's
// first position of each digit comes from the count rows (see kSuper).  The
// keys are loaded first, so that their latency overlaps the reads of the
// count rows.  Ranking: each wave finds, per round, the lanes of each digit
// (ballots over the digit's bits) and records their count for its (round,
// wave, digit); one scan per digit over the 64 (round, wave) counts, in that
// order, then turns the counts into positions, so the whole tile is ranked
// between two barriers.
template <bool BWD>
__global__ __launch_bounds__(kSortBlock) __attribute__((amdgpu_waves_per_eu(8))) void radix_scatter_kernel(Batch Bt, const uint32_t* __restrict__ kin,
                                                                   const uint32_t* __restrict__ vin,
                                                                   uint32_t* __restrict__ kout,
                                                                   uint32_t* __restrict__ vout, int shift,
                                                                   const uint32_t* __restrict__ hist,
                                                                   const uint32_t* __restrict__ sup) {
    __shared__ uint32_t s_key[kSortTile];  // also the scratch of the count-row sums
    __shared__ uint32_t s_val[kSortTile];
    __shared__ uint32_t s_loc[256];   // tile-local first position of each digit
    __shared__ uint32_t s_glob[256];  // global position of the tile's first key of each digit
    __shared__ uint32_t s_run[256];   // the tile's digit counts
    __shared__ uint32_t s_wsum[4];
    __shared__ uint32_t s_part[kSortRounds][256];  // per round: the digit's keys in the round
    // per (round, wave, digit): the count, then the tile-local first position
    __shared__ uint16_t wcnt[kSortRounds][kSortWaves][256];
    static_assert(kSortTile <= 65535, "tile positions are kept in 16 bits");
    static_assert(kSortBlock == 4 * 256 && kSortRounds * kSortWaves == 64, "one scan thread per (round, digit)");
    const int64_t tiles = sort_tiles<BWD>(Bt);
    for (int64_t blk = blockIdx.x; blk < tiles; blk += gridDim.x) {
        const int tid = tile_thread<BWD>(), lane = tid & 63, wave = tid >> 6;
        const SortTile T = sort_tile<BWD>(Bt, blk);
        const int64_t base = T.lt * kSortTile;
        const int64_t nvalid = min((int64_t)kSortTile, T.count - base);
        uint32_t key[kSortRounds], val[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int64_t i = (int64_t)r * kSortBlock + tid;
            const bool valid = i < nvalid;
            key[r] = valid ? kin[T.start + base + i] : 0u;
            val[r] = valid ? vin[T.start + base + i] : 0u;
        }
        uint32_t(*scratch)[256] = reinterpret_cast<uint32_t(*)[256]>(s_key);
        {
            // per digit, in four parts: the asset's count (all super-tile rows)
            // and the count before this tile (earlier super-tiles, then the
            // earlier tiles of its own super-tile)
            // (the loads of a group are all issued before their sums: one load
            // latency per group instead of one per row)
            const int d = tid & 255, part = tid >> 8;
            const int64_t S = T.lt / kSuper, nS = ceil_div(ceil_div(T.count, kSortTile), kSuper);
            uint32_t tot = 0, before = 0;
            uint32_t hv[kSuper / 4];
#pragma unroll
            for (int j = 0; j < kSuper / 4; ++j) {
                const int64_t t = S * kSuper + part + 4 * j;
                hv[j] = t < T.lt ? hist[T.hbase + 256 * t + d] : 0u;
            }
            for (int64_t x0 = part; x0 < nS; x0 += 4 * 8) {
                uint32_t v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int64_t x = x0 + 4 * j;
                    v[j] = x < nS ? sup[T.sbase + 256 * x + d] : 0u;
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    tot += v[j];
                    if (x0 + 4 * j < S) before += v[j];
                }
            }
#pragma unroll
            for (int j = 0; j < kSuper / 4; ++j) before += hv[j];
            scratch[part][d] = tot;
            scratch[4 + part][d] = before;
        }
        __syncthreads();
        uint32_t tot = 0, before = 0;
        if (tid < 256) {
            tot = (scratch[0][tid] + scratch[1][tid]) + (scratch[2][tid] + scratch[3][tid]);
            before = (scratch[4][tid] + scratch[5][tid]) + (scratch[6][tid] + scratch[7][tid]);
            // exclusive scan of the asset's digit counts (waves 0-3)
            uint32_t x = tot;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (lane == 63) s_wsum[wave] = x;
            tot = x - tot;  // exclusive within the wave
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t w = 0;
            for (int k = 0; k < wave; ++k) w += s_wsum[k];
            s_glob[tid] = (uint32_t)T.start + w + tot + before;
            s_run[tid] = 0;
        }
        for (int x = tid; x < kSortRounds * kSortWaves * 256 / 2; x += kSortBlock)
            reinterpret_cast<uint32_t*>(&wcnt[0][0][0])[x] = 0;
        __syncthreads();
        // the tile's digit counts, and every wave's per-round digit counts
        uint32_t rank[kSortRounds];
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const bool valid = (int64_t)r * kSortBlock + tid < nvalid;
            const uint32_t dig = (key[r] >> shift) & 255u;
            if (valid) atomicAdd(&s_run[dig], 1u);
            const uint64_t peers = equal_lanes<8>(dig, valid);
            rank[r] = (uint32_t)__popcll(peers & __lanemask_lt());
            if (valid && rank[r] == 0) wcnt[r][wave][dig] = (uint16_t)__popcll(peers);
        }
        __syncthreads();
        // thread (rr, d): exclusive scan of digit d's counts over the waves of
        // round rr; waves 0-3 also scan the tile's digit counts
        const int sd = tid & 255, rr = tid >> 8;
        uint32_t ex[kSortWaves];
        {
            uint32_t acc = 0;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                ex[w] = acc;
                acc += wcnt[rr][w][sd];
            }
            s_part[rr][sd] = acc;
        }
        uint32_t c = 0, x = 0;
        if (tid < 256) {
            c = s_run[tid];
            x = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (lane == 63) s_wsum[wave] = x;
        }
        __syncthreads();
        if (tid < 256) {
            uint32_t b = 0;
            for (int w = 0; w < wave; ++w) b += s_wsum[w];
            s_loc[tid] = b + x - c;
        }
        __syncthreads();
        {
            uint32_t p = s_loc[sd];
            for (int r = 0; r < rr; ++r) p += s_part[r][sd];
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) wcnt[rr][w][sd] = (uint16_t)(p + ex[w]);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            if ((int64_t)r * kSortBlock + tid < nvalid) {
                const uint32_t dig = (key[r] >> shift) & 255u;
                const uint32_t pos = (uint32_t)wcnt[r][wave][dig] + rank[r];
                s_key[pos] = key[r];
                s_val[pos] = val[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int e = r * kSortBlock + tid;
            if (e >= nvalid) break;
            const uint32_t k = s_key[e];
            const uint32_t d = (k >> shift) & 255u;
            const uint32_t pos = s_glob[d] + ((uint32_t)e - s_loc[d]);
            if ((int64_t)pos < T.start + T.count) {  // always, unless the counts were corrupted
                kout[pos] = k;
                vout[pos] = s_val[e];
            } else {
                set_status(Bt, kStInternal);
            }
        }
        if (BWD) __syncthreads();
    }
}

// Bounds, codes and sort of a small mesh in one workgroup: an asset of at most
// kFrontFaces triangles whose keys and indices stay in LDS over the three passes.
// Wave w holds elements [64 per w, 64 per (w + 1)) of the order before the pass,
// 64 a round; a round's lanes of equal digit are found by ballots, the wave's
// counts of earlier rounds give their rank in the wave, one scan over waves and
// digits the rest: a stable order, as that of the passes over many tiles.
// Bound by the issue rate of one CU (a pass at 5,120 elements is 80 wave-rounds of
// some 80 instructions on four SIMDs) and by the gather of the corners: 28 us at
// 5,120, where bounds, codes and four passes in eleven launches took 54 and
// their gaps.
constexpr int kFrontBlock = 1024;
constexpr int kFrontWaves = kFrontBlock / 64;
constexpr int kFrontBits = 10, kFrontDigits = 1 << kFrontBits;  // three passes over 30-bit codes
constexpr int kFrontPer = kFrontFaces / kFrontBlock;
static_assert(kFrontFaces % kFrontBlock == 0 && kFrontFaces <= 65536, "whole rounds, 16-bit indices");
static_assert(kFrontDigits == kFrontBlock, "a thread per digit");

__global__ __launch_bounds__(kFrontBlock) void front_kernel(Batch Bt, uint32_t* __restrict__ keys,
                                                            uint32_t* __restrict__ vals) {
    __shared__ uint32_t s_key[kFrontFaces];
    __shared__ uint16_t s_idx[kFrontFaces];
    __shared__ uint16_t s_cnt[kFrontWaves][kFrontDigits];
    __shared__ uint32_t s_dig[kFrontDigits];
    __shared__ uint32_t s_w[kFrontWaves];
    __shared__ float s_red[kFrontWaves][6];
    const int a = blockIdx.x;
    const AssetDev& As = Bt.A[a];
    const int n = As.nhf, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (n == 0) return;
    const int per = (n + kFrontBlock - 1) / kFrontBlock;
    const int e0 = wave * 64 * per + lane;  // element of round r: e0 + 64 r
    float3 c[kFrontPer];
    bool anybad = false, nonfin = false;
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    {
        const float* __restrict__ V = As.hi_V;
        const int32_t* __restrict__ F = As.hi_F;
        int3 t[kFrontPer];
#pragma unroll
        for (int r = 0; r < kFrontPer; ++r) {
            bool bad = false;
            const int e = e0 + 64 * r;
            t[r] = r < per && e < n ? tri_idx(F, e, As.nhv, &bad) : make_int3(0, 0, 0);
            anybad |= bad;
        }
#pragma unroll
        for (int r = 0; r < kFrontPer; ++r) {
            c[r] = make_float3(0.f, 0.f, 0.f);
            if (r < per) c[r] = centroid(V, t[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < kFrontPer; ++r) {
        if (r >= per || e0 + 64 * r >= n) continue;
        if (!(isfinite(c[r].x) && isfinite(c[r].y) && isfinite(c[r].z))) {
            nonfin = true;
            continue;
        }
        v[0] = fminf(v[0], c[r].x); v[1] = fminf(v[1], c[r].y); v[2] = fminf(v[2], c[r].z);
        v[3] = fmaxf(v[3], c[r].x); v[4] = fmaxf(v[4], c[r].y); v[5] = fmaxf(v[5], c[r].z);
    }
    if (anybad) set_status(Bt, kStHiIndex);
    if (nonfin) set_status(Bt, kStNonFinite);
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 6; ++k) s_red[wave][k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float x = s_red[lane & (kFrontWaves - 1)][k];
        v[k] = k < 3 ? wave_min(x) : wave_max(x);
    }
    uint32_t key[kFrontPer], idx[kFrontPer];
#pragma unroll
    for (int r = 0; r < kFrontPer; ++r) {
        key[r] = morton(c[r], v);
        idx[r] = (uint32_t)(e0 + 64 * r);
    }
    for (int shift = 0; shift < 30; shift += kFrontBits) {
        for (int x = tid; x < kFrontWaves * kFrontDigits / 2; x += kFrontBlock)
            reinterpret_cast<uint32_t*>(&s_cnt[0][0])[x] = 0;
        __syncthreads();
        uint32_t rank[kFrontPer];
#pragma unroll
        for (int r = 0; r < kFrontPer; ++r) {
            if (r >= per) break;
            const bool valid = e0 + 64 * r < n;
            const uint32_t dig = (key[r] >> shift) & (kFrontDigits - 1);
            const uint64_t peers = equal_lanes<kFrontBits>(dig, valid);
            const uint32_t in = (uint32_t)__popcll(peers & __lanemask_lt());
            const uint32_t was = s_cnt[wave][dig];
            rank[r] = was + in;
            wave_sync();
            if (valid && in == 0) s_cnt[wave][dig] = (uint16_t)(was + __popcll(peers));
            wave_sync();
        }
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kFrontWaves; ++w) {  // exclusive over the waves
            const uint32_t y = s_cnt[w][tid];
            s_cnt[w][tid] = (uint16_t)sum;
            sum += y;
        }
        uint32_t x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) s_w[wave] = x;
        __syncthreads();
        uint32_t before = s_w[lane & (kFrontWaves - 1)];
#pragma unroll
        for (int o = 1; o < kFrontWaves; o <<= 1) {
            const uint32_t y = __shfl_up(before, o, 64);
            if (lane >= o) before += y;
        }
        before = wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)before, wave - 1) : 0u;
        s_dig[tid] = before + x - sum;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kFrontPer; ++r) {
            if (r >= per) break;
            if (e0 + 64 * r >= n) continue;
            const uint32_t dig = (key[r] >> shift) & (kFrontDigits - 1);
            const uint32_t at = s_dig[dig] + s_cnt[wave][dig] + rank[r];
            s_key[at] = key[r];
            s_idx[at] = (uint16_t)idx[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kFrontPer; ++r) {
            const int e = min(e0 + 64 * r, n - 1);
            key[r] = s_key[e];
            idx[r] = s_idx[e];
        }
    }
#pragma unroll
    for (int r = 0; r < kFrontPer; ++r) {
        const int e = e0 + 64 * r;
        if (r < per && e < n) {
            keys[As.hf + e] = key[r];
            vals[As.hf + e] = idx[r];
        }
    }
}

// ---------------------------------------------------------------------------
// 4. hierarchy + leaves + nodes
// ---------------------------------------------------------------------------
//
// The radix tree over the sorted codes, from its leaves up.  A subtree covers
// a leaf range [l, r]; its parent's split lies at r when the prefix common to
// leaves r and r + 1 is longer than that common to l - 1 and l (it is then the
// left child), else at l - 1 (the right child).  Both children leave their box
// at the split; the one that comes second has both boxes and goes on as the
// parent.  A node's index is that of the end of its range towards its sibling
// (Karras: the left child of a node with split s is node or leaf s, the right
// one s + 1; the root is 0), so a node's children and its own index are known as
// it forms, without searches, parent links or a separate refit.
//
// One workgroup does this in LDS for a tile of kBuildTile consecutive leaves.
// The subtrees whose sibling lies in another tile (at most 62 along each edge
// of the tile, about twenty in all) go to the tile's list in order, and a join
// launch does the same over the lists of kJoin tiles, with list entries in place
// of leaves, then over those of kJoin joined groups, until one group is the whole
// asset (the last one takes up to kJoinLast: two joins do for 8M faces).
//
// Bound by the gather of the leaves' corners and the latency of the climb (a
// dozen LDS round trips).  Two workgroups fit a CU.  Before, a hierarchy kernel
// searched every node's range and scattered parent links, a treelet refit read
// them back and climbed with one workgroup per CU, and one workgroup per asset
// finished the top: 1.31M faces 164 -> 104 us, 5.24M 654 -> 246 us, 5,120
// 39 -> 27 us.

__device__ __forceinline__ float pow2f(uint32_t e) { return __uint_as_float(e << 23); }  // 2^(e - 127)

// One axis of a compressed node: the frame [o, o + 255 s] with s a power of
// two, and the bytes of the four child planes.  A decoded plane fmaf(v, s, o)
// rounds lo + v s once, and lo + v s is exact whenever it is representable,
// so it lies on the outer side of a plane c exactly when lo + v s does: the
// bytes come from (c - lo) / s (exact scaling of a once-rounded difference,
// off by at most one) and one check each.
__device__ __forceinline__ uint32_t quantise_axis(float lL, float hL, float lR, float hR, float* o_out,
                                                  uint32_t q_out[4]) {
    const float lo = fminf(lL, lR), hi = fmaxf(hL, hR);
    if (!(isfinite(lo) && isfinite(hi) && lo <= hi)) {
        // NaN planes: an unbounded slab in the box tests
        *o_out = __uint_as_float(0x7FC00000u);
        q_out[0] = q_out[1] = q_out[2] = q_out[3] = 0;
        return 127u;
    }
    // ext / 2^(E - 7) lies in [128, 256) for ext in [2^E, 2^(E+1)); one
    // doubling when 255 steps still fall short of hi
    const float ext = hi - lo;
    const uint32_t eb = (__float_as_uint(ext) >> 23) & 0xFFu;
    uint32_t e = eb > 8u ? eb - 7u : 1u;
    if (e < 254u && fmaf(255.f, pow2f(e), lo) < hi) ++e;
    const float s = pow2f(e), inv = pow2f(254u - e);  // inv = 1 / s
    const float pl[4] = {lL, hL, lR, hR};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float c = pl[j];
        const float x = fminf(fmaxf((c - lo) * inv, 0.f), 255.f);
        uint32_t v;
        if ((j & 1) == 0) {  // lower plane: the largest v with lo + v s <= c
            v = (uint32_t)floorf(x);
            if (v > 0u && fmaf((float)v, s, lo) > c) --v;
        } else {             // upper plane: the smallest v with lo + v s >= c
            v = (uint32_t)ceilf(x);
            if (v < 255u && fmaf((float)v, s, lo) < c) ++v;
        }
        q_out[j] = v;
    }
    *o_out = lo;
    return e;
}

// Writes node p whole: its frame, child planes and child word (the
// hierarchy kernel's), two 16-B stores.
__device__ __forceinline__ void write_compressed(BvhNodeC* node, uint32_t child, const float L[6], const float R[6]) {
    float o[3];
    uint32_t q[3][4], e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) e[k] = quantise_axis(L[k], L[k + 3], R[k], R[k + 3], &o[k], q[k]);
    // byte order: L.lo.xyz, L.hi.xyz, R.lo.xyz, R.hi.xyz
    const uint32_t b[12] = {q[0][0], q[1][0], q[2][0], q[0][1], q[1][1], q[2][1],
                            q[0][2], q[1][2], q[2][2], q[0][3], q[1][3], q[2][3]};
    uint32_t w[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) w[i] = b[4 * i] | (b[4 * i + 1] << 8) | (b[4 * i + 2] << 16) | (b[4 * i + 3] << 24);
    node->a = make_float4(o[0], o[1], o[2], __uint_as_float(e[0] | (e[1] << 8) | (e[2] << 16)));
    node->q = make_uint4(w[0], w[1], w[2], child);
}


// Box of a leaf triangle, widened for the hit rule's edge tolerance: weights
// down to -kLeafEps put the crossing inside the triangle scaled by (1 + 3
// kLeafEps) about its centroid; widen by 4 kLeafEps of the extent (3 plus
// rounding margin) and a few ulps of the coordinates.
__device__ __forceinline__ void leaf_box(const Leaf& L, float box[6]) {
    float ax = L.a.x, ay = L.a.y, az = L.a.z, bx = L.a.w, by = L.b.x, bz = L.b.y;
    float cx = L.b.z, cy = L.b.w, cz = L.c.x;
    box[0] = fminf(fminf(ax, bx), cx); box[1] = fminf(fminf(ay, by), cy); box[2] = fminf(fminf(az, bz), cz);
    box[3] = fmaxf(fmaxf(ax, bx), cx); box[4] = fmaxf(fmaxf(ay, by), cy); box[5] = fmaxf(fmaxf(az, bz), cz);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        float ext = box[q + 3] - box[q];
        float pad = 4.0f * kLeafEps * ext + 4.76837158e-7f * fmaxf(fabsf(box[q]), fabsf(box[q + 3]));
        box[q] -= pad;
        box[q + 3] += pad;
    }
}

// A subtree that waits for a sibling in another tile or group: its first leaf,
// the prefix length before that, and its box (its last leaf is the one before
// the next entry's first).
struct alignas(16) BuildItem {
    float box[6];
    int32_t l, cpl;
};
static_assert(sizeof(BuildItem) == 32, "BuildItem is 32 B");

constexpr int kBuildBlock = 1024;
constexpr int kJoinUnits = 2 * kBuildBlock;  // list entries a join holds at a time
static_assert(kJoinUnits >= 4 * kSpine, "every batch of a join takes some lists");
constexpr uint32_t kNoNode = 0xFFFFFFFFu;

// Common-prefix length of leaves a and a + 1 of an asset of n leaves (-1 past
// its ends).
__device__ __forceinline__ int prefix_len(uint32_t ka, uint32_t kb, int64_t a) {
    return ka == kb ? 32 + __clz((uint32_t)a ^ (uint32_t)(a + 1)) : __clz(ka ^ kb);
}

// The climb's state over UNITS leaves or list entries ("units"); slot k is the
// split before unit k, slot m that after the last one of m.
template <int UNITS>
struct ClimbLds {
    float box[12][UNITS + 1];   // child boxes waiting at a split: left 0-5, right 6-11
    int32_t end[UNITS + 1];     // far end of the child that came first | side << 30, -1: none yet
    uint32_t dest[UNITS + 1];   // node at the split: its index | leaf flags of its children
    int8_t cpl[UNITS + 2];      // prefix common to the leaves before and after a split
    uint16_t item[UNITS];       // slot + 1 where the waiting subtree that starts here left its box
    uint32_t wave_sum[kBuildBlock / 64];
};

// first(k): first leaf of unit k (k = m: one past the last leaf).
template <int UNITS, typename First>
__device__ __forceinline__ void climb(ClimbLds<UNITS>& S, int u, float box[6], First first) {
    int a = u, b = u, slot = -1;
    uint32_t flags = 0;
    for (;;) {
        const int cl = S.cpl[a], cr = S.cpl[b + 1];
        if (cl < 0 && cr < 0) {  // the whole asset
            if (slot >= 0) S.dest[slot] = flags;
            return;
        }
        const bool left = cr > cl;
        if (slot >= 0) S.dest[slot] = (uint32_t)(left ? first(b + 1) - 1 : first(a)) | flags;
        const int si = left ? b + 1 : a;
        const int side = left ? 0 : 6;
#pragma unroll
        for (int q = 0; q < 6; ++q) S.box[side + q][si] = box[q];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        const int32_t old = __hip_atomic_exchange(&S.end[si], (left ? a : b) | (left ? 0 : 1 << 30), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if (old == -1) return;  // the sibling goes on
#pragma unroll
        for (int q = 0; q < 3; ++q) box[q] = fminf(box[q], S.box[6 - side + q][si]);
#pragma unroll
        for (int q = 3; q < 6; ++q) box[q] = fmaxf(box[q], S.box[6 - side + q][si]);
        const int far = old & ~(1 << 30);
        if (left) b = far;
        else a = far;
        slot = si;
        // a child is a leaf when it is one unit of one leaf
        flags = (a == si - 1 && first(si) - first(si - 1) == 1 ? kChildLeafL : 0u) |
                (b == si && first(si + 1) - first(si) == 1 ? kChildLeafR : 0u);
    }
}

// After every unit has climbed: writes the nodes formed, and the subtrees left
// waiting in order; returns their number.
template <int UNITS, typename First>
__device__ uint32_t climb_out(Batch& Bt, ClimbLds<UNITS>& S, int m, BvhNodeC* __restrict__ nodes, BuildItem* items,
                              First first) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int k = tid; k < m; k += kBuildBlock) S.item[k] = 0;
    __syncthreads();
    for (int k = tid; k <= m; k += kBuildBlock) {
        const uint32_t d = S.dest[k];
        if (d != kNoNode) {
            float L[6], R[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                L[q] = S.box[q][k];
                R[q] = S.box[6 + q][k];
            }
            write_compressed(&nodes[d & kChildIndex], (uint32_t)(first(k) - 1) | (d & ~kChildIndex), L, R);
        } else if (S.end[k] != -1) {  // one child waits
            S.item[S.end[k] & (1 << 30) ? k : S.end[k]] = (uint16_t)(k + 1);
        }
    }
    __syncthreads();
    uint32_t base = 0;
    for (int k0 = 0; k0 < m; k0 += kBuildBlock) {
        const int k = k0 + tid;
        const uint32_t it = k < m ? S.item[k] : 0u;
        const uint64_t bal = __ballot(it != 0);
        if (lane == 0) S.wave_sum[wave] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t at = base + (uint32_t)__popcll(bal & __lanemask_lt());
        for (int w = 0; w < kBuildBlock / 64; ++w) {
            const uint32_t c = S.wave_sum[w];
            if (w < wave) at += c;
            base += c;
        }
        if (it != 0) {
            if (at < (uint32_t)kSpine) {
                const int si = (int)it - 1, side = S.end[si] & (1 << 30) ? 6 : 0;
                BuildItem o;
#pragma unroll
                for (int q = 0; q < 6; ++q) o.box[q] = S.box[side + q][si];
                o.l = (int32_t)first(k);
                o.cpl = S.cpl[k];
                items[at] = o;
            } else {
                set_status(Bt, kStInternal);  // the depth bound rules it out
            }
        }
        __syncthreads();
    }
    return min(base, (uint32_t)kSpine);
}

__global__ __launch_bounds__(kBuildBlock) __attribute__((amdgpu_waves_per_eu(8))) void build_tile_kernel(
    Batch Bt, const uint32_t* __restrict__ keys_all, const uint32_t* __restrict__ sorted_idx, Leaf* __restrict__ leaves,
    BvhNodeC* __restrict__ nodes_all, BuildItem* __restrict__ items, uint32_t* __restrict__ counts) {
    static_assert(kBuildTile == kBuildBlock, "a thread per leaf");
    __shared__ ClimbLds<kBuildTile> S;
    int64_t lt;
    const int a = block_asset(Bt, kGBuild, blockIdx.x, &lt);
    const AssetDev& As = Bt.A[a];
    const int64_t n = As.nhf, t0 = lt * kBuildTile;
    const int m = (int)min((int64_t)kBuildTile, n - t0);
    const int tid = threadIdx.x;
    const int64_t i = t0 + tid;
    const uint32_t* __restrict__ keys = keys_all + As.hf;
    const bool on = tid < m;
    float box[6];
    if (on) {
        const uint32_t g = sorted_idx[As.hf + i];
        const uint32_t k0 = keys[i], kl = i > 0 ? keys[i - 1] : 0u;
        bool bad;
        const int3 t = tri_idx(As.hi_F, g, As.nhv, &bad);
        const float3 va = ldv(As.hi_V, t.x), vb = ldv(As.hi_V, t.y), vc = ldv(As.hi_V, t.z);
        Leaf lf;
        lf.a = make_float4(va.x, va.y, va.z, vb.x);
        lf.b = make_float4(vb.y, vb.z, vc.x, vc.y);
        lf.c = make_float4(vc.z, __int_as_float((int32_t)g), 0.f, 0.f);
        leaves[As.hf + i] = lf;
        leaf_box(lf, box);
        S.cpl[tid] = (int8_t)(i > 0 ? prefix_len(kl, k0, i - 1) : -1);
        if (tid == m - 1) S.cpl[m] = (int8_t)(i + 1 < n ? prefix_len(k0, keys[i + 1], i) : -1);
    }
    S.end[tid] = -1;
    S.dest[tid] = kNoNode;
    if (tid == 0) {
        S.end[kBuildTile] = -1;
        S.dest[kBuildTile] = kNoNode;
    }
    __syncthreads();
    auto first = [&](int k) { return (int32_t)t0 + k; };
    if (on) climb(S, tid, box, first);
    __syncthreads();
    const int64_t row = As.tl + lt;
    const uint32_t left = climb_out(Bt, S, m, nodes_all + As.node, items + row * kSpine, first);
    if (tid == 0 && n > kBuildTile) counts[row] = left;  // (a tile that is the whole asset leaves none)
}

// Joins the lists of up to kJoinLast tiles (level 1) or groups (higher levels),
// as many at a time as fit the workgroup's LDS (mostly all of them); what a
// batch leaves waiting goes before the next one.
struct JoinArgs {
    Batch B;
    const uint32_t* keys;
    BvhNodeC* nodes;
    const BuildItem* in;
    const uint32_t* in_count;
    BuildItem* out;
    uint32_t* out_count;
    int level;
};

__global__ __launch_bounds__(kBuildBlock) void build_join_kernel(JoinArgs p) {
    __shared__ ClimbLds<kJoinUnits> S;
    __shared__ int32_t s_first[kJoinUnits + 1];
    __shared__ int32_t s_at[kJoinLast + 1];  // entries before each list
    __shared__ int s_take, s_carry;
    Batch& Bt = p.B;
    int64_t lg;
    const int a = block_asset(Bt, kGJoin1 + p.level - 1, blockIdx.x, &lg);
    const AssetDev& As = Bt.A[a];
    const int64_t n = As.nhf;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t* __restrict__ keys = p.keys + As.hf;
    int64_t span;  // leaves of a list
    const int64_t lists = join_groups(n, p.level - 1, &span), groups = join_groups(n, p.level, nullptr);
    const int64_t c0 = groups == 1 ? 0 : lg * kJoin;
    const int nc = (int)min((int64_t)(groups == 1 ? kJoinLast : kJoin), lists - c0);
    const int64_t row_in = join_row(As.tl, As.join, p.level - 1) + c0, row = join_row(As.tl, As.join, p.level) + lg;
    static_assert(kJoinLast == 128, "two waves sum the list lengths");
    if (tid < 128) {
        int x = tid < nc ? (int)min(p.in_count[row_in + tid], (uint32_t)kSpine) : 0;
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        s_at[tid + 1] = x;
    }
    if (tid == 0) {
        s_at[0] = 0;
        s_carry = 0;
    }
    __syncthreads();
    if (tid >= 64 && tid < 128) s_at[tid + 1] += s_at[64];
    BuildItem* out = p.out + row * kSpine;
    auto first = [&](int k) { return s_first[k]; };
    for (int c = 0; c < nc;) {
        if (tid == 0) s_take = c;
        __syncthreads();
        const int carry = s_carry, before = s_at[c];
        if (tid >= c && tid < nc && carry + s_at[tid + 1] - before <= kJoinUnits) atomicMax(&s_take, tid + 1);
        __syncthreads();
        const int c2 = s_take, m = carry + s_at[c2] - before;
        const int64_t end = min(n, (c0 + c2) * span);  // the batch's last leaf + 1
        float box[kJoinUnits / kBuildBlock][6];
#pragma unroll
        for (int h = 0; h < kJoinUnits / kBuildBlock; ++h) {
            const int u = tid + h * kBuildBlock;
            S.end[u] = -1;
            S.dest[u] = kNoNode;
            if (u < m) {
                const BuildItem* src = out + u;
                if (u >= carry) {
                    const int at = u - carry + before;
                    int lo = c, hi = c2 - 1;  // last list that starts at or before the entry
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (s_at[mid] <= at) lo = mid;
                        else hi = mid - 1;
                    }
                    src = p.in + (row_in + lo) * kSpine + (at - s_at[lo]);
                }
                const BuildItem it = *src;
#pragma unroll
                for (int q = 0; q < 6; ++q) box[h][q] = it.box[q];
                s_first[u] = it.l;
                S.cpl[u] = (int8_t)it.cpl;
            }
        }
        if (tid == 0) {
            S.end[kJoinUnits] = -1;
            S.dest[kJoinUnits] = kNoNode;
            s_first[m] = (int32_t)end;
            S.cpl[m] = (int8_t)(end < n ? prefix_len(keys[end - 1], keys[end], end - 1) : -1);
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kJoinUnits / kBuildBlock; ++h)
            if (tid + h * kBuildBlock < m) climb(S, tid + h * kBuildBlock, box[h], first);
        __syncthreads();
        const uint32_t left = climb_out(Bt, S, m, p.nodes + As.node, out, first);
        if (tid == 0) s_carry = (int)left;
        c = c2;
        __syncthreads();
    }
    if (tid == 0) p.out_count[row] = (uint32_t)s_carry;
}

}  // namespace

int64_t bwd_sort_zero_words(const Layout& L) {
    // the super-tile rows and, behind them, the pair buckets
    return L.save ? (int64_t)(L.bwd_bucket_pf - L.bwd_sup) / 4 : 0;
}

// One asset whose 64-ray batches one workgroup sums at once: the tables of the
// pairs come from the first pass itself, which costs a 256^2 training step 4 us
// less than the launch.
bool pairs_in_one(const BatchHost& H) { return H.L.n == 1 && H.L.t_tex <= 64 * (int64_t)kSortBlock; }

hipError_t launch_sort(const BatchHost& H, int which, int bits, bool* result_in_1, hipStream_t s,
                       hipEvent_t after_first) {
    const Layout& L = H.L;
    const bool bwd = which == kSortBwd;
    const int64_t blocks = H.blocks(bwd ? kGBwdSort : kGSort);
    *result_in_1 = false;
    const int passes = (bits + 7) / 8;
    if (blocks == 0 || passes == 0) return after_first ? hipEventRecord(after_first, s) : hipSuccess;
    uint32_t* kin = (uint32_t*)(H.ws + (bwd ? L.bwd_k0 : L.keys0));
    uint32_t* vin = (uint32_t*)(H.ws + (bwd ? L.bwd_v0 : L.vals0));
    uint32_t* kout = (uint32_t*)(H.ws + (bwd ? L.bwd_k1 : L.keys1));
    uint32_t* vout = (uint32_t*)(H.ws + (bwd ? L.bwd_v1 : L.vals1));
    uint32_t* hist = (uint32_t*)(H.ws + (bwd ? L.bwd_hist : L.hist));
    uint32_t* sup = (uint32_t*)(H.ws + (bwd ? L.bwd_sup : L.sup));
    const int64_t sup_pass = sort_super_rows(bwd ? L.t_btile : L.t_stile, L.n) * 256;
    if (passes > kSortPasses) return hipErrorInvalidValue;
    // the backward's tiles are known on the device: its blocks loop over them
    const dim3 grid((unsigned)(bwd ? std::min<int64_t>(blocks, kBwdSortGrid) : blocks));
    // the super-tile rows start at zero: the BVH sort's lie in the region
    // every forward zeroes first, the backward's are zeroed with the
    // backward's gradient table (bwd_sort_zero_words)
    hipError_t e = hipSuccess;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        uint32_t* sp = sup + sup_pass * p;
        HistArgs h = {H.dev, kin, shift, hist, sp, nullptr, nullptr, nullptr, nullptr, nullptr};
        if (bwd && p == 0) {
            h.keys = kout;
            h.pairs = (const uint32_t*)(H.ws + L.bwd_pairs);
            h.bucket = (const uint32_t*)(H.ws + L.bwd_bucket_pf);
            h.kout = kin;
            h.vout = vin;
            h.bt_pf = (uint32_t*)(H.ws + H.L.bt_pf);
            if (pairs_in_one(H))
                hipLaunchKernelGGL(radix_hist_kernel<kSortPairsOne>, dim3((unsigned)blocks), dim3(kSortBlock), 0, s, h);
            else
                hipLaunchKernelGGL(radix_hist_kernel<kSortPairsFirst>, grid, dim3(kSortBlock), 0, s, h);
        } else if (bwd) {
            hipLaunchKernelGGL(radix_hist_kernel<kSortPairs>, grid, dim3(kSortBlock), 0, s, h);
        } else if (p > 0) {  // code_kernel counted the first pass's digits
            hipLaunchKernelGGL(radix_hist_kernel<kSortBvhKeys>, grid, dim3(kSortBlock), 0, s, h);
        }
        if (p == 0 && after_first && (e = hipEventRecord(after_first, s)) != hipSuccess) return e;
        if (bwd)
            hipLaunchKernelGGL(radix_scatter_kernel<true>, grid, dim3(kSortBlock), 0, s, H.dev,
                               (const uint32_t*)kin, (const uint32_t*)vin, kout, vout, shift,
                               (const uint32_t*)hist, (const uint32_t*)sp);
        else
            hipLaunchKernelGGL(radix_scatter_kernel<false>, grid, dim3(kSortBlock), 0, s, H.dev,
                               (const uint32_t*)kin, (const uint32_t*)vin, kout, vout, shift,
                               (const uint32_t*)hist, (const uint32_t*)sp);
        std::swap(kin, kout);
        std::swap(vin, vout);
        *result_in_1 = !*result_in_1;
    }
    return hipGetLastError();
}

// Faces of an asset past which its partial bounds are reduced by a launch of their
// own: the tiles' reading of all of them grows with the square.  code_kernel with it
// and without, us: 33 and 29 at 2.6M, 59 and 58 at 5.2M, 126 and 150 at 10.5M, 480 and
// 857 at 42M.
constexpr int64_t kBoundsFaces = 6 << 20;

hipError_t launch_bvh_build(const BatchHost& H, hipStream_t s) {
    const Layout& L = H.L;
    if (L.t_hf <= 0) return hipSuccess;
    char* ws = H.ws;
    hipError_t e;
    float* part = (float*)(ws + L.bounds_part);
    uint32_t* k0 = (uint32_t*)(ws + L.keys0);
    uint32_t* v0 = (uint32_t*)(ws + L.vals0);
    BvhNodeC* nodes_c = (BvhNodeC*)(ws + L.nodes_c);
    Leaf* leaves = (Leaf*)(ws + L.leaves);

    if (L.max_hf <= kFrontFaces) {
        hipLaunchKernelGGL(front_kernel, dim3((unsigned)L.n), dim3(kFrontBlock), 0, s, H.dev, k0, v0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(bounds_part_kernel, dim3((unsigned)(H.blocks(kGSort) * kBoundsSplit)), dim3(kBlock), 0, s,
                           H.dev, part);
        const bool one = L.max_hf > kBoundsFaces;
        if (one) hipLaunchKernelGGL(bounds_reduce_kernel, dim3((unsigned)L.n), dim3(kSortBlock), 0, s, H.dev, part);
        hipLaunchKernelGGL(one ? code_kernel<true> : code_kernel<false>, dim3((unsigned)H.blocks(kGSort)),
                           dim3(kSortBlock), 0, s, H.dev, (const float*)part, k0, v0, (uint32_t*)(ws + L.hist),
                           (uint32_t*)(ws + L.sup));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        bool in1 = false;
        if ((e = launch_sort(H, kSortBvh, 30, &in1, s)) != hipSuccess) return e;
    }
    // 30-bit keys take four 8-bit passes: the sorted arrays are back in keys0 / vals0
    BuildItem* items = (BuildItem*)(ws + L.items);
    uint32_t* counts = (uint32_t*)(ws + L.item_cnt);
    hipLaunchKernelGGL(build_tile_kernel, dim3((unsigned)H.blocks(kGBuild)), dim3(kBuildBlock), 0, s, H.dev,
                       (const uint32_t*)k0, (const uint32_t*)v0, leaves, nodes_c, items, counts);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int64_t row = 0;  // first row of the level below
    for (int level = 1; level <= kJoinLevels; ++level) {
        const int64_t blocks = H.blocks(kGJoin1 + level - 1);
        if (blocks == 0) break;  // every asset is whole
        const int64_t next = row + join_rows(L.t_tl, L.n_join, level - 1);
        JoinArgs j;
        j.B = H.dev;
        j.keys = k0;
        j.nodes = nodes_c;
        j.in = items + row * kSpine;
        j.in_count = counts + row;
        j.out = items + next * kSpine;
        j.out_count = counts + next;
        j.level = level;
        hipLaunchKernelGGL(build_join_kernel, dim3((unsigned)blocks), dim3(kBuildBlock), 0, s, j);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        row = next;
    }
    return hipGetLastError();
}

}  // namespace bake
