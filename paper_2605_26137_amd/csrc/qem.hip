// Quadric-error edge-collapse simplification with the edge-constrained optimal
// placement (Sec. 6.1, after Garland & Heckbert 1997), as parallel rounds.
//
// What the section fixes: a quadric Q_v per vertex (squared distances to the
// planes of its faces), the merged quadric Q = Q_v0 + Q_v1 of an edge, the
// placement (solve A x = -b, project onto the edge with t clamped to [0, 1],
// midpoint when A is singular; boundary vertices stay, a boundary edge takes
// its endpoint of lower error), and the same placement for ranking and
// collapse.  The rest are plain rules of this implementation:
//   face quadric      u = (c, -c.p0) with c = (p1 - p0) x (p2 - p0),
//                     K = u u^T / (c.c), nothing for c.c = 0; Q_v sums K over
//                     the faces of v in ascending face order;
//   singular          not (det A > 1e-8 (trace A)^3); solve by the adjugate;
//   cost              max(E(p), 0), E written term by term;
//   valid collapse    one or two faces on the edge, link condition (the rings
//                     share exactly that many vertices), not two endpoints of
//                     three neighbours each (a tetrahedron), not an interior
//                     edge between boundary vertices, and no face around an
//                     endpoint turned to a non-positive dot with its old
//                     normal by the move;
//   a round           edges numbered in (v0, v1) order get the key
//                     (float32(cost) bits, id); eligible = valid with float32
//                     cost <= the k-th smallest, k = ceil(rho n_valid);
//                     m(v) = least eligible key at v, M(v) = least m over v and
//                     its ring; an eligible edge with M(v0) = M(v1) = its key
//                     collapses (no two such edges touch each other's faces);
//                     when they would remove more faces than are left above
//                     the target, only the prefix in key order that fits;
//   collapse          v0 (lower index) survives at p with Q_v0 + Q_v1, faces
//                     holding both endpoints disappear, the others keep their
//                     order.
// All quadric, placement, cost and orientation arithmetic is FP64 with no
// contraction, so every discrete decision (validity, order, singularity)
// follows the plain definition above on the exact FP64 values.
//
// Layout (all in the caller's workspace): positions P [nv][3] and quadrics
// Q [nv][10] in FP64 (q00 q01 q02 q03 q11 q12 q13 q22 q23 q33); face slots
// [3] in their original order, dead ones marked by a negative first corner;
// per vertex a list of its faces (off, num) in an arena; per round the sorted
// unique neighbours (16 slots per vertex, longer rings apart), the edges [ne][2], their float32
// cost bits (0xFFFFFFFF: not collapsible), face counts and FP64 placements, and
// the list of winners.
//
// The lists live from round to round: a collapse moves the faces of v1 to v0
// in place (v0's new list goes to the end of the arena when it outgrows its
// place), and each vertex drops its dead faces as it forms its ring.  When
// half of the vertices are gone (or the arena runs low) the survivors are
// renumbered in their order, the faces compacted and the lists laid out anew:
// the edge order, the keys and the lower-index rule do not change.  A round is
// ten launches (seven of a small mesh): ring, edges, evaluation (two), three
// histogram levels, vertex minima, winners, collapse.  The counts of a round are read back while the
// next one already runs; a round enqueued after the last one finds the `done`
// word set and does nothing.
// Before, every round rebuilt the lists with atomics, scanned and compacted the
// faces (27 launches) and waited for its counts: 1,306,800 -> 10,000 faces
// 32.5 -> 15.9 ms, 20,172 -> 1,000 faces 6.3 -> 3.4 ms.
#pragma clang fp contract(off)

#include <algorithm>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace bake {

namespace {

constexpr int kQB = 256;                    // threads per block of the per-element kernels
constexpr uint32_t kNoKey = 0xFFFFFFFFu;    // cost bits of a non-collapsible edge

constexpr int kRingFaces = 16;              // faces per vertex sorted in registers (see the rings)

// Counter slots
constexpr int kQcEdges = 0, kQcValid = 1, kQcTau = 2, kQcLive = 3, kQcApplied = 4, kQcLiveNext = 5, kQcStatus = 6,
              kQcOut = 7, kQcVerts = 8, kQcDone = 9, kQcDoneNext = 10, kQcArena = 11, kQcPrefix0 = 12, kQcRem0 = 13,
              kQcPrefix1 = 14, kQcRem1 = 15, kQcWinners = 16 /* u64: winners | faces they remove << 32 */,
              kQcRing = 18 /* entries of long rings this round */, kQcGather = 19 /* entries gathered for sorting */,
              kQcLong = 20 /* lists of more than kRingFaces faces */, kQcLongIn = 21 /* of the input */,
              kQcSlots = 32;

inline int64_t blocks_for(int64_t n) { return n <= 0 ? 1 : (n + kQB - 1) / kQB; }


__device__ __forceinline__ bool holds(const int32_t* f, int32_t x) { return f[0] == x || f[1] == x || f[2] == x; }

__device__ __forceinline__ uint32_t f32_bits(double c) { return __float_as_uint((float)c); }

// [x;1]^T Q [x;1]
__device__ __forceinline__ double qerr(const double* q, const double* x) {
    return q[0] * x[0] * x[0] + 2.0 * q[1] * x[0] * x[1] + 2.0 * q[2] * x[0] * x[2] + 2.0 * q[3] * x[0] +
           q[4] * x[1] * x[1] + 2.0 * q[5] * x[1] * x[2] + 2.0 * q[6] * x[1] + q[7] * x[2] * x[2] +
           2.0 * q[8] * x[2] + q[9];
}

// ---- set-up -------------------------------------------------------------

__global__ void qem_init_kernel(const float* __restrict__ V, int64_t nv, const int32_t* __restrict__ Fin,
                                int64_t nf, double* __restrict__ P, int32_t* __restrict__ F,
                                uint32_t* __restrict__ status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nv) {
        P[3 * i] = (double)V[3 * i];
        P[3 * i + 1] = (double)V[3 * i + 1];
        P[3 * i + 2] = (double)V[3 * i + 2];
    }
    if (i < nf) {
        int32_t a = Fin[3 * i], b = Fin[3 * i + 1], c = Fin[3 * i + 2];
        bool bad = a < 0 || b < 0 || c < 0 || a >= nv || b >= nv || c >= nv || a == b || b == c || a == c;
        if (bad) {
            atomicOr(status, 1u);
            a = b = c = 0;  // keep later passes in bounds; the call fails after set-up
        }
        F[3 * i] = a;
        F[3 * i + 1] = b;
        F[3 * i + 2] = c;
    }
}

// ---- vertex -> face lists -------------------------------------------------

// A face with a repeated vertex (only the stand-in for a bad input face, which
// fails the call after set-up) joins no vertex's list: every list then holds
// distinct faces.
__device__ __forceinline__ bool proper(const int32_t* f) { return f[0] != f[1] && f[1] != f[2] && f[0] != f[2]; }

__global__ void qem_deg_kernel(const int32_t* __restrict__ F, int64_t live, uint32_t* __restrict__ deg) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live || !proper(F + 3 * f)) return;
    for (int k = 0; k < 3; ++k) atomicAdd(&deg[F[3 * f + k]], 1u);
}

__global__ void qem_adj_kernel(const int32_t* __restrict__ F, int64_t live, const uint32_t* __restrict__ off,
                               uint32_t* __restrict__ cur, uint32_t* __restrict__ adj) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live || !proper(F + 3 * f)) return;
    for (int k = 0; k < 3; ++k) {
        const int32_t v = F[3 * f + k];
        const uint32_t slot = atomicAdd(&cur[v], 1u);
        adj[off[v] + slot] = (uint32_t)f;
    }
}

// Q_v = sum of the face quadrics around v in ascending face order (the
// unordered list is walked by repeated minimum search).
__global__ void qem_quadric_kernel(const double* __restrict__ P, const int32_t* __restrict__ F, int64_t nv,
                                   const uint32_t* __restrict__ off, const uint32_t* __restrict__ num,
                                   const uint32_t* __restrict__ adj, double* __restrict__ Q, uint32_t* __restrict__ cnt) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const uint32_t b = off[v], n = num[v];
    if (n > (uint32_t)kRingFaces) atomicAdd(&cnt[kQcLongIn], 1u);
    double q[10];
    for (int j = 0; j < 10; ++j) q[j] = 0.0;
    int64_t last = -1;
    for (uint32_t it = 0; it < n; ++it) {
        int64_t f = INT64_MAX;
        for (uint32_t i = 0; i < n; ++i) {
            const int64_t g = adj[b + i];
            if (g > last && g < f) f = g;
        }
        if (f == INT64_MAX) break;  // (the list's faces are distinct: not reached)
        last = f;
        const int32_t* fv = F + 3 * f;
        const double* a = P + 3 * (int64_t)fv[0];
        const double* pb = P + 3 * (int64_t)fv[1];
        const double* pc = P + 3 * (int64_t)fv[2];
        const double e1[3] = {pb[0] - a[0], pb[1] - a[1], pb[2] - a[2]};
        const double e2[3] = {pc[0] - a[0], pc[1] - a[1], pc[2] - a[2]};
        const double c[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                             e1[0] * e2[1] - e1[1] * e2[0]};
        const double cc = c[0] * c[0] + c[1] * c[1] + c[2] * c[2];
        if (cc == 0.0) continue;
        const double u[4] = {c[0], c[1], c[2], -(c[0] * a[0] + c[1] * a[1] + c[2] * a[2])};
        int k = 0;
        for (int i = 0; i < 4; ++i)
            for (int j = i; j < 4; ++j) {
                q[k] = q[k] + (u[i] * u[j]) / cc;
                ++k;
            }
    }
    for (int j = 0; j < 10; ++j) Q[10 * v + j] = q[j];
}

// ---- unique neighbours ----------------------------------------------------

// Is vertex x (taken from the i-th face of v's list) seen in an earlier face?
__device__ __forceinline__ bool seen_before(const int32_t* F, const uint32_t* adj, uint32_t b, uint32_t i,
                                            int32_t x) {
    for (uint32_t j = 0; j < i; ++j)
        if (holds(F + 3 * (int64_t)adj[b + j], x)) return true;
    return false;
}

__device__ __forceinline__ uint32_t shared_count(const int32_t* F, const uint32_t* adj, uint32_t b, uint32_t n,
                                                 int32_t x) {
    uint32_t c = 0;
    for (uint32_t j = 0; j < n; ++j) c += holds(F + 3 * (int64_t)adj[b + j], x) ? 1u : 0u;
    return c;
}

// Cost-bit histograms: digits of 11, 11 and 10 bits.
constexpr int kHistBins = 2048, kHistWords = 2 * kHistBins + 1024;
// Faces of an input up to which one workgroup finds the rank (qem_vmin_small_kernel):
// past them the faces' flags and offsets, idle in the rounds, hold the histograms.
constexpr int64_t kSmallFaces = 2560;
constexpr int kSmallPer = (3 * (int)kSmallFaces + kQB) / kQB;  // cost bits a thread
static_assert(8 * kSmallFaces >= 4 * kHistWords, "keep and koff hold the histograms");
constexpr int kSupBlocks = 32;  // ring blocks whose edge counts are summed together

// The rings.  Around v, the other two corners of every face name v's
// neighbours, each once per face it shares with v: sorted, the runs of that
// list are the unique neighbours in ascending order, and a run of length one
// is an edge with a single face (v is then a boundary vertex).  The lists of up
// to 8 and up to 16 faces are loaded whole (three load latencies) and sorted in
// registers by a network (63 and 191 compare-exchanges; mean valence is six),
// those of up to 24 too where many are that long (384).  A wave sorts one of up to
// 256 faces in LDS, a workgroup a longer one, in LDS or, past 1,024 faces, in
// global memory.
// A ring entry is (x << 3) | min(faces shared with x, 7): the ring carries
// each edge's face count for the per-edge evaluation (vertex indices are
// below 2^28).  Rings of up to kRingKeep vertices are kept in slots of the
// vertex; the first slot of a longer ring says where in RingArgs::longs it lies.
// Only where those run out (many edges of a single face around few vertices) the
// passes walk the face list instead, at a cubic cost.
// 46,080 faces, every ninth vertex with 24 of them, -> 2,304: 5.8 ms, 151 with every
// ring past 16 walked, 10.9 with a wave for each.
constexpr int kRB = 256;        // threads per block of the ring and edge kernels
constexpr int kRingWide = 24;   // faces per vertex sorted in registers where many lists are long
constexpr int kRingWave = 256;  // by a wave
constexpr int kRingLds = 4 * 2 * kRingWave;  // entries a workgroup sorts in LDS
constexpr int kRingKeep = 16;   // ring entries kept per vertex
constexpr uint32_t kBoundary = 1u << 31;  // info: boundary flag, the ring's length below it

__device__ __forceinline__ uint32_t ring_len(uint32_t info) { return info & ~kBoundary; }

template <int N>
__device__ __forceinline__ void sort_network(int32_t e[N]) {  // Batcher's odd-even merge network
#pragma unroll
    for (int p = 1; p < N; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const int32_t a = e[i + j], b = e[i + j + k];
                        e[i + j] = min(a, b);
                        e[i + j + k] = max(a, b);
                    }
}

// The other two corners of face f (corners c0 c1 c2) around v.
__device__ __forceinline__ int2 others(int32_t v, int32_t c0, int32_t c1, int32_t c2) {
    return make_int2(c0 == v ? c1 : c0, c2 == v ? c1 : c2);
}

// Unique neighbours of v from its face list, one at a time (long lists):
// calls fn(x) for each.
template <typename Fn>
__device__ void each_neighbour(const int32_t* F, const uint32_t* adj, uint32_t b, uint32_t n, int32_t v, Fn fn) {
    for (uint32_t i = 0; i < n; ++i) {
        const int32_t* f = F + 3 * (int64_t)adj[b + i];
        for (int k = 0; k < 3; ++k) {
            const int32_t x = f[k];
            if (x != v && !seen_before(F, adj, b, i, x)) fn(x);
        }
    }
}

struct RingArgs {
    const int32_t* F;
    int64_t nv;
    uint32_t *off, *num, *adj;
    int32_t* ring;      // [nv][kRingKeep]
    int32_t* longs;     // [longs_n] longer rings
    uint32_t longs_n;
    int32_t* gather;    // lists that exceed LDS: 2^ceil(log2(2n)) entries each, less than 12 per face in all
    uint32_t* info;     // [nv]
    uint32_t* hcnt;     // [nv] neighbours above v
    uint32_t *part, *sup;  // edges per block and per kSupBlocks blocks
    uint64_t* m;
    uint32_t *hist, *cnt;
    int32_t hist_n;
};

// The ring of a vertex whose ring has no slots of its own, or null where the
// walk over its faces has to do (see above).
__device__ __forceinline__ const int32_t* long_ring(const int32_t* ring, const int32_t* longs, int64_t v) {
    const int32_t at = ring[kRingKeep * v];
    return at >= 0 ? longs + at : nullptr;
}

// Room for a ring of n entries: the vertex's slots or, past them, a place in
// a.longs; null when that is full.
__device__ __forceinline__ int32_t* ring_room(const RingArgs& a, int64_t v, uint32_t n) {
    int32_t* slots = a.ring + (int64_t)kRingKeep * v;
    if (n <= (uint32_t)kRingKeep) return slots;
    const uint32_t at = atomicAdd(&a.cnt[kQcRing], n);
    const bool fits = at <= a.longs_n && n <= a.longs_n - at;
    slots[0] = fits ? (int32_t)at : -1;
    return fits ? a.longs + at : nullptr;
}

// First entry of a sorted ring whose vertex is x or above, when there is one.
__device__ __forceinline__ uint32_t ring_find(const int32_t* ring, uint32_t m, int32_t x) {
    uint32_t at = 0;
    for (uint32_t len = m; len > 1;) {
        const uint32_t half = len >> 1;
        at += (ring[at + half - 1] >> 3) < x ? half : 0u;
        len -= half;
    }
    return at;
}

// What a vertex's ring is known by.
struct RingSums {
    uint32_t uniq, higher, boundary;
};

template <bool BLOCK>
__device__ __forceinline__ void ring_sync() {
    if constexpr (BLOCK) {
        __syncthreads();
    } else {
        wave_sync();
    }
}

// Inclusive count of `on` over the group's threads up to this one, and in all.
template <bool BLOCK>
__device__ __forceinline__ uint32_t ring_count(bool on, uint32_t* s_wave, uint32_t* all) {
    const uint64_t bal = __ballot(on);
    uint32_t before = (uint32_t)__popcll(bal & __lanemask_lt()) + (on ? 1u : 0u), n = (uint32_t)__popcll(bal);
    if constexpr (BLOCK) {
        const int wave = threadIdx.x >> 6;
        __syncthreads();
        if ((threadIdx.x & 63) == 0) s_wave[wave] = n;
        __syncthreads();
        n = 0;
        for (int w = 0; w < kRB / 64; ++w) {
            if (w < wave) before += s_wave[w];
            n += s_wave[w];
        }
    }
    *all = n;
    return before;
}

// The ring of a vertex of many faces, by a wave or by the workgroup: drops the
// dead faces, gathers the other corners into buf (LDS or global, room for
// 2^ceil(log2(2n))), sorts them (bitonic) and writes the runs.
template <bool BLOCK>
__device__ RingSums ring_by_group(const RingArgs& a, int64_t v, int32_t* buf, uint32_t* s_wave, int32_t** s_out) {
    constexpr uint32_t G = BLOCK ? kRB : 64;
    const uint32_t t = threadIdx.x & (G - 1), b = a.off[v], n = a.num[v];
    const int32_t vi = (int32_t)v;
    uint32_t left = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += G) {
        const uint32_t i = i0 + t, f = a.adj[b + min(i, n - 1)];
        const int32_t c0 = a.F[3 * (int64_t)f], c1 = a.F[3 * (int64_t)f + 1], c2 = a.F[3 * (int64_t)f + 2];
        const bool alive = i < n && c0 >= 0;
        uint32_t all;
        const uint32_t at = left + ring_count<BLOCK>(alive, s_wave, &all) - 1;  // (the reads above come first)
        if (alive) {
            a.adj[b + at] = f;
            const int2 xy = others(vi, c0, c1, c2);
            buf[2 * at] = xy.x;
            buf[2 * at + 1] = xy.y;
        }
        left += all;
    }
    uint32_t N = 2;
    while (N < 2 * left) N *= 2;
    for (uint32_t i = 2 * left + t; i < N; i += G) buf[i] = INT32_MAX;
    if (t == 0) a.num[v] = left;
    ring_sync<BLOCK>();
    for (uint32_t k = 2; k <= N; k *= 2)
        for (uint32_t j = k / 2; j > 0; j /= 2) {
            for (uint32_t i = t; i < N / 2; i += G) {
                const uint32_t lo = 2 * i - (i & (j - 1)), hi = lo + j;
                const int32_t x = buf[lo], y = buf[hi];
                if ((x > y) == ((lo & k) == 0)) {
                    buf[lo] = y;
                    buf[hi] = x;
                }
            }
            ring_sync<BLOCK>();
        }
    RingSums r{0, 0, 0};
    int32_t* out = nullptr;
    for (int pass = 0; pass < 2; ++pass) {  // counts, then entries
        uint32_t at = 0;
        for (uint32_t i0 = 0; i0 < 2 * left; i0 += G) {
            const uint32_t i = i0 + t;
            const int32_t x = i < 2 * left ? buf[i] : INT32_MAX;
            const bool head = i < 2 * left && (i == 0 || buf[i - 1] != x);
            uint32_t all, run = 1;
            const uint32_t mine = at + ring_count<BLOCK>(head, s_wave, &all) - 1;
            at += all;
            while (head && run < 7 && i + run < 2 * left && buf[i + run] == x) ++run;
            if (pass == 0) {
                uint32_t some;
                ring_count<BLOCK>(head && x > vi, s_wave, &some);
                r.higher += some;
                ring_count<BLOCK>(head && run == 1, s_wave, &some);
                if (some) r.boundary = kBoundary;
            } else if (head) {
                out[mine] = (x << 3) | (int32_t)run;
            }
        }
        if (pass == 0) {
            r.uniq = at;
            if (t == 0) *s_out = ring_room(a, v, at);
            ring_sync<BLOCK>();
            out = *s_out;
            if (!out) break;
        }
    }
    return r;
}

// Start of a round: drops dead faces from the lists, forms the rings, sums
// the edges per block; clears what the later launches of the round count in.
template <bool WIDE>
__global__ void __launch_bounds__(kRB) qem_ring_kernel(RingArgs a) {
    __shared__ uint32_t s_sum[kRB / 64];
    __shared__ uint64_t s_big[kRB / 64];
    __shared__ int32_t s_buf[kRingLds];
    __shared__ uint32_t s_wave[kRB / 64], s_at;
    __shared__ int32_t* s_out[kRB / 64];
    const int64_t v = (int64_t)blockIdx.x * kRB + threadIdx.x;
    const int t = threadIdx.x;
    if (a.cnt[kQcDoneNext]) {
        if (v == 0) a.cnt[kQcDone] = 1u;
        return;
    }
    for (int64_t i = v; i < a.hist_n; i += (int64_t)gridDim.x * kRB) a.hist[i] = 0u;
    if (v == 0) {
        a.cnt[kQcLive] = a.cnt[kQcLiveNext];
        a.cnt[kQcWinners] = a.cnt[kQcWinners + 1] = 0u;
    }
    uint32_t uniq = 0, higher = 0, boundary = 0, n = 0, b = 0, keep = kRingKeep;
    bool many = false;
    int32_t* ring = a.ring + (int64_t)kRingKeep * v;
    const int32_t vi = (int32_t)v;
    auto emit = [&](int32_t x, uint32_t faces) {
        if (faces == 1) boundary = kBoundary;
        if (uniq < keep) ring[uniq] = (x << 3) | (int32_t)(faces < 7 ? faces : 7);
        ++uniq;
        if (x > vi) ++higher;
    };
    // a list of up to kN faces by its thread, kC loaded at once
    auto sorted = [&](auto faces, auto at_once) {
        constexpr int kN = decltype(faces)::value, kC = decltype(at_once)::value;
        uint32_t left = 0;
        int32_t e[2 * kN];
#pragma unroll
        for (int i0 = 0; i0 < kN; i0 += kC) {
            uint32_t f[kC];
            int32_t c[kC][3];
#pragma unroll
            for (int i = 0; i < kC; ++i) f[i] = a.adj[b + min((uint32_t)(i0 + i), n - 1)];  // (no branch around a load)
#pragma unroll
            for (int i = 0; i < kC; ++i)
#pragma unroll
                for (int k = 0; k < 3; ++k) c[i][k] = a.F[3 * (int64_t)f[i] + k];
#pragma unroll
            for (int i = 0; i < kC; ++i) {
                const bool alive = (uint32_t)(i0 + i) < n && c[i][0] >= 0;
                const int2 xy = others(vi, c[i][0], c[i][1], c[i][2]);
                e[2 * (i0 + i)] = alive ? xy.x : INT32_MAX;
                e[2 * (i0 + i) + 1] = alive ? xy.y : INT32_MAX;
                if (alive) {
                    if (left != (uint32_t)(i0 + i)) a.adj[b + left] = f[i];
                    ++left;
                }
            }
        }
        if (left != n) a.num[v] = left;
        sort_network<2 * kN>(e);
        if constexpr (kN > kRingFaces) {  // the length decides on the place
            uint32_t len = e[0] != INT32_MAX ? 1u : 0u;
#pragma unroll
            for (int i = 1; i < 2 * kN; ++i) len += e[i] != e[i - 1] && e[i] != INT32_MAX ? 1u : 0u;
            ring = ring_room(a, v, len);
            keep = ring ? len : 0u;
        }
        int32_t cur = e[0];
        uint32_t run = 1;
#pragma unroll
        for (int i = 1; i < 2 * kN; ++i) {
            if (e[i] == cur) {
                ++run;
            } else {
                emit(cur, run);
                cur = e[i];
                run = 1;
            }
        }
        if (cur != INT32_MAX) emit(cur, run);
    };
    if (v < a.nv) {
        a.m[v] = ~0ull;
        b = a.off[v];
        n = a.num[v];
        if (n == 0) {
        } else if (n <= 8) {
            sorted(std::integral_constant<int, 8>(), std::integral_constant<int, 8>());
        } else if (n <= (uint32_t)kRingFaces) {
            sorted(std::integral_constant<int, kRingFaces>(), std::integral_constant<int, kRingFaces>());
            many = uniq > (uint32_t)kRingKeep;  // (edges of a single face each)
        } else if (WIDE && n <= (uint32_t)kRingWide) {
            sorted(std::integral_constant<int, WIDE ? kRingWide : 8>(), std::integral_constant<int, 8>());
        } else {
            many = true;
        }
    }
    const int lane = t & 63, wave = t >> 6;
    const bool big = n > (uint32_t)kRingWave;
    const uint64_t longer = __ballot(n > (uint32_t)kRingFaces);
    auto take = [&](const RingSums& x) {
        uniq = x.uniq;
        higher = x.higher;
        boundary = x.boundary;
    };
    for (uint64_t todo = __ballot(many && !big); todo != 0; todo &= todo - 1) {
        const int src = __builtin_ctzll(todo);
        const RingSums x = ring_by_group<false>(a, v - lane + src, s_buf + 2 * kRingWave * wave, nullptr, &s_out[wave]);
        if (lane == src) take(x);
        ring_sync<false>();
    }
    uint32_t s = big ? 0u : higher;
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    const uint64_t bigs = __ballot(big);
    if (lane == 0) {
        s_sum[wave] = s;
        s_big[wave] = bigs;
        if (longer) atomicAdd(&a.cnt[kQcLong], (uint32_t)__popcll(longer));
    }
    __syncthreads();
    uint32_t tot = 0;
    for (int k = 0; k < kRB / 64; ++k) {
        tot += s_sum[k];
        for (uint64_t todo = s_big[k]; todo != 0; todo &= todo - 1) {  // by the workgroup (none, mostly)
            const int src = 64 * k + __builtin_ctzll(todo);
            const int64_t w = v - t + src;
            const uint32_t len = a.num[w];
            int32_t* buf = s_buf;
            if (2 * len > (uint32_t)kRingLds) {
                uint32_t N = 2;
                while (N < 2 * len) N *= 2;
                if (t == 0) s_at = atomicAdd(&a.cnt[kQcGather], N);
                __syncthreads();
                buf = a.gather + s_at;
            }
            const RingSums x = ring_by_group<true>(a, w, buf, s_wave, &s_out[0]);
            if (t == src) take(x);
            tot += x.higher;
            __syncthreads();
        }
    }
    if (v < a.nv) {
        a.info[v] = uniq | boundary;
        a.hcnt[v] = higher;
    }
    if (t == 0) {
        a.part[blockIdx.x] = tot;
        if (tot) atomicAdd(&a.sup[blockIdx.x / kSupBlocks], tot);
    }
}

// Numbers the edges: (v, x) for the neighbours x above v, v ascending, then x.
// A block finds its first edge from the counts of the blocks before it (whole
// groups of kSupBlocks, then single blocks): no scan of its own.
__global__ void __launch_bounds__(kRB) qem_edge_kernel(RingArgs a, uint32_t* __restrict__ eoff,
                                                       int32_t* __restrict__ E) {
    __shared__ uint32_t s_sum[2][kRB / 64];
    if (a.cnt[kQcDone]) return;
    const int64_t v = (int64_t)blockIdx.x * kRB + threadIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t S = blockIdx.x / kSupBlocks;
    uint32_t before = 0;
    for (int64_t i = t; i < S; i += kRB) before += a.sup[i];
    const int64_t b0 = S * kSupBlocks + t;
    if (t < kSupBlocks && b0 < (int64_t)blockIdx.x) before += a.part[b0];
    for (int o = 32; o >= 1; o >>= 1) before += __shfl_xor(before, o, 64);
    const uint32_t h = v < a.nv ? a.hcnt[v] : 0u;
    uint32_t x = h;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) {
        s_sum[0][wave] = before;
        s_sum[1][wave] = x;
    }
    __syncthreads();
    uint32_t base = 0;
    for (int k = 0; k < kRB / 64; ++k) {
        base += s_sum[0][k];
        if (k < wave) base += s_sum[1][k];
    }
    uint32_t e = base + x - h;
    if (blockIdx.x == gridDim.x - 1 && t == kRB - 1) a.cnt[kQcEdges] = e + h;
    uint32_t m = 0;
    const int32_t* ring = a.ring;
    if (v < a.nv) {
        eoff[v] = e;
        m = ring_len(a.info[v]);
        ring = m <= (uint32_t)kRingKeep ? a.ring + (int64_t)kRingKeep * v : long_ring(a.ring, a.longs, v);
    }
    // ascending: those above v come last
    if (m <= (uint32_t)kRingKeep) {
        for (uint32_t j = m - h; j < m; ++j, ++e) {
            E[2 * (int64_t)e] = (int32_t)v;
            E[2 * (int64_t)e + 1] = ring[j] >> 3;
        }
    } else if (!ring) {
        const uint32_t b = a.off[v], n = a.num[v];
        int32_t last = (int32_t)v;
        for (uint32_t j = 0; j < h; ++j, ++e) {
            int32_t next = INT32_MAX;
            each_neighbour(a.F, a.adj, b, n, (int32_t)v, [&](int32_t y) {
                if (y > last && y < next) next = y;
            });
            E[2 * (int64_t)e] = (int32_t)v;
            E[2 * (int64_t)e + 1] = next;
            last = next;
        }
    }
    // a longer ring by the whole wave
    for (uint64_t todo = __ballot(m > (uint32_t)kRingKeep && ring); todo != 0; todo &= todo - 1) {
        const int src = __builtin_ctzll(todo);
        const int64_t w = v - lane + src;
        const uint32_t first = __shfl(e, src, 64), n = __shfl(h, src, 64), below = __shfl(m, src, 64) - n;
        const int32_t* r = long_ring(a.ring, a.longs, w) + below;
        for (uint32_t j = lane; j < n; j += 64) {
            E[2 * (int64_t)(first + j)] = (int32_t)w;
            E[2 * (int64_t)(first + j) + 1] = r[j] >> 3;
        }
    }
}

// ---- per-edge collapse ----------------------------------------------------

// Faces around `moved` that lack `other` keep a positive dot of old and new
// normal when `moved` (now at pm) goes to p; only the other two corners are
// loaded.
__device__ bool no_fold(const double* P, const int32_t* F, const uint32_t* adj, uint32_t b, uint32_t n,
                        int32_t moved, int32_t other, const double* pm, const double* p) {
    for (uint32_t i = 0; i < n; ++i) {
        const int32_t* f = F + 3 * (int64_t)adj[b + i];
        const int32_t f0 = f[0], f1 = f[1], f2 = f[2];
        if (f0 == other || f1 == other || f2 == other) continue;
        const int32_t fk[3] = {f0, f1, f2};
        double a[3][3], q[3][3];
        for (int k = 0; k < 3; ++k) {
            if (fk[k] == moved) {
                for (int c = 0; c < 3; ++c) {
                    a[k][c] = pm[c];
                    q[k][c] = p[c];
                }
            } else {
                const double* src = P + 3 * (int64_t)fk[k];
                for (int c = 0; c < 3; ++c) {
                    a[k][c] = src[c];
                    q[k][c] = src[c];
                }
            }
        }
        double e1[3], e2[3], g1[3], g2[3];
        for (int c = 0; c < 3; ++c) {
            e1[c] = a[1][c] - a[0][c];
            e2[c] = a[2][c] - a[0][c];
            g1[c] = q[1][c] - q[0][c];
            g2[c] = q[2][c] - q[0][c];
        }
        const double n0[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                              e1[0] * e2[1] - e1[1] * e2[0]};
        const double n1[3] = {g1[1] * g2[2] - g1[2] * g2[1], g1[2] * g2[0] - g1[0] * g2[2],
                              g1[0] * g2[1] - g1[1] * g2[0]};
        const double d = n0[0] * n1[0] + n0[1] * n1[1] + n0[2] * n1[2];
        if (!(d > 0.0)) return false;
    }
    return true;
}

struct EvalArgs {
    const double* P;
    const double* Q;
    const int32_t* F;
    const uint32_t *off, *num, *adj, *info, *hcnt, *eoff;
    const int32_t *ring, *longs;
    const int32_t* E;
    const uint32_t* cnt;
    int64_t nv;
    int midpoint;
    uint32_t* bits;     // [cap] float32 cost bits, kNoKey when not collapsible
    uint8_t* faces;     // [cap]
    double* pl;         // [cap][3]
    uint32_t* sup;      // the rings' edge sums, cleared here for the next round
    int64_t sup_n;
    double* cost;       // optional (edge listing): FP64 cost
};

// First half of the evaluation, per edge: link condition, placement and cost.
// The turned-normal test follows per vertex (qem_fold_kernel), except around
// vertices whose ring has no slots.
__global__ void __launch_bounds__(kQB) qem_eval_kernel(EvalArgs a) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a.cnt[kQcDone]) return;
    if (tid < a.sup_n) a.sup[tid] = 0u;
    const int64_t ne = a.cnt[kQcEdges];
    // (one edge per thread of a closed mesh's grid)
    for (int64_t e = tid; e < ne; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v0 = a.E[2 * e], v1 = a.E[2 * e + 1];
        const uint32_t i0 = a.info[v0], i1 = a.info[v1];
        const uint32_t m0 = ring_len(i0), m1 = ring_len(i1);
        const int32_t *ring0 = a.ring + (int64_t)kRingKeep * v0, *ring1 = a.ring + (int64_t)kRingKeep * v1;
        const bool long0 = m0 > (uint32_t)kRingKeep, long1 = m1 > (uint32_t)kRingKeep;
        // faces on the edge (seven stands for more), and common neighbours
        uint32_t c = 0, common = 0;
        if (!long0 && !long1) {
            // both rings whole, compared four entries against four (entries past
            // a ring's end match nothing)
            int32_t r0[kRingKeep], r1[kRingKeep];
#pragma unroll
            for (int q = 0; q < kRingKeep / 4; ++q) {
                const int4 w0 = reinterpret_cast<const int4*>(ring0)[q], w1 = reinterpret_cast<const int4*>(ring1)[q];
                const int32_t x0[4] = {w0.x, w0.y, w0.z, w0.w}, x1[4] = {w1.x, w1.y, w1.z, w1.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    r0[4 * q + k] = (uint32_t)(4 * q + k) < m0 ? x0[k] : -1;
                    r1[4 * q + k] = (uint32_t)(4 * q + k) < m1 ? x1[k] >> 3 : -2;
                }
            }
#pragma unroll
            for (int q = 0; q < kRingKeep; ++q) {
                const int32_t x = r0[q] >> 3;
                if (x == v1) c = (uint32_t)(r0[q] & 7);
                r0[q] = x;
            }
#pragma unroll
            for (int q = 0; q < kRingKeep; q += 4)
#pragma unroll
                for (int t = 0; t < kRingKeep; t += 4)
                    if ((uint32_t)q < m0 && (uint32_t)t < m1) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int l = 0; l < 4; ++l) common += r0[q + k] == r1[t + l] ? 1u : 0u;
                    }
        } else if ((!long0 || (ring0 = long_ring(a.ring, a.longs, v0))) &&
                   (!long1 || (ring1 = long_ring(a.ring, a.longs, v1)))) {
            // the shorter ring's entries looked up in the longer one, eight at a
            // time; the other end's entry holds the edge's faces, and is in
            // neither ring twice
            const bool swap = m0 > m1;
            const int32_t *few = swap ? ring1 : ring0, *all = swap ? ring0 : ring1, other = swap ? v0 : v1;
            const uint32_t mf = swap ? m1 : m0, ma = swap ? m0 : m1;
            for (uint32_t i = 0; i < mf; i += 8) {
                int32_t x[8];
                uint32_t at[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    x[q] = few[min(i + q, mf - 1)];
                    at[q] = 0;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint32_t f = (uint32_t)(x[q] & 7);
                    x[q] = i + q < mf ? x[q] >> 3 : -1;
                    if (x[q] == other) c = f;
                }
                for (uint32_t len = ma; len > 1;) {
                    const uint32_t half = len >> 1;
#pragma unroll
                    for (int q = 0; q < 8; ++q) at[q] += (all[at[q] + half - 1] >> 3) < x[q] ? half : 0u;
                    len -= half;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) common += (all[at[q]] >> 3) == x[q] ? 1u : 0u;
            }
        } else {
            const uint32_t b0 = a.off[v0], n0 = a.num[v0], b1 = a.off[v1], n1 = a.num[v1];
            c = shared_count(a.F, a.adj, b0, n0, v1);
            c = c < 7 ? c : 7;
            if (c >= 1 && c <= 2)
                each_neighbour(a.F, a.adj, b0, n0, v0, [&](int32_t x) {
                    if (x != v1 && shared_count(a.F, a.adj, b1, n1, x) > 0) ++common;
                });
        }
        bool ok = c >= 1 && c <= 2;
        double p[3] = {0.0, 0.0, 0.0}, cost = 0.0;
        if (ok) {
            if (common != c) ok = false;
            if (m0 == 3 && m1 == 3) ok = false;
        }
        const bool bv0 = (i0 & kBoundary) != 0, bv1 = (i1 & kBoundary) != 0, bedge = c == 1;
        if (ok && !bedge && bv0 && bv1) ok = false;
        if (ok) {
            double q[10];
            const double* q0 = a.Q + 10 * (int64_t)v0;
            const double* q1 = a.Q + 10 * (int64_t)v1;
            for (int k = 0; k < 10; ++k) q[k] = q0[k] + q1[k];
            const double* p0 = a.P + 3 * (int64_t)v0;
            const double* p1 = a.P + 3 * (int64_t)v1;
            if (bedge) {
                const double e0 = qerr(q, p0), e1 = qerr(q, p1);
                const double* src = e1 < e0 ? p1 : p0;
                p[0] = src[0];
                p[1] = src[1];
                p[2] = src[2];
            } else if (bv0) {
                p[0] = p0[0];
                p[1] = p0[1];
                p[2] = p0[2];
            } else if (bv1) {
                p[0] = p1[0];
                p[1] = p1[1];
                p[2] = p1[2];
            } else {
                double t = 0.5;
                if (!a.midpoint) {
                    const double det = q[0] * (q[4] * q[7] - q[5] * q[5]) - q[1] * (q[1] * q[7] - q[5] * q[2]) +
                                       q[2] * (q[1] * q[5] - q[4] * q[2]);
                    const double tr = q[0] + q[4] + q[7];
                    if (det > 1e-8 * tr * tr * tr) {
                        const double i00 = q[4] * q[7] - q[5] * q[5], i01 = q[2] * q[5] - q[1] * q[7];
                        const double i02 = q[1] * q[5] - q[2] * q[4], i11 = q[0] * q[7] - q[2] * q[2];
                        const double i12 = q[1] * q[2] - q[0] * q[5], i22 = q[0] * q[4] - q[1] * q[1];
                        double x[3];
                        x[0] = -(i00 * q[3] + i01 * q[6] + i02 * q[8]) / det;
                        x[1] = -(i01 * q[3] + i11 * q[6] + i12 * q[8]) / det;
                        x[2] = -(i02 * q[3] + i12 * q[6] + i22 * q[8]) / det;
                        const double d[3] = {p1[0] - p0[0], p1[1] - p0[1], p1[2] - p0[2]};
                        const double dd = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                        if (dd > 0.0) {
                            t = ((x[0] - p0[0]) * d[0] + (x[1] - p0[1]) * d[1] + (x[2] - p0[2]) * d[2]) / dd;
                            if (!(t > 0.0)) t = 0.0;
                            if (t > 1.0) t = 1.0;
                        } else {
                            t = 0.0;
                        }
                    }
                }
                for (int k = 0; k < 3; ++k) p[k] = (1.0 - t) * p0[k] + t * p1[k];
            }
            const double E = qerr(q, p);
            if (E == E) {
                cost = E > 0.0 ? E : 0.0;
                const double q0c[3] = {p0[0], p0[1], p0[2]}, q1c[3] = {p1[0], p1[1], p1[2]};
                if (long0) ok = no_fold(a.P, a.F, a.adj, a.off[v0], a.num[v0], v0, v1, q0c, p);
                if (ok && long1) ok = no_fold(a.P, a.F, a.adj, a.off[v1], a.num[v1], v1, v0, q1c, p);
            } else {
                ok = false;
            }
        }
        a.bits[e] = ok ? f32_bits(cost) : kNoKey;
        a.faces[e] = (uint8_t)c;
        a.pl[3 * e] = p[0];
        a.pl[3 * e + 1] = p[1];
        a.pl[3 * e + 2] = p[2];
        if (a.cost) a.cost[e] = cost;
    }
}

// Second half: around each vertex, the faces that a collapse of one of its
// edges would keep must not turn.  Eight lanes per vertex: a lane holds one
// face (its corners gathered once for all the edges, not once per edge), the
// vertex's still possible edges pass by in LDS, and an edge that turns a face
// loses its key.  Both ends of an edge clear the same word with the same value.
// Bound by the gathers of the corners: before, every edge gathered the faces
// around both of its ends (110 rounds of 1,306,800 -> 10,000 faces: 8.6 ms,
// now 6.7 ms for both halves).
constexpr int kFoldVerts = kQB / 8;
__global__ void __launch_bounds__(kQB) qem_fold_kernel(EvalArgs a) {
    __shared__ double s_p[kFoldVerts][kRingKeep][3];
    __shared__ int32_t s_x[kFoldVerts][kRingKeep];
    if (a.cnt[kQcDone]) return;
    const int g = threadIdx.x >> 3, l = threadIdx.x & 7, sh = (threadIdx.x & 63) & ~7;
    const int64_t v = (int64_t)blockIdx.x * kFoldVerts + g;
    const int32_t vi = (int32_t)v;
    uint32_t n = 0, m = 0, b = 0;
    if (v < a.nv) {
        n = a.num[v];
        m = ring_len(a.info[v]);
        b = a.off[v];
        if (m > (uint32_t)kRingKeep) n = m = 0;
    }
    // the lane's first face: its loads are independent of the edges'
    int32_t fk[3] = {-1, -1, -1};
    double c[3][3];
    auto load_face = [&](uint32_t i) {
        const int32_t* f = a.F + 3 * (int64_t)a.adj[b + i];
#pragma unroll
        for (int k = 0; k < 3; ++k) fk[k] = f[k];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int d = 0; d < 3; ++d) c[k][d] = a.P[3 * (int64_t)fk[k] + d];
    };
    if ((uint32_t)l < n) load_face(l);
    int32_t x[2];
    uint32_t low = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t j = (uint32_t)(l + 8 * h);
        x[h] = j < m ? a.ring[(int64_t)kRingKeep * v + j] >> 3 : -1;
        low += (uint32_t)__popcll((__ballot(x[h] >= 0 && x[h] < vi) >> sh) & 0xFFull);
    }
    int64_t e[2] = {0, 0};
    bool live[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t j = (uint32_t)(l + 8 * h);
        live[h] = x[h] >= 0;
        if (live[h]) {
            if (x[h] > vi) {
                e[h] = (int64_t)a.eoff[v] + (j - low);
            } else {  // x's edge to v: its rank among x's neighbours above x
                const uint32_t mx = ring_len(a.info[x[h]]);
                uint32_t r = 0;
                if (mx <= (uint32_t)kRingKeep) {
                    const int4* rx = reinterpret_cast<const int4*>(a.ring + (int64_t)kRingKeep * x[h]);
#pragma unroll
                    for (int q = 0; q < kRingKeep / 4; ++q) {
                        const int4 w = rx[q];
                        const int32_t y[4] = {w.x >> 3, w.y >> 3, w.z >> 3, w.w >> 3};
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            r += (uint32_t)(4 * q + k) < mx && y[k] > x[h] && y[k] < vi ? 1u : 0u;
                    }
                } else if (const int32_t* rx = long_ring(a.ring, a.longs, x[h])) {
                    r = ring_find(rx, mx, vi) - (mx - a.hcnt[x[h]]);
                } else {
                    each_neighbour(a.F, a.adj, a.off[x[h]], a.num[x[h]], x[h],
                                   [&](int32_t y) { r += y > x[h] && y < vi ? 1u : 0u; });
                }
                e[h] = (int64_t)a.eoff[x[h]] + r;
            }
        }
    }
    {
        // an edge's placement is loaded beside its key: most edges have one
        uint32_t key[2] = {kNoKey, kNoKey};
        double q[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (live[h]) {
                key[h] = a.bits[e[h]];
#pragma unroll
                for (int k = 0; k < 3; ++k) q[h][k] = a.pl[3 * e[h] + k];
            }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            live[h] = key[h] != kNoKey;
            s_x[g][l + 8 * h] = live[h] ? x[h] : -1;
            if (live[h]) {
#pragma unroll
                for (int k = 0; k < 3; ++k) s_p[g][l + 8 * h][k] = q[h][k];
            }
        }
    }
    wave_sync();
    uint32_t turned = 0;  // bit j: edge j turns a face (the same in all lanes of the vertex)
    for (uint32_t f0 = 0; __ballot(f0 < n) != 0; f0 += 8) {
        const bool has = f0 + l < n;
        if (has && f0 > 0) load_face(f0 + l);
        double n0[3];
        {
            double e1[3], e2[3];
            for (int d = 0; d < 3; ++d) {
                e1[d] = c[1][d] - c[0][d];
                e2[d] = c[2][d] - c[0][d];
            }
            n0[0] = e1[1] * e2[2] - e1[2] * e2[1];
            n0[1] = e1[2] * e2[0] - e1[0] * e2[2];
            n0[2] = e1[0] * e2[1] - e1[1] * e2[0];
        }
        for (uint32_t j = 0; __ballot(j < m) != 0; ++j) {
            const int32_t xj = j < m ? s_x[g][j] : -1;
            bool bad = false;
            if (has && xj >= 0 && fk[0] != xj && fk[1] != xj && fk[2] != xj) {
                double q[3][3], e1[3], e2[3];
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int d = 0; d < 3; ++d) q[k][d] = fk[k] == vi ? s_p[g][j][d] : c[k][d];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    e1[d] = q[1][d] - q[0][d];
                    e2[d] = q[2][d] - q[0][d];
                }
                const double n1[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                                      e1[0] * e2[1] - e1[1] * e2[0]};
                const double d = n0[0] * n1[0] + n0[1] * n1[1] + n0[2] * n1[2];
                bad = !(d > 0.0);
            }
            if ((__ballot(bad) >> sh) & 0xFFull) turned |= 1u << j;
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (live[h] && (turned >> (l + 8 * h)) & 1u) a.bits[e[h]] = kNoKey;
}

// ---- round selection ------------------------------------------------------

// The k-th smallest cost bits, digit by digit: each level's histogram counts
// the valid edges whose upper digits match the prefix chosen so far, and the
// next launch picks the digit where the running count first reaches the rank
// still to find.  Every workgroup picks for itself; block 0 leaves the choice
// for the launches after it.
struct Select {
    uint32_t prefix;  // digits chosen so far
    uint32_t rem;     // rank still to find within the chosen prefix (1-based)
};

// The digit of a level's histogram (nb = 1024 or 2048 bins), by a whole block
// of kQB threads; the result in every thread.  rho >= 0: the first level, the
// rank is ceil(rho * total) and *total_out takes the total.
__device__ Select select_digit(const uint32_t* __restrict__ h, int nb, Select in, double rho, uint32_t* total_out) {
    __shared__ uint32_t s_wave[kQB / 64];
    __shared__ Select s_out;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, per = nb / kQB;
    uint32_t c[kHistBins / kQB], sum = 0;
    for (int k = 0; k < kHistBins / kQB; ++k) {
        c[k] = k < per ? h[per * t + k] : 0u;
        sum += c[k];
    }
    uint32_t inc = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    __syncthreads();
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t total = 0;
    for (int k = 0; k < kQB / 64; ++k) {
        if (k < wave) inc += s_wave[k];
        total += s_wave[k];
    }
    uint32_t rem = in.rem;
    if (rho >= 0.0) {
        int64_t k = (int64_t)ceil(rho * (double)total);
        if (k < 1) k = 1;
        if (k > (int64_t)total) k = total;
        rem = (uint32_t)k;
    }
    const uint32_t before = inc - sum;
    if (total == 0) {
        if (t == 0) s_out = Select{0u, 0u};
    } else if (before < rem && rem <= inc) {
        uint32_t acc = before;
        for (int k = 0; k < kHistBins / kQB; ++k) {
            if (k < per && rem <= acc + c[k]) {
                s_out = Select{in.prefix * (uint32_t)nb + (uint32_t)(per * t + k), rem - acc};
                break;
            }
            acc += c[k];
        }
    }
    __syncthreads();
    const Select out = s_out;
    __syncthreads();
    if (total_out) *total_out = total;
    return out;
}

// What the levels before `level` chose (block-wide): level 1 picks digit 0,
// level 2 digit 1, level 3 (vertex minima) digit 2, the earlier ones are read.
__device__ Select selection(const uint32_t* __restrict__ hist, uint32_t* __restrict__ cnt, int level, double rho) {
    Select st{0u, 0u};
    if (level == 1) {
        uint32_t total = 0;
        st = select_digit(hist, kHistBins, st, rho, &total);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            cnt[kQcPrefix0] = st.prefix;
            cnt[kQcRem0] = st.rem;
            cnt[kQcValid] = total;
        }
    } else if (level == 2) {
        st = select_digit(hist + kHistBins, kHistBins, Select{cnt[kQcPrefix0], cnt[kQcRem0]}, -1.0, nullptr);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            cnt[kQcPrefix1] = st.prefix;
            cnt[kQcRem1] = st.rem;
        }
    } else if (level == 3) {
        st = select_digit(hist + 2 * kHistBins, 1024, Select{cnt[kQcPrefix1], cnt[kQcRem1]}, -1.0, nullptr);
        if (blockIdx.x == 0 && threadIdx.x == 0) cnt[kQcTau] = st.prefix;
    }
    return st;
}

// Level l histogram of the valid cost bits whose upper digits match the
// prefix chosen from levels 0..l-1.  Few blocks: each merges its bins with
// global atomics.
template <int LEVEL>
__global__ void __launch_bounds__(kQB) qem_hist_kernel(const uint32_t* __restrict__ bits, uint32_t* __restrict__ hist,
                                                       uint32_t* __restrict__ cnt, double rho) {
    constexpr int kBins = LEVEL == 2 ? 1024 : kHistBins;
    constexpr int kShift = LEVEL == 0 ? 21 : (LEVEL == 1 ? 10 : 0), kUp = LEVEL == 1 ? 21 : 10;
    __shared__ uint32_t h[kBins];
    if (cnt[kQcDone]) return;
    for (int i = threadIdx.x; i < kBins; i += kQB) h[i] = 0;
    Select st{0u, 0u};
    if (LEVEL > 0) st = selection(hist, cnt, LEVEL, rho);
    else __syncthreads();
    if (LEVEL > 0 && st.rem == 0) return;  // no valid edge
    const int64_t ne = cnt[kQcEdges];
    constexpr int kU = 4;
    const int64_t stride = (int64_t)gridDim.x * kQB;
    for (int64_t e0 = (int64_t)blockIdx.x * kQB + threadIdx.x; e0 < ne; e0 += kU * stride) {
        uint32_t x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = e0 + u * stride < ne ? bits[e0 + u * stride] : kNoKey;
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (x[u] != kNoKey && (LEVEL == 0 || (x[u] >> kUp) == st.prefix))
                atomicAdd(&h[(x[u] >> kShift) & (kBins - 1)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kBins; i += kQB)
        if (h[i]) atomicAdd(&hist[LEVEL * kHistBins + i], h[i]);
}

// m(v): least key of the eligible edges at v.
__device__ __forceinline__ void vertex_min(const int32_t* __restrict__ E, int64_t e, uint32_t x, uint64_t* __restrict__ m) {
    const unsigned long long key = ((unsigned long long)x << 32) | (unsigned long long)(uint32_t)e;
    const int2 v = reinterpret_cast<const int2*>(E)[e];
    atomicMin((unsigned long long*)&m[v.x], key);
    atomicMin((unsigned long long*)&m[v.y], key);
}

__global__ void __launch_bounds__(kQB) qem_vmin_kernel(const int32_t* __restrict__ E,
                                                       const uint32_t* __restrict__ bits,
                                                       const uint32_t* __restrict__ hist, uint32_t* __restrict__ cnt,
                                                       uint64_t* __restrict__ m) {
    if (cnt[kQcDone]) return;
    const Select st = selection(hist, cnt, 3, -1.0);
    if (st.rem == 0) return;  // no valid edge
    const int64_t ne = cnt[kQcEdges];
    for (int64_t e = (int64_t)blockIdx.x * kQB + threadIdx.x; e < ne; e += (int64_t)gridDim.x * kQB) {
        const uint32_t x = bits[e];
        if (x > st.prefix) continue;  // kNoKey too: it is above every cost
        vertex_min(E, e, x, m);
    }
}

// The three levels and the minima of a small mesh by one workgroup, which keeps the
// edges' cost bits in registers and the histograms in LDS: no memory for them in
// the workspace, whose 20 KB would be most of a small mesh's.
__global__ void __launch_bounds__(kQB) qem_vmin_small_kernel(const int32_t* __restrict__ E,
                                                             const uint32_t* __restrict__ bits,
                                                             uint32_t* __restrict__ cnt, double rho,
                                                             uint64_t* __restrict__ m) {
    __shared__ uint32_t h[kHistBins];
    if (cnt[kQcDone]) return;
    const int64_t ne = cnt[kQcEdges];
    uint32_t x[kSmallPer];
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k) {
        const int64_t e = (int64_t)k * kQB + threadIdx.x;
        x[k] = e < ne ? bits[e] : kNoKey;
    }
    Select st{0u, 0u};
    uint32_t total = 0;
    for (int level = 0; level < 3; ++level) {
        const int bins = level == 2 ? 1024 : kHistBins, shift = level == 0 ? 21 : (level == 1 ? 10 : 0),
                  up = level == 1 ? 21 : 10;
        for (int i = threadIdx.x; i < bins; i += kQB) h[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSmallPer; ++k)
            if (x[k] != kNoKey && (level == 0 || (x[k] >> up) == st.prefix)) atomicAdd(&h[(x[k] >> shift) & (bins - 1)], 1u);
        __syncthreads();
        st = select_digit(h, bins, st, level == 0 ? rho : -1.0, level == 0 ? &total : nullptr);
    }
    if (threadIdx.x == 0) {
        cnt[kQcValid] = total;
        cnt[kQcTau] = st.prefix;
    }
    if (total == 0) return;
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k)
        if (x[k] <= st.prefix) vertex_min(E, (int64_t)k * kQB + threadIdx.x, x[k], m);  // (kNoKey is above every cost)
}

struct WinArgs {
    const int32_t *E, *F, *ring, *longs;
    const uint32_t *bits, *info, *off, *num, *adj;
    const uint8_t* faces;
    const uint64_t* m;
    uint32_t* cnt;
    uint32_t* list;  // winners, in no order
};

// Winners: an eligible edge whose key is the least at both ends and at every
// neighbour of them.  m(v0) = m(v1) = key leaves few edges (a few in a hundred):
// a workgroup gathers those of its 2,048 edges in LDS, so that whole waves walk
// their rings and not single lanes of every wave, collects the winners in LDS
// too and takes their places in the list with one atomic.
constexpr int kWinBlock = 512, kWinEdges = 4, kWinTile = kWinBlock * kWinEdges;
__global__ void __launch_bounds__(kWinBlock) qem_win_kernel(WinArgs a) {
    __shared__ uint32_t s_list[kWinBlock + kWinTile];
    __shared__ uint32_t s_cand[kWinTile];
    __shared__ uint32_t s_n, s_f, s_c, s_base;
    if (a.cnt[kQcDone]) return;
    const uint32_t tau = a.cnt[kQcTau], valid = a.cnt[kQcValid];
    const int64_t ne = valid ? a.cnt[kQcEdges] : 0;
    if (threadIdx.x == 0) s_n = s_f = s_c = 0;
    __syncthreads();
    auto flush = [&]() {  // block-uniform
        const uint32_t n = s_n;
        if (n == 0) return;
        if (threadIdx.x == 0)
            s_base = (uint32_t)atomicAdd((unsigned long long*)&a.cnt[kQcWinners],
                                         (unsigned long long)n | ((unsigned long long)s_f << 32));
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < n; i += kWinBlock) a.list[s_base + i] = s_list[i];
        __syncthreads();
        if (threadIdx.x == 0) s_n = s_f = 0;
        __syncthreads();
    };
    // no m below key in the ring of v?
    auto clear_around = [&](int32_t v, uint32_t m, uint64_t key) {
        if (m <= (uint32_t)kRingKeep) {
            const int4* r = reinterpret_cast<const int4*>(a.ring + (int64_t)kRingKeep * v);
            int4 w[kRingKeep / 4];
#pragma unroll
            for (int q = 0; q < kRingKeep / 4; ++q) w[q] = r[q];
            uint64_t least = ~0ull;
            uint64_t x[kRingKeep];
#pragma unroll
            for (int q = 0; q < kRingKeep / 4; ++q) {
                const int32_t y[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
#pragma unroll
                for (int k = 0; k < 4; ++k)  // past the ring's end: v itself, whose m is key
                    x[4 * q + k] = a.m[(uint32_t)(4 * q + k) < m ? y[k] >> 3 : v];
            }
#pragma unroll
            for (int k = 0; k < kRingKeep; ++k) least = x[k] < least ? x[k] : least;
            return least >= key;
        }
        if (const int32_t* r = long_ring(a.ring, a.longs, v)) {
            for (uint32_t i = 0; i < m; i += kRingKeep) {
                uint64_t x[kRingKeep], least = ~0ull;
#pragma unroll
                for (int k = 0; k < kRingKeep; ++k) x[k] = a.m[r[min(i + k, m - 1)] >> 3];
#pragma unroll
                for (int k = 0; k < kRingKeep; ++k) least = x[k] < least ? x[k] : least;
                if (least < key) return false;
            }
            return true;
        }
        const uint32_t b = a.off[v], n = a.num[v];
        for (uint32_t i = 0; i < n; ++i)
            for (int k = 0; k < 3; ++k)
                if (a.m[a.F[3 * (int64_t)a.adj[b + i] + k]] < key) return false;
        return true;
    };
    for (int64_t e0 = (int64_t)blockIdx.x * kWinTile; e0 < ne; e0 += (int64_t)gridDim.x * kWinTile) {
        uint64_t key[kWinEdges], ma[kWinEdges], mb[kWinEdges];
        int2 v[kWinEdges];
        uint32_t x[kWinEdges];
#pragma unroll
        for (int u = 0; u < kWinEdges; ++u) {
            const int64_t e = e0 + u * kWinBlock + threadIdx.x;
            const int64_t ec = e < ne ? e : ne - 1;
            x[u] = a.bits[ec];
            v[u] = reinterpret_cast<const int2*>(a.E)[ec];
            key[u] = ((uint64_t)x[u] << 32) | (uint64_t)(uint32_t)e;
            if (e >= ne) x[u] = kNoKey;
        }
#pragma unroll
        for (int u = 0; u < kWinEdges; ++u) {
            ma[u] = mb[u] = 0;
            if (x[u] <= tau) {
                ma[u] = a.m[v[u].x];
                mb[u] = a.m[v[u].y];
            }
        }
#pragma unroll
        for (int u = 0; u < kWinEdges; ++u)
            if (x[u] <= tau && ma[u] == key[u] && mb[u] == key[u]) s_cand[atomicAdd(&s_c, 1u)] = (uint32_t)key[u];
        __syncthreads();
        const uint32_t nc = s_c;
        for (uint32_t i = threadIdx.x; i < nc; i += kWinBlock) {
            const uint32_t e = s_cand[i];
            const int2 w = reinterpret_cast<const int2*>(a.E)[e];
            const uint64_t k = ((uint64_t)a.bits[e] << 32) | (uint64_t)e;
            const uint32_t f = a.faces[e], la = ring_len(a.info[w.x]), lb = ring_len(a.info[w.y]);
            const bool ca = clear_around(w.x, la, k), cb = clear_around(w.y, lb, k);
            if (ca && cb) {
                s_list[atomicAdd(&s_n, 1u)] = e;
                atomicAdd(&s_f, f);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) s_c = 0;
        if (s_n > (uint32_t)kWinBlock) flush();
        else __syncthreads();
    }
    flush();
}

// The smallest winner key that no longer fits when the winners together
// remove more than `budget` faces (keys ascending, face counts summed): a
// radix descent over the winners' 64-bit keys, 8 bits per level, by a whole
// block; also the collapses kept and the faces they remove.
struct Cut {
    unsigned long long key;
    uint32_t applied, removed;
};
__device__ Cut find_cut(const uint32_t* __restrict__ list, uint32_t n, const uint32_t* __restrict__ bits,
                        const uint8_t* __restrict__ faces, uint32_t budget) {
    __shared__ uint32_t h[256], hc[256];
    __shared__ unsigned long long s_prefix;
    __shared__ uint32_t s_budget, s_kf, s_kn;
    if (threadIdx.x == 0) {
        s_prefix = 0;
        s_budget = budget;
        s_kf = 0;
        s_kn = 0;
    }
    for (int level = 0; level < 8; ++level) {
        const int shift = 56 - 8 * level;
        if (threadIdx.x < 256) {
            h[threadIdx.x] = 0;
            hc[threadIdx.x] = 0;
        }
        __syncthreads();
        const unsigned long long pre = s_prefix;
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
            const uint32_t e = list[i];
            const uint64_t k = ((uint64_t)bits[e] << 32) | (uint64_t)e;
            if (level > 0 && (k >> (shift + 8)) != pre) continue;
            atomicAdd(&h[(k >> shift) & 255u], (uint32_t)faces[e]);
            atomicAdd(&hc[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t acc = 0, accn = 0, d = 0;
            for (; d < 256; ++d) {
                if (acc + h[d] > s_budget) break;
                acc += h[d];
                accn += hc[d];
            }
            // the winners under the prefix weigh more than the budget, so a digit overflows
            s_prefix = (pre << 8) | (d < 256 ? d : 255u);
            s_budget -= acc;
            s_kf += acc;
            s_kn += accn;
        }
        __syncthreads();
    }
    return Cut{s_prefix, s_kn, s_kf};
}

struct ApplyArgs {
    const uint32_t *list, *bits;
    const int32_t* E;
    const uint8_t* faces;
    const double* pl;
    uint32_t* cnt;
    double *P, *Q;
    int32_t* F;
    uint32_t *off, *num, *adj;
    uint32_t arena;   // entries of adj
    int64_t target;
    uint32_t* rec;    // host memory: the counts of the round
};

// The collapses.  Winners touch disjoint faces and vertices, so each thread
// changes its own: position and quadric of v0, the faces of v1 (dead when they
// hold v0, else v1 becomes v0), and v0's list.  Block 0 closes the round.
__global__ void __launch_bounds__(kQB) qem_apply_kernel(ApplyArgs a) {
    if (a.cnt[kQcDone]) return;
    const uint32_t nw = a.cnt[kQcWinners], nf = a.cnt[kQcWinners + 1];
    const int64_t live = a.cnt[kQcLive];
    Cut cut{~0ull, nw, nf};
    if ((int64_t)nf > live - a.target)
        cut = find_cut(a.list, nw, a.bits, a.faces, (uint32_t)(live > a.target ? live - a.target : 0));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.rec[kQcLong] = a.cnt[kQcLong];
        a.cnt[kQcRing] = a.cnt[kQcGather] = a.cnt[kQcLong] = 0u;  // for the next round's rings
        a.cnt[kQcApplied] = cut.applied;
        a.cnt[kQcLiveNext] = (uint32_t)(live - cut.removed);
        const uint32_t done = cut.applied == 0 || live - cut.removed <= a.target ? 1u : 0u;
        if (done) a.cnt[kQcDoneNext] = 1u;
        a.rec[kQcEdges] = a.cnt[kQcEdges];
        a.rec[kQcValid] = a.cnt[kQcValid];
        a.rec[kQcApplied] = cut.applied;
        a.rec[kQcLiveNext] = (uint32_t)(live - cut.removed);
        a.rec[kQcDoneNext] = done;
        a.rec[kQcArena] = a.cnt[kQcArena];  // this round's own entries may be in it or not
    }
    const int lane = threadIdx.x & 63;
    for (uint32_t i0 = blockIdx.x * kQB; i0 < nw; i0 += gridDim.x * kQB) {
        const uint32_t i = i0 + threadIdx.x;
        bool on = i < nw;
        uint32_t e = 0, b0 = 0, n0 = 0, b1 = 0, n1 = 0, c = 0;
        int32_t v0 = 0, v1 = 0;
        if (on) {
            e = a.list[i];
            on = (((uint64_t)a.bits[e] << 32) | (uint64_t)e) < cut.key;
        }
        if (on) {
            v0 = a.E[2 * (int64_t)e];
            v1 = a.E[2 * (int64_t)e + 1];
            c = a.faces[e];
            b0 = a.off[v0];
            n0 = a.num[v0];
            b1 = a.off[v1];
            n1 = a.num[v1];
        }
        const uint32_t nn = on ? n0 + n1 - 2 * c : 0u;  // v0's new list
        const uint32_t need = nn > n0 ? nn : 0u;
        uint32_t x = need;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        uint32_t base = 0;
        if (lane == 63 && x) base = atomicAdd(&a.cnt[kQcArena], x);
        base = __shfl(base, 63, 64) + x - need;
        const uint32_t to = need ? base : b0;
        if (need && (base + need > a.arena || base + need < base)) {  // the host keeps room for every round
            atomicOr(&a.cnt[kQcStatus], 2u);
            on = false;
        }
        const bool many = on && n0 + n1 > 64;
        if (on) {
            for (int k = 0; k < 3; ++k) a.P[3 * (int64_t)v0 + k] = a.pl[3 * (int64_t)e + k];
            for (int k = 0; k < 10; ++k) a.Q[10 * (int64_t)v0 + k] = a.Q[10 * (int64_t)v0 + k] + a.Q[10 * (int64_t)v1 + k];
        }
        if (on && !many) {
            // both lists eight faces at a time, their loads issued together (the
            // faces of a batch are distinct, and only this thread changes them)
            uint32_t w = 0;
            auto walk = [&](uint32_t b, uint32_t n, bool second) {
                for (uint32_t q0 = 0; q0 < n; q0 += 8) {
                    uint32_t f[8];
                    int32_t x[8][3];
#pragma unroll
                    for (int q = 0; q < 8; ++q) f[q] = a.adj[b + min(q0 + q, n - 1)];
#pragma unroll
                    for (int q = 0; q < 8; ++q)
#pragma unroll
                        for (int k = 0; k < 3; ++k) x[q][k] = a.F[3 * (int64_t)f[q] + k];
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        if (q0 + q >= n || x[q][0] < 0) continue;  // past the end, or dead with v0's list
                        if (holds(x[q], v1) && holds(x[q], v0)) {
                            a.F[3 * (int64_t)f[q]] = -1;
                            continue;
                        }
                        if (second) {
#pragma unroll
                            for (int k = 0; k < 3; ++k)
                                if (x[q][k] == v1) a.F[3 * (int64_t)f[q] + k] = v0;
                        }
                        if (w < nn) a.adj[to + w++] = f[q];
                    }
                }
            };
            walk(b0, n0, false);
            walk(b1, n1, true);
            a.off[v0] = to;
            a.num[v0] = w;
            a.num[v1] = 0u;
        }
        // long lists by the whole wave, 64 faces at a time (a place written is
        // never past the faces read; a face of both lists is met in each)
        for (uint64_t todo = __ballot(many); todo != 0; todo &= todo - 1) {
            const int src = __builtin_ctzll(todo);
            const int32_t u0 = __shfl(v0, src, 64), u1 = __shfl(v1, src, 64);
            const uint32_t at = __shfl(to, src, 64), room = __shfl(nn, src, 64);
            uint32_t w = 0;
            for (int list = 0; list < 2; ++list) {
                const uint32_t b = __shfl(list ? b1 : b0, src, 64), n = __shfl(list ? n1 : n0, src, 64);
                for (uint32_t q0 = 0; q0 < n; q0 += 64) {
                    const uint32_t f = a.adj[b + min(q0 + lane, n - 1)];
                    const int32_t x[3] = {a.F[3 * (int64_t)f], a.F[3 * (int64_t)f + 1], a.F[3 * (int64_t)f + 2]};
                    const bool in = q0 + lane < n && x[0] >= 0, both = in && holds(x, u0) && holds(x, u1);
                    const uint64_t kept = __ballot(in && !both);
                    const uint32_t o = w + (uint32_t)__popcll(kept & __lanemask_lt());
                    if (both) a.F[3 * (int64_t)f] = -1;
                    if (in && !both) {
                        for (int k = 0; k < 3; ++k)
                            if (list && x[k] == u1) a.F[3 * (int64_t)f + k] = u0;
                        if (o < room) a.adj[at + o] = f;
                    }
                    w += (uint32_t)__popcll(kept);
                }
                wave_sync();
            }
            if (lane == src) {
                a.off[v0] = to;
                a.num[v0] = min(w, nn);
                a.num[v1] = 0u;
            }
        }
    }
}

// ---- compaction of the faces ------------------------------------------------

__global__ void qem_alive_kernel(const int32_t* __restrict__ F, int64_t slots, uint32_t* __restrict__ keep) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f < slots) keep[f] = F[3 * f] >= 0 ? 1u : 0u;
}

__global__ void qem_face_scatter_kernel(const int32_t* __restrict__ F2, int64_t live, const uint32_t* __restrict__ keep,
                                        const uint32_t* __restrict__ koff, int32_t* __restrict__ F) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live || !keep[f]) return;
    const int64_t o = koff[f];
    F[3 * o] = F2[3 * f];
    F[3 * o + 1] = F2[3 * f + 1];
    F[3 * o + 2] = F2[3 * f + 2];
}

// ---- renumbering -----------------------------------------------------------
// New index = rank among the vertices a live face references.

__global__ void qem_vmove_kernel(const double* __restrict__ P, const double* __restrict__ Q, int64_t nv,
                                 const uint32_t* __restrict__ ref, const uint32_t* __restrict__ vid,
                                 double* __restrict__ P2, double* __restrict__ Q2) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv || !ref[v]) return;
    const int64_t o = vid[v];
    for (int k = 0; k < 3; ++k) P2[3 * o + k] = P[3 * v + k];
    for (int k = 0; k < 10; ++k) Q2[10 * o + k] = Q[10 * v + k];
}

__global__ void qem_frenum_kernel(int32_t* __restrict__ F, int64_t live, const uint32_t* __restrict__ vid) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live) return;
    for (int k = 0; k < 3; ++k) F[3 * f + k] = (int32_t)vid[F[3 * f + k]];
}

// ---- output ---------------------------------------------------------------

__global__ void qem_ref_kernel(const int32_t* __restrict__ F, int64_t live, uint32_t* __restrict__ ref) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live) return;
    for (int k = 0; k < 3; ++k) ref[F[3 * f + k]] = 1u;
}

__global__ void qem_vout_kernel(const double* __restrict__ P, int64_t nv, const uint32_t* __restrict__ ref,
                                const uint32_t* __restrict__ vid, float* __restrict__ V_out) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv || !ref[v]) return;
    const int64_t o = vid[v];
    V_out[3 * o] = (float)P[3 * v];
    V_out[3 * o + 1] = (float)P[3 * v + 1];
    V_out[3 * o + 2] = (float)P[3 * v + 2];
}

__global__ void qem_fout_kernel(const int32_t* __restrict__ F, int64_t live, const uint32_t* __restrict__ vid,
                                int32_t* __restrict__ F_out) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= live) return;
    for (int k = 0; k < 3; ++k) F_out[3 * f + k] = (int32_t)vid[F[3 * f + k]];
}

__global__ void qem_edge_out_kernel(const int32_t* __restrict__ E, const uint8_t* __restrict__ faces,
                                    const uint32_t* __restrict__ bits, const double* __restrict__ pl,
                                    const uint32_t* __restrict__ n_edges, int64_t cap, int32_t* __restrict__ E_out,
                                    uint8_t* __restrict__ valid_out, int32_t* __restrict__ faces_out,
                                    double* __restrict__ p_out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)*n_edges || e >= cap) return;
    E_out[2 * e] = E[2 * e];
    E_out[2 * e + 1] = E[2 * e + 1];
    faces_out[e] = faces[e];
    valid_out[e] = bits[e] != kNoKey ? 1 : 0;
    for (int k = 0; k < 3; ++k) p_out[3 * e + k] = pl[3 * e + k];
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Vertex slots up to which the survivors are not renumbered: the passes over
// that many vertices take one wave of workgroups anyway, while a renumbering
// costs about twenty launches and two waits (20,172 faces: 4.9 ms with it, 4.4
// without, before the later launches were shortened).
constexpr int64_t kRenumber = 1 << 15;


size_t qem_layout(int64_t nv, int64_t nf, QemLayout* L) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const int64_t cap = 3 * nf + 1;  // edges: every edge has a face, every face three edges
    const int64_t scan_n = std::max<int64_t>(nv, nf) + 1;
    const int64_t rblocks = (nv + kRB - 1) / kRB + 1;
    L->nv = nv;
    L->nf = nf;
    L->edge_cap = cap;
    // face lists: three entries per face, and room for what two rounds may
    // append (each at most one entry per live face) and for those before them
    L->arena = std::min<int64_t>(7 * nf + 64, (int64_t)0xFFFFFFF0);
    L->cnt = take(4 * kQcSlots);
    L->P = take(24 * (size_t)nv);
    L->Q = take(80 * (size_t)nv);
    L->P2 = take(24 * (size_t)nv);
    L->Q2 = take(80 * (size_t)nv);
    L->F = take(12 * (size_t)nf);
    L->F2 = take(12 * (size_t)nf);
    L->hist = L->keep = take(4 * (size_t)nf);
    L->koff = take(4 * (size_t)(nf + 1));
    L->num = take(4 * (size_t)(nv + 1));
    L->off = take(4 * (size_t)(nv + 1));
    L->cur = take(4 * (size_t)(nv + 1));
    L->adj = take(4 * (size_t)L->arena);
    L->ring = take(4 * (size_t)kRingKeep * (size_t)nv);
    L->info = take(4 * (size_t)(nv + 1));
    L->hcnt = take(4 * (size_t)(nv + 1));
    L->eoff = take(4 * (size_t)(nv + 1));
    L->part = take(4 * (size_t)rblocks);
    L->sup = take(4 * (size_t)(rblocks / kSupBlocks + 1));
    L->E = take(8 * (size_t)cap);
    L->bits = take(4 * (size_t)cap);
    L->faces = take((size_t)cap);
    L->pl = take(24 * (size_t)cap);
    L->m = take(8 * (size_t)nv);
    L->list = take(4 * (size_t)(nf + 1));  // a winner removes at least one face of its own
    L->scan_tmp = take(4 * (size_t)(scan_tmp_elems(scan_n) + 1));
    L->total = off;
    return off;
}

namespace {

struct QemPtrs {
    uint32_t *cnt, *hist, *keep, *koff, *num, *off, *cur, *adj, *info, *hcnt, *eoff, *part, *sup, *bits, *list, *scan_tmp;
    double *P, *Q, *P2, *Q2, *pl;
    int32_t *F, *F2, *ring, *E;
    uint8_t* faces;
    uint64_t* m;
};

QemPtrs ptrs(const QemLayout& L, char* ws) {
    QemPtrs p;
    p.cnt = (uint32_t*)(ws + L.cnt);
    p.hist = (uint32_t*)(ws + L.hist);
    p.keep = (uint32_t*)(ws + L.keep);
    p.koff = (uint32_t*)(ws + L.koff);
    p.num = (uint32_t*)(ws + L.num);
    p.off = (uint32_t*)(ws + L.off);
    p.cur = (uint32_t*)(ws + L.cur);
    p.adj = (uint32_t*)(ws + L.adj);
    p.ring = (int32_t*)(ws + L.ring);
    p.info = (uint32_t*)(ws + L.info);
    p.hcnt = (uint32_t*)(ws + L.hcnt);
    p.eoff = (uint32_t*)(ws + L.eoff);
    p.part = (uint32_t*)(ws + L.part);
    p.sup = (uint32_t*)(ws + L.sup);
    p.bits = (uint32_t*)(ws + L.bits);
    p.list = (uint32_t*)(ws + L.list);
    p.scan_tmp = (uint32_t*)(ws + L.scan_tmp);
    p.P = (double*)(ws + L.P);
    p.Q = (double*)(ws + L.Q);
    p.P2 = (double*)(ws + L.P2);
    p.Q2 = (double*)(ws + L.Q2);
    p.pl = (double*)(ws + L.pl);
    p.F = (int32_t*)(ws + L.F);
    p.F2 = (int32_t*)(ws + L.F2);
    p.E = (int32_t*)(ws + L.E);
    p.faces = (uint8_t*)(ws + L.faces);
    p.m = (uint64_t*)(ws + L.m);
    return p;
}

#define QEM_TRY(expr)                        \
    do {                                     \
        hipError_t e_ = (expr);              \
        if (e_ != hipSuccess) return e_;     \
    } while (0)

// vertex -> face lists of the `live` current faces, at the arena's start
hipError_t build_lists(int64_t nv, const QemPtrs& p, int64_t live, hipStream_t s) {
    QEM_TRY(fill_u32(p.num, 0, nv + 1, s));
    QEM_TRY(fill_u32(p.cur, 0, nv + 1, s));
    hipLaunchKernelGGL(qem_deg_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, p.num);
    QEM_TRY(hipGetLastError());
    QEM_TRY(exclusive_scan_u32(p.num, p.off, nv, p.scan_tmp, p.cnt + kQcArena, s));
    hipLaunchKernelGGL(qem_adj_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, p.off, p.cur, p.adj);
    return hipGetLastError();
}

// Where the rings that have no slots go: the spare positions and quadrics or, if
// that is more, the spare faces, which only a renumbering or the output write,
// with no round in flight.  All rings together have at most six entries per face:
// the former holds them from 0.23 vertices per face on, the latter those of
// vertices whose edges have two faces each.
bool longs_by_vertex(const QemLayout& L) { return 26 * L.nv >= 3 * L.nf; }
int32_t* longs_at(const QemLayout& L, const QemPtrs& p) { return longs_by_vertex(L) ? (int32_t*)p.P2 : p.F2; }
uint32_t longs_room(const QemLayout& L) {
    return (uint32_t)std::min<int64_t>(longs_by_vertex(L) ? 26 * L.nv : 3 * L.nf, INT32_MAX);
}

// Lists of more than kRingFaces faces from which a thread sorts those of up to
// kRingWide by itself.  Otherwise a wave does, one after the other, 2 us each; but
// the wider network costs every launch registers (9.2 -> 12.4 us at 20,172 faces,
// 17 -> 25 us a round of 1,306,800 -> 10,000) and few long lists lie apart.
constexpr uint32_t kManyLong = 16;

// rings and edges of the current mesh; edge count at cnt[kQcEdges].  longs: about
// the lists of more than kRingFaces faces
hipError_t build_edges(const QemLayout& L, int64_t nv, const QemPtrs& p, uint32_t longs, hipStream_t s) {
    const int64_t g = std::max<int64_t>((nv + kRB - 1) / kRB, 1);
    RingArgs a{};
    a.F = p.F;
    a.nv = nv;
    a.off = p.off;
    a.num = p.num;
    a.adj = p.adj;
    a.ring = p.ring;
    a.longs = longs_at(L, p);
    a.longs_n = longs_room(L);
    a.gather = (int32_t*)p.pl;  // placements are written after the rings
    a.info = p.info;
    a.hcnt = p.hcnt;
    a.part = p.part;
    a.sup = p.sup;
    a.m = p.m;
    a.hist = p.hist;
    a.hist_n = L.nf > kSmallFaces ? kHistWords : 0;
    a.cnt = p.cnt;
    if (longs > kManyLong)
        hipLaunchKernelGGL(qem_ring_kernel<true>, dim3(g), dim3(kRB), 0, s, a);
    else
        hipLaunchKernelGGL(qem_ring_kernel<false>, dim3(g), dim3(kRB), 0, s, a);
    QEM_TRY(hipGetLastError());
    hipLaunchKernelGGL(qem_edge_kernel, dim3(g), dim3(kRB), 0, s, a, p.eoff, p.E);
    return hipGetLastError();
}

// `edges`: about the mesh's edge count (the kernel strides over all of them)
hipError_t eval_edges(const QemLayout& L, int64_t nv, const QemPtrs& p, int64_t edges, int midpoint, double* cost,
                      hipStream_t s) {
    EvalArgs a{};
    a.P = p.P;
    a.Q = p.Q;
    a.F = p.F;
    a.off = p.off;
    a.num = p.num;
    a.adj = p.adj;
    a.info = p.info;
    a.hcnt = p.hcnt;
    a.eoff = p.eoff;
    a.ring = p.ring;
    a.longs = longs_at(L, p);
    a.E = p.E;
    a.cnt = p.cnt;
    a.nv = nv;
    a.midpoint = midpoint;
    a.bits = p.bits;
    a.faces = p.faces;
    a.pl = p.pl;
    a.sup = p.sup;
    a.sup_n = (nv + kRB - 1) / kRB / kSupBlocks + 1;
    a.cost = cost;
    hipLaunchKernelGGL(qem_eval_kernel, dim3(blocks_for(std::max(edges, a.sup_n))), dim3(kQB), 0, s, a);
    QEM_TRY(hipGetLastError());
    const int64_t g = std::max<int64_t>((nv + kFoldVerts - 1) / kFoldVerts, 1);
    hipLaunchKernelGGL(qem_fold_kernel, dim3(g), dim3(kQB), 0, s, a);
    return hipGetLastError();
}

hipError_t set_up(const QemLayout& L, const QemPtrs& p, const float* V, const int32_t* F, hipStream_t s) {
    QEM_TRY(fill_u32(p.cnt, 0, kQcSlots, s));
    QEM_TRY(fill_u32(p.cnt + kQcLiveNext, (uint32_t)L.nf, 1, s));
    QEM_TRY(fill_u32(p.sup, 0, (L.nv + kRB - 1) / kRB / kSupBlocks + 1, s));
    const int64_t n = std::max(L.nv, L.nf);
    hipLaunchKernelGGL(qem_init_kernel, dim3(blocks_for(n)), dim3(kQB), 0, s, V, L.nv, F, L.nf, p.P, p.F,
                       p.cnt + kQcStatus);
    QEM_TRY(hipGetLastError());
    QEM_TRY(build_lists(L.nv, p, L.nf, s));
    hipLaunchKernelGGL(qem_quadric_kernel, dim3(blocks_for(L.nv)), dim3(kQB), 0, s, p.P, p.F, L.nv, p.off, p.num,
                       p.adj, p.Q, p.cnt);
    return hipGetLastError();
}

// The live faces of the `slots` face slots, in their order, into F2 (then
// swapped with F); their number at cnt[kQcOut].
hipError_t compact_faces(QemPtrs& p, int64_t slots, hipStream_t s) {
    hipLaunchKernelGGL(qem_alive_kernel, dim3(blocks_for(slots)), dim3(kQB), 0, s, p.F, slots, p.keep);
    QEM_TRY(hipGetLastError());
    QEM_TRY(exclusive_scan_u32(p.keep, p.koff, slots, p.scan_tmp, p.cnt + kQcOut, s));
    hipLaunchKernelGGL(qem_face_scatter_kernel, dim3(blocks_for(slots)), dim3(kQB), 0, s, p.F, slots, p.keep, p.koff,
                       p.F2);
    QEM_TRY(hipGetLastError());
    std::swap(p.F, p.F2);
    return hipSuccess;
}

// One round: ten launches (seven of a small mesh).  `live` bounds the live faces from above.
hipError_t enqueue_round(const QemLayout& L, const QemPtrs& p, int64_t nv, int64_t live, uint32_t longs, int64_t target,
                         double rho, int midpoint, uint32_t* rec, hipEvent_t before_eval, hipEvent_t after_eval, hipStream_t s) {
    QEM_TRY(build_edges(L, nv, p, longs, s));
    const int64_t edges = 3 * live / 2 + 1;  // of a closed mesh; an open one has more, and the kernels stride
    if (before_eval) QEM_TRY(hipEventRecord(before_eval, s));
    QEM_TRY(eval_edges(L, nv, p, edges, midpoint, nullptr, s));
    if (after_eval) QEM_TRY(hipEventRecord(after_eval, s));
    if (L.nf <= kSmallFaces) {
        hipLaunchKernelGGL(qem_vmin_small_kernel, dim3(1), dim3(kQB), 0, s, p.E, p.bits, p.cnt, rho, p.m);
    } else {
        const int64_t hgrid = std::min<int64_t>(blocks_for(edges), 512);
        hipLaunchKernelGGL(qem_hist_kernel<0>, dim3(hgrid), dim3(kQB), 0, s, p.bits, p.hist, p.cnt, rho);
        hipLaunchKernelGGL(qem_hist_kernel<1>, dim3(hgrid), dim3(kQB), 0, s, p.bits, p.hist, p.cnt, rho);
        hipLaunchKernelGGL(qem_hist_kernel<2>, dim3(hgrid), dim3(kQB), 0, s, p.bits, p.hist, p.cnt, rho);
        hipLaunchKernelGGL(qem_vmin_kernel, dim3(std::min<int64_t>(blocks_for(edges), 2048)), dim3(kQB), 0, s, p.E,
                           p.bits, p.hist, p.cnt, p.m);
    }
    QEM_TRY(hipGetLastError());
    WinArgs w{};
    w.E = p.E;
    w.F = p.F;
    w.ring = p.ring;
    w.longs = longs_at(L, p);
    w.bits = p.bits;
    w.info = p.info;
    w.off = p.off;
    w.num = p.num;
    w.adj = p.adj;
    w.faces = p.faces;
    w.m = p.m;
    w.cnt = p.cnt;
    w.list = p.list;
    hipLaunchKernelGGL(qem_win_kernel, dim3(std::min<int64_t>((edges + kWinTile - 1) / kWinTile, 1024)), dim3(kWinBlock),
                       0, s, w);
    QEM_TRY(hipGetLastError());
    ApplyArgs a{};
    a.list = p.list;
    a.bits = p.bits;
    a.E = p.E;
    a.faces = p.faces;
    a.pl = p.pl;
    a.cnt = p.cnt;
    a.P = p.P;
    a.Q = p.Q;
    a.F = p.F;
    a.off = p.off;
    a.num = p.num;
    a.adj = p.adj;
    a.arena = (uint32_t)L.arena;
    a.target = target;
    a.rec = rec;
    hipLaunchKernelGGL(qem_apply_kernel, dim3(std::min<int64_t>(blocks_for(edges / 16), 256)), dim3(kQB), 0, s, a);
    return hipGetLastError();
}

struct Event {  // one per call: an event belongs to its device
    hipEvent_t e = nullptr;
    hipError_t make(unsigned flags) { return hipEventCreateWithFlags(&e, flags); }
    ~Event() {
        if (e) (void)hipEventDestroy(e);
    }
};

}  // namespace

hipError_t qem_edges_run(const QemLayout& L, char* ws, const float* V, const int32_t* F, int midpoint,
                         double* Q_out, int64_t cap, int32_t* E_out, uint8_t* valid_out, int32_t* faces_out,
                         double* cost_out, double* p_out, uint32_t* status, int64_t* n_edges, hipStream_t s) {
    const QemPtrs p = ptrs(L, ws);
    QEM_TRY(set_up(L, p, V, F, s));
    QEM_TRY(build_edges(L, L.nv, p, ~0u, s));
    uint32_t h[kQcSlots];
    QEM_TRY(hipMemcpyAsync(h, p.cnt, sizeof h, hipMemcpyDeviceToHost, s));
    QEM_TRY(hipStreamSynchronize(s));
    *status = h[kQcStatus];
    *n_edges = h[kQcEdges];
    if (h[kQcStatus] || (int64_t)h[kQcEdges] > cap) return hipSuccess;
    QEM_TRY(eval_edges(L, L.nv, p, h[kQcEdges], midpoint, cost_out, s));
    hipLaunchKernelGGL(qem_edge_out_kernel, dim3(blocks_for(h[kQcEdges])), dim3(kQB), 0, s, p.E, p.faces, p.bits, p.pl,
                       p.cnt + kQcEdges, cap, E_out, valid_out, faces_out, p_out);
    QEM_TRY(hipGetLastError());
    if (Q_out) QEM_TRY(hipMemcpyAsync(Q_out, p.Q, 80 * (size_t)L.nv, hipMemcpyDeviceToDevice, s));
    return hipStreamSynchronize(s);
}

hipError_t qem_simplify_run(const QemLayout& L, char* ws, const float* V, const int32_t* F, int64_t target, double rho,
                            int32_t max_rounds, int midpoint, float* V_out, int32_t* F_out, int64_t* counts,
                            int32_t* rounds_out, int64_t* stats, float* times_ms, uint32_t* status, hipStream_t s) {
    QemPtrs p = ptrs(L, ws);
    // optional timing: the whole call, and the per-edge evaluation launches
    // summed (each round is then waited for before the next)
    Event tev[4], ready[2];
    if (times_ms) {
        for (int k = 0; k < 4; ++k) QEM_TRY(tev[k].make(hipEventDefault));
        times_ms[0] = times_ms[1] = 0.f;
        QEM_TRY(hipEventRecord(tev[2].e, s));
    }
    for (int k = 0; k < 2; ++k) QEM_TRY(ready[k].make(hipEventDisableTiming));
    QEM_TRY(set_up(L, p, V, F, s));
    // the counts come back into pinned host memory (one buffer per calling
    // thread, kept for the process): the last launch of a round writes them
    // there itself, two rounds' in turn (a copy per round took 4 us of its
    // stream time)
    static thread_local uint32_t* h = nullptr;
    if (!h)
        QEM_TRY(hipHostMalloc((void**)&h, 4 * 3 * kQcSlots,
                              hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent));
    constexpr size_t kCountBytes = 4 * kQcSlots;
    QEM_TRY(hipMemcpyAsync(h, p.cnt, kCountBytes, hipMemcpyDeviceToHost, s));
    QEM_TRY(hipStreamSynchronize(s));
    *status = h[kQcStatus];
    if (h[kQcStatus]) return hipSuccess;
    int64_t nv = L.nv;       // vertex slots in use (shrinks when the survivors are renumbered)
    int64_t slots = L.nf;    // face slots in use
    int64_t live = L.nf;     // live faces after the last round that was read back
    int64_t arena = h[kQcArena];  // list entries in use then
    uint32_t longs = h[kQcLongIn];  // lists of more than kRingFaces faces then
    int32_t done = 0, queued = 0;  // rounds read back and rounds enqueued
    bool more = live > target && max_rounds > 0;
    // reads round `done` back
    auto take = [&]() -> hipError_t {
        QEM_TRY(hipEventSynchronize(ready[done & 1].e));
        const volatile uint32_t* c = h + kQcSlots * (1 + (done & 1));
        live = c[kQcLiveNext];
        arena = c[kQcArena];
        longs = c[kQcLong];
        if (stats) {
            stats[4 * done] = c[kQcEdges];
            stats[4 * done + 1] = c[kQcValid];
            stats[4 * done + 2] = c[kQcApplied];
            stats[4 * done + 3] = live;
        }
        ++done;
        if (c[kQcDoneNext]) more = false;
        return hipSuccess;
    };
    while (more) {
        if (queued < max_rounds) {
            // every round may append an entry per live face: the one this
            // would enqueue, those in flight, and the last one read back
            const bool tight = arena + (int64_t)(queued - done + 2) * live > L.arena;
            if (tight || (done == queued && live < nv && nv > kRenumber)) {
                while (done < queued && more) QEM_TRY(take());
                if (!more) break;
                // about twice as many slots as live vertices (a closed mesh has
                // about two faces per vertex): renumber the survivors
                uint32_t* ref = p.info;  // per-round scratch until the next rings
                uint32_t* vid = p.eoff;
                QEM_TRY(compact_faces(p, slots, s));
                QEM_TRY(fill_u32(ref, 0, nv + 1, s));
                hipLaunchKernelGGL(qem_ref_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, ref);
                QEM_TRY(hipGetLastError());
                QEM_TRY(exclusive_scan_u32(ref, vid, nv, p.scan_tmp, p.cnt + kQcVerts, s));
                hipLaunchKernelGGL(qem_vmove_kernel, dim3(blocks_for(nv)), dim3(kQB), 0, s, p.P, p.Q, nv, ref, vid,
                                   p.P2, p.Q2);
                QEM_TRY(hipGetLastError());
                hipLaunchKernelGGL(qem_frenum_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, vid);
                QEM_TRY(hipGetLastError());
                QEM_TRY(build_lists(nv, p, live, s));
                QEM_TRY(hipMemcpyAsync(h, p.cnt, kCountBytes, hipMemcpyDeviceToHost, s));
                QEM_TRY(hipStreamSynchronize(s));
                nv = h[kQcVerts];
                slots = live;
                arena = h[kQcArena];
                std::swap(p.P, p.P2);
                std::swap(p.Q, p.Q2);
            }
            QEM_TRY(enqueue_round(L, p, nv, live, longs, target, rho, midpoint, h + kQcSlots * (1 + (queued & 1)), tev[0].e,
                                  tev[1].e, s));
            QEM_TRY(hipEventRecord(ready[queued & 1].e, s));
            ++queued;
        }
        // a round stays in flight while the one before it is read, unless the
        // renumbering is near, no more may follow, or the rounds are timed
        const int32_t keep = queued == max_rounds || times_ms || (nv > kRenumber && live - live / 8 < nv) ? 0 : 1;
        while (more && queued - done > keep) {
            QEM_TRY(take());
            if (times_ms) {
                float ms = 0.f;
                QEM_TRY(hipEventElapsedTime(&ms, tev[0].e, tev[1].e));
                times_ms[0] += ms;
            }
            if (done == max_rounds) more = false;
        }
    }
    *rounds_out = done;
    // output: referenced vertices in ascending index, faces in their order
    // (a round enqueued after the last one changed nothing)
    uint32_t* ref = p.info;
    uint32_t* vid = p.eoff;
    QEM_TRY(compact_faces(p, slots, s));
    QEM_TRY(fill_u32(ref, 0, nv + 1, s));
    hipLaunchKernelGGL(qem_ref_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, ref);
    QEM_TRY(hipGetLastError());
    QEM_TRY(exclusive_scan_u32(ref, vid, nv, p.scan_tmp, p.cnt + kQcVerts, s));
    hipLaunchKernelGGL(qem_vout_kernel, dim3(blocks_for(nv)), dim3(kQB), 0, s, p.P, nv, ref, vid, V_out);
    QEM_TRY(hipGetLastError());
    hipLaunchKernelGGL(qem_fout_kernel, dim3(blocks_for(live)), dim3(kQB), 0, s, p.F, live, vid, F_out);
    QEM_TRY(hipGetLastError());
    QEM_TRY(hipMemcpyAsync(h, p.cnt, kCountBytes, hipMemcpyDeviceToHost, s));
    if (times_ms) QEM_TRY(hipEventRecord(tev[3].e, s));
    QEM_TRY(hipStreamSynchronize(s));
    if (times_ms) QEM_TRY(hipEventElapsedTime(&times_ms[1], tev[2].e, tev[3].e));
    if (h[kQcStatus]) return hipErrorUnknown;  // a list outgrew the arena: the room kept above rules it out
    counts[0] = h[kQcVerts];
    counts[1] = live;
    return hipSuccess;
}

}  // namespace bake
