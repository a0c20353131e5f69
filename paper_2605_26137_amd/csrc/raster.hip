// Low-poly preparation, UV-space rasteriser, uncovered-texel fill, chart
// dilation and RGB8 encoding.
//
// The rasteriser produces the G-buffer of the paper's bake (Sec. 6.4): for
// every texel centre covered by a low-poly face in UV space, the face and the
// barycentric weights, from which the world position and the interpolated
// smooth normal follow.  Coverage is decided exactly in integers: corners are
// snapped to 1/256 texel (exact in FP32 since res is a power of two) and the
// three edge functions are evaluated in int64 at the texel centre.
#include "internal.h"

namespace bake {

namespace {

constexpr uint32_t kFaceReliable = 1u;  // UV det != 0, 3D area != 0, indices and data valid
constexpr uint32_t kFaceRaster = 2u;    // may cover texels (indices valid, UV in range, det != 0)

__device__ __forceinline__ float3 ld3(const float* p, int64_t i) {
    return make_float3(p[3 * i], p[3 * i + 1], p[3 * i + 2]);
}
__device__ __forceinline__ float3 sub3(float3 a, float3 b) {
    return make_float3(a.x - b.x, a.y - b.y, a.z - b.z);
}
__device__ __forceinline__ float3 cross3(float3 a, float3 b) {
    return make_float3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float dot3(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ bool finite3(float3 a) {
    return isfinite(a.x) && isfinite(a.y) && isfinite(a.z);
}

// ---------------------------------------------------------------------------
// Low-poly preparation
// ---------------------------------------------------------------------------

// Per face: snapped UV corners, tangent T_f = sgn(det) (e1 dv2 - e2 dv1) and
// handedness h_f = sign(((e1 x e2) x T_f) . B_f) with B_f = sgn(det)(e2 du1 -
// e1 du2); reliability flags; vertex degrees for the vertex -> face CSR.
__global__ __launch_bounds__(256) void lo_face_kernel(Batch Bt, float4* __restrict__ face_t,
                                                      int4* __restrict__ face_uv,
                                                      uint32_t* __restrict__ deg) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGLoF, blockIdx.x, &lb)];
    const int64_t f = lb * 256 + threadIdx.x;
    if (f >= As.nlf) return;
    const float* __restrict__ V = As.lo_V;
    const int32_t* __restrict__ F = As.lo_F;
    const float* __restrict__ UV = As.lo_UV;
    const int64_t nv = As.nlv;
    int32_t a = F[3 * f], b = F[3 * f + 1], c = F[3 * f + 2];
    bool idx_ok = a >= 0 && b >= 0 && c >= 0 && a < nv && b < nv && c < nv;
    uint32_t st = 0;
    if (!idx_ok) st |= kStLoIndex;
    float u[6];
    bool uv_ok = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        u[k] = UV[6 * f + k];
        uv_ok = uv_ok && isfinite(u[k]) && u[k] >= -1.0f && u[k] <= 2.0f;
    }
    if (!uv_ok) st |= kStBadUV;
    const float sc = (float)As.res * 256.0f;
    int32_t X[3], Y[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        X[k] = uv_ok ? (int32_t)rintf(u[2 * k] * sc) : 0;
        Y[k] = uv_ok ? (int32_t)rintf(u[2 * k + 1] * sc) : 0;
    }
    int64_t du1 = X[1] - X[0], dv1 = Y[1] - Y[0], du2 = X[2] - X[0], dv2 = Y[2] - Y[0];
    int64_t det = du1 * dv2 - du2 * dv1;
    float sg = det > 0 ? 1.0f : (det < 0 ? -1.0f : 0.0f);
    float4 T4 = make_float4(0.f, 0.f, 0.f, 1.f);
    bool rel = false;
    if (idx_ok) {
        float3 A = ld3(V, a), B = ld3(V, b), C = ld3(V, c);
        bool fin = finite3(A) && finite3(B) && finite3(C);
        if (!fin) st |= kStNonFinite;
        float3 e1 = sub3(B, A), e2 = sub3(C, A);
        float fdu1 = (float)du1, fdv1 = (float)dv1, fdu2 = (float)du2, fdv2 = (float)dv2;
        float3 T = make_float3(sg * (e1.x * fdv2 - e2.x * fdv1), sg * (e1.y * fdv2 - e2.y * fdv1),
                               sg * (e1.z * fdv2 - e2.z * fdv1));
        float3 Bt3 = make_float3(sg * (e2.x * fdu1 - e1.x * fdu2), sg * (e2.y * fdu1 - e1.y * fdu2),
                                 sg * (e2.z * fdu1 - e1.z * fdu2));
        float3 n = cross3(e1, e2);
        float hs = dot3(cross3(n, T), Bt3);
        T4 = make_float4(T.x, T.y, T.z, hs < 0.f ? -1.f : 1.f);
        bool area = n.x != 0.f || n.y != 0.f || n.z != 0.f;
        rel = fin && uv_ok && det != 0 && area;
        atomicAdd(&deg[As.lv + a], 1u);
        atomicAdd(&deg[As.lv + b], 1u);
        atomicAdd(&deg[As.lv + c], 1u);
    }
    uint32_t flags = (rel ? kFaceReliable : 0u) | ((idx_ok && uv_ok && det != 0) ? kFaceRaster : 0u);
    const int64_t fg = As.lf + f;
    face_t[fg] = T4;
    face_uv[2 * fg] = make_int4(X[0], Y[0], X[1], Y[1]);
    face_uv[2 * fg + 1] = make_int4(X[2], Y[2], (int32_t)flags, 0);
    if (st) set_status(Bt, st);
}

// Adjacency entries hold asset-local face indices at the positions given by
// the (batch-wide) exclusive scan of the degrees.
__global__ __launch_bounds__(256) void lo_adj_kernel(Batch Bt, const uint32_t* __restrict__ off,
                                                     uint32_t* __restrict__ cur, int32_t* __restrict__ adj) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGLoF, blockIdx.x, &lb)];
    const int64_t f = lb * 256 + threadIdx.x;
    if (f >= As.nlf) return;
    const int32_t* __restrict__ F = As.lo_F;
    const int64_t nv = As.nlv;
    int32_t v[3] = {F[3 * f], F[3 * f + 1], F[3 * f + 2]};
    if (v[0] < 0 || v[1] < 0 || v[2] < 0 || v[0] >= nv || v[1] >= nv || v[2] >= nv) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int64_t g = As.lv + v[k];
        uint32_t slot = atomicAdd(&cur[g], 1u);
        adj[off[g] + slot] = (int32_t)f;
    }
}

// Per vertex: sort its incident faces ascending (fixed summation order, so the
// result does not depend on the order the adjacency was filled in), then
// n_v = normalise(sum (V1 - V0) x (V2 - V0)).  The blocks past the vertices' clear
// the face map, which the next launch claims texels in: a launch of its own took
// 1.6 us at 128^2 and the gap before it; from the first low-poly launch the 67 MB
// of 4096^2 held up the bounds on the other stream.
constexpr int kFillPer = 4 * 256 * 4;  // texels a block and trip
__global__ __launch_bounds__(256) void lo_normal_kernel(Batch Bt, int32_t vertex_blocks,
                                                        const uint32_t* __restrict__ off, int32_t* __restrict__ adj,
                                                        float4* __restrict__ lo_n, uint4* __restrict__ facemap,
                                                        int64_t texels) {
    if ((int32_t)blockIdx.x >= vertex_blocks) {
        const uint4 none = make_uint4(kNoFace, kNoFace, kNoFace, kNoFace);
        const int64_t step = (int64_t)(gridDim.x - vertex_blocks) * 256, quads = texels / 4;
        const int64_t i0 = (int64_t)(blockIdx.x - vertex_blocks) * 256 + threadIdx.x;
        for (int64_t i = i0; i < quads; i += step) facemap[i] = none;
        if (i0 < texels - 4 * quads) reinterpret_cast<uint32_t*>(facemap)[4 * quads + i0] = kNoFace;
        return;
    }
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGLoV, blockIdx.x, &lb)];
    const int64_t v = lb * 256 + threadIdx.x;
    if (v >= As.nlv) return;
    const float* __restrict__ V = As.lo_V;
    const int32_t* __restrict__ F = As.lo_F;
    const int64_t g = As.lv + v;
    uint32_t b = off[g], e = off[g + 1];
    for (uint32_t i = b + 1; i < e; ++i) {
        int32_t x = adj[i];
        uint32_t j = i;
        while (j > b && adj[j - 1] > x) {
            adj[j] = adj[j - 1];
            --j;
        }
        adj[j] = x;
    }
    float3 s = make_float3(0.f, 0.f, 0.f);
    for (uint32_t i = b; i < e; ++i) {
        int32_t f = adj[i];
        float3 A = ld3(V, F[3 * f]), B = ld3(V, F[3 * f + 1]), C = ld3(V, F[3 * f + 2]);
        float3 c = cross3(sub3(B, A), sub3(C, A));
        s.x += c.x;
        s.y += c.y;
        s.z += c.z;
    }
    float l2 = dot3(s, s);
    float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
    if (l2 > 0.f && isfinite(l2)) {
        float r = 1.0f / sqrtf(l2);
        out = make_float4(s.x * r, s.y * r, s.z * r, 1.f);
    }
    lo_n[g] = out;
}

// ---------------------------------------------------------------------------
// Rasteriser: one wave (64 lanes) per face, lanes stride over the face's
// texel bounding box.
// ---------------------------------------------------------------------------

struct FaceBox {
    int32_t X[3], Y[3];
    int32_t i0, j0, w, h;
    bool ok;
};

__device__ __forceinline__ int32_t floor_div256(int32_t x) { return x >> 8; }  // arithmetic shift

__device__ __forceinline__ FaceBox load_face_box(const int4* __restrict__ face_uv, int64_t fg,
                                                 int32_t res) {
    FaceBox fb;
    int4 p = face_uv[2 * fg], q = face_uv[2 * fg + 1];
    fb.X[0] = p.x; fb.Y[0] = p.y; fb.X[1] = p.z; fb.Y[1] = p.w; fb.X[2] = q.x; fb.Y[2] = q.y;
    fb.ok = (q.z & kFaceRaster) != 0;
    int32_t xmin = min(min(fb.X[0], fb.X[1]), fb.X[2]), xmax = max(max(fb.X[0], fb.X[1]), fb.X[2]);
    int32_t ymin = min(min(fb.Y[0], fb.Y[1]), fb.Y[2]), ymax = max(max(fb.Y[0], fb.Y[1]), fb.Y[2]);
    // texel centres 256 j + 128 inside [xmin, xmax]
    int32_t j0 = floor_div256(xmin - 128 + 255), j1 = floor_div256(xmax - 128);
    int32_t i0 = floor_div256(ymin - 128 + 255), i1 = floor_div256(ymax - 128);
    j0 = max(j0, 0); i0 = max(i0, 0);
    j1 = min(j1, res - 1); i1 = min(i1, res - 1);
    fb.j0 = j0; fb.i0 = i0;
    fb.w = j1 - j0 + 1; fb.h = i1 - i0 + 1;
    if (fb.w <= 0 || fb.h <= 0) fb.ok = false;
    return fb;
}

// Edge functions at texel (i, j); true when the face covers it.
__device__ __forceinline__ bool cover(const FaceBox& fb, int32_t i, int32_t j, int64_t E[3], int64_t* S) {
    return cover_at(fb.X, fb.Y, i, j, E, S);
}

constexpr int kRasterBlock = 256;
constexpr int kWavesPerBlock = kRasterBlock / 64;

// The face of a raster wave, or -1 past the asset's faces.
__device__ __forceinline__ int64_t raster_face(const Batch& Bt, const AssetDev** As) {
    int64_t lb;
    *As = &Bt.A[block_asset(Bt, kGLoFWave, blockIdx.x, &lb)];
    const int64_t f = lb * kWavesPerBlock + (threadIdx.x >> 6);
    return f < (*As)->nlf ? f : -1;
}

__global__ __launch_bounds__(kRasterBlock) void raster_claim_kernel(Batch Bt, const int4* __restrict__ face_uv,
                                                                    uint32_t* __restrict__ facemap) {
    const AssetDev* As;
    const int64_t f = raster_face(Bt, &As);
    const int lane = threadIdx.x & 63;
    if (f < 0) return;
    const int32_t res = As->res;
    FaceBox fb = load_face_box(face_uv, As->lf + f, res);
    if (!fb.ok) return;
    uint32_t* fm = facemap + As->tex;
    int64_t total = (int64_t)fb.w * fb.h;
    for (int64_t k = lane; k < total; k += 64) {
        int32_t i = fb.i0 + (int32_t)(k / fb.w), j = fb.j0 + (int32_t)(k % fb.w);
        int64_t E[3], S;
        if (cover(fb, i, j, E, &S)) atomicMin(&fm[(int64_t)i * res + j], (uint32_t)f);
    }
}

__global__ __launch_bounds__(kRasterBlock) void raster_count_kernel(Batch Bt, const int4* __restrict__ face_uv,
                                                                    const uint32_t* __restrict__ facemap,
                                                                    uint32_t* __restrict__ cnt) {
    const AssetDev* As;
    const int64_t f = raster_face(Bt, &As);
    const int lane = threadIdx.x & 63;
    if (f < 0) return;
    const int32_t res = As->res;
    FaceBox fb = load_face_box(face_uv, As->lf + f, res);
    const uint32_t* fm = facemap + As->tex;
    uint32_t c = 0;
    if (fb.ok) {
        int64_t total = (int64_t)fb.w * fb.h;
        for (int64_t k0 = 0; k0 < total; k0 += 64) {
            int64_t k = k0 + lane;
            bool win = false;
            if (k < total) {
                int32_t i = fb.i0 + (int32_t)(k / fb.w), j = fb.j0 + (int32_t)(k % fb.w);
                int64_t E[3], S;
                win = cover(fb, i, j, E, &S) && fm[(int64_t)i * res + j] == (uint32_t)f;
            }
            c += (uint32_t)__popcll(__ballot(win));
        }
    }
    if (lane == 0) cnt[As->lf + f] = c;
}

__global__ __launch_bounds__(kRasterBlock) void raster_emit_kernel(Batch Bt, const int4* __restrict__ face_uv,
                                                                   const uint32_t* __restrict__ facemap,
                                                                   const uint32_t* __restrict__ off,
                                                                   Ray* __restrict__ rays) {
    const AssetDev* As;
    const int64_t f = raster_face(Bt, &As);
    const int lane = threadIdx.x & 63;
    if (f < 0) return;
    const int32_t res = As->res;
    FaceBox fb = load_face_box(face_uv, As->lf + f, res);
    if (!fb.ok) return;
    const uint32_t* fm = facemap + As->tex;
    int64_t total = (int64_t)fb.w * fb.h;
    uint32_t run = off[As->lf + f];
    for (int64_t k0 = 0; k0 < total; k0 += 64) {
        int64_t k = k0 + lane;
        bool win = false;
        int64_t E[3] = {0, 0, 0}, S = 1;
        int32_t i = 0, j = 0;
        if (k < total) {
            i = fb.i0 + (int32_t)(k / fb.w);
            j = fb.j0 + (int32_t)(k % fb.w);
            win = cover(fb, i, j, E, &S) && fm[(int64_t)i * res + j] == (uint32_t)f;
        }
        uint64_t m = __ballot(win);
        if (win) {
            uint32_t r = run + (uint32_t)__popcll(m & __lanemask_lt());
            Ray ray;
            ray.texel = i * res + j;
            ray.face = (int32_t)f;
            bary_of(E, S, &ray.b1, &ray.b2);
            rays[r] = ray;
        }
        run += (uint32_t)__popcll(m);
    }
}

// ---------------------------------------------------------------------------
// Uncovered texels, dilation, RGB8
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void fill_uncovered_kernel(Batch Bt, const uint32_t* __restrict__ facemap,
                                                             uint8_t* __restrict__ level) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGTex, blockIdx.x, &lb)];
    const int64_t t = lb * 256 + threadIdx.x;
    if (t >= (int64_t)As.res * As.res) return;
    bool cov = facemap[As.tex + t] != kNoFace;
    level[As.tex + t] = cov ? 0 : 255;
    if (!cov) {
        As.out_map[3 * t] = 0.f;
        As.out_map[3 * t + 1] = 0.f;
        As.out_map[3 * t + 2] = 1.f;
        As.out_hit[t] = kUncovered;
    }
}

// The uncovered texels alone (no dilation): (0,0,1) and the uncovered status.
__global__ __launch_bounds__(256) void uncovered_kernel(Batch Bt, const uint32_t* __restrict__ facemap) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGTex, blockIdx.x, &lb)];
    const int64_t t = lb * 256 + threadIdx.x;
    if (t >= (int64_t)As.res * As.res || facemap[As.tex + t] != kNoFace) return;
    As.out_map[3 * t] = 0.f;
    As.out_map[3 * t + 1] = 0.f;
    As.out_map[3 * t + 2] = 1.f;
    As.out_hit[t] = kUncovered;
}

// Written out, so that the fused and the per-pass fill round alike.
__device__ __forceinline__ float sumsq(float x, float y, float z) { return fmaf(z, z, fmaf(y, y, x * x)); }

// Pass k: a still-empty texel takes the normalised sum of its 8 neighbours
// that had a value before this pass (level < k).  Texels written in this pass
// are never read in it, so the map is updated in place.
__global__ __launch_bounds__(256) void dilate_kernel(Batch Bt, int pass, uint8_t* __restrict__ level_all) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGTex, blockIdx.x, &lb)];
    const int32_t res = As.res;
    const int64_t t = lb * 256 + threadIdx.x;
    if (t >= (int64_t)res * res) return;
    uint8_t* __restrict__ level = level_all + As.tex;
    float* __restrict__ map = As.out_map;
    if (level[t] != 255) return;
    const int32_t i = (int32_t)(t >> As.log2res), j = (int32_t)(t & (res - 1));
    float sx = 0.f, sy = 0.f, sz = 0.f;
    int cnt = 0;
#pragma unroll
    for (int di = -1; di <= 1; ++di) {
#pragma unroll
        for (int dj = -1; dj <= 1; ++dj) {
            if (di == 0 && dj == 0) continue;
            int32_t ii = i + di, jj = j + dj;
            if (ii < 0 || jj < 0 || ii >= res || jj >= res) continue;
            int64_t u = (int64_t)ii * res + jj;
            if (level[u] < pass) {
                sx += map[3 * u];
                sy += map[3 * u + 1];
                sz += map[3 * u + 2];
                ++cnt;
            }
        }
    }
    if (cnt == 0) return;
    float l2 = sumsq(sx, sy, sz);
    if (!(l2 > 0.f)) return;
    float r = 1.0f / sqrtf(l2);
    map[3 * t] = sx * r;
    map[3 * t + 1] = sy * r;
    map[3 * t + 2] = sz * r;
    level[t] = (uint8_t)pass;
}

__device__ __forceinline__ uint8_t rgb8_of(float v) {
    float c = floorf((v + 1.0f) * 127.5f + 0.5f);
    c = fminf(fmaxf(c, 0.0f), 255.0f);
    return (uint8_t)c;
}

// Uncovered fill, 1 <= k <= kMaxFusedPasses dilation passes and the 8-bit map in
// one launch.  A workgroup takes a tile of kFinishCols x kFinishRows texels plus a
// k-texel halo; a region row is a wave's, a lane per column.  Its rows become
// 64-bit masks: inside the image, and has a value before the pass (covered, or
// filled in an earlier pass).  Covered texels beside an uncovered one go to
// LDS with their traced value (all of them where the 8-bit map is written),
// uncovered ones as (0,0,1).  A pass fills, with the pass rule of dilate_kernel,
// only the empty texels that the masks show to have a valued neighbour: they go to
// a list that the workgroup shares out.  A texel's twenty-four neighbour values
// are read whether valued or not and selected, so that they arrive together
// instead of one after the other behind eight branches (adding the +0 of an
// unvalued one changes no sum that starts at +0).  A value at distance d from the
// region's edge is exact through pass d, so the tile (d >= k) is exact after k
// passes: the result is bitwise that of the fill + per-pass launches (same
// neighbours, same order of sums).
//
// Bound by latency: coverage, values, then k passes of two LDS trips each.  A
// tile of 28 rows gives a small image workgroups enough and a wave four rows.
// 128^2 with 2 passes 16.7 -> 8.8 us, 512^2 with 4 and the bytes 34 -> 16, 2048^2
// 53 -> 46, 4096^2 176 -> 158 (before: 56 rows, a coverage load awaited per row,
// every covered value read, a separate launch for the bytes).  12 rows: 6.7, 14, 55
// and 196 us; 56 rows: 13, 24, 56 and 179.
constexpr int kFinishBlock = 512;
constexpr int kFinishWaves = kFinishBlock / 64;
static_assert(kFinishCols + 2 * kMaxFusedPasses <= 64, "a region row fits one wave");

template <int PASSES>
__global__ __launch_bounds__(kFinishBlock) void finish_kernel(Batch Bt, const uint32_t* __restrict__ facemap_all) {
    static_assert(PASSES >= 1 && PASSES <= kMaxFusedPasses, "fused pass count");
    constexpr int R = kFinishRows + 2 * PASSES;                   // region rows
    constexpr int kRows = (R + kFinishWaves - 1) / kFinishWaves;  // region rows per wave
    __shared__ float s_map[R][3][64];
    __shared__ uint64_t s_in[R], s_val[2][R];
    __shared__ uint16_t s_list[R * 64];
    __shared__ int s_n[2];
    int64_t lt;
    const AssetDev& As = Bt.A[block_asset(Bt, kGTile, blockIdx.x, &lt)];
    const int32_t res = As.res;
    const int32_t tiles_x = (res + kFinishCols - 1) / kFinishCols;
    const int32_t oi = (int32_t)(lt / tiles_x) * kFinishRows - PASSES;  // region origin
    const int32_t oj = (int32_t)(lt % tiles_x) * kFinishCols - PASSES;
    const uint32_t* __restrict__ facemap = facemap_all + As.tex;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t j = oj + lane;
    const bool col_in = lane < kFinishCols + 2 * PASSES && j >= 0 && j < res;
    uint8_t* const rgb8 = As.out_rgb8;
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    int32_t t[kRows];
    uint32_t f[kRows];
    bool cov[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const int r = wave + u * kFinishWaves;
        const int32_t i = oi + r;
        const bool in = r < R && col_in && i >= 0 && i < res;
        t[u] = in ? i * res + j : -1;
        f[u] = facemap[max(t[u], 0)];  // no branch: the rows' loads go out together
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        cov[u] = t[u] >= 0 && f[u] != kNoFace;
        const int r = wave + u * kFinishWaves;
        if (r >= R) break;  // wave-uniform
        const uint64_t bin = __ballot(t[u] >= 0), bcov = __ballot(cov[u]);
        if (lane == 0) {
            s_in[r] = bin;
            s_val[0][r] = bcov;
        }
    }
    __syncthreads();
    float m[kRows][3];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const int r = wave + u * kFinishWaves;
        m[u][0] = 0.f;
        m[u][1] = 0.f;
        m[u][2] = 1.f;
        if (r >= R) break;
        uint64_t near = 0;  // uncovered texels, then their neighbours
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
            const int rr = min(max(r + d, 0), R - 1);
            near |= s_in[rr] & ~s_val[0][rr];
        }
        near |= (near << 1) | (near >> 1);
        if (cov[u] && (rgb8 || ((near >> lane) & 1ull))) {
            m[u][0] = As.out_map[3 * t[u]];
            m[u][1] = As.out_map[3 * t[u] + 1];
            m[u][2] = As.out_map[3 * t[u] + 2];
        }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const int r = wave + u * kFinishWaves;
        if (r >= R) break;
#pragma unroll
        for (int q = 0; q < 3; ++q) s_map[r][q][lane] = m[u][q];
    }
    __syncthreads();
    for (int pass = 1; pass <= PASSES; ++pass) {
        const uint64_t* cur = s_val[(pass - 1) & 1];
        uint64_t* nxt = s_val[pass & 1];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int r = wave + u * kFinishWaves;
            if (r >= R) break;  // wave-uniform
            const uint64_t vu = r > 0 ? cur[r - 1] : 0ull, vc = cur[r], vd = r + 1 < R ? cur[r + 1] : 0ull;
            const uint64_t vm = vu | vc | vd;
            const uint64_t cand = (vm | (vm << 1) | (vm >> 1)) & s_in[r] & ~vc;
            int at = 0;
            if (lane == 0) {
                nxt[r] = vc;
                if (cand) at = atomicAdd(&s_n[pass & 1], __popcll(cand));
            }
            at = __builtin_amdgcn_readfirstlane(at);
            if ((cand >> lane) & 1ull)
                s_list[at + __popcll(cand & ((1ull << lane) - 1ull))] = (uint16_t)(r * 64 + lane);
        }
        __syncthreads();
        const int todo = s_n[pass & 1];
        if (threadIdx.x == 0) s_n[(pass & 1) ^ 1] = 0;  // read before the barrier that opened this pass
        for (int e = threadIdx.x; e < todo; e += kFinishBlock) {
            const int r = s_list[e] >> 6, c = s_list[e] & 63;
            float sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
            for (int di = -1; di <= 1; ++di) {
                const int ii = min(max(r + di, 0), R - 1);
                const uint32_t has = ii == r + di ? (uint32_t)(c > 0 ? cur[ii] >> (c - 1) : cur[ii] << 1) & 7u : 0u;
#pragma unroll
                for (int dj = -1; dj <= 1; ++dj) {
                    if (di == 0 && dj == 0) continue;
                    const int jj = min(max(c + dj, 0), 63);
                    const bool on = (has >> (dj + 1)) & 1u;
                    const float x = s_map[ii][0][jj], y = s_map[ii][1][jj], z = s_map[ii][2][jj];
                    sx += on ? x : 0.f;
                    sy += on ? y : 0.f;
                    sz += on ? z : 0.f;
                }
            }
            // at least one neighbour had a value (the candidate mask)
            const float l2 = sumsq(sx, sy, sz);
            if (l2 > 0.f) {
                // texels filled in this pass are read by no one in it: the
                // pass reads the masks of `cur` and writes those of `nxt`
                const float inv = 1.0f / sqrtf(l2);
                s_map[r][0][c] = sx * inv;
                s_map[r][1][c] = sy * inv;
                s_map[r][2][c] = sz * inv;
                atomicOr((unsigned long long*)&nxt[r], 1ull << c);
            }
        }
        __syncthreads();
    }
    // the tile's uncovered texels, filled or (0,0,1); every texel's bytes
    const bool col_tile = lane >= PASSES && lane < PASSES + kFinishCols;
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const int r = wave + u * kFinishWaves;
        if (r < PASSES || r >= PASSES + kFinishRows || !col_tile || t[u] < 0) continue;
        const float x = s_map[r][0][lane], y = s_map[r][1][lane], z = s_map[r][2][lane];
        if (!cov[u]) {
            As.out_map[3 * t[u]] = x;
            As.out_map[3 * t[u] + 1] = y;
            As.out_map[3 * t[u] + 2] = z;
            As.out_hit[t[u]] = kUncovered;
        }
        if (rgb8) {
            const int64_t at = 3 * (int64_t)t[u];
            rgb8[at] = rgb8_of(x);
            rgb8[at + 1] = rgb8_of(y);
            rgb8[at + 2] = rgb8_of(z);
        }
    }
}

__global__ __launch_bounds__(256) void rgb8_kernel(Batch Bt) {
    int64_t lb;
    const AssetDev& As = Bt.A[block_asset(Bt, kGTex3, blockIdx.x, &lb)];
    const int64_t k = lb * 256 + threadIdx.x;
    if (!As.out_rgb8 || k >= 3 * (int64_t)As.res * As.res) return;
    As.out_rgb8[k] = rgb8_of(As.out_map[k]);
}

inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_lo_prep(const BatchHost& H, hipStream_t s) {
    const Layout& L = H.L;
    char* ws = H.ws;
    uint32_t* deg = (uint32_t*)(ws + L.lo_deg);
    uint32_t* off = (uint32_t*)(ws + L.lo_off);
    uint32_t* cur = (uint32_t*)(ws + L.lo_cur);
    hipError_t e;
    if (H.blocks(kGLoF) > 0) {
        hipLaunchKernelGGL(lo_face_kernel, dim3((unsigned)H.blocks(kGLoF)), dim3(256), 0, s, H.dev,
                           (float4*)(ws + L.face_t), (int4*)(ws + L.face_uv), deg);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // batch-wide scan: vertex g's faces sit at [off[g], off[g + 1])
    if ((e = exclusive_scan_u32(deg, off, L.t_lv, (uint32_t*)(ws + L.scan_tmp), off + L.t_lv, s)) !=
        hipSuccess)
        return e;
    if (H.blocks(kGLoF) > 0) {
        hipLaunchKernelGGL(lo_adj_kernel, dim3((unsigned)H.blocks(kGLoF)), dim3(256), 0, s, H.dev,
                           (const uint32_t*)off, cur, (int32_t*)(ws + L.lo_adj));
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int64_t vertices = H.blocks(kGLoV), fill = std::min<int64_t>((L.t_tex + kFillPer - 1) / kFillPer, 2048);
    if (vertices + fill > 0) {
        hipLaunchKernelGGL(lo_normal_kernel, dim3((unsigned)(vertices + fill)), dim3(256), 0, s, H.dev,
                           (int32_t)vertices, (const uint32_t*)off, (int32_t*)(ws + L.lo_adj), (float4*)(ws + L.lo_n),
                           (uint4*)(ws + L.facemap), L.t_tex);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_raster(const BatchHost& H, hipStream_t s, bool emit) {
    const Layout& L = H.L;
    char* ws = H.ws;
    uint32_t* facemap = (uint32_t*)(ws + L.facemap);
    uint32_t* cnt = (uint32_t*)(ws + L.face_cnt);
    uint32_t* off = (uint32_t*)(ws + L.face_off);
    const int4* fuv = (const int4*)(ws + L.face_uv);
    hipError_t e;
    const unsigned g = (unsigned)H.blocks(kGLoFWave);
    if (g > 0) {
        hipLaunchKernelGGL(raster_claim_kernel, dim3(g), dim3(kRasterBlock), 0, s, H.dev, fuv, facemap);
        hipLaunchKernelGGL(raster_count_kernel, dim3(g), dim3(kRasterBlock), 0, s, H.dev, fuv,
                           (const uint32_t*)facemap, cnt);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // batch-wide scan: the face-ordered ray lists of the assets, concatenated
    if ((e = launch_ray_spaces(H, s)) != hipSuccess) return e;
    if (g > 0 && emit) {
        hipLaunchKernelGGL(raster_emit_kernel, dim3(g), dim3(kRasterBlock), 0, s, H.dev, fuv,
                           (const uint32_t*)facemap, (const uint32_t*)off, (Ray*)(ws + L.rays));
    }
    return hipGetLastError();
}

hipError_t launch_fill_uncovered(const BatchHost& H, hipStream_t s) {
    if (H.blocks(kGTex) == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_uncovered_kernel, dim3((unsigned)H.blocks(kGTex)), dim3(256), 0, s, H.dev,
                       (const uint32_t*)(H.ws + H.L.facemap), (uint8_t*)(H.ws + H.L.level));
    return hipGetLastError();
}

// After the traversal: uncovered fill and dilation, fused for few passes.
hipError_t launch_dilate(const BatchHost& H, int passes, hipStream_t s) {
    const uint32_t* fm = (const uint32_t*)(H.ws + H.L.facemap);
    if (passes == 0) {
        if (H.blocks(kGTex) == 0) return hipSuccess;
        hipLaunchKernelGGL(uncovered_kernel, dim3((unsigned)H.blocks(kGTex)), dim3(256), 0, s, H.dev, fm);
        return hipGetLastError();
    }
    if (passes <= kMaxFusedPasses) {
        if (H.blocks(kGTile) == 0) return hipSuccess;
        const dim3 grid((unsigned)H.blocks(kGTile)), block(kFinishBlock);
        switch (passes) {
            case 1: hipLaunchKernelGGL(finish_kernel<1>, grid, block, 0, s, H.dev, fm); break;
            case 2: hipLaunchKernelGGL(finish_kernel<2>, grid, block, 0, s, H.dev, fm); break;
            case 3: hipLaunchKernelGGL(finish_kernel<3>, grid, block, 0, s, H.dev, fm); break;
            default: hipLaunchKernelGGL(finish_kernel<4>, grid, block, 0, s, H.dev, fm); break;
        }
        static_assert(kMaxFusedPasses == 4, "one finish_kernel instance per fused pass count");
        return hipGetLastError();
    }
    hipError_t e = launch_fill_uncovered(H, s);
    if (e != hipSuccess || H.blocks(kGTex) == 0) return e;
    for (int k = 1; k <= passes; ++k) {
        hipLaunchKernelGGL(dilate_kernel, dim3((unsigned)H.blocks(kGTex)), dim3(256), 0, s, H.dev, k,
                           (uint8_t*)(H.ws + H.L.level));
    }
    return hipGetLastError();
}

hipError_t launch_rgb8(const BatchHost& H, hipStream_t s) {
    if (H.blocks(kGTex3) == 0) return hipSuccess;
    hipLaunchKernelGGL(rgb8_kernel, dim3((unsigned)H.blocks(kGTex3)), dim3(256), 0, s, H.dev);
    return hipGetLastError();
}

}  // namespace bake
