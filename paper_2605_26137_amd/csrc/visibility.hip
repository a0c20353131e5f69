// Hidden-face removal (Sec. 6.2), second half: the flood fill.  Seeds are the
// faces some camera ray hit first; an exterior face f promotes a face g that
// shares an edge with it (two distinct vertex indices in common) when their
// normals agree in direction, n_f . n_g > 0 with n = (V1 - V0) x (V2 - V0).
// The sign is taken in FP64 from the float vertices with no fused
// operations, in a fixed order (x, y, z), so it is the same decision
// wherever it is evaluated.  The condition is symmetric, so the exterior is
// the set of faces joined to a seed by such edges; the traversal order (and
// the order of the per-vertex face lists, filled with atomics) does not
// change it.
//
// Layout: per-vertex face lists (CSR: deg -> off by a scan, adj filled with
// per-vertex cursors), and per face a union-find parent.  Visible faces are
// exterior as they are, and most faces are visible; a hidden face joins the
// hidden faces it agrees with (union-find over the whole device: the later root
// hooks onto the earlier, in a fixed order, with a compare-and-swap, so parents
// only ever move forward in it and every search ends) and notes whether it agrees
// with a visible one.  A hidden face is then exterior when any face of its set
// noted that.
// The sets, and with them the result, do not depend on the order of the
// unions.  Bound by the latency of a handful of dependent gathers: lists and
// fill of 21,425 faces 1.06 -> 0.10 ms and of 106,254 faces 4.39 -> 0.14 ms
// (8 views of 96^2, which leave most faces to the fill), 0.37 -> 0.10 ms after
// 512 views of 1024^2, against the breadth-first expansion in one workgroup
// that it replaced; a hidden fan of 20,000 faces in a shell of 20,480 0.69 -> 0.51
// (11.0 with the tip's list walked for each face, 1.3 with roots hooked by index).
#include "internal.h"

namespace bake {

namespace {

__device__ __forceinline__ bool face_verts(const AssetDev& As, int64_t f, int32_t v[3]) {
    v[0] = As.hi_F[3 * f];
    v[1] = As.hi_F[3 * f + 1];
    v[2] = As.hi_F[3 * f + 2];
    return v[0] >= 0 && v[1] >= 0 && v[2] >= 0 && v[0] < As.nhv && v[1] < As.nhv && v[2] < As.nhv;
}

struct d3 {
    double x, y, z;
};

__device__ __forceinline__ d3 face_normal(const AssetDev& As, const int32_t v[3]) {
#pragma clang fp contract(off)
    const float* V = As.hi_V;
    const double ax = V[3 * (int64_t)v[0]], ay = V[3 * (int64_t)v[0] + 1], az = V[3 * (int64_t)v[0] + 2];
    const double bx = (double)V[3 * (int64_t)v[1]] - ax, by = (double)V[3 * (int64_t)v[1] + 1] - ay,
                 bz = (double)V[3 * (int64_t)v[1] + 2] - az;
    const double cx = (double)V[3 * (int64_t)v[2]] - ax, cy = (double)V[3 * (int64_t)v[2] + 1] - ay,
                 cz = (double)V[3 * (int64_t)v[2] + 2] - az;
    d3 n;
    n.x = by * cz - bz * cy;
    n.y = bz * cx - bx * cz;
    n.z = bx * cy - by * cx;
    return n;
}

__device__ __forceinline__ bool agree(const d3& a, const d3& b) {
#pragma clang fp contract(off)
    const double d = a.x * b.x + a.y * b.y + a.z * b.z;
    return d > 0.0;
}

// Vertex degrees; every face starts as a set of its own that has met nothing.
__global__ __launch_bounds__(256) void fv_count_kernel(Batch B, FillRun r) {
    const AssetDev& As = B.A[0];
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= As.nhf) return;
    r.parent[f] = (uint32_t)f;
    r.seen[f] = 0u;
    uint32_t* __restrict__ deg = r.deg;
    int32_t v[3];
    if (!face_verts(As, f, v)) {
        set_status(B, kStHiIndex);
        return;
    }
    for (int i = 0; i < 3; ++i)
        if ((i < 1 || v[i] != v[0]) && (i < 2 || v[i] != v[1])) atomicAdd(&deg[v[i]], 1u);
}

__global__ __launch_bounds__(256) void fv_fill_kernel(Batch B, const uint32_t* __restrict__ off,
                                                      uint32_t* __restrict__ cur, uint32_t* __restrict__ adj) {
    const AssetDev& As = B.A[0];
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= As.nhf) return;
    int32_t v[3];
    if (!face_verts(As, f, v)) return;
    for (int i = 0; i < 3; ++i)
        if ((i < 1 || v[i] != v[0]) && (i < 2 || v[i] != v[1])) adj[off[v[i]] + atomicAdd(&cur[v[i]], 1u)] = (uint32_t)f;
}

// Parents are read and written by workgroups on every XCD while the unions
// run, so both go past the XCDs' own caches (device scope).
__device__ __forceinline__ uint32_t ld_parent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The order in which roots hook onto each other.  By index, faces numbered along a
// strip or a fan would hook each onto the one before it, all at once, and the
// first search through them would walk the whole chain.
__device__ __forceinline__ bool before(uint32_t a, uint32_t b) { return a * 2654435761u < b * 2654435761u; }

// Root of x, halving the path on the way (only links of non-roots are moved,
// to an ancestor).
__device__ __forceinline__ uint32_t find_root(uint32_t* parent, uint32_t x) {
    uint32_t p = ld_parent(&parent[x]);
    while (p != x) {
        const uint32_t g = ld_parent(&parent[p]);
        if (g != p) __hip_atomic_store(&parent[x], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = p;
        p = g;
    }
    return x;
}

__global__ __launch_bounds__(256) void fill_union_kernel(Batch B, FillRun r) {
    const AssetDev& As = B.A[0];
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= As.nhf || r.visible[f]) return;
    int32_t fv[3];
    if (!face_verts(As, f, fv)) return;
    const d3 nf_ = face_normal(As, fv);
    bool met = false;
    // the faces across an edge are in both its ends' lists: the shorter is walked
    // (the tip of a fan of n faces would cost each of them n)
    for (int i = 0; i < 3; ++i) {
        const int32_t p = fv[i], q = fv[i == 2 ? 0 : i + 1];
        if (p == q) continue;
        const bool swap = r.off[q + 1] - r.off[q] < r.off[p + 1] - r.off[p];
        const int32_t at = swap ? q : p, other = swap ? p : q;
        for (uint32_t e = r.off[at]; e < r.off[at + 1]; ++e) {
            const int64_t g = r.adj[e];
            const bool vis = r.visible[g] != 0u;
            // a pair of hidden faces is joined by the larger of the two
            if (vis ? met : g >= f) continue;
            int32_t gv[3];
            if (!face_verts(As, g, gv) || (gv[0] != other && gv[1] != other && gv[2] != other) ||
                !agree(nf_, face_normal(As, gv)))
                continue;
            if (vis) {
                met = true;
                continue;
            }
            uint32_t a = find_root(r.parent, (uint32_t)f), b = find_root(r.parent, (uint32_t)g);
            while (a != b) {
                if (before(a, b)) {
                    const uint32_t t = a;
                    a = b;
                    b = t;
                }
                const uint32_t old = atomicCAS(&r.parent[a], a, b);
                if (old == a) break;
                a = find_root(r.parent, old);
                b = find_root(r.parent, b);
            }
        }
    }
    r.met[f] = met ? 1u : 0u;
}

__global__ __launch_bounds__(256) void fill_mark_kernel(Batch B, FillRun r) {
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= B.A[0].nhf || r.visible[f]) return;
    int32_t fv[3];
    if (face_verts(B.A[0], f, fv) && r.met[f]) r.seen[find_root(r.parent, (uint32_t)f)] = 1u;
}

__global__ __launch_bounds__(256) void fill_out_kernel(Batch B, FillRun r) {
    const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (f >= B.A[0].nhf) return;
    const bool vis = r.visible[f] != 0u;
    if (r.visible_out) r.visible_out[f] = vis ? 1 : 0;
    if (r.exterior_out) r.exterior_out[f] = vis || r.seen[find_root(r.parent, (uint32_t)f)] ? 1 : 0;
}

}  // namespace

hipError_t launch_flood_fill(const BatchHost& H, const FillRun& r, hipStream_t s) {
    const AssetDev& As = H.A[0];
    const int64_t nf = As.nhf, nv = As.nhv;
    hipError_t e;
    if ((e = fill_u32(r.deg, 0, nv + 1, s)) != hipSuccess) return e;
    if ((e = fill_u32(r.cur, 0, nv + 1, s)) != hipSuccess) return e;
    const unsigned g = (unsigned)((nf + 255) / 256);
    if (g > 0) hipLaunchKernelGGL(fv_count_kernel, dim3(g), dim3(256), 0, s, H.dev, r);
    if ((e = exclusive_scan_u32(r.deg, r.off, nv, r.scan_tmp, r.off + nv, s)) != hipSuccess) return e;
    if (g > 0) {
        hipLaunchKernelGGL(fv_fill_kernel, dim3(g), dim3(256), 0, s, H.dev, (const uint32_t*)r.off, r.cur, r.adj);
        hipLaunchKernelGGL(fill_union_kernel, dim3(g), dim3(256), 0, s, H.dev, r);
        hipLaunchKernelGGL(fill_mark_kernel, dim3(g), dim3(256), 0, s, H.dev, r);
        hipLaunchKernelGGL(fill_out_kernel, dim3(g), dim3(256), 0, s, H.dev, r);
    }
    return hipGetLastError();
}

}  // namespace bake
