// mesh.hip -- triangle meshes: host construction of the BVH (binned
// surface-area heuristic splits, 16 bins per axis over the centroid bounds; a
// median split where the bins cannot separate the triangles; leaves of up to
// four triangles, preorder layout with skip links for stackless traversal),
// and the FP16 distance grid of a mesh on the device.
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "host.hpp"
#include "mesh.hpp"

namespace msst {
namespace {

// Splits are binned surface-area costs over all three axes in one pass, on
// triangle bounds and centroids worked out once: a bin's bounds are folded from
// both ends instead of anew for each split, and a split that moves no triangle
// is not priced again (20 480 triangles on one core 11.7 -> 3.5 ms, for 75
// bytes of host memory a triangle beside the nodes instead of 4).  A minimum
// keeps the earlier of equal values and skips NaN, in the order of the
// triangles, so that a node's bytes, signs of zeros included, depend on the
// triangles alone.
struct Builder {
    typedef float F4 __attribute__((ext_vector_type(4)));
    static constexpr int kBins = 16;
    struct Tri {
        F4 lo, hi;    // bounds
        F4 sum, mid;  // of the vertices, and a third of it (the fourth entry is unused)
    };
    std::vector<Tri> tri;
    std::vector<int32_t> idx, right;
    std::vector<uint8_t> bin[3];  // of the node's triangles, by position
    std::vector<BvhNode> nodes;

    static F4 min4(F4 a, F4 b) { return b < a ? b : a; }
    static F4 max4(F4 a, F4 b) { return a < b ? b : a; }
    static double area(F4 lo, F4 hi) {
        const double dx = hi.x - lo.x, dy = hi.y - lo.y, dz = hi.z - lo.z;
        return dx < 0 ? 0.0 : dx * dy + dy * dz + dz * dx;
    }

    void init(const float* tris, int n) {
        tri.resize(n);
        idx.resize(n);
        right.resize(n);
        for (auto& k : bin) k.resize(n);
        nodes.reserve(2 * (size_t)n);
        for (int i = 0; i < n; ++i) {
            const float* t = tris + 9 * (size_t)i;
            const F4 v[3] = {{t[0], t[1], t[2], 0.0f}, {t[3], t[4], t[5], 0.0f}, {t[6], t[7], t[8], 0.0f}};
            Tri& r = tri[i];
            r.lo = min4(min4(min4((F4)INFINITY, v[0]), v[1]), v[2]);
            r.hi = max4(max4(max4((F4)-INFINITY, v[0]), v[1]), v[2]);
            r.sum = v[0] + v[1] + v[2];
            r.mid = r.sum / 3.0f;
            idx[i] = i;
        }
    }

    void build(int b, int e, int depth) {
        const int self = (int)nodes.size();
        nodes.push_back(BvhNode{});
        BvhNode nd{};
        F4 lo = INFINITY, hi = -INFINITY, clo = INFINITY, chi = -INFINITY;
        for (int i = b; i < e; ++i) {
            const Tri& t = tri[idx[i]];
            lo = min4(lo, t.lo);
            hi = max4(hi, t.hi);
            clo = min4(clo, t.mid);
            chi = max4(chi, t.mid);
        }
        for (int a = 0; a < 3; ++a) {
            nd.lo[a] = lo[a];
            nd.hi[a] = hi[a];
        }
        if (e - b <= kBvhLeafMax) {
            nd.leaf = (b << 4) | (e - b);
            nd.skip = self + 1;
            nodes[self] = nd;
            return;
        }
        const F4 ext = chi - clo;
        const bool wide[3] = {ext.x > 0.0f, ext.y > 0.0f, ext.z > 0.0f};
        F4 blo[3][kBins], bhi[3][kBins];
        int cnt[3][kBins] = {};
        for (int a = 0; a < 3; ++a)
            for (int k = 0; k < kBins; ++k) {
                blo[a][k] = INFINITY;
                bhi[a][k] = -INFINITY;
            }
        for (int i = b; i < e; ++i) {
            const Tri& t = tri[idx[i]];
            const F4 at = (t.mid - clo) / ext * (float)kBins;
            for (int a = 0; a < 3; ++a) {
                const int k = wide[a] ? std::min(kBins - 1, std::max(0, (int)at[a])) : 0;
                bin[a][i] = (uint8_t)k;
                ++cnt[a][k];
                blo[a][k] = min4(blo[a][k], t.lo);
                bhi[a][k] = max4(bhi[a][k], t.hi);
            }
        }
        // cost of a split = area(left) n_left + area(right) n_right
        int best_axis = -1, best_bin = 0;
        double best_cost = INFINITY;
        for (int a = 0; a < 3; ++a) {
            if (!wide[a]) continue;
            F4 rlo[kBins], rhi[kBins];
            F4 l = INFINITY, h = -INFINITY;
            for (int k = kBins - 1; k > 0; --k) {
                rlo[k] = l = min4(l, blo[a][k]);
                rhi[k] = h = max4(h, bhi[a][k]);
            }
            l = INFINITY;
            h = -INFINITY;
            int nl = 0;
            for (int split = 1; split < kBins; ++split) {
                if (cnt[a][split - 1] == 0) continue;  // the cost of the split before, or nothing on the left
                l = min4(l, blo[a][split - 1]);
                h = max4(h, bhi[a][split - 1]);
                nl += cnt[a][split - 1];
                const int nr = e - b - nl;
                if (nr == 0) break;
                const double cost = area(l, h) * nl + area(rlo[split], rhi[split]) * nr;
                if (cost < best_cost) {
                    best_cost = cost;
                    best_axis = a;
                    best_bin = split;
                }
            }
        }
        int mid = b;
        if (best_axis >= 0 && depth < 48) {
            int nr = 0;
            for (int i = b; i < e; ++i) {
                if (bin[best_axis][i] < best_bin) idx[mid++] = idx[i];
                else right[nr++] = idx[i];
            }
            std::copy(right.begin(), right.begin() + nr, idx.begin() + mid);
        } else {
            // no separating bin (or a deep, lopsided branch): split the index
            // range at its median along the longest centroid axis
            int axis = 0;
            for (int a = 1; a < 3; ++a)
                if (chi[a] - clo[a] > chi[axis] - clo[axis]) axis = a;
            mid = b + (e - b) / 2;
            std::nth_element(idx.begin() + b, idx.begin() + mid, idx.begin() + e, [&](int32_t x, int32_t y) {
                const float cx = tri[x].sum[axis], cy = tri[y].sum[axis];
                return cx < cy || (cx == cy && x < y);
            });
        }
        build(b, mid, depth + 1);
        build(mid, e, depth + 1);
        nd.leaf = -1;
        nd.skip = (int)nodes.size();
        nodes[self] = nd;
    }
};

}  // namespace

// ---------------------------------------------------------------------------
// Distance grid of a mesh: at every voxel centre the FP64 distance to the
// nearest triangle, negative where the ray from there along
// (1, 2, 3) / sqrt(14) crosses the mesh an odd number of times.
//
// Testing every triangle for every voxel is 4.3e10 FP64 distances for 20 480
// triangles on 128^3 voxels.  A block takes a brick of 4^3 voxels and narrows
// the triangles down in two steps before the FP64 tests: bounding spheres
// against the brick's (lanes over triangles, lists in LDS), then per voxel
// (lanes over voxels, the eight waves sharing the lists) the sphere and an
// FP32 distance.  Every step keeps whatever its rounding could misjudge
// (margins far above the FP32 error; triangles too thin for FP32 pass all
// filters and bound nothing), so the smallest distance and the parity of the
// crossings come from the same FP64 arithmetic as testing all of them, and
// neither depends on the order: the grid is the same bit for bit.
//
// VALU-bound, half on reading the triangles once and a quarter per brick and
// half on the per-voxel filters.  20 480 triangles: 128^3 voxels 153 -> 5.4
// ms, 97^3 72 -> 2.8 ms; 1 280 triangles on 33^3 0.82 -> 0.09 ms; never slower
// down to one triangle on 9^3.  Bricks of 8^3 read the triangles less often, but
// their lists overflow near the medial axis (the centre of a round body keeps
// nearly every triangle): 15.8 ms.
constexpr int kGridWaves = 8, kGridThreads = 64 * kGridWaves;
constexpr int kBrick = 4;
// Triangles listed in LDS at a time, 20 bytes each, so that two blocks fit a
// CU: those of the distances from the front, those of the rays from the
// back; a brick with more works them off in parts.
constexpr int kGridList = 3584;

// Bounding sphere about the centroid; unbounded for a triangle so thin that
// the FP32 tests mean nothing (the FP64 test then always runs).
__device__ __forceinline__ void tri_sphere(const float* t, V3& m, float& r) {
    const V3 a = v3(t[0], t[1], t[2]), b = v3(t[3], t[4], t[5]), c = v3(t[6], t[7], t[8]);
    m = (1.0f / 3.0f) * (a + b + c);
    const V3 da = a - m, db = b - m, dc = c - m, e1 = b - a, e2 = c - a, nv = cross(e1, e2);
    const float q = __builtin_fmaxf(dot(da, da), __builtin_fmaxf(dot(db, db), dot(dc, dc)));
    r = dot(nv, nv) > 1e-10f * dot(e1, e1) * dot(e2, e2) ? fast_sqrt(q) : INFINITY;
}

// The same for the crossing test: unbounded where the triangle is nearly
// parallel to the ray direction u.
__device__ __forceinline__ float tri_ray_radius(const float* t, V3 u, float r) {
    const V3 a = v3(t[0], t[1], t[2]), e1 = v3(t[3], t[4], t[5]) - a, e2 = v3(t[6], t[7], t[8]) - a;
    const float det = dot(e1, cross(u, e2));
    return det * det > 1e-10f * dot(e1, e1) * dot(e2, e2) ? r : INFINITY;
}

// Squared FP32 distance from p to a triangle (the nearest of its edges, or
// its plane where p projects inside), and shape, the relative error of its
// normal in units of the FP32 rounding.  The edges are differences of exact
// values, good to a rounding; what is left grows with |p - a|, which the
// triangle's size bounds.  (The unit normal keeps its products in range: edges
// too long for the square of their cross product give a shape of 0 with a
// distance of 0, or one that is not a number.)
__device__ __forceinline__ float edge_dist2(V3 p, V3 e, float ee) {
    const float s = __builtin_fminf(1.0f, __builtin_fmaxf(0.0f, dot(p, e) * fast_rcp(ee)));
    const V3 q = p - s * e;
    return dot(q, q);
}
__device__ __forceinline__ float tri_distance32(const float* t, V3 p, float& shape) {
    const V3 a = v3(t[0], t[1], t[2]), b = v3(t[3], t[4], t[5]), c = v3(t[6], t[7], t[8]);
    const V3 e1 = b - a, e2 = c - b, e3 = a - c, cr = cross(e1, e2);
    const float l1 = dot(e1, e1), l2 = dot(e2, e2), l3 = dot(e3, e3), inv = fast_rsq(dot(cr, cr));
    const V3 nv = inv * cr;
    const V3 pa = p - a, pb = p - b, pc = p - c;
    float d2 = __builtin_fminf(edge_dist2(pa, e1, l1), __builtin_fminf(edge_dist2(pb, e2, l2), edge_dist2(pc, e3, l3)));
    const bool in = dot(cross(e1, nv), pa) <= 0.0f && dot(cross(e2, nv), pb) <= 0.0f && dot(cross(e3, nv), pc) <= 0.0f;
    const float h = dot(nv, pa);
    d2 = in ? __builtin_fminf(d2, h * h) : d2;
    shape = (l1 + l2 + l3) * inv;
    return d2;
}

__global__ __launch_bounds__(kGridThreads) void sdf_grid_mesh_kernel(const float* __restrict__ tris, int n_tris,
                                                                     int res, double lox, double loy, double loz,
                                                                     double hx, double hy, double hz, uint16_t* out) {
    __shared__ float4 list_s[kGridList];    // bounding sphere
    __shared__ uint32_t list_i[kGridList];  // triangle
    __shared__ int n_dist, n_ray;
    __shared__ float near_w[kGridWaves], bound_w[kGridWaves][64];
    __shared__ double dmin_w[kGridWaves][64];
    __shared__ uint64_t odd_w[kGridWaves];
    const double u64[3] = {0.2672612419124244, 0.5345224838248488, 0.8017837257372732};
    const V3 u = v3((float)u64[0], (float)u64[1], (float)u64[2]);
    const int wave = uniform_u32(threadIdx.x >> 6), lane = lane_id();
    const int64_t nb = (res + kBrick - 1) / kBrick;
    // half diagonal between the voxel centres of a brick; the largest
    // coordinate of the grid, the scale of the rounding errors
    const float r_brick = 0.5f * (kBrick - 1) * (float)sqrt(hx * hx + hy * hy + hz * hz) * 1.0001f;
    const double end = fmax(fmax(fmax(fabs(lox), fabs(lox + res * hx)), fmax(fabs(loy), fabs(loy + res * hy))),
                            fmax(fabs(loz), fabs(loz + res * hz)));
    const float scale = (float)end, slack = 1e-5f * scale;
    // may the ray from within `pad` of c meet the sphere (m, r)?
    auto meets = [&](V3 m, float r, V3 c, float pad) __attribute__((always_inline)) {
        const V3 v = m - c;
        const float along = dot(v, u);
        const V3 x = v - along * u;
        const float lim = r + pad + slack + 1e-5f * (__builtin_fabsf(v.x) + __builtin_fabsf(v.y) + __builtin_fabsf(v.z));
        return !(dot(x, x) > lim * lim) && !(along < -lim);
    };

    for (int64_t brick = blockIdx.x; brick < nb * nb * nb; brick += gridDim.x) {
        const int64_t bi = brick % nb * kBrick, bj = brick / nb % nb * kBrick, bk = brick / (nb * nb) * kBrick;
        const int64_t i = bi + (lane & 3), j = bj + ((lane >> 2) & 3), k = bk + (lane >> 4);
        const double p64[3] = {lox + (i + 0.5) * hx, loy + (j + 0.5) * hy, loz + (k + 0.5) * hz};
        const V3 p = v3((float)p64[0], (float)p64[1], (float)p64[2]);
        const V3 cb = v3((float)(lox + (bi + 0.5 * kBrick) * hx), (float)(loy + (bj + 0.5 * kBrick) * hy),
                         (float)(loz + (bk + 0.5 * kBrick) * hz));
        // A centroid's distance from the brick's centre, the smallest of all
        // or of every fourth triangle: no voxel is farther than that plus
        // r_brick from the mesh.  (A centroid is off by up to 4e-7 of its
        // triangle's size, however near it is: 1e-6 of the radius is added to
        // its distance, here and below.)
        const int stride = n_tris >= 4 * kGridThreads ? 4 : 1;
        float near = INFINITY;
        for (int q = stride * threadIdx.x; q < n_tris; q += stride * kGridThreads) {
            V3 m;
            float r;
            tri_sphere(tris + 9 * (int64_t)q, m, r);
            near = __builtin_fminf(near, __builtin_fmaf(1e-6f, r, fast_sqrt(dot(m - cb, m - cb))));
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) near = __builtin_fminf(near, __shfl_xor(near, off));
        if (lane == 0) near_w[wave] = near;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kGridWaves; ++w) near = __builtin_fminf(near, near_w[w]);

        // Lists the triangles from `first` on that pass the brick's tests;
        // returns where the next part starts (n_tris: all done).
        auto list_from = [&](int first) __attribute__((always_inline)) -> int {
            __syncthreads();
            if (threadIdx.x == 0) n_dist = n_ray = 0;
            __syncthreads();
            int at = first;
            while (at < n_tris) {
                const int q = at + (int)threadIdx.x;
                V3 m = v3(0, 0, 0);
                float r = 0.0f, rr = 0.0f;
                bool dist = false, ray = false;
                if (q < n_tris) {
                    const float* t = tris + 9 * (int64_t)q;
                    tri_sphere(t, m, r);
                    rr = tri_ray_radius(t, u, r);
                    const float lim = 1.00001f * (r + near + 2.0f * r_brick) + slack;
                    dist = !(dot(m - cb, m - cb) > lim * lim);
                    ray = meets(m, rr, cb, r_brick);
                }
                const uint64_t dmask = ballot(dist), rmask = ballot(ray);
                int d0 = 0, r0 = 0;
                if (lane == 0) {
                    if (dmask) d0 = atomicAdd(&n_dist, __popcll(dmask));
                    if (rmask) r0 = atomicAdd(&n_ray, __popcll(rmask));
                }
                d0 = __builtin_amdgcn_readfirstlane(d0);
                r0 = __builtin_amdgcn_readfirstlane(r0);
                if (dist) {
                    const int slot = d0 + rank_in(dmask);
                    list_s[slot] = make_float4(m.x, m.y, m.z, r);
                    list_i[slot] = (uint32_t)q;
                }
                if (ray) {
                    const int slot = kGridList - 1 - (r0 + rank_in(rmask));
                    list_s[slot] = make_float4(m.x, m.y, m.z, rr);
                    list_i[slot] = (uint32_t)q;
                }
                at += kGridThreads;
                __syncthreads();
                const int n_now = n_dist + n_ray;
                __syncthreads();
                if (n_now > kGridList - 2 * kGridThreads) break;
            }
            return at < n_tris ? at : n_tris;
        };

        // First pass: an upper bound of each voxel's distance from the
        // centroids, and the ray's crossings.
        float bound = INFINITY;
        bool odd = false;
        int next = 0;
        bool one_part = false;  // the lists hold all of the brick's triangles
        for (int first = 0; first < n_tris; first = next) {
            next = list_from(first);
            for (int e = wave; e < n_dist; e += kGridWaves) {
                const float4 s = list_s[e];
                const V3 v = v3(s.x, s.y, s.z) - p;
                bound = __builtin_fminf(bound, __builtin_fmaf(1e-6f, s.w, fast_sqrt(dot(v, v))));
            }
            for (int e = wave; e < n_ray; e += kGridWaves) {
                const float4 s = list_s[kGridList - 1 - e];
                const bool test = meets(v3(s.x, s.y, s.z), s.w, p, 0.0f);
                if (ballot(test) == 0) continue;
                const int q = (int)uniform_u32(list_i[kGridList - 1 - e]);
                if (test) odd ^= tri_ray_crosses64(tris + 9 * (int64_t)q, p64, u64);
            }
            one_part = first == 0 && next == n_tris;
        }
        bound_w[wave][lane] = bound;
        const uint64_t mask = ballot(odd);
        if (lane == 0) odd_w[wave] = mask;
        __syncthreads();
        bound = bound_w[0][lane];
#pragma unroll
        for (int w = 1; w < kGridWaves; ++w) bound = __builtin_fminf(bound, bound_w[w][lane]);
        // Second pass: FP64 for the triangles that neither their sphere nor
        // their FP32 distance rules out.
        double dmin = INFINITY;
        for (int first = 0; first < n_tris; first = next) {
            next = one_part ? n_tris : list_from(first);
            for (int e = wave; e < n_dist; e += kGridWaves) {
                const float4 s = list_s[e];
                const V3 v = v3(s.x, s.y, s.z) - p;
                const float lim = 1.00001f * (s.w + bound) + slack;
                bool need = !(dot(v, v) > lim * lim);
                if (ballot(need) == 0) continue;
                const float* t = tris + 9 * (int64_t)uniform_u32(list_i[e]);
                if (s.w < INFINITY) {
                    float shape;
                    const float d2 = tri_distance32(t, p, shape);
                    const float most = bound + 1e-6f * (8.0f + shape) * (scale + bound + s.w);
                    need = need && !(d2 > most * most);
                    if (ballot(need) == 0) continue;
                }
                if (need) {
                    dmin = fmin(dmin, tri_distance64(t, p64));
                    bound = __builtin_fminf(bound, (float)dmin + slack);
                }
            }
        }
        dmin_w[wave][lane] = dmin;
        __syncthreads();
        if (wave == 0 && i < res && j < res && k < res) {
            uint64_t sign = 0;
#pragma unroll
            for (int w = 0; w < kGridWaves; ++w) {
                dmin = fmin(dmin, dmin_w[w][lane]);
                sign ^= odd_w[w];
            }
            out[(k * res + j) * res + i] = fp16_bits_rtz((sign >> lane) & 1 ? -dmin : dmin);
        }
        __syncthreads();
    }
}

void launch_mesh_grid(const float* tris, int n_tris, int res, const float* lo, const double* h, uint16_t* grid,
                      int cus, hipStream_t stream) {
    const int64_t nb = (res + kBrick - 1) / kBrick;
    int64_t blocks = nb * nb * nb;
    if (blocks > (int64_t)cus * 64) blocks = (int64_t)cus * 64;
    hipLaunchKernelGGL(sdf_grid_mesh_kernel, dim3((unsigned)blocks), dim3(kGridThreads), 0, stream, tris, n_tris, res,
                       (double)lo[0], (double)lo[1], (double)lo[2], h[0], h[1], h[2], grid);
}

}  // namespace msst

extern "C" {

ms_status ms_mesh_bvh_size(int32_t n_tris, size_t* node_bytes) {
    MS_REQUIRE(node_bytes != nullptr, "ms_mesh_bvh_size: node_bytes is NULL");
    MS_REQUIRE(n_tris >= 1 && n_tris < (1 << 26), "ms_mesh_bvh_size: n_tris must be in [1, 2^26)");
    *node_bytes = (size_t)(2 * n_tris) * sizeof(msst::BvhNode);
    return MS_OK;
}

ms_status ms_build_mesh_bvh(const float* tris_host, int32_t n_tris, void* nodes_host, size_t node_bytes,
                            float* tris_sorted_host, int32_t* n_nodes) {
    using namespace msst;
    MS_REQUIRE(tris_host && nodes_host && tris_sorted_host && n_nodes, "ms_build_mesh_bvh: NULL argument");
    MS_REQUIRE(n_tris >= 1 && n_tris < (1 << 26), "ms_build_mesh_bvh: n_tris must be in [1, 2^26)");
    for (int64_t i = 0; i < 9 * (int64_t)n_tris; ++i)
        MS_REQUIRE(std::isfinite(tris_host[i]), "ms_build_mesh_bvh: vertex coordinates must be finite");
    size_t need = 0;
    ms_mesh_bvh_size(n_tris, &need);
    if (node_bytes < need) return set_error(MS_ERR_WORKSPACE_TOO_SMALL, "ms_build_mesh_bvh: nodes need %zu bytes", need);
    Builder bld;
    try {
        bld.init(tris_host, n_tris);
        bld.build(0, n_tris, 0);
    } catch (const std::bad_alloc&) {
        return set_error(MS_ERR_UNSUPPORTED, "ms_build_mesh_bvh: no host memory for %d triangles", n_tris);
    }
    std::memcpy(nodes_host, bld.nodes.data(), bld.nodes.size() * sizeof(BvhNode));
    for (int i = 0; i < n_tris; ++i)
        std::memcpy(tris_sorted_host + 9 * (size_t)i, tris_host + 9 * (size_t)bld.idx[i], 9 * sizeof(float));
    *n_nodes = (int32_t)bld.nodes.size();
    clear_error();
    return MS_OK;
}

}  // extern "C"
