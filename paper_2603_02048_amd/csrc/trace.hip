// trace.hip -- curved-ray marching through the refractive-index field on gfx950.
//
// Paper Sec. 3.3.2-3.3.3.  Inside the volume every ray follows the explicit
// update of Eq. 16,
//     omega_{k+1} = normalize(omega_k + ds_k / n_k (I - omega_k omega_k^T) g_k)
//     C_{k+1}     = C_k + ds_k omega_{k+1},
// with n_k and g_k trilinearly sampled from the gridded (delta_n, grad n)
// (Sec. 3.3.1) and the step of Eq. 18,
//     ds_k = clamp(n_k theta_max / (|(I - omega omega^T) g_k| + eps), ds_min, ds_max),
// or the fixed step of Sec. 4.1.  Outside the volume rays are straight (Fig. 1
// caption); the image is formed only by bending (Sec. 3.3.2): the exit ray is
// intersected with a backdrop plane and re-projected through the same pinhole.
//
// Three launches per trace:
//   k_raygen  one thread per queue slot: pinhole ray, slab test against the
//             volume; rays that miss are finished at once, rays that enter
//             are binned by their chord length (longest first) and counted;
//             it also clears the counter set of the next launch
//   k_raygen_place  places the entering rays in a hit list sorted by bin
//             (wave ballots + mbcnt ranks, one atomic per workgroup and bin)
//   k_march   persistent waves pull hit rays from the list in batches of
//             64 (fewer where that leaves waves without work); once refill_min lanes have finished (by default all of
//             them), the idle lanes are refilled together (ballot of idle
//             lanes, one atomic per batch, mbcnt rank); finished rays write
//             their outputs at the next refill.  The length sort keeps the
//             lanes of a batch finishing together, and whole-batch refills
//             keep a wave's lanes one 8x8 pixel tile, whose rays gather from
//             few cache lines (see sample_field).
//             Each ray's arithmetic is independent of which lane or wave runs
//             it, so results are bitwise repeatable.
//
// Positions are float32 metres with a compensated (Kahan) sum of the steps.
// The direction is carried as an unnormalised vector p = wr + dw (entry
// direction plus accumulated turns); since normalize() ignores scale, adding
// |p| ds/n P g to p reproduces Eq. 16 exactly while dw keeps the low-order bits
// of many small turns that a unit vector would round away.
#include "haze_device.h"
#include "ray_geom.h"

#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cstring>

namespace haze {

// Exit distance along w from a point in the volume (clamped at 0).
__device__ __forceinline__ float exit_distance(const TraceGrid &G, const float c[3], const float w[3])
{
    // per axis the face the ray heads for, chosen by value (a per-lane choice
    // of address would turn the uniform bounds into vector loads), and the
    // distance by the hardware reciprocal (~2 ulp); axes with w = 0 never exit
    float t = INFINITY;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float face = w[k] > 0.0f ? G.hi[k] : G.lo[k];
        const float tk = (face - c[k]) * __builtin_amdgcn_rcpf(w[k]);
        if (w[k] != 0.0f) t = fminf(t, tk);
    }
    return fmaxf(t, 0.0f);
}

__device__ __forceinline__ float quad_side(const SceneQuad &Q, const float x[3])
{
    return fmaf(Q.n[0], x[0], fmaf(Q.n[1], x[1], fmaf(Q.n[2], x[2], -Q.n0)));
}

// The same with the plane (n, n0) as one vector.
__device__ __forceinline__ float plane_side(const float4 &P, const float x[3])
{
    return fmaf(P.x, x[0], fmaf(P.y, x[1], fmaf(P.z, x[2], -P.w)));
}

__device__ __forceinline__ bool in_quad(const SceneQuad &Q, const float h[3])
{
    const float u = fmaf(Q.du[0], h[0], fmaf(Q.du[1], h[1], fmaf(Q.du[2], h[2], -Q.du0)));
    const float v = fmaf(Q.dv[0], h[0], fmaf(Q.dv[1], h[1], fmaf(Q.dv[2], h[2], -Q.dv0)));
    return u >= 0.0f && u <= 1.0f && v >= 0.0f && v <= 1.0f;
}

// First board met by the straight ray x + t w, t in [0, tmax]; ties go to the
// lower index.  Returns the board index or -1, and t.
__device__ __forceinline__ int cast_quads(const SceneQuad *quads, int nquads, const float x[3], const float w[3],
                                          float tmax, float &thit)
{
    int best = -1;
    float bt = tmax;
    for (int k = 0; k < nquads; ++k) {
        const SceneQuad &Q = quads[k];
        const float dn = Q.n[0] * w[0] + Q.n[1] * w[1] + Q.n[2] * w[2];
        if (dn == 0.0f) continue;
        const float t = -quad_side(Q, x) / dn;
        if (!(t >= 0.0f) || t > bt || (t == bt && best >= 0)) continue;
        const float h[3] = {fmaf(t, w[0], x[0]), fmaf(t, w[1], x[1]), fmaf(t, w[2], x[2])};
        if (!in_quad(Q, h)) continue;
        best = k;
        bt = t;
    }
    thit = bt;
    return best;
}

// ---- triangle-mesh scenes ----

__device__ __forceinline__ bool in_tri(const SceneQuad &T, const float h[3])
{
    const float u = fmaf(T.du[0], h[0], fmaf(T.du[1], h[1], fmaf(T.du[2], h[2], -T.du0)));
    const float v = fmaf(T.dv[0], h[0], fmaf(T.dv[1], h[1], fmaf(T.dv[2], h[2], -T.dv0)));
    return u >= 0.0f && v >= 0.0f && u + v <= 1.0f;
}

// The tests' loads are gathers, served by the texture-address unit a lane (or
// what shares its line) at a time: list entries are read four and ranges two to
// a load (global loads need the words' own alignment), and the planes of a mesh
// of up to kLdsTriangles, 32 KB, come from LDS (five workgroups of the march
// then just fit a compute unit).  The march of 2 x 640x360 with 448 triangles:
// 136 us with the planes in memory, 126 from LDS.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(4)));
constexpr int kLdsTriangles = 2048;
extern __shared__ float4 mesh_planes[];

// Plane (n, n0) of triangle k.
__device__ __forceinline__ float4 tri_plane(const MeshLaunch &M, int k)
{
    if (M.ntris <= kLdsTriangles) return mesh_planes[k];
    return *reinterpret_cast<const float4 *>(M.tris[k].n);
}

// Fills them; all threads of the workgroup, before its first tri_plane().
__device__ __forceinline__ void load_planes(const MeshLaunch &M)
{
    if (M.ntris > kLdsTriangles) return;
    for (int k = (int)threadIdx.x; k < M.ntris; k += (int)blockDim.x)
        mesh_planes[k] = *reinterpret_cast<const float4 *>(M.tris[k].n);
    __syncthreads();
}

static size_t mesh_lds(const TraceLaunch &L)
{
    return L.mesh.ntris <= kLdsTriangles ? sizeof(float4) * (size_t)L.mesh.ntris : 0;
}

// f(k, plane) for those triangles of M.list[e0, e1), in its order, for which
// may(plane) holds.  Sorted out 32 at a time first: a wave then takes f as often
// as its busiest lane has candidates, not at every entry that is one for any
// lane.  (The load of a list's last entries begins before the list where it
// can, and reads past it in an array of less than four, which hz_mesh_create
// fills up; neither counts.)
template <class G, class F>
__device__ __forceinline__ void for_list(const MeshLaunch &M, uint32_t e0, uint32_t e1, const G &may, const F &f)
{
    for (uint32_t b = e0; b < e1; b += 32u) {
        const uint32_t be = min(b + 32u, e1);
        uint32_t cand = 0u;
        for (uint32_t e = b; e < be; e += 4u) {
            const uint32_t g = max(min(e + 4u, e1), 4u) - 4u;
            const u32x4 k4 = *reinterpret_cast<const u32x4 *>(M.list + g);
            const int k[4] = {(int)k4.x, (int)k4.y, (int)k4.z, (int)k4.w};
            float4 P[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) P[j] = tri_plane(M, k[j]);
            uint32_t m = 0u;
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j)
                if (may(P[j])) m |= 1u << j;
            cand |= (m >> (e - g)) << (e - b);
        }
        if (be - b < 32u) cand &= (1u << (be - b)) - 1u;
        while (cand) {
            const int k = (int)M.list[b + (uint32_t)__builtin_ctz(cand)];
            cand &= cand - 1u;
            f(k, tri_plane(M, k));
        }
    }
}

// Straight ray x + t w against triangle k of plane P (n, n0): keeps the first
// hit in (best, bt), ties to the lower triangle index.
__device__ __forceinline__ void cast_tri(const MeshLaunch &M, int k, const float4 &P, const float x[3],
                                         const float w[3], int &best, float &bt)
{
    const float dn = P.x * w[0] + P.y * w[1] + P.z * w[2];
    if (dn == 0.0f) return;
    const float t = -plane_side(P, x) / dn;
    if (!(t >= 0.0f) || t > bt || (t == bt && best >= 0 && k >= best)) return;
    const float h[3] = {fmaf(t, w[0], x[0]), fmaf(t, w[1], x[1]), fmaf(t, w[2], x[2])};
    if (!in_tri(M.tris[k], h)) return;
    best = k;
    bt = t;
}

// First triangle met by the straight ray x + t w, t in [0, tmax]: the ray
// walks the shell cells it crosses (3D DDA) and tests their lists, until the
// next cell starts beyond the best hit.  A cell lists every triangle within
// reach of it, so a hit inside a cell is found there whatever the rounding of
// the walk.  Returns the triangle or -1, and t; counts the exact tests.
__device__ int cast_mesh(const MeshLaunch &M, const float x[3], const float w[3], float tmax, float &thit,
                         uint32_t &ntests)
{
    int best = -1;
    float bt = tmax;
    if (M.brute) {
        for (int k = 0; k < M.ntris; ++k) cast_tri(M, k, tri_plane(M, k), x, w, best, bt);
        ntests += (uint32_t)M.ntris;
        thit = bt;
        return best;
    }
    float ta = 0.0f, tb = tmax;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float lo = M.lo[a], hi = M.lo[a] + (float)M.res[a] * M.cell;
        if (w[a] == 0.0f) {
            if (x[a] < lo || x[a] > hi) ta = INFINITY;
            continue;
        }
        const float inv = 1.0f / w[a];
        const float t1 = (lo - x[a]) * inv, t2 = (hi - x[a]) * inv;
        ta = fmaxf(ta, fminf(t1, t2));
        tb = fminf(tb, fmaxf(t1, t2));
    }
    if (!(ta <= tb)) {
        thit = bt;
        return -1;
    }
    // per-axis walk state in scalars (an array indexed by the axis chosen at
    // run time would live in private memory)
    auto axis_start = [&](int a, int &ci, int &stp, float &tn, float &td) {
        const float p = fmaf(ta, w[a], x[a]);
        ci = min(max((int)floorf((p - M.lo[a]) * M.inv_cell), 0), M.res[a] - 1);
        if (w[a] > 0.0f) {
            stp = 1;
            tn = (M.lo[a] + (float)(ci + 1) * M.cell - x[a]) / w[a];
            td = M.cell / w[a];
        } else if (w[a] < 0.0f) {
            stp = -1;
            tn = (M.lo[a] + (float)ci * M.cell - x[a]) / w[a];
            td = -M.cell / w[a];
        } else {
            stp = 0;
            tn = INFINITY;
            td = INFINITY;
        }
    };
    int cx, cy, cz, sx, sy, sz;
    float tnx, tny, tnz, tdx, tdy, tdz;
    axis_start(0, cx, sx, tnx, tdx);
    axis_start(1, cy, sy, tny, tdy);
    axis_start(2, cz, sz, tnz, tdz);
    const int rx = M.res[0], ry = M.res[1], rz = M.res[2];
    float tenter = ta;
    uint32_t cell = ((uint32_t)cz * (uint32_t)ry + (uint32_t)cy) * (uint32_t)rx + (uint32_t)cx;
    const auto cell_list = [&](uint32_t &e0, uint32_t &e1) {
        const u32x2 se = *reinterpret_cast<const u32x2 *>(M.start + cell);
        e0 = se.x;
        e1 = se.y;
    };
    // cells left along each axis, and the steps in the cell numbers
    int lx = sx > 0 ? rx - 1 - cx : cx, ly = sy > 0 ? ry - 1 - cy : cy, lz = sz > 0 ? rz - 1 - cz : cz;
    const uint32_t jx = (uint32_t)sx, jy = (uint32_t)(sy * rx), jz = (uint32_t)(sz * (rx * ry));
    uint32_t e0, e1;
    cell_list(e0, e1);
    for (int it = 0; it < rx + ry + rz + 3; ++it) {
        if (tenter > bt) break;
        // the next cell, and its list's range while this cell's list is tested
        const bool ax = tnx <= tny && tnx <= tnz, ay = !ax && tny <= tnz, az = !ax && !ay;
        tenter = ax ? tnx : ay ? tny : tnz;
        tnx = ax ? tnx + tdx : tnx;
        tny = ay ? tny + tdy : tny;
        tnz = az ? tnz + tdz : tnz;
        cell += ax ? jx : ay ? jy : jz;
        lx -= ax;
        ly -= ay;
        lz -= az;
        const bool last = min(min(lx, ly), lz) < 0 || tenter > tb;
        uint32_t f0 = 0u, f1 = 0u;
        if (!last) cell_list(f0, f1);
        for (uint32_t e = e0; e < e1; e += 2u) {
            const int k0 = (int)M.list[e], k1 = (int)M.list[min(e + 1u, e1 - 1u)];
            const float4 P0 = tri_plane(M, k0), P1 = tri_plane(M, k1);
            cast_tri(M, k0, P0, x, w, best, bt);
            cast_tri(M, k1, P1, x, w, best, bt);   // (k0 once more changes nothing)
        }
        ntests += e1 - e0;
        if (last) break;
        e0 = f0;
        e1 = f1;
    }
    thit = bt;
    return best;
}

// The chord a -> b = a + ds w of one march step against triangle k: the side
// value changes sign (or reaches zero) along it; keeps the first crossing
// (fraction lam, then the lower index) in (best, bl, hp).
__device__ __forceinline__ void chord_tri(const MeshLaunch &M, int k, const float4 &P, const float a[3],
                                          const float b[3], const float w[3], float ds, int &best, float &bl,
                                          float hp[3])
{
    const float s0 = plane_side(P, a), s1 = plane_side(P, b);
    if (s0 == 0.0f || (s0 > 0.0f && s1 > 0.0f) || (s0 < 0.0f && s1 < 0.0f)) return;
    const float lam = s0 / (s0 - s1);
    if (!(lam < bl || (lam == bl && k < best))) return;
    const float back = (1.0f - lam) * ds;
    const float h[3] = {fmaf(-back, w[0], b[0]), fmaf(-back, w[1], b[1]), fmaf(-back, w[2], b[2])};
    if (!in_tri(M.tris[k], h)) return;
    best = k;
    bl = lam;
    hp[0] = h[0]; hp[1] = h[1]; hp[2] = h[2];
}

// Writes a finished ray.  With surf >= 0 the ray already met scene board surf
// at hp; otherwise the straight ray (x, w) is cast against the boards and the
// view's backdrop plane (front side only) and the nearest wins, boards on
// ties.  The image point is re-projected through the pinhole: displacement =
// projected point - pixel centre (Sec. 3.3.2).
// Per-ray count of exact triangle tests of the ray's output, or null.
__device__ __forceinline__ uint32_t *tri_tests_of(const TraceLaunch &L, const Ray &r)
{
    return L.subset ? L.flat.tri_tests : L.jobs[r.job].tri_tests;
}

// SCENE 0: no scene; 1, 2: boards (surf is a board); 3: triangle mesh (surf
// is a triangle, reported by its surface id, and ntests counts the exact
// triangle tests the ray took so far).
template <int SCENE>
__device__ __forceinline__ void finish_ray(const TraceLaunch &L, const SceneQuad *quads, const TraceJob &J, const Ray &r, const float x[3],
                                           const float w[3], uint32_t steps, int status, const float *hp = nullptr,
                                           int surf = -1, uint32_t ntests = 0u)
{
    constexpr bool BOARDS = SCENE == 1 || SCENE == 2;
    float disp0 = __builtin_nanf(""), disp1 = __builtin_nanf("");
    int sid = 255;
    if (status != 3) {
        float h[3];
        bool hit = surf >= 0;
        if (hit) {
            h[0] = hp[0]; h[1] = hp[1]; h[2] = hp[2];
            sid = (SCENE == 3 ? (int)L.mesh.surf[surf] : surf) + 1;
        } else {
            const float denom = w[0] * J.plane_n[0] + w[1] * J.plane_n[1] + w[2] * J.plane_n[2];
            float tb = -1.0f;
            if (denom < 0.0f) {
                tb = ((J.plane_p[0] - x[0]) * J.plane_n[0] + (J.plane_p[1] - x[1]) * J.plane_n[1] +
                      (J.plane_p[2] - x[2]) * J.plane_n[2]) / denom;
                if (!(tb >= 0.0f)) tb = -1.0f;
            }
            float t = tb;
            hit = tb >= 0.0f;
            sid = 0;
            if (BOARDS) {
                float tq;
                const int q = cast_quads(quads, L.nquads, x, w, hit ? tb : INFINITY, tq);
                if (q >= 0) {
                    t = tq;
                    hit = true;
                    sid = q + 1;
                }
            }
            if (SCENE == 3) {
                float tq;
                const int q = cast_mesh(L.mesh, x, w, hit ? tb : INFINITY, tq, ntests);
                if (q >= 0) {
                    t = tq;
                    hit = true;
                    sid = (int)L.mesh.surf[q] + 1;
                }
            }
            if (hit) {
                h[0] = x[0] + t * w[0];
                h[1] = x[1] + t * w[1];
                h[2] = x[2] + t * w[2];
            }
        }
        float zc = 0.0f, xc = 0.0f, yc = 0.0f;
        if (hit) {
            const float hx = h[0] - J.eye[0];
            const float hy = h[1] - J.eye[1];
            const float hz = h[2] - J.eye[2];
            xc = hx * J.r[0] + hy * J.r[1] + hz * J.r[2];
            yc = hx * J.u[0] + hy * J.u[1] + hz * J.u[2];
            zc = hx * J.f[0] + hy * J.f[1] + hz * J.f[2];
            hit = zc > 0.0f;
        }
        if (hit) {
            disp0 = (J.half_w + J.fpx * xc / zc) - ((float)r.p + 0.5f);
            disp1 = (J.half_h - J.fpx * yc / zc) - ((float)r.q + 0.5f);
        } else {
            sid = 255;
            if (status == 0) status = 2;
        }
    }
    float *disp, *ep, *ed;
    uint32_t *st, *tt;
    uint8_t *stat, *sf;
    if (L.subset) {
        disp = L.flat.disp; ep = L.flat.exit_pos; ed = L.flat.exit_dir; st = L.flat.steps; stat = L.flat.status;
        sf = L.flat.surface; tt = L.flat.tri_tests;
    } else {
        disp = J.disp; ep = J.exit_pos; ed = J.exit_dir; st = J.steps; stat = J.status; sf = J.surface;
        tt = J.tri_tests;
    }
    if (BOARDS || sf) {
        if (sf) sf[r.out] = (uint8_t)sid;
    }
    if (SCENE == 3 && tt) tt[r.out] = ntests;   // the whole ray's exact triangle tests
    const int64_t o = r.out;
    if (disp) {
        disp[2 * o] = disp0;
        disp[2 * o + 1] = disp1;
    }
    if (ep) {
        ep[3 * o] = x[0];
        ep[3 * o + 1] = x[1];
        ep[3 * o + 2] = x[2];
    }
    if (ed) {
        ed[3 * o] = w[0];
        ed[3 * o + 1] = w[1];
        ed[3 * o + 2] = w[2];
    }
    if (st) st[o] = steps;
    if (stat) stat[o] = (uint8_t)status;
}

// Part of a job table carried in the kernel arguments: the tracer's view
// table reaches the device without a host staging buffer.
constexpr int kTableChunkWords = 240;
struct TableChunk {
    uint32_t offset;   // destination word offset
    uint32_t nwords;
    uint32_t w[kTableChunkWords];
};

__global__ __launch_bounds__(256) void k_put_table(uint32_t *__restrict__ dst, TableChunk c)
{
    for (uint32_t i = threadIdx.x; i < c.nwords; i += blockDim.x) dst[c.offset + i] = c.w[i];
}

// Zero the bin totals, the placement cursors and the march batch head.
__global__ void k_trace_init(uint32_t *counters)
{
    for (int k = threadIdx.x; k <= kMarchHead; k += blockDim.x) *hit_counter(counters, k) = 0u;
}

// Per-wave counts of each bin among the lanes' bins (255: none) into
// wcnt[wave][bin]; returns the lane's rank among the wave's lanes of its bin.
__device__ __forceinline__ uint32_t bin_rank(int bin, uint32_t (*wcnt)[kRayBins])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < kRayBins) wcnt[wave][lane] = 0u;
    // only the bins present in the wave (a wave is a pixel tile, whose rays
    // have similar chords: usually one to three bins)
    uint32_t rank = 0;
    uint64_t todo = __ballot(bin < kRayBins);
    while (todo) {
        const int first = (int)__builtin_ctzll(todo);
        const int b = __builtin_amdgcn_readlane(bin, first);
        const uint64_t m = __ballot(bin == b);
        if (lane == 0) wcnt[wave][b] = (uint32_t)__popcll(m);
        if (bin == b)
            rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        todo &= ~m;
    }
    return rank;
}

// SCENE: 0 no scene, 1 boards, 3 triangle mesh (the launch's scene kind, so
// that the common case carries no scene code).
template <int SCENE, int B>
__global__ __launch_bounds__(B) void k_raygen(TraceLaunch L, const TraceJob *__restrict__ jobs,
                                                                const SceneQuad *__restrict__ quads)
{
    if (SCENE == 3) load_planes(L.mesh);
    // A tile's slots run down its columns (decode_slot), but the rays that
    // miss write their outputs here, by pixel: the 64 threads of a tile take
    // its slots transposed, so neighbouring threads write neighbouring pixels
    // of a row.  (Which thread takes a slot changes nothing else: the counts
    // are per workgroup, and the hit list is placed in slot order.)
    const int l = (int)(threadIdx.x & 63);
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u) +
                         (L.subset ? l : (((l & 7) << 3) | (l >> 3)));
    bool enters = false;
    int bin = 255;
    // one ray: pinhole direction, entry into the volume, the rays that miss
    // (or meet the scene first) finished here
    const auto generate = [&](const TraceJob &J, Ray &r) {
        const float3 d3 = pixel_dir(J, r.p, r.q);
        const float d[3] = {d3.x, d3.y, d3.z};
        float t0, t1 = 0.0f;
        enters = enter_volume(L.grid, J.eye, d, t0, &t1);
        if (enters) bin = kRayBins - 1 - min(kRayBins - 1, max(0, (int)((t1 - t0) * L.inv_len_bin)));
        if (SCENE == 3) {
            if (enters) {
                // the mesh in front of the volume ends the ray before it enters;
                // otherwise the march continues the test count from here
                float tq;
                uint32_t nt = 0u;
                const int q = cast_mesh(L.mesh, J.eye, d, t0, tq, nt);
                if (q >= 0) {
                    const float hp[3] = {J.eye[0] + tq * d[0], J.eye[1] + tq * d[1], J.eye[2] + tq * d[2]};
                    finish_ray<3>(L, quads, J, r, J.eye, d, 0u, 0, hp, q, nt);
                    enters = false;
                } else if (uint32_t *tt = tri_tests_of(L, r)) {
                    tt[r.out] = nt;
                }
            } else {
                finish_ray<3>(L, quads, J, r, J.eye, d, 0u, 0);
            }
        } else if (SCENE == 1 && enters) {
            // a board in front of the volume ends the ray before it enters
            float tq;
            const int q = cast_quads(quads, L.nquads, J.eye, d, t0, tq);
            if (q >= 0) {
                const float hp[3] = {J.eye[0] + tq * d[0], J.eye[1] + tq * d[1], J.eye[2] + tq * d[2]};
                finish_ray<1>(L, quads, J, r, J.eye, d, 0u, 0, hp, q);
                enters = false;
            }
        } else if (!enters) {
            finish_ray<SCENE == 1 ? 1 : 0>(L, quads, J, r, J.eye, d, 0u, 0);
        }
    };
    if (!L.subset) {
        // a wave's 64 slots are one 8x8 tile of one view: the view is found,
        // and read, with scalar loads (`jobs` is L.jobs, which nothing here
        // writes)
        const uint32_t base =
            __builtin_amdgcn_readfirstlane((uint32_t)(blockIdx.x * blockDim.x + (threadIdx.x & ~63u)));
        if ((int64_t)base < L.nslots) {
            const int job = job_of_slot(jobs, L.njobs, base);
            const TraceJob &J = jobs[job];
            Ray r;
            if (slot < L.nslots && decode_tile_slot(J, job, slot, r)) generate(J, r);
        }
    } else if (slot < L.nslots) {
        Ray r;
        if (decode_slot(L, slot, r)) {
            generate(L.jobs[r.job], r);
        } else {
            // ray id outside the views: flag it, leave no stale values behind
            const float nan = __builtin_nanf("");
            if (L.flat.disp) L.flat.disp[2 * slot] = L.flat.disp[2 * slot + 1] = nan;
            if (L.flat.exit_pos)
                L.flat.exit_pos[3 * slot] = L.flat.exit_pos[3 * slot + 1] = L.flat.exit_pos[3 * slot + 2] = nan;
            if (L.flat.exit_dir)
                L.flat.exit_dir[3 * slot] = L.flat.exit_dir[3 * slot + 1] = L.flat.exit_dir[3 * slot + 2] = nan;
            if (L.flat.steps) L.flat.steps[slot] = 0u;
            if (L.flat.status) L.flat.status[slot] = 4u;
            if (L.flat.surface) L.flat.surface[slot] = 255u;
            if (L.flat.tri_tests) L.flat.tri_tests[slot] = 0u;
        }
    }
    // the next launch's counter set (this launch's march uses the other one)
    static_assert(kMarchHead < B, "one workgroup clears a counter set");
    if (blockIdx.x == 0 && threadIdx.x <= kMarchHead) *hit_counter(L.counters_next, threadIdx.x) = 0u;
    // pass 1 of the length sort: remember the bin, count the bins of the
    // workgroup (wave ballots), one atomic per non-empty bin
    if (!enters) bin = 255;
    if (slot < L.nslots) L.slot_bin[slot] = (uint8_t)bin;
    __shared__ uint32_t wcnt[B / 64][kRayBins];
    bin_rank(bin, wcnt);
    __syncthreads();
    if (threadIdx.x < kRayBins) {
        uint32_t total = 0;
        for (int w = 0; w < B / 64; ++w) total += wcnt[w][threadIdx.x];
        if (total) atomicAdd(hit_counter(L.counters, threadIdx.x), total);
    }
}

// Pass 2 of the length sort: each entering ray takes its place in its bin's
// range of the hit list (bins in order, longest rays first).  The order inside
// a bin depends on the atomics, which changes no ray's result.
__global__ __launch_bounds__(kRaygenBlock) void k_raygen_place(TraceLaunch L)
{
    const int64_t slot = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int bin = slot < L.nslots ? (int)L.slot_bin[slot] : 255;
    constexpr int W = kRaygenBlock / 64;
    __shared__ uint32_t wcnt[W][kRayBins];
    __shared__ uint4 tot4[kRayBins / 4];
    uint32_t *const tot = (uint32_t *)tot4;
    if (threadIdx.x < kRayBins) tot[threadIdx.x] = *hit_counter(L.counters, threadIdx.x);
    const uint32_t rank = bin_rank(bin, wcnt);
    __syncthreads();
    // a thread for each bin: the place of each wave's first ray of the bin
    // (unrolled, with the counts read at once: every workgroup waits for these
    // few threads.  8 x 1280x720 29 -> 25 us, 4 x 1920x1080 38 -> 28.5)
    if (threadIdx.x < kRayBins) {
        const int b = threadIdx.x;
        uint32_t cnt[W], total = 0, start = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            cnt[w] = wcnt[w][b];
            total += cnt[w];
        }
        if (total) {
            uint32_t at = atomicAdd(hit_counter(L.counters, kRayBins + b), total);
#pragma unroll
            for (int q = 0; q < kRayBins / 4; ++q) {
                const uint4 v = tot4[q];
                start += (4 * q < b ? v.x : 0u) + (4 * q + 1 < b ? v.y : 0u) + (4 * q + 2 < b ? v.z : 0u) +
                         (4 * q + 3 < b ? v.w : 0u);
            }
            at += start;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                wcnt[w][b] = at;
                at += cnt[w];
            }
        }
    }
    __syncthreads();
    if (bin < kRayBins) L.hits[wcnt[threadIdx.x >> 6][bin] + rank] = (uint32_t)slot;
}

__device__ __forceinline__ void wsum(float4 &v, float wgt, const float4 &c)
{
    v.x = fmaf(wgt, c.x, v.x);
    v.y = fmaf(wgt, c.y, v.y);
    v.z = fmaf(wgt, c.z, v.z);
    v.w = fmaf(wgt, c.w, v.w);
}

// Grid constants of the march, those of 16-bit float fields in vector registers
// where there is room: an FMA, add or multiply with a scalar-register operand
// takes the slower of the two issue paths (4.4 against 2.5 cycles of a SIMD
// measured), and two scalar operands cost a move.  All of them where boards leave
// five waves to a SIMD (2 x 960x540: 89.7 us with none, 87.5); else the offsets of
// the cell only, which save that move (nine requests over four 256^3 F16 fields
// 3,993 us with none, 3,907 with the offsets), since with all of them, the same
// within 0.5%, kernels spill, and fewer waves fit; none with a mesh.
struct MarchConst {
    float inv_sp[3], off[3];
    float magic;       // 2^23
    float inv_scale;
    float ds_max;
};

__device__ __forceinline__ float in_vgpr(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}

template <bool ALL, bool OFF>
__device__ __forceinline__ MarchConst march_const(const TraceGrid &G, const TraceStep &S)
{
    const auto put = [](float x) { return ALL ? in_vgpr(x) : x; };
    MarchConst K;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        K.inv_sp[a] = put(G.inv_sp[a]);
        K.off[a] = OFF ? in_vgpr(G.off[a]) : G.off[a];
    }
    K.magic = put(8388608.0f);
    K.inv_scale = put(G.inv_scale);
    K.ds_max = put(S.ds_max);
    return K;
}

// Cell of x and the trilinear weights in it: cell index (as a float) clamped
// to [0, R-2], so the outer half-voxel extrapolates linearly.  (A NaN
// coordinate gives a NaN weight, which poisons the sample and is caught by the
// march's finiteness test, and cell 0.)
__device__ __forceinline__ void cell_of(const TraceGrid &G, const MarchConst &K, const float x[3], float fl[3], float t[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float u = fmaf(x[a], K.inv_sp[a], K.off[a]);
        fl[a] = __builtin_amdgcn_fmed3f(floorf(u), 0.0f, G.maxi[a]);
        t[a] = u - fl[a];
    }
}

// F16/BF16 voxels are 8 bytes; the two z-neighbours of a cell row are one
// 16-byte load (8-byte aligned, which the hardware serves as one dwordx4).
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));
// The field pointer reaches the kernel through the job table, so the compiler
// cannot prove it is global memory; say so, to get global (not flat) loads.
typedef const u32x4_a8 __attribute__((address_space(1))) *gpair_ptr;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const f32x4 __attribute__((address_space(1))) *gfloat4_ptr;

__device__ __forceinline__ float4 load_f32x4(gfloat4_ptr F, uint32_t i)
{
    const f32x4 v = F[i];
    return make_float4(v.x, v.y, v.z, v.w);
}

template <int DT>
__device__ __forceinline__ float4 half4_to_float4(uint32_t lo, uint32_t hi)
{
    if (DT == DT_F16) {
        return make_float4(__half2float(__ushort_as_half((unsigned short)(lo & 0xffffu))),
                           __half2float(__ushort_as_half((unsigned short)(lo >> 16))),
                           __half2float(__ushort_as_half((unsigned short)(hi & 0xffffu))),
                           __half2float(__ushort_as_half((unsigned short)(hi >> 16))));
    } else {
        return make_float4(__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16),
                           __uint_as_float(hi & 0xffff0000u));
    }
}

template <int DT>
__device__ __forceinline__ void load_pair_at(gpair_ptr p, float4 &a, float4 &b)
{
    const u32x4_a8 v = *p;
    a = half4_to_float4<DT>(v.x, v.y);
    b = half4_to_float4<DT>(v.z, v.w);
}

// A field read by every ray of a launch (ONE): the bases of a cell's four rows
// (x, x + 1 at y; x, x + 1 at y + 1), which wave-uniform registers hold, each
// less kFieldBias, so that a cell needs one 32-bit offset and no address per
// row: 12 fewer instructions of a step's about 150.  4 x 1920x1080 of 256^3 F16,
// bound by issue, 3,520 -> 3,320 us; 8 x 1280x720 of 128^3 F32, bound by its
// gathers, 1,057 -> 1,039.  Batches that mix fields, and fields past
// one_field(), keep an address per view and row; so do scenes in the volume.
struct FieldRows {
    uint64_t row[4];
    uint32_t row_x;      // voxels along x
    uint32_t row_z;      // bytes of a column along z
};

template <int DT>
__device__ __forceinline__ FieldRows field_rows(const TraceGrid &G, const void *field)
{
    constexpr uint32_t B = DT == DT_F32 ? 16u : 8u;
    FieldRows R;
    const uint64_t base = (uint64_t)field - kFieldBias;
    R.row_x = (uint32_t)G.res[0];
    R.row_z = (uint32_t)G.res[2] * B;
    const uint64_t sx = R.row_z, sy = (uint64_t)R.row_x * R.row_z;
    R.row[0] = base;
    R.row[1] = base + sx;
    R.row[2] = base + sy;
    R.row[3] = base + sx + sy;
    // four bases, not one and three differences to add per lane
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+s"(R.row[k]));
    return R;
}

// Trilinear sample of (delta_n, grad n) at x (Sec. 3.3.1): 8 corners, 4 row
// loads of a z-neighbour pair each.  The gathers are bound by how the
// texture-address unit serves a wave's 64 addresses: lanes next to each other
// that fall in one cache line are served together.  The packed field keeps z
// (the cameras' up axis) fastest and the queue orders a tile's pixels
// column-major, so neighbouring lanes are vertically adjacent pixels whose
// rows share lines whatever horizontal direction the view looks along.  (With
// x fastest and row-major tiles only views along y coalesced: single 1280x720
// views along x took 1.8x as long.)
template <int DT, bool ONE>
__device__ __forceinline__ float4 sample_field(const TraceGrid &G, const MarchConst &K, const FieldRows &R,
                                               const void *__restrict__ f, const float x[3])
{
    float fl[3], t[3];
    cell_of(G, K, x, fl, t);
    float4 c000, c100, c010, c110, c001, c101, c011, c111;
    if (ONE) {
        // Indices below 2^23 are the low bits of index + 2^23 in a float: x and
        // y go into 24-bit products as they are, z already in bytes, with the
        // exponent bits of that sum (kFieldBias) taken off the bases.
        constexpr float B = DT == DT_F32 ? 16.0f : 8.0f;
        const uint32_t ix = __float_as_uint(fl[0] + K.magic), iy = __float_as_uint(fl[1] + K.magic);
        const uint32_t zb = __float_as_uint(fmaf(fl[2], B, K.magic));
        const uint32_t row = __umul24(iy, R.row_x) + (ix & 0xffffffu);
        const uint32_t o = __umul24(row, R.row_z) + zb;
        if (DT == DT_F32) {
            const gfloat4_ptr p0 = (gfloat4_ptr)(R.row[0] + o), q0 = (gfloat4_ptr)(R.row[1] + o),
                              p1 = (gfloat4_ptr)(R.row[2] + o), q1 = (gfloat4_ptr)(R.row[3] + o);
            c000 = load_f32x4(p0, 0);
            c001 = load_f32x4(p0, 1);
            c100 = load_f32x4(q0, 0);
            c101 = load_f32x4(q0, 1);
            c010 = load_f32x4(p1, 0);
            c011 = load_f32x4(p1, 1);
            c110 = load_f32x4(q1, 0);
            c111 = load_f32x4(q1, 1);
        } else {
            load_pair_at<DT>((gpair_ptr)(R.row[0] + o), c000, c001);
            load_pair_at<DT>((gpair_ptr)(R.row[1] + o), c100, c101);
            load_pair_at<DT>((gpair_ptr)(R.row[2] + o), c010, c011);
            load_pair_at<DT>((gpair_ptr)(R.row[3] + o), c110, c111);
        }
    } else {
        // The cell's corner voxel in the packed field, whose fastest axis is z
        // (fields hold fewer than 2^31 voxels: 32-bit indices), then 64-bit
        // pointer steps: the z-neighbour is the load's immediate offset, and the
        // x and y rows one add each.
        const uint32_t b = ((uint32_t)fl[1] * (uint32_t)G.res[0] + (uint32_t)fl[0]) * (uint32_t)G.res[2] + (uint32_t)fl[2];
        const uint32_t sx = (uint32_t)G.res[2], sy = (uint32_t)G.res[0] * (uint32_t)G.res[2];
        if (DT == DT_F32) {
            const gfloat4_ptr p0 = (gfloat4_ptr)f + b, p1 = p0 + sy;
            const gfloat4_ptr q0 = p0 + sx, q1 = p1 + sx;
            c000 = load_f32x4(p0, 0);
            c001 = load_f32x4(p0, 1);
            c100 = load_f32x4(q0, 0);
            c101 = load_f32x4(q0, 1);
            c010 = load_f32x4(p1, 0);
            c011 = load_f32x4(p1, 1);
            c110 = load_f32x4(q1, 0);
            c111 = load_f32x4(q1, 1);
        } else {
            typedef const uint16_t __attribute__((address_space(1))) *ghalf_ptr;
            const gpair_ptr p0 = (gpair_ptr)(reinterpret_cast<const uint16_t *>(f) + 4 * (size_t)b);
            const gpair_ptr p1 = (gpair_ptr)((ghalf_ptr)p0 + 4 * (size_t)sy);
            const gpair_ptr q0 = (gpair_ptr)((ghalf_ptr)p0 + 4 * (size_t)sx);
            const gpair_ptr q1 = (gpair_ptr)((ghalf_ptr)p1 + 4 * (size_t)sx);
            load_pair_at<DT>(p0, c000, c001);
            load_pair_at<DT>(q0, c100, c101);
            load_pair_at<DT>(p1, c010, c011);
            load_pair_at<DT>(q1, c110, c111);
        }
    }
    // trilinear weights, then one FMA per corner and channel
    const float ux = 1.0f - t[0], uy = 1.0f - t[1], uz = 1.0f - t[2];
    const float a00 = ux * uy, a10 = t[0] * uy, a01 = ux * t[1], a11 = t[0] * t[1];
    const float w000 = a00 * uz, w100 = a10 * uz, w010 = a01 * uz, w110 = a11 * uz;
    const float w001 = a00 * t[2], w101 = a10 * t[2], w011 = a01 * t[2], w111 = a11 * t[2];
    float4 v;
    if (DT == DT_F16) {
        // (with an addend of zero the product takes its 16-bit factor without a
        // conversion of its own)
        v.x = fmaf(w000, c000.x, 0.0f);
        v.y = fmaf(w000, c000.y, 0.0f);
        v.z = fmaf(w000, c000.z, 0.0f);
        v.w = fmaf(w000, c000.w, 0.0f);
    } else {
        v.x = w000 * c000.x;
        v.y = w000 * c000.y;
        v.z = w000 * c000.z;
        v.w = w000 * c000.w;
    }
    wsum(v, w100, c100);
    wsum(v, w010, c010);
    wsum(v, w110, c110);
    wsum(v, w001, c001);
    wsum(v, w101, c101);
    wsum(v, w011, c011);
    wsum(v, w111, c111);
    if (DT != DT_F32) {
        // stored values are scaled; interpolation is linear, so unscale once
        v.x *= K.inv_scale;
        v.y *= K.inv_scale;
        v.z *= K.inv_scale;
        v.w *= K.inv_scale;
    }
    return v;
}

// Distance from c to the nearest face of the box (negative outside).
__device__ __forceinline__ float face_distance(const TraceGrid &G, const float c[3])
{
    return fminf(fminf(fminf(c[0] - G.lo[0], G.hi[0] - c[0]), fminf(c[1] - G.lo[1], G.hi[1] - c[1])),
                 fminf(c[2] - G.lo[2], G.hi[2] - c[2]));
}

// How a march steps: plain, lean (see march()), or lean with a second wave walking
// ahead.  (16-bit fields without a scene in the volume always take the lean step;
// plain is then the kernel of large launches, where it is another one.)
enum { kStepPlain = 0, kStepLean = 1, kStepWalk = 2 };

// In launches of few rays the second wave of a workgroup walks straight along
// the rays that the first one marches, a voxel (or a longer step) at a time and
// as many steps side by side as its lanes allow, and loads a word of each of a
// cell's four rows: the march's gathers then find their lines in the caches, and
// a ray's steps, which such a launch lasts as long as, wait less.  (The march
// itself cannot: its loads return in order.)  The walk only reads, inside the
// field, and ends with the rays' chords or with the march, whichever is first.
// It naps for about 0.4 us per step of the march, so as not to push out of the
// L2 what it fetched: 4,096 chosen rays of 128^3 113 us without the walk, 112
// without naps, 99 with 0.2 us, 94 to 98 with these, 95 with 0.5; 64x36 rays 85 ->
// 78, 320x180 113 -> 105, 128x128 of 64^3 61 -> 55.
template <int DT, bool ONE>
__device__ __forceinline__ void walk_ahead(const TraceLaunch &L, uint32_t first, uint32_t sb, uint32_t nh,
                                           const uint32_t *over)
{
    const TraceGrid &G = L.grid;
    const uint32_t lane = threadIdx.x & 63u, ray = lane & (sb - 1u), sub = lane / sb, nsub = 64u / sb;
    if (first + ray >= nh) return;
    Ray r{0, 0, 0, 0};
    decode_slot(L, L.hits[first + ray], r);
    const TraceJob &J = L.jobs[r.job];
    const char *field = (const char *)(ONE ? L.field : J.field);
    const float3 d3 = pixel_dir(J, r.p, r.q);
    const float w[3] = {d3.x, d3.y, d3.z};
    float t0 = 0.0f, t1 = 0.0f;
    if (!enter_volume(G, J.eye, w, t0, &t1)) return;
    const float ds = L.step.uniform ? L.step.ds_uniform : L.step.ds_max;
    const float h = fmaxf(ds, fminf(fminf(1.0f / G.inv_sp[0], 1.0f / G.inv_sp[1]), 1.0f / G.inv_sp[2]));
    const int naps = (int)fminf(1024.0f, 1.2f * (float)nsub * h / ds);   // at least one
    constexpr uint32_t B = DT == DT_F32 ? 16u : 8u;
    const uint32_t sx = (uint32_t)G.res[2], sy = (uint32_t)G.res[0] * (uint32_t)G.res[2];
    const int n = (int)fminf((t1 - t0) / h + 1.0f, 131072.0f);
    for (int k = (int)sub; k < n; k += (int)nsub) {
        const float t = t0 + (float)k * h;
        uint32_t i[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            i[a] = (uint32_t)__builtin_amdgcn_fmed3f(floorf(fmaf(J.eye[a] + t * w[a], G.inv_sp[a], G.off[a])), 0.0f,
                                                     G.maxi[a]);
        const char *p = field + (size_t)((i[1] * (uint32_t)G.res[0] + i[0]) * (uint32_t)G.res[2] + i[2]) * B;
        const uint32_t v0 = *(const uint32_t *)p, v1 = *(const uint32_t *)(p + (size_t)sx * B);
        const uint32_t v2 = *(const uint32_t *)(p + (size_t)sy * B), v3 = *(const uint32_t *)(p + (size_t)(sx + sy) * B);
        asm volatile("" ::"v"(v0), "v"(v1), "v"(v2), "v"(v3));
        for (int s = 0; s < naps; ++s) {
            if (__hip_atomic_load(over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) return;
            __builtin_amdgcn_s_sleep(13);
        }
    }
}

// SCENE 0: no scene boards; 1: boards, none near the volume (met only by the
// straight exit ray); 2: some boards may cross the volume, so the chord of
// every step is tested against those (L.ninner of them) and the first one
// crossed ends the ray at the crossing point.
// ONE: every ray reads field L.field (see FieldRows), else its view's.
template <int DT, int SCENE, bool ONE, int STEP>
__device__ __forceinline__ void march(const TraceLaunch &L)
{
    const TraceGrid &G = L.grid;
    const TraceStep &S = L.step;
    const MarchConst K = march_const<DT == DT_F16 && SCENE == 2, DT == DT_F16 && SCENE != 3>(G, S);
    const FieldRows rows = ONE ? field_rows<DT>(G, L.field) : FieldRows{};
    // LEAN: a step asks once per wave whether any ray is near a face and once per
    // ray whether anything ends it, and sorts these out only then.
    constexpr bool LEAN = STEP != kStepPlain || (SCENE < 2 && DT != DT_F32);
    uint32_t nh = 0;
    for (int k = 0; k < kRayBins; ++k) nh += *hit_counter(L.counters, k);
    nh = __builtin_amdgcn_readfirstlane(nh);
    const uint32_t refill_min = (uint32_t)max(1, min(64, L.refill_min));
    const int lane = threadIdx.x & 63;

    // Work distribution over the length-sorted hits.  Wave w first takes
    // hits [sb w, sb w + sb) with no atomic; later batches of 64 come from one
    // counter past the static range, fetched ahead (the atomic's latency hides
    // behind the march).  Each wave keeps its reserve
    // [next, end) of hit indices.  With no more batches than workgroups the
    // waves are numbered across the workgroups, else along them (neighbouring
    // tiles then share a compute unit's L1).
    const uint32_t blk = blockIdx.x, nblk = gridDim.x;
    const uint32_t wpb = blockDim.x >> 6, nwaves = nblk * wpb;
    const uint32_t sb = march_batch(nh);
    const bool across = (uint64_t)nblk * sb >= nh;
    const uint32_t wib = threadIdx.x >> 6;
    const uint32_t wave_id = __builtin_amdgcn_readfirstlane(across ? blk + nblk * wib : blk * wpb + wib);
    const uint32_t dyn0 = nwaves * sb;
    uint32_t next = min(wave_id * sb, nh);
    uint32_t end = min(next + sb, nh);
    // With less than a second batch for each wave, a batch goes to the wave that
    // has finished its first: reserved while its rays were young, the last
    // batches began after the longest rays had ended.  One F32 view of 1600x900
    // on 128^3, 1.1 batches a wave, 271 -> 247 us, one of 1920x1080, 1.6 batches,
    // 365 -> 338; BF16 with fixed steps 639 -> 570 and 898 -> 800.  From about two batches a wave on the
    // rounds even out by themselves, and F32 is 2% slower with it.
    const bool late = nh < dyn0 + nwaves * 64u;
    __shared__ uint32_t over;   // the first wave's rays have ended
    const bool walk = STEP == kStepWalk && across && sb < 64u;
    if (walk) {
        if (threadIdx.x == 0) over = 0u;
        __syncthreads();
        if (wib == 1u) {
            if (blk * sb < nh) walk_ahead<DT, ONE>(L, blk * sb, sb, nh, &over);
            return;
        }
    }
    bool done = next >= nh && dyn0 >= nh;
    bool pending = false;
    uint32_t pend_v = 0;

    bool active = false;
    Ray r{0, 0, 0, 0};
    const void *field = nullptr;
    // direction omega = p / |p| with p = wr + dw: wr is the entry direction and
    // dw accumulates the turns, so small turns keep their low-order bits
    float c[3] = {0, 0, 0}, cc[3] = {0, 0, 0}, w[3] = {0, 0, 1}, wr[3] = {0, 0, 1}, dw[3] = {0, 0, 0};
    float pnorm = 1.0f;
    float safe = 0.0f;   // lower bound of the distance from c to the box faces
    uint32_t steps = 0;
    float side[SCENE == 2 ? kMaxInner : 1];   // side values of the inner boards at c
    // A finished ray keeps its end state (c, w, steps) and writes its outputs
    // only when the wave refills or stops, so the output code runs once for
    // all lanes finished since, not once per finishing lane.
    int fin = -1;        // status of a finished ray not yet written (-1: none)
    int fin_surf = -1;   // its board or triangle (c is then the hit point), -1 for none
    uint32_t ntests = 0u;   // SCENE 3: the ray's exact triangle tests so far

    // Outer loop: refill the wave's idle lanes (wave-uniform bookkeeping);
    // inner loop: step the active lanes until enough of them have finished.
    // The refill and the step are separate loops, so the step loop carries
    // the rays' state alone (no joins with the refill code on every step).
    for (;;) {
        const uint64_t idle = __ballot(!active);
        const uint32_t nidle = (uint32_t)__popcll(idle);
        if (!done) {
            if (fin >= 0) {
                finish_ray<SCENE>(L, L.quads, L.jobs[r.job], r, c, w, steps, fin, c, fin_surf, ntests);
                fin = -1;
            }
            if (next == end) {
                uint32_t b;
                if (pending) {
                    b = __shfl(pend_v, 0);
                    pending = false;
                } else {
                    uint32_t v = 0;
                    if (lane == 0) v = dyn0 + atomicAdd(hit_counter(L.counters, kMarchHead), 64u);
                    b = __shfl(v, 0);
                }
                b = __builtin_amdgcn_readfirstlane(b);
                if (b >= nh) {
                    done = true;   // next == end: nothing left to hand out below
                } else {
                    next = b;
                    end = min(b + 64u, nh);
                }
            }
            if (!active && next < end) {
                const uint32_t k = next + __builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
                if (k < end) {
                    const int64_t slot = L.hits[k];
                    decode_slot(L, slot, r);
                    const TraceJob &J = L.jobs[r.job];
                    if (!ONE) field = J.field;
                    const float3 d3 = pixel_dir(J, r.p, r.q);
                    w[0] = d3.x; w[1] = d3.y; w[2] = d3.z;
                    wr[0] = d3.x; wr[1] = d3.y; wr[2] = d3.z;
                    dw[0] = dw[1] = dw[2] = 0.0f;
                    pnorm = sqrtf(d3.x * d3.x + d3.y * d3.y + d3.z * d3.z);
                    float t0 = 0.0f;
                    enter_volume(G, J.eye, w, t0);
                    c[0] = J.eye[0] + t0 * w[0];
                    c[1] = J.eye[1] + t0 * w[1];
                    c[2] = J.eye[2] + t0 * w[2];
                    cc[0] = cc[1] = cc[2] = 0.0f;
                    safe = face_distance(G, c);
                    steps = 0;
                    active = true;
                    if (SCENE == 3) {
                        const uint32_t *tt = tri_tests_of(L, r);
                        ntests = tt ? tt[r.out] : 0u;   // the straight part before the volume
                    }
                    if (SCENE == 2) {
#pragma unroll
                        for (int j = 0; j < kMaxInner; ++j)
                            side[j] = j < L.ninner ? plane_side(L.inner[j], c) : 0.0f;
                    }
                }
            }
            next = min(next + nidle, end);
            if (!done && next == end && !pending) {
                if (dyn0 >= nh) {
                    done = true;   // the static batches hold every hit: no dynamic work
                } else if (!late) {
                    if (lane == 0) pend_v = dyn0 + atomicAdd(hit_counter(L.counters, kMarchHead), 64u);
                    pending = true;
                }
            }
        }
        if (done && __ballot(active) == 0ull) {
            if (fin >= 0) finish_ray<SCENE>(L, L.quads, L.jobs[r.job], r, c, w, steps, fin, c, fin_surf, ntests);
            if (walk && wib == 0u) __hip_atomic_store(&over, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            break;
        }
        // once nothing is left to hand out, step until every lane is done
        const uint32_t want_idle = done ? 64u : refill_min;
        for (;;) {
            if (active) {
                // ---- one step of Eq. 16 with the step of Eq. 18 ----
                // Only a step that starts near a face needs the exit distance te
                // (LEAN: it is left unset while no lane of the wave is near one).
                float te;
                if (LEAN) asm volatile("" : "=v"(te));
                int status = -1, hit_surf = -1;
                const bool any_near = !LEAN || __ballot(safe <= S.near_cap) != 0ull;
                if (any_near) {
                    te = INFINITY;
                    if (safe <= S.near_cap) {
                        safe = face_distance(G, c);
                        if (safe <= S.near_cap) {
                            te = exit_distance(G, c, w);
                            if (te <= S.tau) status = 0;
                        }
                    }
                }
                if (status < 0) {
                    // the shell cell of C_k, its bound and list with the field's loads
                    float shell = INFINITY;
                    uint32_t e0 = 0u, e1 = 0u;
                    if (SCENE == 3 && !L.mesh.brute) {
                        const MeshLaunch &M = L.mesh;
                        int ci[3];
                        bool in = true;
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            ci[a] = (int)floorf((c[a] - M.lo[a]) * M.inv_cell);
                            in = in && ci[a] >= 0 && ci[a] < M.res[a];
                        }
                        if (in) {
                            const uint32_t cell = ((uint32_t)ci[2] * (uint32_t)M.res[1] + (uint32_t)ci[1]) *
                                                      (uint32_t)M.res[0] + (uint32_t)ci[0];
                            shell = M.dlow[cell];
                            const u32x2 se = *reinterpret_cast<const u32x2 *>(M.start + cell);
                            e0 = se.x;
                            e1 = se.y;
                        }
                    }
                    const float4 s = sample_field<DT, ONE>(G, K, rows, field, c);
                    const float n = 1.0f + s.x;
                    const float rn = __builtin_amdgcn_rcpf(n);
                    const float wg = w[0] * s.y + w[1] * s.z + w[2] * s.w;
                    const float pg0 = s.y - wg * w[0], pg1 = s.z - wg * w[1], pg2 = s.w - wg * w[2];
                    float ds;
                    if (S.uniform) {
                        ds = LEAN ? in_vgpr(S.ds_uniform) : S.ds_uniform;
                    } else {
                        const float pgn = __builtin_amdgcn_sqrtf(pg0 * pg0 + pg1 * pg1 + pg2 * pg2);
                        // clamp to [ds_min, ds_max] (ds_min <= ds_max, checked on the host) in
                        // one med3: fminf/fmaxf would also canonicalize both bounds every step
                        ds = __builtin_amdgcn_fmed3f(n * S.theta_max * __builtin_amdgcn_rcpf(pgn + S.eps), S.ds_min,
                                                     K.ds_max);
                    }
                    if (any_near) {   // a branch (the asm keeps it one); in it
                        if (LEAN) asm volatile("" : "+v"(te));
                        ds = te < ds ? te : ds;   // min(ds, te) as a select: fminf would canonicalize both
                    }
                    // omega_{k+1} = normalize(omega_k + ds/n P g) = normalize(p + |p| ds/n P g)
                    const float a = ds * rn * pnorm;
                    dw[0] = fmaf(a, pg0, dw[0]);
                    dw[1] = fmaf(a, pg1, dw[1]);
                    dw[2] = fmaf(a, pg2, dw[2]);
                    const float p0 = wr[0] + dw[0], p1 = wr[1] + dw[1], p2 = wr[2] + dw[2];
                    const float pn2 = p0 * p0 + p1 * p1 + p2 * p2;
                    const float inv = __builtin_amdgcn_rsqf(pn2);
                    pnorm = pn2 * inv;
                    w[0] = p0 * inv;
                    w[1] = p1 * inv;
                    w[2] = p2 * inv;
                    float cp[3];   // C_k (SCENE 3)
                    if (SCENE == 3) {
                        cp[0] = c[0]; cp[1] = c[1]; cp[2] = c[2];
                    }
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        // compensated C += ds * w
                        const float y = fmaf(ds, w[k], -cc[k]);
                        const float t = c[k] + y;
                        cc[k] = (t - c[k]) - y;
                        c[k] = t;
                    }
                    ++steps;
                    safe -= ds;
                    int surf = -1;
                    float hp[3];
                    if (SCENE == 3) {
                        // chord C_k -> C_{k+1} against the triangles that the shell
                        // cell of C_k lists, unless the cell's distance bound
                        // exceeds the step (then no triangle is within reach)
                        const MeshLaunch &M = L.mesh;
                        float bl = 2.0f;
                        if (M.brute) {
                            for (int k = 0; k < M.ntris; ++k)
                                chord_tri(M, k, tri_plane(M, k), cp, c, w, ds, surf, bl, hp);
                            ntests += (uint32_t)M.ntris;
                        } else if (shell <= ds * 1.001f) {
                            for_list(
                                M, e0, e1,
                                [&](const float4 &P) { return plane_side(P, cp) * plane_side(P, c) <= 0.0f; },
                                [&](int k, const float4 &P) { chord_tri(M, k, P, cp, c, w, ds, surf, bl, hp); });
                            ntests += e1 - e0;
                        }
                    }
                    if (SCENE == 2) {
                        // (The planes come with the kernel's arguments, in scalar registers:
                        // from memory they were a vector load and its wait per board and
                        // step, 98 us of march at 2 x 960x540 with two boards against 87.)
                        // chord C_k -> C_{k+1} = C_{k+1} - ds w: the board whose side value
                        // changes sign (or reaches zero) first along it; ties go to the
                        // lower board index
                        float best = 2.0f;
#pragma unroll
                        for (int j = 0; j < kMaxInner; ++j) {
                            if (j >= L.ninner) continue;
                            const int k = (int)((L.inner_idx >> (8 * j)) & 255u);
                            const float s0 = side[j], s1 = plane_side(L.inner[j], c);
                            side[j] = s1;
                            if (s0 == 0.0f || (s0 > 0.0f && s1 > 0.0f) || (s0 < 0.0f && s1 < 0.0f)) continue;
                            const float lam = s0 / (s0 - s1);
                            if (!(lam < best)) continue;
                            const float back = (1.0f - lam) * ds;
                            const float h[3] = {fmaf(-back, w[0], c[0]), fmaf(-back, w[1], c[1]),
                                                fmaf(-back, w[2], c[2])};
                            if (!in_quad(L.quads[k], h)) continue;
                            best = lam;
                            surf = k;
                            hp[0] = h[0]; hp[1] = h[1]; hp[2] = h[2];
                        }
                    }
                    // a non-finite sample makes n or the direction vector p non-finite
                    // (or p zero); otherwise the step, direction and position stay finite.
                    const bool finite = pn2 > 0.0f && pn2 < INFINITY && fabsf(n) < INFINITY;
                    const bool on = finite && safe > S.pos_eps && (int32_t)steps < S.max_steps;
                    if (!LEAN || !on) {
                        if (!finite)
                            status = 3;
                        else if ((SCENE == 2 || SCENE == 3) && surf >= 0) {
                            c[0] = hp[0]; c[1] = hp[1]; c[2] = hp[2];
                            status = 0;
                            hit_surf = surf;
                        } else if (safe <= S.pos_eps &&
                                   (c[0] < G.lo[0] || c[0] > G.hi[0] || c[1] < G.lo[1] || c[1] > G.hi[1] ||
                                    c[2] < G.lo[2] || c[2] > G.hi[2]))
                            status = 0;
                        else if ((int32_t)steps >= S.max_steps)
                            status = 1;
                    }
                }
                if (status >= 0) {
                    fin = status;
                    fin_surf = hit_surf;
                    active = false;
                }
            }
            if ((uint32_t)__popcll(__ballot(!active)) >= want_idle) break;
        }
    }
}

// Waves per SIMD: six (at most 80 registers a lane, where some kernels spill up to
// 18), five with boards or a mesh in the volume.  Seven (72 registers) for F16 up
// to kLeanSlots, without scene: the chip then holds 458,752 rays at once and not
// 393,216.  900x506 with 413,000 rays entering 181 us with six, 160 with seven;
// 1280x720 with 330,000 117 and 120.  Large launches run several rounds either way,
// and within 72 registers a step takes 1.5% more instructions: 4 x 1920x1080 of
// 256^3 3,288 us and 3,397.
template <int DT, int SCENE, int STEP>
constexpr int march_waves = DT == DT_F16 && SCENE == 0 && STEP == kStepLean ? 7 : 6;

template <int DT, int SCENE, bool ONE, int STEP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(march_waves<DT, SCENE, STEP>)))
void k_march(TraceLaunch L)
{
    march<DT, SCENE, ONE, STEP>(L);
}

template <int DT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_march_boards(TraceLaunch L)
{
    march<DT, 2, false, kStepPlain>(L);
}

template <int DT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_march_mesh(TraceLaunch L)
{
    load_planes(L.mesh);
    march<DT, 3, false, kStepPlain>(L);
}

// With a scene in the volume the scene's tests bound a step: the boards' march
// lost 2% by the rows' registers (97.4 -> 99.7 us at 2 x 960x540).
template <int SCENE>
constexpr bool one_field_march = SCENE < 2;

// The lean step (see march()) is for marches bound by instruction issue or by one
// ray's steps: of 16-bit fields (4 x 1920x1080 of 256^3 3,320 us against 3,510)
// and of F32 fields up to 2^20 slots (64x36 rays of 128^3 78 against 83, 640x360
// 114 against 117, 1280x720 the same).  Larger F32 launches may be bound by their
// gathers (1920x1080 with 1.4 M rays entering 807 against 788, with 0.55 M 336 and
// 337, 2 x 1280x720 with every ray entering 967 and 950), and with a scene in the
// volume its tests count most (boards 103 against 99.5).
constexpr int64_t kLeanSlots = (int64_t)1 << 20;
// The walk ahead is for launches of at most 32,768 entering rays; larger ones don't
// carry its code (640x360 of 128^3, 71,000 rays, 114 us without and 116 with it).
constexpr int64_t kWalkSlots = (int64_t)1 << 17;

template <int DT, int SCENE, bool ONE, int STEP>
static constexpr auto march_kernel()
{
    if constexpr (SCENE == 2)
        return &k_march_boards<DT>;
    else if constexpr (SCENE == 3)
        return &k_march_mesh<DT>;
    else
        return &k_march<DT, SCENE, ONE,
                        STEP == kStepPlain && DT != DT_F32 &&
                                march_waves<DT, SCENE, kStepLean> == march_waves<DT, SCENE, kStepPlain>
                            ? kStepLean
                            : STEP>;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------

// Copy `bytes` (a multiple of 4) of host memory to device memory at `dst`
// through kernel arguments, in chunks of kTableChunkWords words.
hipError_t launch_put_table(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    TableChunk c;
    const uint32_t total = (uint32_t)(bytes / 4);
    for (uint32_t off = 0; off < total; off += kTableChunkWords) {
        c.offset = off;
        c.nwords = std::min<uint32_t>(kTableChunkWords, total - off);
        std::memcpy(c.w, (const uint32_t *)src + off, 4u * c.nwords);
        hipLaunchKernelGGL(k_put_table, dim3(1), dim3(256), 0, s, (uint32_t *)dst, c);
    }
    return hipGetLastError();
}

// Ray generation for L.nslots > 0 slots; `clear_counters` when the set
// L.counters was not cleared by the previous launch's ray generation (new
// memory, or after a failed launch).
template <int SCENE, int B>
static void launch_raygen_t(const TraceLaunch &L, size_t lds, hipStream_t s, hipEvent_t e0)
{
    hipExtLaunchKernelGGL((k_raygen<SCENE, B>), dim3((unsigned)((L.nslots + B - 1) / B)), dim3(B), lds, s, e0, nullptr,
                          0, L, L.jobs, L.quads);
}

hipError_t launch_raygen(const TraceLaunch &L, bool clear_counters, hipStream_t s, const KTimer &t)
{
    if (L.nslots <= 0) return hipSuccess;
    if (clear_counters)
        hipExtLaunchKernelGGL(k_trace_init, dim3(1), dim3(64), 0, s, t.start, nullptr, 0, L.counters);
    const dim3 g((unsigned)((L.nslots + kRaygenBlock - 1) / kRaygenBlock));
    hipEvent_t e0 = clear_counters ? nullptr : t.start;
    // The mesh's ray generation holds 76 registers a lane: one workgroup of 1,024
    // to a compute unit, and 450 of them (2 x 640x360) took two rounds, 53 us
    // against 44 in workgroups of 256.  The others run in 512 (2 x 960x540 with
    // boards 19.5 us in 1,024, 18.8 in 512), but large launches in 1,024: each
    // workgroup adds to the same counters, once for each bin among its entering
    // rays.  1,024 / 512: 1280x720 18.2 / 16.3 us when a third enters and 22.0 /
    // 24.4 when all do, 1920x1080 27.4 / 24.4 and 31.7 / 41.0.  Chosen rays enter
    // all and lie in many bins: 100,000 of them 13.6 / 12.6 us, 200,000 15.9 / 16.0,
    // 400,000 20.9 / 24.4, 2,500,000 72 / 92.
    const bool large = L.nslots > (int64_t)1 << (L.subset ? 18 : 20);
    if (L.mesh.ntris > 0)
        launch_raygen_t<3, 256>(L, mesh_lds(L), s, e0);
    else if (L.nquads > 0)
        large ? launch_raygen_t<1, 1024>(L, 0, s, e0) : launch_raygen_t<1, 512>(L, 0, s, e0);
    else
        large ? launch_raygen_t<0, 1024>(L, 0, s, e0) : launch_raygen_t<0, 512>(L, 0, s, e0);
    hipExtLaunchKernelGGL(k_raygen_place, g, dim3(kRaygenBlock), 0, s, nullptr, t.stop, 0, L);
    return hipGetLastError();
}

static int march_scene_mode(const TraceLaunch &L) { return L.mesh.ntris > 0 ? 3 : L.ninner > 0 ? 2 : L.nquads > 0 ? 1 : 0; }

template <int DT, int SCENE, bool ONE, int STEP>
static void launch_march_k(const TraceLaunch &L, int march_blocks, hipStream_t s, const KTimer &t)
{
    hipExtLaunchKernelGGL((march_kernel<DT, SCENE, ONE, STEP>()), dim3(march_blocks), dim3(256),
                          SCENE == 3 ? mesh_lds(L) : 0, s, t.start, t.stop, 0, L);
}

template <int DT, int SCENE, bool ONE>
static void launch_march_o(const TraceLaunch &L, int march_blocks, hipStream_t s, const KTimer &t)
{
    if (L.nslots <= kWalkSlots)
        launch_march_k<DT, SCENE, ONE, kStepWalk>(L, march_blocks, s, t);
    else if (L.nslots <= kLeanSlots)
        launch_march_k<DT, SCENE, ONE, kStepLean>(L, march_blocks, s, t);
    else
        launch_march_k<DT, SCENE, ONE, kStepPlain>(L, march_blocks, s, t);
}

template <int DT, int SCENE>
static void launch_march_t(const TraceLaunch &L, int march_blocks, hipStream_t s, const KTimer &t)
{
    if (one_field_march<SCENE> && L.field)
        launch_march_o<DT, SCENE, one_field_march<SCENE>>(L, march_blocks, s, t);
    else
        launch_march_o<DT, SCENE, false>(L, march_blocks, s, t);
}

template <int DT>
static void launch_march_scene(const TraceLaunch &L, int march_blocks, hipStream_t s, const KTimer &t)
{
    switch (march_scene_mode(L)) {
    case 3: launch_march_t<DT, 3>(L, march_blocks, s, t); break;
    case 2: launch_march_t<DT, 2>(L, march_blocks, s, t); break;
    case 1: launch_march_t<DT, 1>(L, march_blocks, s, t); break;
    default: launch_march_t<DT, 0>(L, march_blocks, s, t);
    }
}

hipError_t launch_march(int dtype, const TraceLaunch &L, int march_blocks, hipStream_t s, const KTimer &t)
{
    if (dtype == DT_F32)
        launch_march_scene<DT_F32>(L, march_blocks, s, t);
    else if (dtype == DT_F16)
        launch_march_scene<DT_F16>(L, march_blocks, s, t);
    else
        launch_march_scene<DT_BF16>(L, march_blocks, s, t);
    return hipGetLastError();
}

template <int DT, int SCENE>
static hipError_t occupancy(bool large, int *nb)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        nb, large ? march_kernel<DT, SCENE, true, kStepPlain>() : march_kernel<DT, SCENE, true, kStepLean>(), 256, 0);
}

template <int SCENE>
static hipError_t occupancy(int dtype, bool large, int *nb)
{
    return dtype == DT_F32   ? occupancy<DT_F32, SCENE>(large, nb)
           : dtype == DT_F16 ? occupancy<DT_F16, SCENE>(large, nb)
                             : occupancy<DT_BF16, SCENE>(large, nb);
}

// Whether a march of that many slots takes the kernels of large launches.
bool march_large(int64_t nslots) { return nslots > kLeanSlots; }

int march_blocks_per_cu(int dtype, int scene_mode, bool large)
{
    int nb = 0;
    const hipError_t e = scene_mode == 3   ? occupancy<3>(dtype, large, &nb)
                         : scene_mode == 2 ? occupancy<2>(dtype, large, &nb)
                         : scene_mode == 1 ? occupancy<1>(dtype, large, &nb)
                                           : occupancy<0>(dtype, large, &nb);
    if (e != hipSuccess || nb < 1) nb = 1;
    return nb;
}

}  // namespace haze
