// Tetrahedral parts: volume ray casting of unstructured meshes split into
// (possibly non-convex) parts, the parts standing in for the ranks that own
// a share of a finite-element data set.
//
// A frame, for n parts and the context camera:
//   march     one workgroup per 8 x 8 tile of a part's ROI (the part's
//             bounding box projected), its wavefronts taking stretches of the
//             tile's rays, or, where tiles are many, one wavefront per tile.
//             Every lattice sample t_k = (k + 1/2) dt of the ray inside the
//             part's bounding box is located in the part: by a short walk
//             from the tetrahedron that held the ray's previous sample (to the
//             neighbour across the face that rejects the sample most), else
//             among the tetrahedra listed in the sample's cell of the part's
//             uniform grid.  A tetrahedron holds p when its four signed sub-volumes
//             are positive, a zero one counting when the tie direction enters
//             across that face, so a sample has one owner in the whole mesh
//             and the first tetrahedron found is that owner.  The value is
//             the barycentric interpolation of the vertex values, classified
//             and accumulated front to back as in the brick march.  A part
//             that is not convex can hold several stretches of a ray: each
//             maximal run of consecutive held samples becomes a run
//             (first sample index, premultiplied colour, alpha).
//   resolve   per pixel, the runs of all parts in sample-index order with
//             "over", then the background.  Runs of different parts never
//             share a sample, so this equals accumulating the whole ray.
// With one directional light, before the march: a count pass (held samples
// per ROI pixel of every part), an exclusive scan (a slot per held sample), a
// record pass (each slot's sample index), then the shadow pass, in which every
// slot's shadow ray visits part home, home + 1, ... (mod n), and the march
// scales each held sample's emission by a0 + (1 - a0) S from its slot.
// Locations are those of float64 planes with contraction off (float32 planes
// with an error bound settle what they can), so the owner of a sample does
// not depend on the launch.
// Measured (1280x720, 2.0 M tetrahedra in 8 parts, 20.6 M held samples): one
// lane per ray, in step, float64 planes 3.91 ms a frame; as here 1.60 ms.
// 384x384, 246 K in 4 parts with shadows: 21.7 -> 5.5 ms; 14.6 K in 3 parts,
// 317x241: 0.48 -> 0.18 ms.
#include "march_common.h"
#include "tet_kernels.h"

#include <algorithm>
#include <cmath>

namespace dpvr {
namespace {

typedef __attribute__((address_space(1))) const int32_t gint;
typedef __attribute__((address_space(1))) const uint32_t guint;
typedef double double2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef int int4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const double2_t gdouble2;
typedef __attribute__((address_space(1))) const float4_t gfloat4;
typedef int4_t int4_unaligned __attribute__((aligned(4)));
typedef __attribute__((address_space(1))) const int4_unaligned gint4_unaligned;

// Value of vertex v: given, or (a cell centre) the mean of its cell's
// nodes, summed in node order.
__device__ inline float vertex_value(const float* __restrict__ vv, int32_t n_input,
                                     const int32_t* __restrict__ centre_nodes, int32_t v) {
    if (v < n_input) return vv[v];
    const int32_t* c = centre_nodes + 8 * (long long)(v - n_input);
    float s = 0.0f;
    int n = 0;
    for (; n < 8 && c[n] >= 0; ++n) s += vv[c[n]];
    return s / (float)n;
}

__global__ __launch_bounds__(256) void tet_values(const float* __restrict__ vv, int32_t n_input,
                                                  const int32_t* __restrict__ centre_nodes,
                                                  const int4* __restrict__ tets, int32_t n,
                                                  float4* __restrict__ vals) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const int4 t = tets[e];
    vals[e] = make_float4(vertex_value(vv, n_input, centre_nodes, t.x), vertex_value(vv, n_input, centre_nodes, t.y),
                          vertex_value(vv, n_input, centre_nodes, t.z), vertex_value(vv, n_input, centre_nodes, t.w));
}

// Candidate sample indices [k0, k1] of the ray against the closed box
// [lo, hi], widened by two samples on each side (rounding of the slab
// parameters never drops a sample; ownership is decided per sample).
__device__ inline bool box_range(const CamRay& r, const double lo[3], const double hi[3], double dt,
                                 long long& k0, long long& k1) {
#pragma clang fp contract(off)
    double tin = 0.0, tout = INFINITY;
    for (int c = 0; c < 3; ++c) {
        if (r.d[c] == 0.0) {
            if (r.o[c] < lo[c] || r.o[c] > hi[c]) return false;
            continue;
        }
        const double ta = (lo[c] - r.o[c]) / r.d[c], tb = (hi[c] - r.o[c]) / r.d[c];
        tin = fmax(tin, fmin(ta, tb));
        tout = fmin(tout, fmax(ta, tb));
    }
    if (!(tout >= tin - 2.0 * dt)) return false;
    const double a = fmax(floor(tin / dt - 0.5) - 2.0, 0.0), b = ceil(tout / dt - 0.5) + 2.0;
    if (!(b >= a)) return false;
    k0 = (long long)a;
    k1 = (long long)b;
    return true;
}

// The four sub-volumes D of p in tetrahedron e, and the face to leave it by when it does not hold p: of the faces that reject p, the one
// with the most negative sub-volume (-1: e holds p).
__device__ inline int reject_face(const TetPartK& P, int e, double p0, double p1, double p2, double D[4]) {
#pragma clang fp contract(off)
    gdouble2* pl = ((gdouble2*)P.planes) + 8 * (long long)e;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double2_t a = pl[2 * i], b = pl[2 * i + 1];
        D[i] = ((a.x * p0 + a.y * p1) + b.x * p2) - b.y;
    }
    const double least = fmin(fmin(D[0], D[1]), fmin(D[2], D[3]));
    int face = D[0] == least ? 0 : D[1] == least ? 1 : D[2] == least ? 2 : 3;
    if (least > 0.0) face = -1;
    if (least == 0.0) {                  // on a face (rare): the tie rule
        const uint32_t own = ((guint*)P.owned)[e];
        face = -1;
#pragma unroll
        for (int i = 3; i >= 0; --i) face = D[i] == 0.0 && !((own >> i) & 1u) ? i : face;
    }
    return face;
}

// reject_face in float32 (x: p relative to the part's grid origin; pl: the
// tetrahedron's float32 record, the first three barycentric coordinates as
// planes), where the smallest coordinate is beyond the error bound;
// kUndecided otherwise (also for records marked with an infinity).
constexpr int kUndecided = 4;
__device__ inline int reject_face32(const TetPartK& P, const float4_t (&pl)[3], float x0, float x1, float x2) {
    float l[4], e = 0.0f;
    l[3] = 1.0f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float4_t n = pl[i];
        l[i] = fmaf(n.x, x0, fmaf(n.y, x1, fmaf(n.z, x2, -n.w)));
        l[3] -= l[i];
        e = fmaf(fabsf(n.x), P.err32[0], fmaf(fabsf(n.y), P.err32[1], fmaf(fabsf(n.z), P.err32[2], e)));
    }
    const float least = fminf(fminf(l[0], l[1]), fminf(l[2], l[3]));
    const int face = l[0] == least ? 0 : l[1] == least ? 1 : l[2] == least ? 2 : 3;
    return least + e < 0.0f ? face : least - e > 0.0f ? -1 : kUndecided;
}

// Steps of the walk from the previous sample's tetrahedron across rejecting
// faces before the grid is searched.
constexpr int kWalkSteps = 4;

// Adds every lane's n to *counter (one atomic per wavefront); all lanes of
// the wavefront call it.
__device__ inline void count_held(unsigned long long* counter, unsigned long long n) {
    if (!counter) return;
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    if ((threadIdx.x & 63) == 0 && n) atomicAdd(counter, n);
}

// The tetrahedron of part P that holds p (-1: none), by the BVH: from the
// root, a node whose box holds p is entered (its first child follows it; a
// leaf's tetrahedra are tested), any other is skipped through its skip link.
// (A leaf's tetrahedra by the float32 planes first: with the float64 ones alone,
// 128 bytes a test for 48, frames took 1.2 to 1.3 times as long.)
__device__ inline int bvh_locate(const TetPartK& P, double p0, double p1, double p2) {
    const float x0 = (float)(p0 - P.glo[0]), x1 = (float)(p1 - P.glo[1]), x2 = (float)(p2 - P.glo[2]);
    double D[4];
    int node = P.n_tets > 0 ? 0 : -1;
    while (node >= 0) {
        gint* nd = ((gint*)P.bvh_nodes) + 8 * (long long)node;
        const int skip = nd[3], leaf = nd[7];
        const bool in = p0 >= (double)__int_as_float(nd[0]) && p1 >= (double)__int_as_float(nd[1]) &&
                        p2 >= (double)__int_as_float(nd[2]) && p0 <= (double)__int_as_float(nd[4]) &&
                        p1 <= (double)__int_as_float(nd[5]) && p2 <= (double)__int_as_float(nd[6]);
        if (!in) {
            node = skip;
        } else if (leaf >= 0) {
            const int first = leaf >> 3, count = leaf & 7;
            for (int i = 0; i < count; ++i) {
                const int e = ((gint*)P.bvh_tets)[first + i];
                gfloat4* rec = ((gfloat4*)P.planes32) + 3 * (long long)e;
                const float4_t pl[3] = {rec[0], rec[1], rec[2]};
                int face = reject_face32(P, pl, x0, x1, x2);
                if (face == kUndecided) face = reject_face(P, e, p0, p1, p2, D);
                if (face < 0) return e;
            }
            node = skip;
        } else {
            node = node + 1;
        }
    }
    return -1;
}

// Value of a point in tetrahedron e: the affine function of the part's
// records (x: the point relative to the grid origin), in float64.  Where a
// vertex value is not finite the record is NaN and the barycentric sum of
// the sub-volumes of p takes its place.
__device__ inline float tet_value(const TetPartK& P, int e, const double x[3], const double p[3]) {
#pragma clang fp contract(off)
    gdouble2* rec = ((gdouble2*)P.affine) + e;
    const double2_t a = rec[0], b = rec[P.n_tets];
    const double v = ((a.x * x[0] + a.y * x[1]) + b.x * x[2]) + b.y;
    if (v == v) return (float)v;
    double D[4];
    (void)reject_face(P, e, p[0], p[1], p[2], D);
    const float4_t w = ((gfloat4*)P.vals)[e];
    const double s = ((D[0] + D[1]) + D[2]) + D[3];
    const double num = ((D[0] * (double)w.x + D[1] * (double)w.y) + D[2] * (double)w.z) + D[3] * (double)w.w;
    return __fdividef((float)num, (float)s);
}

// The records of a part's affine values: value(x) = g . x + c with x
// relative to the grid origin, from the planes and the vertex values
// (v0 + sum (v_i - v0) D_i(x) / sum D_i; the D_i sum to the same volume at
// every x).  Bound by memory: 176 bytes a tetrahedron.  Once per time step of a
// part: 2.0 M tetrahedra in one part, setting the values 17 us without the
// records, 77 with them (8 parts 47 and 117), for a 1280x720 frame of 2.35 ms
// before and 0.72 now (3.9 and 1.7), 96x72 pixels of 246 K 1.30 and 0.27.
__global__ __launch_bounds__(256) void tet_affine(TetPartK P, double2_t* __restrict__ out) {
#pragma clang fp contract(off)
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= P.n_tets) return;
    gdouble2* pl = ((gdouble2*)P.planes) + 8 * (long long)e;
    const float4_t v = ((gfloat4*)P.vals)[e];
    double n[4][3], d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double2_t a = pl[2 * i], b = pl[2 * i + 1];
        n[i][0] = a.x;
        n[i][1] = a.y;
        n[i][2] = b.x;
        d[i] = ((a.x * P.glo[0] + a.y * P.glo[1]) + b.x * P.glo[2]) - b.y;   // D_i at x = 0
    }
    const double S = ((d[0] + d[1]) + d[2]) + d[3];
    const double w[3] = {((double)v.y - (double)v.x) / S, ((double)v.z - (double)v.x) / S,
                         ((double)v.w - (double)v.x) / S};
    double g[3], c = (double)v.x;
#pragma unroll
    for (int a = 0; a < 3; ++a) g[a] = (w[0] * n[1][a] + w[1] * n[2][a]) + w[2] * n[3][a];
    c += (w[0] * d[1] + w[1] * d[2]) + w[2] * d[3];
    const float all = ((v.x - v.x) + (v.y - v.y)) + ((v.z - v.z) + (v.w - v.w));   // NaN unless all are finite
    if (!(all == 0.0f)) c = __builtin_nan("");
    out[e] = double2_t{g[0], g[1]};
    out[(long long)P.n_tets + e] = double2_t{g[2], c};
}

// The samples k0 .. k1 (none if k1 < k0; k0 >= 0, fewer than 2^31 of them) of
// ray r in part P, in order: held(k, value) for a sample that a tetrahedron
// holds, gap() for a stretch of samples that none holds; k is a double (exact;
// a shadow ray may meet a part after more than 2^31 samples).  A sample is
// sought by a walk from the previous sample's tetrahedron (kWalkSteps tests,
// each step across the face that rejects it most), then among the tetrahedra
// listed in its grid cell (or in the BVH).
//
// Vector-memory instructions bound this (a 16-byte load of 64 scattered lanes
// takes the L1 33 to 65 cycles, 17 where four neighbouring lanes share a
// line; measured), so a test reads 48 bytes of float32 barycentric planes and
// only a sample that they leave undecided reads the 128 bytes of float64 ones.
// A loop trip waits once: it issues what every lane needs next -- one 16-byte
// load per lane of its tetrahedron's neighbours, its list's next candidates or
// its cell's head, and the planes -- and then settles what it can.  Every
// lane is at its own sample: one whose sample is settled goes on while others
// still search (with the lanes in step, a wavefront took the longest search
// of its 64 lanes at every sample).  A sample in an empty cell, d cells from
// the nearest listed one, also settles the following ones that stay within
// d - 1 cells of it.
//
// The BVH's lanes wait for each other instead, since a search of the hierarchy
// costs by the nodes that any lane of the wavefront meets: kInStep, every lane at
// its next sample; else a lane waits until none of the wavefront walks, and all
// waiting ones search at once.  In step takes 0.84 to 0.92 of the time of waiting
// where tiles go to a wavefront each (24^3 to 128 x 96 x 96 cells in 3 to 16 parts,
// 28000 tiles and more; one part of 80 x 64 x 64 1.27), 0.98 to 1.56 in stretches.
// One lane a ray with float64 planes, then waiting with them in the leaves, and
// as here: 7.1 M in 16 parts at 1920x1080 35.5, 39.4 and 28.6 ms, 2.0 M in 16 at
// 2560x1440 27.1, 34.6 and 25.6, 83 K in 6 at 2560x1440 5.69, 6.96 and 5.33.
template <int kLocator, bool kValues, bool kInStep, typename Held, typename Gap>
__device__ __forceinline__ void walk_part(const TetPartK& P, const CamRay& r, double dt, long long k0, long long k1,
                                          Held held, Gap gap) {
#pragma clang fp contract(off)
    double k = (double)k0;
    int left = k1 >= k0 ? (int)(k1 - k0) : -1;           // samples after this one
    int cand = -1;                                       // tetrahedron to test (-1: look the sample's cell up)
    int walk = 0;                                        // walk steps left (0: cand is from the cell's list)
    int next = -1, q = 0, qend = 0;                      // the list's candidate after cand, and the rest [q, qend)
    const int cells = P.gdim[0] * P.gdim[1] * P.gdim[2];
    // (0.999: below the true ratio whatever the rounding)
    const double move = fmax(fmax(fabs(r.d[0] * dt * P.ginv[0]), fabs(r.d[1] * dt * P.ginv[1])),
                             fabs(r.d[2] * dt * P.ginv[2]));     // cells per sample, at most
    const float per_cell = (float)fmin(0.999 / move, 1e6);       // samples per cell moved
    double x[3];                                         // the sample relative to the grid origin
    auto point = [&](double p[3]) {
        const double t = (k + 0.5) * dt;
        for (int c = 0; c < 3; ++c) p[c] = r.o[c] + t * r.d[c];
    };
    auto place = [&]() {
        double p[3];
        point(p);
        for (int c = 0; c < 3; ++c) x[c] = p[c] - P.glo[c];
    };
    if constexpr (kLocator == kTetBvh && kInStep) {
        for (; left >= 0; --left, k += 1.0) {
            double p[3], D[4];
            place();
            point(p);
            int found = -1;
            for (walk = kWalkSteps; cand >= 0;) {
                const int4_t aux = *(gint4_unaligned*)((gint*)P.nbr + 4 * (long long)cand);
                gfloat4* rec = ((gfloat4*)P.planes32) + 3 * (long long)cand;
                const float4_t pl[3] = {rec[0], rec[1], rec[2]};
                int face = reject_face32(P, pl, (float)x[0], (float)x[1], (float)x[2]);
                if (face == kUndecided) face = reject_face(P, cand, p[0], p[1], p[2], D);
                if (face < 0) {
                    found = cand;
                    break;
                }
                cand = --walk > 0 ? (face == 0 ? aux.x : face == 1 ? aux.y : face == 2 ? aux.z : aux.w) : -1;
            }
            if (found < 0) found = bvh_locate(P, p[0], p[1], p[2]);
            if (found >= 0) held(k, kValues ? tet_value(P, found, x, p) : 0.0f);
            else gap();
            cand = found;
        }
        return;
    }
    place();
    while (left >= 0) {
        const bool walking = kLocator == kTetBvh && __any(cand >= 0);
        int settle = 0;                                  // samples to go on by
        int found = -1;
        // (a point outside the grid takes the head after the last cell's, of
        // an empty cell; one less than a cell below the grid looks cell 0 up,
        // whose tetrahedra reject it)
        gint* src = (gint*)P.cell_head;
        float4_t pl[3];
        if (cand >= 0) {
            src = walk > 0 ? (gint*)P.nbr + 4 * (long long)cand : (gint*)P.cell_tets + q;
            gfloat4* rec = ((gfloat4*)P.planes32) + 3 * (long long)cand;
#pragma unroll
            for (int i = 0; i < 3; ++i) pl[i] = rec[i];
        } else if (kLocator == kTetGrid) {
            const int c0 = (int)(x[0] * P.ginv[0]), c1 = (int)(x[1] * P.ginv[1]), c2 = (int)(x[2] * P.ginv[2]);
            const bool in = ((unsigned)c0 < (unsigned)P.gdim[0]) & ((unsigned)c1 < (unsigned)P.gdim[1]) &
                            ((unsigned)c2 < (unsigned)P.gdim[2]);
            src += 4 * (long long)(in ? (c2 * P.gdim[1] + c1) * P.gdim[0] + c0 : cells);
        }
        const int4_t aux = *(gint4_unaligned*)src;
        if (cand >= 0) {
            int face = reject_face32(P, pl, (float)x[0], (float)x[1], (float)x[2]);
            if (face == kUndecided) {
                double p[3], D[4];
                point(p);
                face = reject_face(P, cand, p[0], p[1], p[2], D);
            }
            if (face < 0) {
                found = cand;
                settle = 1;
            } else if (walk > 0) {
                cand = --walk > 0 ? (face == 0 ? aux.x : face == 1 ? aux.y : face == 2 ? aux.z : aux.w) : -1;
            } else {
                cand = next;
                next = q < qend ? aux.x : -1;
                ++q;
                if (cand < 0) settle = 1;                // the cell's list is through
            }
        } else if (kLocator == kTetBvh) {
            // (once every lane waits for it: the hierarchy is searched by all of
            // them at once)
            if (!walking) {
                double p[3];
                point(p);
                found = bvh_locate(P, p[0], p[1], p[2]);
                settle = 1;
            }
        } else if (aux.x < 0) {
            settle = 1 + (int)((float)(-aux.x - 1) * per_cell);
        } else {
            cand = aux.x;
            next = aux.y;
            walk = 0;
            q = aux.z;
            qend = aux.w;
        }
        if (settle > 0) {
            if (found >= 0) {
                float v = 0.0f;
                if (kValues) {
                    double p[3];
                    point(p);
                    v = tet_value(P, found, x, p);
                }
                held(k, v);
            } else {
                gap();
            }
            cand = found;
            walk = kWalkSteps;
            q = qend;
            k += (double)settle;
            left = settle > left ? -1 : left - settle;
            place();
        }
    }
}

// A tile's rays are cut into kStretches stretches of equal length, which the
// kWaves wavefronts of its workgroup take one after another: a wavefront
// alone waits for its slowest ray through every search, and a small frame has
// too few tiles to fill the GPU.  (One fixed stretch per wavefront leaves most
// of them idle: a part fills its bounding box unevenly.)  The stretches' runs
// wait in a pool of kPool entries in LDS, chained per ray and stretch, and are
// joined in order afterwards.  (A tile that needs more is taken again by one
// wavefront: 32 layers of cells in turn from two parts, 16 runs a ray and part,
// 2.95 ms, 2.36 with one lane a ray in step; 16 layers fit, 0.38 and 1.07 ms.
// Four wavefronts taking 16 rays each: 2.73, but 48 layers 4.43 against 4.28.)
constexpr int kWaves = 4;
constexpr int kStretches = 8;
constexpr int kPool = 704;

// Part and ROI pixel of this thread (its lane) in tile `wg` of the frame's
// tiles.  A part's tiles are numbered down the columns of bands 8 tiles high,
// so that tiles in flight together are a compact block of the image whose
// rays share tetrahedra.  (Giving each XCD runs of 64 consecutive tiles cut
// the L2 misses to a sixth but left the XCDs unevenly loaded: 2.18 against
// 1.85 ms for 2.0 M tetrahedra at 1280x720.)
__device__ inline int tile_pixel(const TetFrameParams& f, int wg, int& lx, int& ly) {
    int lo = 0, hi = f.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (f.tile_start[mid] <= wg) lo = mid; else hi = mid - 1;
    }
    const int j = uniform_i(lo);
    const int tile = wg - uniform_i(f.tile_start[j]);
    const TetPartK& P = const_entry(f.parts, j);
    const int tiles_x = (P.roi_w + kTetTile - 1) / kTetTile, tiles_y = (P.roi_h + kTetTile - 1) / kTetTile;
    const int band = tile / (8 * tiles_x), r = tile - band * 8 * tiles_x;
    const int rows = min(8, tiles_y - 8 * band);
    const int lane = threadIdx.x & 63;
    // lanes in Z order: four consecutive lanes are 2 x 2 pixels
    lx = r / rows * kTetTile + ((lane & 1) | (lane >> 1 & 2) | (lane >> 2 & 4));
    ly = (8 * band + r % rows) * kTetTile + ((lane >> 1 & 1) | (lane >> 2 & 2) | (lane >> 3 & 4));
    return j;
}

// The march of every part's ROI rays, in one of four modes: kTetMarch
// (runs), kTetCount (held samples per frame entry into offsets), kTetRecord
// (the sample index of every held sample into its slot) and kTetShaded (runs
// with every held sample's emission scaled by a0 + (1 - a0) S from its slot).
template <int kMode>
constexpr bool tet_runs() { return kMode == kTetMarch || kMode == kTetShaded; }

// kAlone: every wavefront takes a tile of its own, its rays whole (api.cpp's
// tet_alone chooses).
template <int kMode, int kLocator, bool kAlone>
__global__ __launch_bounds__(tet_runs<kMode>() ? 64 * kWaves : 64, 5) void tet_march(TetFrameParams f) {
    constexpr bool kRuns = tet_runs<kMode>();
    constexpr bool kPooled = kRuns && !kAlone;
    __shared__ TFTable tft;
    __shared__ int run_key[kPooled ? kPool : 1], run_end[kPooled ? kPool : 1];
    __shared__ float run_rgb[kPooled ? 3 * kPool : 1], run_T[kPooled ? kPool : 1];
    __shared__ short run_next[kPooled ? kPool : 1];
    __shared__ short first_run[kPooled ? kStretches * 64 : 1];
    __shared__ int pool_used, taken;
    const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
    if (kRuns) {
        load_tf(tft, f.tf, f.dt, threadIdx.x, 64 * kWaves);
        if (kPooled && threadIdx.x == 0) {
            pool_used = 0;
            taken = kWaves;
        }
        __syncthreads();
    }
    int lx, ly;
    const int tile = f.tile0 + (kRuns && kAlone ? kWaves * (int)blockIdx.x + wave : (int)blockIdx.x);
    const int j = tile_pixel(f, min(tile, f.total_tiles - 1), lx, ly);
    const TetPartK& P = const_entry(f.parts, j);
    const bool live = lx < P.roi_w && ly < P.roi_h && tile < f.total_tiles;
    const long long npix = (long long)P.roi_w * P.roi_h;
    const long long li = (long long)ly * P.roi_w + lx;
    const float tf_k = 255.0f / (f.tf.vmax - f.tf.vmin);
    const float tf_o = -f.tf.vmin * tf_k;
    const float a0 = f.ambient, a1 = 1.0f - f.ambient;
    long long k0 = 0, k1 = -1, slot0 = 0, slots = 0;
    CamRay r{};
    if (live) {
        r = camera_ray(f.cam, P.roi_x0 + lx, P.roi_y0 + ly);
        if (box_range(r, P.lo, P.hi, f.dt, k0, k1) && k1 > 0x7fffffffLL) {
            if (f.err) atomicOr(f.err, kErrRange);
            k1 = k0 - 1;
        }
        if (kMode == kTetRecord || kMode == kTetShaded) {
            slot0 = f.offsets[P.entry0 + li];
            slots = f.offsets[P.entry0 + li + 1] - slot0;   // the count pass's held samples of this ray
        }
    }
    if constexpr (!kRuns) {
        unsigned long long held = 0;
        walk_part<kLocator, false, true>(P, r, f.dt, k0, k1, [&](double k, float) {
            // the passes locate alike, so a ray holds as many samples as
            // counted; a mismatch (which only a logic error could cause) is
            // reported and never writes outside the ray's slots
            if (kMode == kTetRecord) {
                if ((long long)held < slots) f.slot_k[slot0 + (long long)held] = (int)k;
                else if (f.err) atomicOr(f.err, kErrRange);
            }
            ++held;
        }, []() {});
        if (kMode == kTetCount && live) f.offsets[P.entry0 + li] = (long long)held;
        return;
    }
    auto store = [&](int n, int key, float c0, float c1, float c2, float T) {
        const long long q = (long long)n * npix + li;
        P.rkey[q] = key;
        reinterpret_cast<float4*>(P.rcol)[q] = make_float4(c0, c1, c2, 1.0f - T);
    };
    unsigned long long held = 0, counted = 0;   // of a stretch, of all that this wavefront took
    int nrun = 0;
    bool overflow = false;
    // the stretches of this wavefront; should the pool not hold the tile's
    // runs, wavefront 0 takes its rays again, whole, and stores their runs as
    // they end
    bool whole = kAlone;
    for (int piece = wave;;) {
        const long long n = k1 - k0 + 1;
        long long ka = k0 + n * piece / kStretches, kb = k0 + n * (piece + 1) / kStretches - 1;
        if (whole) {
            ka = k0;
            kb = k1;
        }
        long long slot = slot0;                 // of this stretch's first held sample: slots are in sample order
        if (kMode == kTetShaded && ka > k0) {
            long long lo = 0, hi = slots;
            while (lo < hi) {
                const long long mid = (lo + hi) >> 1;
                if ((long long)f.slot_k[slot0 + mid] < ka) lo = mid + 1; else hi = mid;
            }
            slot += lo;
        }
        held = 0;
        nrun = 0;
        int first = -1, last = -1;              // this stretch's chain
        bool in_run = false;
        int key = 0, end = 0;
        float C0 = 0.f, C1 = 0.f, C2 = 0.f, T = 1.f;
        auto close_run = [&]() {
            if (whole) {
                if (nrun < f.max_runs) store(nrun, key, C0, C1, C2, T);
                else overflow = true;
            } else {
                const int i = atomicAdd(&pool_used, 1);
                if (i < kPool) {
                    run_key[i] = key;
                    run_end[i] = end;
                    run_rgb[3 * i] = C0;
                    run_rgb[3 * i + 1] = C1;
                    run_rgb[3 * i + 2] = C2;
                    run_T[i] = T;
                    run_next[i] = -1;
                    if (last >= 0) run_next[last] = (short)i;
                    else first = i;
                    last = i;
                }
            }
            ++nrun;
            in_run = false;
        };
        walk_part<kLocator, true, kAlone>(P, r, f.dt, ka, kb, [&](double sample, float v) {
#pragma clang fp contract(off)
            const int k = (int)sample;
            if (!in_run) {
                in_run = true;
                key = k;
                C0 = C1 = C2 = 0.f;
                T = 1.f;
            }
            end = k;
            const Classified c = classify(tft, v, tf_k, tf_o);
            float sh = 1.0f;
            if (kMode == kTetShaded) {
                const long long q = slot + (long long)held;
                sh = a0 + a1 * (q < slot0 + slots ? f.shade[q] : 1.0f);
            }
            const float Tn = T * trans_exp2(-c.a);
            const float w = T - Tn;
            C0 = fmaf(w, c.r * sh, C0);
            C1 = fmaf(w, c.g * sh, C1);
            C2 = fmaf(w, c.b * sh, C2);
            T = Tn;
            ++held;
        }, [&]() {
            if (in_run) close_run();
        });
        if (in_run) close_run();
        counted += held;
        if (kAlone || whole) break;
        first_run[piece * 64 + lane] = (short)first;
        if (lane == 0) piece = atomicAdd(&taken, 1);
        piece = uniform_i(piece);
        if (piece < kStretches) continue;
        __syncthreads();
        whole = uniform_i(pool_used) > kPool;
        if (!whole || wave > 0) break;
        counted = 0;
    }
    if (!kAlone && whole && wave > 0) counted = 0;
    if ((kAlone || wave == 0) && live) {
        if (!whole) {
            // join the stretches: a run that goes on in the next one is one run
            nrun = 0;
            bool open = false;
            int key = 0, end = 0;
            float C0 = 0.f, C1 = 0.f, C2 = 0.f, T = 1.f;
            auto put = [&]() {
                if (nrun < f.max_runs) {
                    store(nrun, key, C0, C1, C2, T);
                    ++nrun;
                } else {
                    overflow = true;
                }
            };
            for (int s = 0; s < kStretches; ++s) {
                for (int i = first_run[s * 64 + lane]; i >= 0; i = run_next[i]) {
                    const int nk = run_key[i];
                    const float n0 = run_rgb[3 * i], n1 = run_rgb[3 * i + 1], n2 = run_rgb[3 * i + 2];
                    if (open && nk == end + 1) {
                        C0 = fmaf(T, n0, C0);
                        C1 = fmaf(T, n1, C1);
                        C2 = fmaf(T, n2, C2);
                        T *= run_T[i];
                    } else {
                        if (open) put();
                        open = true;
                        key = nk;
                        C0 = n0;
                        C1 = n1;
                        C2 = n2;
                        T = run_T[i];
                    }
                    end = run_end[i];
                }
            }
            if (open) put();
        }
        P.rcount[li] = min(nrun, f.max_runs);
        if (overflow && f.err) atomicOr(f.err, kErrRuns);
    }
    count_held(f.samples, counted);
}

// The shadow rays of one tile of a home part's ROI (the tiles of the march):
// the ray of every held primary sample (its slot) cycles through the parts
// home, home + 1, ... (mod n), multiplying its transmittance by each one's.  A
// lane takes every split-th held sample of its pixel (split: the wavefronts of
// a tile, from its wavefront's place among them), so that a wavefront's 64 rays
// start at the same depth behind 8 x 8 neighbouring pixels and cross the same
// tetrahedra; with the lanes on 64 consecutive samples of one primary ray their
// loads touched as many lines as lanes.
constexpr int kMaxShadowSplit = 256;

template <int kLocator>
__global__ __launch_bounds__(256, 5) void tet_shadow(TetFrameParams f) {
    __shared__ TFTable tft;
    load_tf(tft, f.tf, f.dt, threadIdx.x, 256);
    __syncthreads();
    const float tf_k = 255.0f / (f.tf.vmax - f.tf.vmin);
    const float tf_o = -f.tf.vmin * tf_k;
    int lx, ly;
    const int j = tile_pixel(f, f.tile0 + (int)blockIdx.x, lx, ly);
    const TetPartK& home = const_entry(f.parts, j);
    const bool live = lx < home.roi_w && ly < home.roi_h;
    long long slot0 = 0, slots = 0;
    CamRay cr{};
    if (live) {
        const long long e = home.entry0 + (long long)ly * home.roi_w + lx;
        slot0 = f.offsets[e];
        slots = f.offsets[e + 1] - slot0;
        cr = camera_ray(f.cam, home.roi_x0 + lx, home.roi_y0 + ly);
    }
    unsigned long long evaluated = 0;
    for (long long i = 4 * blockIdx.y + (threadIdx.x >> 6); i < slots; i += 4 * gridDim.y) {
        CamRay sr;
        {
#pragma clang fp contract(off)
            const double t = ((double)f.slot_k[slot0 + i] + 0.5) * f.dt;
            for (int a = 0; a < 3; ++a) {
                sr.o[a] = cr.o[a] + t * cr.d[a];
                sr.d[a] = f.light[a];
            }
        }
        float all = 1.0f;
        for (int s = 0; s < f.n; ++s) {
            int h = j + s;
            h = h >= f.n ? h - f.n : h;
            const TetPartK& at = const_entry(f.parts, h);
            float S = 1.0f;
            long long j0 = 0, j1 = -1;
            if (at.n_tets > 0 && box_range(sr, at.lo, at.hi, f.dt, j0, j1) && j1 - j0 > 0x7ffffffeLL) {
                if (f.err) atomicOr(f.err, kErrRange);
                j1 = j0 - 1;
            }
            walk_part<kLocator, true, false>(at, sr, f.dt, j0, j1, [&](double, float v) {
                S = S * trans_exp2(-classify(tft, v, tf_k, tf_o).a);
                ++evaluated;
            }, []() {});
            all = s == 0 ? S : all * S;
        }
        f.shade[slot0 + i] = all;
    }
    count_held(f.samples, evaluated);
}

// Per pixel: the runs of every part whose ROI holds the pixel, merged by
// first sample index (each part's runs are already in ray order), each
// "over" the result so far, then over the background.
__global__ __launch_bounds__(256) void tet_resolve(TetFrameParams f) {
    __shared__ uint8_t head[kMaxTetParts * 256];
    const int tid = threadIdx.x;
    for (int q = 0; q < f.n; ++q) head[q * 256 + tid] = 0;
    const long long npx = (long long)f.width * f.height;
    const long long pix = (long long)blockIdx.x * 256 + tid;
    if (pix >= npx) return;
    const int px = (int)(pix % f.width), py = (int)(pix / f.width);
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, A = 0.f;
    for (;;) {
        int best = 0x7fffffff, bq = -1;
        long long bslot = 0;
        for (int q = 0; q < f.n; ++q) {
            const TetPartK& P = f.parts[q];
            const int lx = px - P.roi_x0, ly = py - P.roi_y0;
            if (lx < 0 || ly < 0 || lx >= P.roi_w || ly >= P.roi_h) continue;
            const long long li = (long long)ly * P.roi_w + lx;
            const int h = head[q * 256 + tid];
            if (h >= min(P.rcount[li], f.max_runs)) continue;
            const long long slot = (long long)h * P.roi_w * P.roi_h + li;
            const int k = P.rkey[slot];
            if (k < best) {
                best = k;
                bq = q;
                bslot = slot;
            }
        }
        if (bq < 0) break;
        const float4 c = reinterpret_cast<const float4*>(f.parts[bq].rcol)[bslot];
        const float w = 1.0f - A;
        C0 = fmaf(w, c.x, C0);
        C1 = fmaf(w, c.y, C1);
        C2 = fmaf(w, c.z, C2);
        A = fmaf(w, c.w, A);
        ++head[bq * 256 + tid];
    }
    const float w = 1.0f - A;
    reinterpret_cast<float4*>(f.out)[pix] =
        make_float4(fmaf(w, f.bg[0], C0), fmaf(w, f.bg[1], C1), fmaf(w, f.bg[2], C2), fmaf(w, f.bg[3], A));
}

// Wavefronts per tile of the shadow rays: 6 for each held sample of the ROIs'
// mean pixel (24 where tiles are few, and the GPU waits for the fullest pixel), at
// most kMaxShadowSplit (a lane past its pixel's samples only loads the table, but
// a pixel may hold many times the mean).  Always 256, a frame of short rays spent
// its time on workgroups without work: 16^3 cells in 4 parts at 800x600, step 8,
// 1571 us, 289 so; step 0.5 4.51 and 3.46 ms; 40^3 in 4 parts at 384x288, step 0.5,
// 5.48 and 5.45 (2.5 a sample: 5.66).  27 x 23 x 17 in 4 parts at 172x135, step
// 0.5, 1.41 ms at 256, 1.60 at 6 a sample.
int shadow_split(const TetFrameParams& p) {
    const double mean = (double)p.total / ((double)kTetTile * kTetTile * p.total_tiles);
    const double each = p.total_tiles < 1024 ? 24.0 : 6.0;
    return 4 * (int)std::min(kMaxShadowSplit / 4.0, 1.0 + std::ceil(each * mean / 4.0));
}

template <int kLocator>
void launch_tet_stages(TetFrameParams p, int stages, hipStream_t stream) {
    const dim3 one(64), threads(64 * kWaves);
    auto pieces = [&](auto launch) {
        for (p.tile0 = 0; p.tile0 < p.total_tiles; p.tile0 += kMaxLaunchTiles)
            launch(min(p.total_tiles - p.tile0, kMaxLaunchTiles));
    };
    if (stages & kTetCount)
        pieces([&](int n) { hipLaunchKernelGGL((tet_march<kTetCount, kLocator, true>), dim3(n), one, 0, stream, p); });
    if (stages & kTetRecord)
        pieces([&](int n) { hipLaunchKernelGGL((tet_march<kTetRecord, kLocator, true>), dim3(n), one, 0, stream, p); });
    if ((stages & kTetShadow) && p.total > 0)
        pieces([&](int n) {
            hipLaunchKernelGGL(tet_shadow<kLocator>, dim3(n, shadow_split(p) / 4), dim3(256), 0, stream, p);
        });
    auto runs = [&](auto pooled, auto alone) {
        pieces([&](int n) {
            if (p.alone) hipLaunchKernelGGL(alone, dim3((n + kWaves - 1) / kWaves), threads, 0, stream, p);
            else hipLaunchKernelGGL(pooled, dim3(n), threads, 0, stream, p);
        });
    };
    if (stages & kTetMarch) runs(tet_march<kTetMarch, kLocator, false>, tet_march<kTetMarch, kLocator, true>);
    if (stages & kTetShaded) runs(tet_march<kTetShaded, kLocator, false>, tet_march<kTetShaded, kLocator, true>);
}

}  // namespace

hipError_t launch_tet_values(const float* vertex_values, int32_t n_input, const int32_t* centre_nodes,
                             const int32_t* tets, int32_t n_tets, float* vals, hipStream_t stream) {
    if (n_tets <= 0) return hipSuccess;
    hipLaunchKernelGGL(tet_values, dim3((n_tets + 255) / 256), dim3(256), 0, stream, vertex_values, n_input,
                       centre_nodes, reinterpret_cast<const int4*>(tets), n_tets, reinterpret_cast<float4*>(vals));
    return hipGetLastError();
}

hipError_t launch_tet_frame(TetFrameParams p, int stages, hipStream_t stream) {
    if (stages == kTetAffine) {
        if (p.one.n_tets > 0)
            hipLaunchKernelGGL(tet_affine, dim3((p.one.n_tets + 255) / 256), dim3(256), 0, stream, p.one,
                               reinterpret_cast<double2_t*>(const_cast<double*>(p.one.affine)));
        return hipGetLastError();
    }
    if (p.locator == kTetBvh)
        launch_tet_stages<kTetBvh>(p, stages, stream);
    else
        launch_tet_stages<kTetGrid>(p, stages, stream);
    const long long npx = (long long)p.width * p.height;
    if (stages & kTetResolve)
        hipLaunchKernelGGL(tet_resolve, dim3((unsigned)((npx + 255) / 256)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace dpvr
