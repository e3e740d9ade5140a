// Ray-queue cycling (RQC) on one GPU, with shadow rays.
//
// The bricks play the ranks of a data-parallel renderer: every ray is
// traced through every brick's data by cycling ray queues from brick to
// brick, so the data never moves and its decomposition can be arbitrary.
// One directional light: each primary sample's emitted colour is scaled by
// a0 + (1 - a0) S, S the transmittance of its shadow ray toward the light,
// which has to visit the bricks that hold the occluders.
//
// A frame, for n bricks (ranks) and the context camera:
//   plan      one entry per (brick b, ROI pixel of b): the first owned sample
//             index of the pixel's ray in b and the number of owned samples;
//             an exclusive scan gives every owned primary sample a slot.
//   shadow    the shadow rays spawned by the samples that brick b owns form
//             b's queue, which cycles through bricks b, b + 1, ... (mod n),
//             multiplying each ray's transmittance in its slot (one launch:
//             on one GPU a cycle step is a change of which brick is read).
//   primary   the primary ray of every pixel through every brick, giving the
//             segment (premultiplied colour, alpha, depth key) of the samples
//             that brick owns, with the shaded emission; segments go to the
//             pixel's slot of that brick.
//   resolve   per pixel, the n segments in (key, brick index) order with
//             "over", then the background.
// For emission-absorption on disjoint bricks this equals sort-last
// compositing of per-brick partials: with shadows off (a0 = 1) every segment
// is bit-identical to the brick's partial pixel and the resolve repeats the
// composite's arithmetic, so the image equals the sort-last image exactly.
#include "march_common.h"

#include <algorithm>
#include <cmath>

namespace dpvr {
namespace {

constexpr int kScanBlock = 1024;     // elements per workgroup of the scan (256 threads x 4)

// Brick of an entry: the largest b with entry0[b] <= e.
__device__ inline int brick_of_entry(const RqcParams& p, long long e) {
    int lo = 0, hi = p.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.bricks[mid].entry0 <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Adds every lane's n to *counter (one atomic per wavefront); all lanes of
// the wavefront must call it.
__device__ inline void count_samples(unsigned long long* counter, unsigned long long n) {
    if (!counter) return;
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    if ((threadIdx.x & 63) == 0 && n) atomicAdd(counter, n);
}

// ----------------------------------------------------------------- plan
__global__ __launch_bounds__(256) void rqc_count(RqcParams p) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= p.n_entries) return;
    const int b = brick_of_entry(p, e);
    const RqcBrick& rb = p.bricks[b];
    const long long r = e - rb.entry0;
    const int px = rb.roi_x0 + (int)(r % rb.roi_w), py = rb.roi_y0 + (int)(r / rb.roi_w);
    RaySetup rs;
    long long cnt = 0;
    int kf = -1;
    if (setup_ray(p.cam, rb.brick, p.dt, px, py, rs)) {
        if (rs.kl > 0x7fffffffLL) {
            if (p.err) atomicOr(p.err, kErrRange);
        } else {
            cnt = rs.kl - rs.kf + 1;
            kf = (int)rs.kf;
        }
    }
    p.kf[e] = kf;
    p.offsets[e] = cnt;
}

// Exclusive scan of offsets[0 .. n) in place (offsets[n] = total), in three
// launches: per-block scans with block totals, a scan of the totals, and the
// block carries added back.
__global__ __launch_bounds__(256) void scan_blocks(long long* v, long long n, long long* sums) {
    __shared__ long long s[256];
    const long long base = (long long)blockIdx.x * kScanBlock + threadIdx.x * 4;
    long long x[4], run = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = base + i < n ? v[base + i] : 0;
        run += x[i];
    }
    s[threadIdx.x] = run;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {      // inclusive scan of the thread totals
        const long long add = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += add;
        __syncthreads();
    }
    long long acc = s[threadIdx.x] - run;          // exclusive prefix of this thread
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (base + i < n) v[base + i] = acc;
        acc += x[i];
    }
    if (threadIdx.x == 255) sums[blockIdx.x] = s[255];
}

__global__ __launch_bounds__(256) void scan_sums(long long* sums, long long nb, long long* total) {
    __shared__ long long s[256];
    __shared__ long long carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (long long b0 = 0; b0 < nb; b0 += 256) {
        const long long i = b0 + threadIdx.x;
        const long long x = i < nb ? sums[i] : 0;
        s[threadIdx.x] = x;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const long long add = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
            __syncthreads();
            s[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nb) sums[i] = carry + s[threadIdx.x] - x;
        __syncthreads();
        if (threadIdx.x == 255) carry += s[255];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(256) void scan_add(long long* v, long long n, const long long* sums) {
    const long long i = (long long)blockIdx.x * kScanBlock + threadIdx.x;
    const long long c = sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i + k * 256 < n) v[i + k * 256] += c;
}

// ------------------------------------------------------ one brick's samples
// The 8 corner values of cell c, in lerp3's order.
template <typename TS>
__device__ inline void corners(const TS* __restrict__ vox, const Cell& c, int pitch, long long sxy, float (&v)[8]) {
    const long long base = (long long)c.iz * sxy + (long long)c.iy * pitch + c.ix;
    v[0] = ld(vox, base);
    v[1] = ld(vox, base + 1);
    v[2] = ld(vox, base + pitch);
    v[3] = ld(vox, base + pitch + 1);
    v[4] = ld(vox, base + sxy);
    v[5] = ld(vox, base + sxy + 1);
    v[6] = ld(vox, base + sxy + pitch);
    v[7] = ld(vox, base + sxy + pitch + 1);
}

// The samples kf .. kl of ray rs in a brick (wavefront-uniform), block by
// block as the partial march takes them (same anchors, same float32
// positions, same trilinear arithmetic), each passed to fn(k, value).  Two
// samples' corner loads are in flight together.  bl, st: the ray's anchor
// blocks and step.  Returns false if fn stops the walk.
template <typename TS, typename Fn>
__device__ __forceinline__ bool walk_rows(const BrickK& b, double dt, double inv_dt, const RaySetup& rs,
                                          const Blocks& bl, const Step& st, Fn fn) {
    const Rows<TS> rows = make_rows<TS>(b);
    long long n = block_of(bl, dt, inv_dt, rs.kf);
    long long k = rs.kf;
    while (k <= rs.kl) {
        const long long kend = min(block_start(bl, inv_dt, n + 1) - 1, rs.kl);
        if (kend >= k) {
            const Anchor an = make_anchor(rs, b, dt, k);
            const unsigned base = anchor_offset(rows, an);
            const int m = (int)(kend - k) + 1;
            for (int j = 0; j < m; j += 2) {
                const Spot s0 = locate_rows(rows, base, an, st, (float)j);
                const Spot s1 = locate_rows(rows, base, an, st, (float)(j + 1));
                const Corners<TS> c0 = gather_rows(rows, s0.off);
                const Corners<TS> c1 = gather_rows(rows, s1.off);
                __builtin_amdgcn_sched_barrier(0);
                if (!fn(k + j, lerp_rows(s0, c0))) return false;
                if (j + 1 < m && !fn(k + j + 1, lerp_rows(s1, c1))) return false;
            }
            k = kend + 1;
        }
        ++n;
    }
    return true;
}

// The same walk for any brick (64-bit addresses): the next sample's corner
// loads are issued before fn runs on the current one.
template <typename TS, typename Fn>
__device__ inline bool walk_any(const BrickK& b, double dt, double inv_dt, const RaySetup& rs, const Blocks& bl,
                                const Step& st, Fn fn) {
    const TS* __restrict__ vox = reinterpret_cast<const TS*>(b.data);
    const int snx = b.sdim[0], sny = b.sdim[1], snz = b.sdim[2];
    const int pitch = row_pitch(snx);
    const long long sxy = (long long)pitch * sny;
    long long n = block_of(bl, dt, inv_dt, rs.kf);
    long long k = rs.kf;
    while (k <= rs.kl) {
        const long long knext = block_start(bl, inv_dt, n + 1);
        const long long kend = min(knext - 1, rs.kl);
        if (kend >= k) {
            const Anchor an = make_anchor(rs, b, dt, k);
            float fj = 0.0f;
            Cell c = locate(an, st, fj, snx, sny, snz);
            float v[8];
            corners(vox, c, pitch, sxy, v);
            for (long long kk = k; kk <= kend; ++kk) {
                const Cell cur = c;
                const float w[8] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
                if (kk < kend) {
                    fj += 1.0f;
                    c = locate(an, st, fj, snx, sny, snz);
                    corners(vox, c, pitch, sxy, v);
                }
                if (!fn(kk, lerp3(cur, w[0], w[1], w[2], w[3], w[4], w[5], w[6], w[7]))) return false;
            }
            k = kend + 1;
        }
        ++n;
    }
    return true;
}

template <typename Fn>
__device__ __forceinline__ void walk(const RqcBrick& rb, double dt, double inv_dt, const RaySetup& rs,
                                     const Blocks& bl, const Step& st, Fn fn) {
    const BrickK& b = rb.brick;
    if (rb.storage == kF16) {
        if (fits_rows(b, 2)) walk_rows<__half>(b, dt, inv_dt, rs, bl, st, fn);
        else walk_any<__half>(b, dt, inv_dt, rs, bl, st, fn);
    } else {
        if (fits_rows(b, 4)) walk_rows<float>(b, dt, inv_dt, rs, bl, st, fn);
        else walk_any<float>(b, dt, inv_dt, rs, bl, st, fn);
    }
}

// --------------------------------------------------------------- shadows
// What the shadow rays of a frame share in a brick: they have one direction.
struct LightBrick {
    Step st;
    int axis, sg;
    double c0, inv_dw;       // plane n = 0 is crossed at (c0 - o_w) / d_w
    double c1;
};

// The shadow rays of one 8 x 8 tile of a home brick's ROI: the ray of every
// owned primary sample (its slot) cycles through the bricks home, home + 1,
// ... (mod n), multiplying its transmittance by each one's.  A lane takes
// every split-th sample of its pixel (split: the wavefronts of a tile), so
// that a wavefront's 64 rays start at one depth behind 8 x 8 neighbouring
// pixels: neighbouring lanes read neighbouring voxels of a few rows.  (With the
// lanes on 64 consecutive samples of one primary ray every lane read rows of
// its own, 33 cycles of the L1 a load instead of 17.)  Bound by those vector
// loads, 4 a sample.
// Measured (96^3 in 6 bricks, 384x384, 896 M shadow and primary samples): the
// frame 7.48 ms with one launch per cycle step and slot-ordered lanes, 3.49
// so; 3.78 with the lanes in rows of 8.
constexpr int kMaxShadowSplit = 64;

__global__ __launch_bounds__(256, 5) void rqc_shadow(RqcParams p) {
    __shared__ TFTable tft;
    __shared__ LightBrick light[kMaxPartials];
    load_tf(tft, p.tf, p.dt, threadIdx.x, blockDim.x);
    if ((int)threadIdx.x < p.n) {
#pragma clang fp contract(off)
        const BrickK& b = p.bricks[threadIdx.x].brick;
        RaySetup rs;
        for (int c = 0; c < 3; ++c) {
            rs.o[c] = 0.0;
            rs.d[c] = p.light[c];
        }
        const Blocks bl = make_blocks(rs, b);
        LightBrick L;
        L.st = make_step(rs, b, p.dt);
        L.axis = bl.axis;
        L.sg = bl.sg;
        L.c0 = (0.5 - (double)b.ghost) * pick3(b.spacing, bl.axis) + pick3(b.origin, bl.axis);
        L.inv_dw = 1.0 / pick3(rs.d, bl.axis);
        L.c1 = bl.c1;
        light[threadIdx.x] = L;
    }
    __syncthreads();
    // the tile's brick: the last whose tiles begin at or before it
    int tile = p.tile0 + (int)blockIdx.x, h = 0;
    for (; h + 1 < p.n; ++h) {
        const RqcBrick& rb = const_entry(p.bricks, h);
        const int t = (rb.roi_w + 7) / 8 * ((rb.roi_h + 7) / 8);
        if (tile < t) break;
        tile -= t;
    }
    const RqcBrick& home = const_entry(p.bricks, h);
    const int tiles_x = (home.roi_w + 7) / 8;
    const int lane = threadIdx.x & 63;
    // lanes in Z order: four consecutive lanes are 2 x 2 pixels
    const int lx = tile % tiles_x * 8 + ((lane & 1) | (lane >> 1 & 2) | (lane >> 2 & 4));
    const int ly = tile / tiles_x * 8 + ((lane >> 1 & 1) | (lane >> 2 & 2) | (lane >> 3 & 4));
    const float tf_k = 255.0f / (p.tf.vmax - p.tf.vmin);
    const float tf_o = -p.tf.vmin * tf_k;
    long long q0 = 0, slots = 0, kf = 0;
    CamRay cr{};
    if (lx < home.roi_w && ly < home.roi_h) {
        const long long e = home.entry0 + (long long)ly * home.roi_w + lx;
        q0 = p.offsets[e];
        slots = p.offsets[e + 1] - q0;
        kf = p.kf[e];
        cr = camera_ray(p.cam, home.roi_x0 + lx, home.roi_y0 + ly);
    }
    unsigned long long evaluated = 0;
    for (long long i = 4 * blockIdx.y + (threadIdx.x >> 6); i < slots; i += p.split) {
        RaySetup rs;
        {
#pragma clang fp contract(off)
            const double t = ((double)(kf + i) + 0.5) * p.dt;
            for (int c = 0; c < 3; ++c) {
                rs.o[c] = cr.o[c] + t * cr.d[c];
                rs.d[c] = p.light[c];
            }
        }
        float all = 1.0f;
        for (int s = 0; s < p.n; ++s) {
            const int at = h + s < p.n ? h + s : h + s - p.n;
            const RqcBrick& rb = const_entry(p.bricks, at);
            float T = 1.0f;
            if (owned_run(rs, rb.brick, p.dt, p.inv_dt, p.inv_light)) {
                const LightBrick L = light[at];
                Blocks bl;
                bl.axis = L.axis;
                bl.sg = L.sg;
                bl.c0 = (L.c0 - pick3(rs.o, L.axis)) * L.inv_dw;
                bl.c1 = L.c1;
                walk(rb, p.dt, p.inv_dt, rs, bl, L.st, [&](long long, float v) {
                    T = T * trans_exp2(-classify(tft, v, tf_k, tf_o).a);
                    return true;
                });
                evaluated += (unsigned long long)(rs.kl - rs.kf + 1);
            }
            all = s == 0 ? T : all * T;
        }
        p.shade[q0 + i] = all;
    }
    count_samples(p.samples, evaluated);
}

// --------------------------------------------------------------- primary
// The primary rays of four 8 x 8 pixel tiles (one wavefront each) through
// brick blockIdx.y: each ray's segment (key, C, alpha) goes to its pixel's
// slot of that brick.  The accumulation is the partial march's
// (emission-absorption, the same early-termination rule), the emitted colour
// scaled by a0 + (1 - a0) S.
__global__ __launch_bounds__(256) void rqc_primary(RqcParams p) {
    __shared__ TFTable tft;
    load_tf(tft, p.tf, p.dt, threadIdx.x, blockDim.x);
    __syncthreads();
    const int c = blockIdx.y;
    const RqcBrick& rb = const_entry(p.bricks, c);
    const int tiles_x = (p.width + 7) / 8, lane = threadIdx.x & 63;
    const int tile = 4 * blockIdx.x + uniform_i(threadIdx.x >> 6);
    const int px = tile % tiles_x * 8 + (lane & 7), py = tile / tiles_x * 8 + (lane >> 3);
    const bool live = px < p.width && py < p.height;
    const float tf_k = 255.0f / (p.tf.vmax - p.tf.vmin);
    const float tf_o = -p.tf.vmin * tf_k;
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, T = 1.f, key = INFINITY;
    unsigned long long evaluated = 0;
    const int lx = px - rb.roi_x0, ly = py - rb.roi_y0;
    RaySetup rs;
    if (live && lx >= 0 && ly >= 0 && lx < rb.roi_w && ly < rb.roi_h &&
        setup_ray(p.cam, rb.brick, p.dt, px, py, rs)) {
        key = (float)(((double)rs.kf + 0.5) * p.dt);
        const long long q0 = p.offsets[rb.entry0 + (long long)ly * rb.roi_w + lx];
        const float a0 = p.ambient, a1 = 1.0f - p.ambient;
        walk(rb, p.dt, p.inv_dt, rs, make_blocks(rs, rb.brick), make_step(rs, rb.brick, p.dt),
             [&](long long k, float v) {
#pragma clang fp contract(off)
            const Classified e = classify(tft, v, tf_k, tf_o);
            float f = 1.0f;
            if (p.shadows) f = a0 + a1 * p.shade[q0 + (k - rs.kf)];
            const float Tn = T * trans_exp2(-e.a);
            const float w = T - Tn;
            C0 = fmaf(w, e.r * f, C0);
            C1 = fmaf(w, e.g * f, C1);
            C2 = fmaf(w, e.b * f, C2);
            T = Tn;
            ++evaluated;
            // the partial march tests termination after odd offsets
            return !(((k - rs.kf) & 1) && T < p.ert_eps);
        });
    }
    count_samples(p.samples, evaluated);
    if (!live) return;
    float* sg = p.segs + (((long long)py * p.width + px) * p.n + c) * 5;
    sg[0] = key;
    sg[1] = C0;
    sg[2] = C1;
    sg[3] = C2;
    sg[4] = 1.0f - T;
}

// --------------------------------------------------------------- resolve
// The pixel's n segments with finite keys in (key, brick index) order, each
// "over" the result so far, then over the background (the composite's
// arithmetic).
__global__ __launch_bounds__(256) void rqc_resolve(RqcParams p) {
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= (long long)p.width * p.height) return;
    const float* sg = p.segs + pix * p.n * 5;
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, A = 0.f;
    float lk = -INFINITY;
    int li = -1;
    for (int m = 0; m < p.n; ++m) {
        float bk = INFINITY;
        int bi = -1;
        for (int c = 0; c < p.n; ++c) {
            const float z = sg[c * 5];
            const bool after = z > lk || (z == lk && c > li);
            if (z < INFINITY && after && (z < bk || (z == bk && c < bi))) {
                bk = z;
                bi = c;
            }
        }
        if (bi < 0) break;
        const float w = 1.0f - A;
        C0 = fmaf(w, sg[bi * 5 + 1], C0);
        C1 = fmaf(w, sg[bi * 5 + 2], C1);
        C2 = fmaf(w, sg[bi * 5 + 3], C2);
        A = fmaf(w, sg[bi * 5 + 4], A);
        lk = bk;
        li = bi;
    }
    const float w = 1.0f - A;
    reinterpret_cast<float4*>(p.out)[pix] =
        make_float4(fmaf(w, p.bg[0], C0), fmaf(w, p.bg[1], C1), fmaf(w, p.bg[2], C2), fmaf(w, p.bg[3], A));
}

// Wavefronts per tile of the shadow rays: 1.5 for each sample of the ROIs'
// mean pixel (6 where tiles are few and their samples must fill the GPU), at
// most kMaxShadowSplit; a lane past its pixel's samples only loads the tables.
// Always 64, a frame of short rays spent its time on workgroups without work:
// 32^3 in one brick at 1920x1080, step 8, 565 us, 149 so (256 at 6 a sample); in 4
// bricks 1110 and 375; 96^3 in 6 bricks at 384x384, step 0.5, 3.50 ms either way;
// 32^3 in 4 bricks at 96x72, step 0.5, 147 at 1.5, 111 at 6.
int shadow_split(long long total, int tiles) {
    const double mean = (double)total / (64.0 * tiles), each = tiles < 1024 ? 6.0 : 1.5;
    return 4 * (int)std::min(kMaxShadowSplit / 4.0, 1.0 + std::ceil(each * mean / 4.0));
}

inline int grid_for(long long n, int per) { return (int)((n + per - 1) / per); }

}  // namespace

hipError_t launch_exclusive_scan(long long* v, long long n, long long* sums, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const long long nb = (n + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(scan_blocks, dim3((unsigned)nb), dim3(256), 0, stream, v, n, sums);
    hipLaunchKernelGGL(scan_sums, dim3(1), dim3(256), 0, stream, sums, nb, v + n);
    hipLaunchKernelGGL(scan_add, dim3((unsigned)nb), dim3(256), 0, stream, v, n, sums);
    return hipGetLastError();
}

long long scan_blocks(long long n) { return (n + kScanBlock - 1) / kScanBlock; }

hipError_t launch_rqc_plan(const RqcParams& p, long long* scan_sums_buf, long long* total, hipStream_t stream) {
    if (p.n_entries <= 0) return hipSuccess;
    hipLaunchKernelGGL(rqc_count, dim3(grid_for(p.n_entries, 256)), dim3(256), 0, stream, p);
    (void)total;   // the scan leaves the total in p.offsets[n_entries]
    return launch_exclusive_scan(p.offsets, p.n_entries, scan_sums_buf, stream);
}

long long rqc_scan_blocks(long long n_entries) { return scan_blocks(n_entries); }

hipError_t launch_rqc_frame(RqcParams p, int cus, hipStream_t stream) {
    (void)cus;
    const long long npx = (long long)p.width * p.height;
    if (p.shadows && p.total > 0) {
        p.split = shadow_split(p.total, p.tiles);
        for (p.tile0 = 0; p.tile0 < p.tiles; p.tile0 += kMaxLaunchTiles)
            hipLaunchKernelGGL(rqc_shadow, dim3(min(p.tiles - p.tile0, kMaxLaunchTiles), p.split / 4), dim3(256), 0,
                               stream, p);
    }
    const int tiles = (p.width + 7) / 8 * ((p.height + 7) / 8);
    hipLaunchKernelGGL(rqc_primary, dim3((tiles + 3) / 4, p.n), dim3(256), 0, stream, p);
    hipLaunchKernelGGL(rqc_resolve, dim3(grid_for(npx, 256)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace dpvr
