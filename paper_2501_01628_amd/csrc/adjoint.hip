// Adjoint of the per-brick ray march for gfx950: gradients of a loss with
// respect to the transfer-function table and the global voxel array, given
// the loss gradient of the brick's partial image (dL/dC_rgb, dL/dA per ROI
// pixel).
//
// kParts lanes share a ray, each a stretch of its owned samples; a workgroup
// takes an 8x8 tile, a wavefront kParts lanes for each of 64 / kParts pixels
// of it.  A lane walks its stretch forward for its colour and transmittance,
// exchanges them with the ray's other lanes (transmittance in front of the
// stretch, colour and transmittance of what lies behind it), then walks it
// backwards with
//   R_k = a_k rgb_k + (1 - a_k) R_{k+1},  Q_k = (1 - a_k) Q_{k+1}
// (R = colour, Q = transmittance of what lies behind sample k in the brick),
//   dC/drgb_k = T_k a_k,  dC/da_k = T_k (rgb_k - R_{k+1}),  dA/da_k = T_k Q_{k+1}.
// The transmittance T_k in front of a sample is exp2 of the a' summed up to it:
// forward over the ray's stretches, taken off again on the way back, the sum as
// an integer and a fraction, so that T_k is nearly as exact as one exponential
// (a product over the ray gathers two roundings a sample).
// One lane per ray, from transmittance checkpoints, left the GPU to its
// longest rays: at 512x512 on 128^3 the slowest of 3,016 wavefronts ran 3.4
// times the average, 2 to 3 per SIMD.  Bound by the vector ALU (76 % of its
// issue slots while a CU is busy, 56 % of the lanes active; 16 bricks of 512 x
// 256 x 256 at 384x384 65 % and 51 %) and by the voxel atomics (13 % of the time
// of the former, 36 % of the latter).  Forward and backward of 8 views of the
// former, step 0.5: 7.2 ms before, 4.4 now; of one view of the latter, float16,
// step 0.25: 7.4 ms before, 6.4 now, of which 3.0 here.  8 lanes a ray: 1 % and
// 12 % slower (set-up, partly filled stretches).  A view into a few voxels, bound
// by the atomics alone, pays for the corners at the stretches' ends: 128 x 112 x
// 96 in 6 bricks, a tenth of the field of view over 256x192, 2.5 ms before, 2.65
// now; 80 x 60 x 90 in 8, half of it over 343x245, 1.31 and 1.37.
// The opacity a_k = 1 - exp2(-a'_k) with a' the pre-scaled table opacity;
// table gradients are summed per lane while consecutive samples use one
// table segment, accumulated per workgroup in LDS (ds_add_f32) and flushed
// with one global atomic per touched entry; voxel gradients are
// scattered with the 8 trilinear weights to the global voxels that the stored
// (ghost-padded) voxels copy, so ghost contributions fold back to their source
// (summed per lane per corner while the walk stays in one cell; moving to a
// neighbouring cell keeps the sums of the shared corners, so a corner is
// added with one atomic when the walk leaves it).
#include "march_common.h"

namespace dpvr {
namespace {

constexpr int kTile = 8;
constexpr int kParts = 4;               // lanes per ray
constexpr int kThreads = 64 * kParts;   // an 8x8 tile
// A workgroup takes kSeries tiles one after the other where that leaves kFill
// workgroups (4 on each of 256 CUs; many partials: always): the table gradient
// is added to global memory once a workgroup, and every such float add rounds
// at the size of the whole sum.  One tile a workgroup is 2 % (one brick) to 5 %
// (16 bricks) faster, but the gradients' error against float64 grew from 2.8e-7
// to 4.6e-7 on a scene of several bricks, where this leaves it as it was.
constexpr int kSeries = 4;
constexpr int kFill = 1024;
constexpr float kLn2 = 0.6931471805599453f;

// Where a ray's samples lie: position, corner reads and stored cell of sample
// j after an anchor.  RowReads by 32-bit offsets (bricks that fits_rows
// accepts), AnyReads by 64-bit indices.
template <typename TS>
struct RowReads {
    Rows<TS> rows;
    unsigned base;
    struct At {
        Spot s;
        Corners<TS> c;
    };
    __device__ RowReads(const BrickK& b) : rows(make_rows<TS>(b)), base(0) {}
    __device__ void anchor(const Anchor& an) { base = anchor_offset(rows, an); }
    __device__ At read(const Anchor& an, const Step& st, float fj) const {
        At a;
        a.s = locate_rows(rows, base, an, st, fj);
        a.c = gather_rows(rows, a.s.off);
        return a;
    }
    __device__ float value(const At& a) const { return lerp_rows(a.s, a.c); }
    __device__ static float fx(const At& a) { return a.s.fx; }
    __device__ static float fy(const At& a) { return a.s.fy; }
    __device__ static float fz(const At& a) { return a.s.fz; }
};
template <typename TS>
struct AnyReads {
    const TS* vox;
    int snx, sny, snz, pitch;
    long long sxy;
    struct At {
        Cell c;
        float v;
    };
    __device__ AnyReads(const BrickK& b)
        : vox(reinterpret_cast<const TS*>(b.data)), snx(b.sdim[0]), sny(b.sdim[1]), snz(b.sdim[2]),
          pitch(row_pitch(b.sdim[0])), sxy((long long)row_pitch(b.sdim[0]) * b.sdim[1]) {}
    __device__ void anchor(const Anchor&) {}
    __device__ At read(const Anchor& an, const Step& st, float fj) const {
        At a;
        a.c = locate(an, st, fj, snx, sny, snz);
        a.v = trilinear(vox, a.c, pitch, sxy);
        return a;
    }
    __device__ float value(const At& a) const { return a.v; }
    __device__ static float fx(const At& a) { return a.c.fx; }
    __device__ static float fy(const At& a) { return a.c.fy; }
    __device__ static float fz(const At& a) { return a.c.fz; }
};

// One lane's share of a ray (part: its stretch; g: the loss gradient, zero
// for lanes without a ray), table gradients into gtf.  All lanes of the
// wavefront call it.
template <typename Reads>
__device__ __forceinline__ void backward_ray(const MarchParams& p, const BackwardParams& bp, const TFTable& tft,
                                             float* gtf, const RaySetup& rs, bool has, int part, const float4 g,
                                             float tf_k, float tf_o, Reads reads) {
    const BrickK& b = p.brick;
    // d a' / d alpha_table: converts pre-scaled opacity gradients to table units
    const float a_scale = p.tf.opacity_scale * (float)p.dt * kLog2e;
    const int gnx = bp.vol_dims[0], gny = bp.vol_dims[1], gnz = bp.vol_dims[2];
    Step st{};
    Blocks bl{0.0, 1.0, 2, 1};
    long long k0 = 0, k1 = -1;
    if (has) {
        st = make_step(rs, b, p.dt);
        bl = make_blocks(rs, b);
        const long long N = rs.kl - rs.kf + 1;
        k0 = rs.kf + N * part / kParts;
        k1 = rs.kf + N * (part + 1) / kParts - 1;
    }
    // the samples [ka, kb] in runs of one anchor block each, in order or
    // (kBack) last first: run(anchor, first sample of the block's run, lo, hi)
    // with samples kA + lo .. kA + hi
    auto blocks_forward = [&](long long ka, long long kb, auto run) {
        if (kb < ka) return;
        long long n = block_of(bl, p.dt, p.inv_dt, ka);
        for (long long k = ka; k <= kb; ++n) {
            const long long kA = max(rs.kf, block_start(bl, p.inv_dt, n));
            const long long kend = min(block_start(bl, p.inv_dt, n + 1) - 1, kb);
            if (kend < k) continue;
            run(kA, (int)(k - kA), (int)(kend - kA));
            k = kend + 1;
        }
    };
    auto blocks_back = [&](long long ka, long long kb, auto run) {
        if (kb < ka) return;
        long long n = block_of(bl, p.dt, p.inv_dt, kb);
        for (long long k = kb; k >= ka; --n) {
            const long long kA = max(rs.kf, block_start(bl, p.inv_dt, n));
            const long long kbeg = max(kA, ka);
            if (kbeg > k) continue;
            run(kA, (int)(kbeg - kA), (int)(k - kA));
            k = kbeg - 1;
        }
    };
    // voxel-gradient contributions of the current cell's 8 corners, not
    // yet added (acc[cx + 2 cy + 4 cz] for corner (ix + cx, iy + cy,
    // iz + cz) of the stored grid)
    bool pending = false;
    int pend_ix = 0, pend_iy = 0, pend_iz = 0;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float* G = bp.grad_vox;
    const int glo0 = bp.lo[0] - b.ghost, glo1 = bp.lo[1] - b.ghost, glo2 = bp.lo[2] - b.ghost;
    // stored index s -> global index clamp(lo + s - ghost)
    auto add_voxel = [&](int sx, int sy, int sz, float v) {
        if (v == 0.0f) return;
        const int gx = min(max(glo0 + sx, 0), gnx - 1);
        const int gy = min(max(glo1 + sy, 0), gny - 1);
        const int gz = min(max(glo2 + sz, 0), gnz - 1);
        atomicAdd(G + ((long long)gz * gny + gy) * gnx + gx, v);
    };
    auto flush = [&]() {
        if (!pending) return;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            add_voxel(pend_ix + (i & 1), pend_iy + ((i >> 1) & 1), pend_iz + (i >> 2), acc[i]);
            acc[i] = 0.f;
        }
    };
    // the walk moves to cell (nx, ny, nz): a corner the two cells share
    // keeps its sum (moving by one cell along an axis keeps the 4 corners
    // of the face crossed); the corners left behind are added now, one
    // axis at a time; a jump of more than one cell adds all 8
    auto move_to = [&](int nx, int ny, int nz) {
        const int dx = nx - pend_ix, dy = ny - pend_iy, dz = nz - pend_iz;
        if (!pending || dx < -1 || dx > 1 || dy < -1 || dy > 1 || dz < -1 || dz > 1) {
            flush();
        } else {
            if (dx != 0) {
#pragma unroll
                for (int yz = 0; yz < 4; ++yz) {   // corner pairs along x: acc[2 yz], acc[2 yz + 1]
                    const int cy = yz & 1, cz = yz >> 1;
                    const float a0 = acc[2 * yz], a1 = acc[2 * yz + 1];
                    add_voxel(pend_ix + (dx > 0 ? 0 : 1), pend_iy + cy, pend_iz + cz, dx > 0 ? a0 : a1);
                    acc[2 * yz] = dx > 0 ? a1 : 0.f;
                    acc[2 * yz + 1] = dx > 0 ? 0.f : a0;
                }
            }
            if (dy != 0) {
#pragma unroll
                for (int xz = 0; xz < 4; ++xz) {   // pairs along y: acc[i], acc[i + 2], i = cx + 4 cz
                    const int cx = xz & 1, cz = xz >> 1, i = cx + 4 * cz;
                    const float a0 = acc[i], a1 = acc[i + 2];
                    add_voxel(nx + cx, pend_iy + (dy > 0 ? 0 : 1), pend_iz + cz, dy > 0 ? a0 : a1);
                    acc[i] = dy > 0 ? a1 : 0.f;
                    acc[i + 2] = dy > 0 ? 0.f : a0;
                }
            }
            if (dz != 0) {
#pragma unroll
                for (int xy = 0; xy < 4; ++xy) {   // pairs along z: acc[i], acc[i + 4], i = cx + 2 cy
                    const float a0 = acc[xy], a1 = acc[xy + 4];
                    add_voxel(nx + (xy & 1), ny + (xy >> 1), pend_iz + (dz > 0 ? 0 : 1), dz > 0 ? a0 : a1);
                    acc[xy] = dz > 0 ? a1 : 0.f;
                    acc[xy + 4] = dz > 0 ? 0.f : a0;
                }
            }
        }
        pending = true;
        pend_ix = nx;
        pend_iy = ny;
        pend_iz = nz;
    };
    // table-gradient contributions of the current segment index, not
    // yet added (entries seg and seg + 1): consecutive samples mostly
    // use one segment, so LDS atomics happen once per change
    int tseg = -1;
    float tacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto tflush = [&]() {
        if (tseg < 0) return;
        float* g0 = &gtf[4 * tseg];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (tacc[i] != 0.0f) atomicAdd(g0 + i, tacc[i]);
            tacc[i] = 0.f;
        }
    };
    // a' summed over samples, as sn + sf (an a' above 160, which leaves no
    // transmittance that float32 holds, counts as 160: sn fits an int for 13 M
    // samples of a ray).  The integer part is split off before the addition:
    // adding a whole dense a' to the fraction would round it at the size of
    // that a', and the walk back would leave the rounding in front of the dense
    // sample, where T_k is still near 1.
    int sn = 0;
    float sf = 0.0f;
    auto sum_a = [&](float a) {
        const float most = rintf(a);
        sf += a - most;                  // |a - most| <= 1/2, exact
        const float carry = rintf(sf);
        sf -= carry;
        sn += (int)(most + carry);
    };
    constexpr float kMostA = 160.0f;
    // forward: colour and transmittance of the stretch, and its sum of a'
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, F = 1.f;
    auto ahead = [&](const auto& a) {
        const Classified e = classify(tft, reads.value(a), tf_k, tf_o);
        const float Fn = F * trans_exp2(-e.a);
        const float w = F - Fn;
        C0 = fmaf(w, e.r, C0);
        C1 = fmaf(w, e.g, C1);
        C2 = fmaf(w, e.b, C2);
        F = Fn;
        sum_a(fminf(e.a, kMostA));
    };
    blocks_forward(k0, k1, [&](long long kA, int lo, int hi) {
        const Anchor an = make_anchor(rs, b, p.dt, kA);
        reads.anchor(an);
        for (int j = lo; j <= hi; j += 2) {
            const auto a0 = reads.read(an, st, (float)j);
            const auto a1 = reads.read(an, st, (float)(j + 1));
            __builtin_amdgcn_sched_barrier(0);
            ahead(a0);
            if (j < hi) ahead(a1);
        }
    });
    // the ray's stretches: a' in front of this one, and R, Q behind it
    const int own_n = sn;
    const float own_f = sf;
    float R0 = 0.f, R1 = 0.f, R2 = 0.f, Q = 1.f;
    const int first = (threadIdx.x & 63) - part * (64 / kParts);
#pragma unroll
    for (int q = 0; q < kParts; ++q) {
        const int nq = __shfl(own_n, first + q * (64 / kParts));
        const float fq = __shfl(own_f, first + q * (64 / kParts));
        if (q < part) {
            sn += nq;
            sum_a(fq);
        }
    }
#pragma unroll
    for (int q = kParts - 1; q > 0; --q) {
        const int lane = first + q * (64 / kParts);
        const float c0 = __shfl(C0, lane), c1 = __shfl(C1, lane), c2 = __shfl(C2, lane), Fq = __shfl(F, lane);
        if (q > part) {
            R0 = fmaf(Fq, R0, c0);
            R1 = fmaf(Fq, R1, c1);
            R2 = fmaf(Fq, R2, c2);
            Q *= Fq;
        }
    }
    {
        auto back = [&](const auto& a, const Anchor& an, float fj) {
            const Classified e = classify(tft, reads.value(a), tf_k, tf_o);
            const float om = trans_exp2(-e.a);          // 1 - alpha
            const float al = 1.0f - om;
            sum_a(-fminf(e.a, kMostA));
            const float Tk = ldexpf(trans_exp2(-sf), -sn);
            const float ta = Tk * al;
            const float d_r = g.x * ta, d_g = g.y * ta, d_b = g.z * ta;
            const float d_al = Tk * (g.x * (e.r - R0) + g.y * (e.g - R1) + g.z * (e.b - R2) + g.w * Q);
            const float d_ap = d_al * kLn2 * om;   // dL/da'
            const float w1 = e.phi, w0 = 1.0f - e.phi;
            if (e.seg != tseg) {
                tflush();
                tseg = e.seg;
            }
            tacc[0] += w0 * d_r;
            tacc[1] += w0 * d_g;
            tacc[2] += w0 * d_b;
            tacc[3] += w0 * d_ap * a_scale;
            tacc[4] += w1 * d_r;
            tacc[5] += w1 * d_g;
            tacc[6] += w1 * d_b;
            tacc[7] += w1 * d_ap * a_scale;
            if (e.inside) {
                const float4 D = tft.diff[e.seg];
                const float dv = tf_k * (d_r * D.x + d_g * D.y + d_b * D.z + d_ap * D.w);
                if (dv != 0.0f) {
                    // consecutive samples mostly share a cell: sum their
                    // corner weights here, one set of atomics per cell
                    const int ix = an.ia0 + floor_int(fmaf(fj, st.s0, an.uf0));
                    const int iy = an.ia1 + floor_int(fmaf(fj, st.s1, an.uf1));
                    const int iz = an.ia2 + floor_int(fmaf(fj, st.s2, an.uf2));
                    if (!pending || ix != pend_ix || iy != pend_iy || iz != pend_iz) move_to(ix, iy, iz);
                    const float fx = Reads::fx(a), fy = Reads::fy(a), fz = Reads::fz(a);
                    const float ux = 1.0f - fx, uy = 1.0f - fy, uz = 1.0f - fz;
                    acc[0] += dv * ux * uy * uz;
                    acc[1] += dv * fx * uy * uz;
                    acc[2] += dv * ux * fy * uz;
                    acc[3] += dv * fx * fy * uz;
                    acc[4] += dv * ux * uy * fz;
                    acc[5] += dv * fx * uy * fz;
                    acc[6] += dv * ux * fy * fz;
                    acc[7] += dv * fx * fy * fz;
                }
            }
            R0 = fmaf(al, e.r, om * R0);
            R1 = fmaf(al, e.g, om * R1);
            R2 = fmaf(al, e.b, om * R2);
            Q = om * Q;
        };
        blocks_back(k0, k1, [&](long long kA, int lo, int hi) {
            const Anchor an = make_anchor(rs, b, p.dt, kA);
            reads.anchor(an);
            for (int j = hi; j >= lo; j -= 2) {
                const float f0 = (float)j, f1 = (float)(j - 1);
                const auto a0 = reads.read(an, st, f0);
                const auto a1 = reads.read(an, st, f1);
                __builtin_amdgcn_sched_barrier(0);
                back(a0, an, f0);
                if (j > lo) back(a1, an, f1);
            }
        });
    }
    flush();
    tflush();
}

// One workgroup's work: tiles block, block + blocks, ... of the partial (p, bp).
template <typename TS>
__device__ __forceinline__ void backward_tiles(const MarchParams& p, const BackwardParams& bp, int block, int blocks) {
    __shared__ TFTable tft;
    __shared__ float gtf[256 * 4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    load_tf(tft, p.tf, p.dt, threadIdx.x, kThreads);
    for (int e = threadIdx.x; e < 1024; e += kThreads) gtf[e] = 0.0f;
    __syncthreads();

    // a wavefront's 64 / kParts pixels: a 4 x 4 quarter of the tile
    static_assert(kParts == 4, "a wavefront takes a 4 x 4 quarter of the tile");
    const int q = lane & 15, part = lane >> 4;
    const float tf_k = 255.0f / (p.tf.vmax - p.tf.vmin);
    const float tf_o = -p.tf.vmin * tf_k;
    for (int tile = block; tile < p.tiles_x * p.tiles_y; tile += blocks) {
        const int lx = tile % p.tiles_x * kTile + (wave & 1) * 4 + (q & 3);
        const int ly = tile / p.tiles_x * kTile + (wave >> 1) * 4 + (q >> 2);
        RaySetup rs;
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
        bool has = lx < p.roi_w && ly < p.roi_h && setup_ray(p.cam, p.brick, p.dt, p.roi_x0 + lx, p.roi_y0 + ly, rs);
        if (has) {
            g = reinterpret_cast<const float4*>(bp.d_part)[(long long)ly * p.roi_w + lx];
            has = g.x != 0.f || g.y != 0.f || g.z != 0.f || g.w != 0.f;
        }
        if (fits_rows(p.brick, sizeof(TS)))
            backward_ray(p, bp, tft, gtf, rs, has, part, g, tf_k, tf_o, RowReads<TS>(p.brick));
        else
            backward_ray(p, bp, tft, gtf, rs, has, part, g, tf_k, tf_o, AnyReads<TS>(p.brick));
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 1024; e += kThreads) {
        const float v = gtf[e];
        if (v != 0.0f) atomicAdd(bp.grad_tf + e, v);
    }
}

template <typename TS>
__global__ __launch_bounds__(kThreads, 4) void march_backward(MarchParams p, BackwardParams bp) {
    backward_tiles<TS>(p, bp, blockIdx.x, gridDim.x);
}

// Many partials in one launch: workgroup b takes tiles of job j, the last j
// with block_start[j] <= b (so that partials of few tiles still fill the GPU
// together).
template <typename TS>
__global__ __launch_bounds__(kThreads, 4) void march_backward_many(const BackwardJob* __restrict__ jobs,
                                                                const int32_t* __restrict__ block_start,
                                                                int32_t n_jobs) {
    const int b = blockIdx.x;
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (block_start[mid] <= b) lo = mid; else hi = mid - 1;
    }
    lo = uniform_i(lo);      // uniform: the job's fields load as scalars
    const BackwardJob& J = const_entry(jobs, lo);
    const int first = uniform_i(block_start[lo]);
    backward_tiles<TS>(J.p, J.bp, b - first, uniform_i(block_start[lo + 1]) - first);
}

}  // namespace

int backward_many_waves() { return kSeries; }

hipError_t launch_march_backward_many(const BackwardJob* jobs, const int32_t* block_start, int32_t n_jobs,
                                      int32_t total_blocks, StorageK storage, hipStream_t stream) {
    if (n_jobs <= 0 || total_blocks <= 0) return hipSuccess;
    if (storage == kF16)
        hipLaunchKernelGGL(march_backward_many<__half>, dim3(total_blocks), dim3(kThreads), 0, stream, jobs,
                           block_start, n_jobs);
    else
        hipLaunchKernelGGL(march_backward_many<float>, dim3(total_blocks), dim3(kThreads), 0, stream, jobs,
                           block_start, n_jobs);
    return hipGetLastError();
}

hipError_t launch_march_backward(const MarchParams& p, const BackwardParams& bp, StorageK storage,
                                 hipStream_t stream) {
    const int tiles = p.tiles_x * p.tiles_y;
    if (tiles == 0) return hipSuccess;
    const int blocks = max((tiles + kSeries - 1) / kSeries, min(tiles, kFill));
    if (storage == kF16)
        hipLaunchKernelGGL(march_backward<__half>, dim3(blocks), dim3(kThreads), 0, stream, p, bp);
    else
        hipLaunchKernelGGL(march_backward<float>, dim3(blocks), dim3(kThreads), 0, stream, p, bp);
    return hipGetLastError();
}

}  // namespace dpvr
