// Brick ingest for gfx950: copy the caller's ghost-padded float32 voxels into
// the brick's workspace at the brick's storage precision (float32, or IEEE
// binary16 rounded to nearest even), re-pitching rows to a multiple of 8
// elements (16-byte aligned rows for the staged march).  Pure streaming, one
// pass over HBM.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include "dpvr_kernels.h"

namespace dpvr {
namespace {

// Both kernels write the workspace in units of kUnit consecutive elements of a
// row (the row pitch is a multiple of 8): one store of 16 bytes (float16: 8) a
// unit, and one unaligned load of 16 bytes where the unit lies inside the
// source row.  Index: unsigned, or 64-bit for bricks of 2^32 units and more
// (a 64-bit division an element bound the copy: 8 bricks of 384 x 384 x 256
// took 117 us, 72 now, 63 at the rate of a large copy).
constexpr int kUnit = 4;
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef floatx4 floatx4_unaligned __attribute__((aligned(4)));

__device__ inline void store_unit(float* dst, floatx4 v) { *reinterpret_cast<floatx4*>(dst) = v; }
__device__ inline void store_unit(__half* dst, floatx4 v) {
    auto bits = [](float x) { return (unsigned)__half_as_ushort(__float2half_rn(x)); };
    *reinterpret_cast<uint2*>(dst) = make_uint2(bits(v.x) | bits(v.y) << 16, bits(v.z) | bits(v.w) << 16);
}

// Re-pitch the caller's x-fastest voxels (row length snx) into the workspace
// (row pitch P = snx rounded up to 8, pad columns zeroed).  One thread per
// unit; reads and writes are both row-contiguous.
template <typename TD, typename Index>
__global__ __launch_bounds__(256) void ingest_kernel(const float* __restrict__ src,
                                                     TD* __restrict__ dst, int snx, int units,
                                                     Index total) {
    const Index stride = (Index)gridDim.x * blockDim.x;
    for (Index i = (Index)blockIdx.x * blockDim.x + threadIdx.x; i < total;) {
        const Index row = i / (Index)units;
        const int x = (int)(i - row * (Index)units) * kUnit;
        const float* in = src + (long long)row * snx + x;
        floatx4 v;
        if (x + kUnit <= snx) {
            v = *reinterpret_cast<const floatx4_unaligned*>(in);
        } else {
#pragma unroll
            for (int k = 0; k < kUnit; ++k) v[k] = x + k < snx ? in[k] : 0.0f;
        }
        store_unit(dst + (long long)i * kUnit, v);
        if (total - i <= stride) break;      // (an unsigned index may not pass the total)
        i += stride;
    }
}

// Gather a brick's ghost-padded box out of a global voxel array (indices
// clamped to the grid, i.e. edge replication at the domain boundary).  One
// thread per unit of a stored row, x fastest: reads of a stored row are one
// contiguous global row.
template <typename TD, typename Index>
__global__ __launch_bounds__(256) void gather_kernel(GatherParams g, TD* __restrict__ dst, int units, Index total) {
    const long long gnx = g.vol_dims[0], gny = g.vol_dims[1], gnz = g.vol_dims[2];
    const Index stride = (Index)gridDim.x * blockDim.x;
    for (Index i = (Index)blockIdx.x * blockDim.x + threadIdx.x; i < total;) {
        const Index row = i / (Index)units, slice = row / (Index)g.sdim[1];
        const int sx = (int)(i - row * (Index)units) * kUnit;
        const long long sy = (long long)(row - slice * (Index)g.sdim[1]), sz = (long long)slice;
        const long long y = min(max((long long)g.lo[1] + sy - g.ghost, 0LL), gny - 1);
        const long long z = min(max((long long)g.lo[2] + sz - g.ghost, 0LL), gnz - 1);
        const float* in = g.volume + (z * gny + y) * gnx;
        const long long x = (long long)g.lo[0] + sx - g.ghost;
        floatx4 v;
        if (sx + kUnit <= g.sdim[0] && x >= 0 && x + kUnit <= gnx) {
            v = *reinterpret_cast<const floatx4_unaligned*>(in + x);
        } else {
#pragma unroll
            for (int k = 0; k < kUnit; ++k) v[k] = sx + k < g.sdim[0] ? in[min(max(x + k, 0LL), gnx - 1)] : 0.0f;
        }
        store_unit(dst + (long long)i * kUnit, v);
        if (total - i <= stride) break;
        i += stride;
    }
}

int unit_blocks(long long total) { return (int)min((total + 255) / 256, 1LL << 20); }

}  // namespace

hipError_t launch_gather(const GatherParams& g, void* dst, StorageK storage, hipStream_t stream) {
    const int units = ((g.sdim[0] + 7) & ~7) / kUnit;
    const long long total = (long long)units * g.sdim[1] * g.sdim[2];
    if (total <= 0) return hipSuccess;
    const dim3 grid(unit_blocks(total)), block(256);
    const bool wide = total > 0xffffffffLL;
    if (storage == kF16) {
        __half* d = reinterpret_cast<__half*>(dst);
        if (wide) hipLaunchKernelGGL((gather_kernel<__half, long long>), grid, block, 0, stream, g, d, units, total);
        else hipLaunchKernelGGL((gather_kernel<__half, unsigned>), grid, block, 0, stream, g, d, units, (unsigned)total);
    } else {
        float* d = reinterpret_cast<float*>(dst);
        if (wide) hipLaunchKernelGGL((gather_kernel<float, long long>), grid, block, 0, stream, g, d, units, total);
        else hipLaunchKernelGGL((gather_kernel<float, unsigned>), grid, block, 0, stream, g, d, units, (unsigned)total);
    }
    return hipGetLastError();
}

hipError_t launch_ingest(const float* src, void* dst, const int32_t sdim[3], StorageK storage,
                         hipStream_t stream) {
    const int snx = sdim[0], units = ((snx + 7) & ~7) / kUnit;
    const long long total = (long long)units * sdim[1] * sdim[2];
    if (total <= 0) return hipSuccess;
    const dim3 grid(unit_blocks(total)), block(256);
    const bool wide = total > 0xffffffffLL;
    if (storage == kF16) {
        __half* d = reinterpret_cast<__half*>(dst);
        if (wide) hipLaunchKernelGGL((ingest_kernel<__half, long long>), grid, block, 0, stream, src, d, snx, units, total);
        else hipLaunchKernelGGL((ingest_kernel<__half, unsigned>), grid, block, 0, stream, src, d, snx, units, (unsigned)total);
    } else {
        float* d = reinterpret_cast<float*>(dst);
        if (wide) hipLaunchKernelGGL((ingest_kernel<float, long long>), grid, block, 0, stream, src, d, snx, units, total);
        else hipLaunchKernelGGL((ingest_kernel<float, unsigned>), grid, block, 0, stream, src, d, snx, units, (unsigned)total);
    }
    return hipGetLastError();
}

}  // namespace dpvr
