// Upload of a plan's int32 tables: one workgroup reads them from pinned host memory over the host link
// and writes them to the workspace, then tells the host that the staging buffer is free again.
//
// Bound by latency: a copy command in the stream hands the transfer to a copy engine and waits for it
// on both sides, some 20 us during which the compute units stand still; a kernel starts like any other
// behind the one before it.  (Re-layout, decode and merge of a new batch of 48 requests: 129 -> 113.5 us a
// pass; a bind of 76 KB of tables and a small kernel 24.9 -> 14.6.)  One workgroup
// of 1024 lanes keeps 64 KiB of reads in flight, which is what the link delivers in one round trip, and
// lets a single barrier say that the whole table has been read.
#include "common.hip.h"
#include "kernels.h"

namespace pk {
namespace {

constexpr int kLanes = 1024, kUnroll = 4;

// `chunks`: 16-byte pieces
__global__ __launch_bounds__(kLanes) void upload_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int chunks,
                                                        uint32_t* done, uint32_t stamp) {
    for (int c0 = threadIdx.x; c0 < chunks; c0 += kLanes * kUnroll) {
        u32x4 v[kUnroll];
#pragma unroll
        for (int i = 0; i < kUnroll; ++i)
            if (c0 + i * kLanes < chunks) v[i] = src[c0 + i * kLanes];
#pragma unroll
        for (int i = 0; i < kUnroll; ++i)
            if (c0 + i * kLanes < chunks) dst[c0 + i * kLanes] = v[i];
    }
    // every lane has its data here (the stores took it): the host may write the buffer again
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(done, stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

int launch_upload(const void* src, void* dst, int64_t bytes, uint32_t* done, uint32_t stamp, void* stream) {
    if (bytes % 16 != 0 || bytes > 0x7FFFFFFF) return static_cast<int>(hipErrorInvalidValue);
    hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(kLanes), 0, static_cast<hipStream_t>(stream),
                       static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), static_cast<int>(bytes / 16), done, stamp);
    return static_cast<int>(hipGetLastError());
}

}  // namespace pk
