// Packed prefill attention, bf16 MFMA, head dimensions 128 and 64 (Sec. 3.1): the launches.  The
// kernels' device code is in prefill_body.hip.h, included once per head dimension.
#define PK_WAVES 4
#define PK_D 128
#define PK_DNS d128
#include "prefill_body.hip.h"
#undef PK_D
#undef PK_DNS
#define PK_D 64
#define PK_DNS d64
#include "prefill_body.hip.h"
#undef PK_D
#undef PK_DNS
#define PK_D 128
#define PK_DNS few128
#include "prefill_few_body.hip.h"
#undef PK_D
#undef PK_DNS
#define PK_D 64
#define PK_DNS few64
#include "prefill_few_body.hip.h"
#undef PK_D
#undef PK_DNS
#undef PK_WAVES
#define PK_WAVES 8
#define PK_D 128
#define PK_DNS d128x2
#include "prefill_body.hip.h"
#undef PK_D
#undef PK_DNS
#undef PK_WAVES

namespace pk {
namespace {

// Two query heads of a KV head per workgroup: they work on the same K/V tiles, which are copied into LDS once
// for both.
__global__ __launch_bounds__(512, 2) void prefill_bf16_pair_kernel(PrefillArgs a) {
    __shared__ __align__(1024) unsigned char lds[5 * d128x2::TILE_BYTES];
    d128x2::prefill_tile_body(a, static_cast<int>(blockIdx.x), lds);
}

__global__ __launch_bounds__(256, 2) void prefill_bf16_dma_kernel(PrefillArgs a) {
    __shared__ __align__(1024) unsigned char lds[5 * d128::TILE_BYTES];
    d128::prefill_tile_body(a, static_cast<int>(blockIdx.x), lds);
}

__global__ __launch_bounds__(256, 3) void prefill_bf16_dma64_kernel(PrefillArgs a) {
    __shared__ __align__(1024) unsigned char lds[5 * d64::TILE_BYTES];
    d64::prefill_tile_body(a, static_cast<int>(blockIdx.x), lds);
}

// Launches of little work (PrefillArgs::light).
__global__ __launch_bounds__(256, 2) void prefill_bf16_few_kernel(PrefillArgs a) {
    __shared__ __align__(1024) unsigned char lds[5 * few128::TILE_BYTES];
    few128::prefill_tile_body(a, static_cast<int>(blockIdx.x), lds);
}

__global__ __launch_bounds__(256, 2) void prefill_bf16_few64_kernel(PrefillArgs a) {
    __shared__ __align__(1024) unsigned char lds[5 * few64::TILE_BYTES];
    few64::prefill_tile_body(a, static_cast<int>(blockIdx.x), lds);
}

// Behind a launch of few workgroups whose lists are cut into pieces.
__global__ __launch_bounds__(64 * few128::DB) void prefill_merge_kernel(PrefillArgs a) { few128::prefill_merge(a, static_cast<int>(blockIdx.x)); }
__global__ __launch_bounds__(64 * few64::DB) void prefill_merge64_kernel(PrefillArgs a) { few64::prefill_merge(a, static_cast<int>(blockIdx.x)); }

}  // namespace

int launch_prefill_merge_bf16(const PrefillArgs& a, void* stream) {
    const int64_t grid = static_cast<int64_t>(a.n_merges) * a.Hkv * a.heads_per_kv * 4;
    if (grid == 0) return 0;
    if (grid > 0x7FFFFFFF) return static_cast<int>(hipErrorInvalidValue);
    if (a.d == 128)
        hipLaunchKernelGGL(prefill_merge_kernel, dim3(static_cast<unsigned>(grid)), dim3(64 * few128::DB), 0, static_cast<hipStream_t>(stream), a);
    else
        hipLaunchKernelGGL(prefill_merge64_kernel, dim3(static_cast<unsigned>(grid)), dim3(64 * few64::DB), 0, static_cast<hipStream_t>(stream), a);
    return static_cast<int>(hipGetLastError());
}

int launch_prefill_bf16_pipe(const PrefillArgs& args, void* stream) {
    PrefillArgs a = args;
    a.heads_per_kv = a.Hq / a.Hkv;
    a.by_hkv = FastDiv::by(static_cast<uint32_t>(a.Hkv));
    // Copying each K/V tile once for two heads halves the copies (a tile step of two four-wave workgroups on a
    // compute unit reads 256 KiB of LDS and writes 64), and the energy they take.  What it costs: nothing runs beside a workgroup's first loads
    // and last stores, and a chip that is not full has fewer compute units at work.  Four / eight waves with 128 rows and one head / two (the
    // padded launch; on query tiles of several heads ahead_with_eight in schedule.cpp weighs the two):
    //   32 chunks of a 70B-shaped layer (140 key tiles on average)  10.42 / 10.32 ms
    //   1 x 4096 rows behind 8192 (160 tiles, 1024 four-wave workgroups)  573 / 549 us
    //   2 x 3000 behind 3000 with 16 heads (71 tiles, 752 workgroups)     252 / 225 us
    //   32 x 1024 behind 2048 (40 tiles)  1225 / 1216 us;  8 x 4096 (32 tiles)  979 / 981 us;  32 x 1024 behind 1024 (24 tiles)  782 / 786 us
    //   16 x 2048 (16 tiles)  561 / 558 us;  64 ragged prompts (10 tiles)  379 / 380 us
    //   1 x 2048 behind 8192 (144 tiles, 512 workgroups)  271 / 265 us;  1 x 1024 (256 workgroups)  152 / 206 us
    // D = 64 stays with four waves: with 168 registers a wave, three such workgroups share a compute unit, of eight waves
    // only one does:
    //   8 x 4096  575 / 627 us;  16 x 2048  326 / 363 us;  32 x 512 behind 8192 with 64 heads  2205 / 2342 us
    //   1 x 1024 behind 8192  123 / 149 us;  1 x 4096 behind 8192  363 / 348 us;  2 x 3000 behind 3000 with 16 heads  187 / 164 us
    const int mates = (a.eight ? 8 : 4) >> a.row_shift;     // heads of a workgroup
    if (a.heads_per_kv % mates != 0) return static_cast<int>(hipErrorInvalidValue);
    a.heads_per_kv /= mates;
    a.by_r = FastDiv::by(static_cast<uint32_t>(a.heads_per_kv));
    const int64_t pairs = static_cast<int64_t>(a.n_tiles) * a.Hkv;
    const int64_t grid = (pairs + 7) / 8 * 8 * a.heads_per_kv;
    if (grid == 0) return 0;
    if (grid > 0x7FFFFFFF) return static_cast<int>(hipErrorInvalidValue);
    if (a.light && a.d == 128)
        hipLaunchKernelGGL(prefill_bf16_few_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), a);
    else if (a.light && a.d == 64)
        hipLaunchKernelGGL(prefill_bf16_few64_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), a);
    else if (a.eight)
        hipLaunchKernelGGL(prefill_bf16_pair_kernel, dim3(static_cast<unsigned>(grid)), dim3(512), 0,
                           static_cast<hipStream_t>(stream), a);
    else if (a.d == 128)
        hipLaunchKernelGGL(prefill_bf16_dma_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), a);
    else if (a.d == 64)
        hipLaunchKernelGGL(prefill_bf16_dma64_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), a);
    else
        return static_cast<int>(hipErrorInvalidValue);
    const int e = static_cast<int>(hipGetLastError());
    return e != 0 ? e : launch_prefill_merge_bf16(a, stream);
}

}  // namespace pk
