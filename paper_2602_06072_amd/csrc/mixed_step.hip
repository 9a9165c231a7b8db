// Fused mixed step (Sec. 3, overview: prefill and decode requests of one continuous-batching step
// share the packed execution): the packed prefill tiles and the packed decode work items of one
// step in ONE launch.  Prefill is bound by the matrix pipe, decode by HBM; side by side on a
// compute unit they use what the other leaves idle.  The two kernels launched one after the other
// cannot do that, and launched on two streams they hardly overlap: the prefill workgroups take
// every register and LDS slot first.  Here the roles are dealt by workgroup number instead: runs of
// prefill workgroups and runs of decode workgroups (four waves: a (work item, KV head) pair each or, as
// the decode plan has it, one pair together),
// the decode runs spread evenly over the launch; the prefill workgroups keep their numbers modulo 8,
// i.e. their XCD, so the heads of a KV head still share an L2.  The LSE merge of the decode partials
// is a second, short launch.
// What bounds it (32 chunks of a 70B-shaped layer + 480 decode rows, 11.5 to 12.4 ms on different cards): the prefill tiles alone take 9.6 to 10.6 ms, the
// decode alone 2.6; what decode workgroups cost is the slots that they take and 17.9 GB streaming next to
// prefill tiles, about half of it each.  Eight-wave prefill workgroups here, with 128 rows to a tile: 12.15 to 12.7 against 12.2 ms.
// The query tiles are the prefill call's, also where that has eight waves and with fewer than eight heads per KV head twice the rows: 8 chunks with 32/8 heads
// and 200 decode rows 2136 us with tiles of 64 rows and two heads, 2129 with 32 and four; 16 x 128 rows behind some 9000 tokens 512 and 515.
#include "decode_body.hip.h"
#include "mixed_order.h"
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

namespace pk {
namespace {

// one kernel per head dimension and kind of decode workgroup (NS: the namespace of the prefill body, D: the head
// dimension); the work items and the arithmetic are those of the decode launch
#define PK_MIXED_STEP_KERNEL(NAME, NS, D, WPE, DECODE)                                                \
    __global__ __launch_bounds__(256, WPE) void NAME(PrefillArgs pa, DecodeArgs da, MixedOrder m) {   \
        __shared__ __align__(1024) unsigned char lds[5 * NS::TILE_BYTES];                             \
        const int x = static_cast<int>(blockIdx.x);                                                   \
        bool decode;                                                                                  \
        const int block = m.set_of(x >> 3, decode) * 8 + (x & 7);                                     \
        if (decode) {                                                                                 \
            DECODE<D>(pa.by_hkv, da, block, lds);                                                     \
            return;                                                                                   \
        }                                                                                             \
        if (block < m.n_prefill) NS::prefill_tile_body(pa, block, lds);                               \
    }
// four (work item, KV head) pairs, a wave each
template <int D>
__device__ __forceinline__ void decode_by_waves(const FastDiv& by_hkv, const DecodeArgs& da, const int block, unsigned char*) {
    const int unit = block * 4 + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int item = by_hkv(unit), kvh = unit - item * da.Hkv;
    if (item >= da.n_items) return;
    if (item < da.n_wide) decode_body<D, 2, 1>(da, item, kvh);
    else decode_body<D, 1, 2>(da, item, kvh);
}
// one pair
template <int D>
__device__ __forceinline__ void decode_by_workgroup(const FastDiv& by_hkv, const DecodeArgs& da, const int block, unsigned char* lds) {
    const int item = by_hkv(block), kvh = block - item * da.Hkv;
    if (item < da.n_items) decode_group_body<D>(da, item, kvh, lds);
}
static_assert(kGroupLds<128> <= 5 * d128::TILE_BYTES && kGroupLds<64> <= 5 * d64::TILE_BYTES && kGroupWaves == 4, "decode_by_workgroup");
PK_MIXED_STEP_KERNEL(mixed_step_kernel, d128, 128, 2, decode_by_waves)
PK_MIXED_STEP_KERNEL(mixed_step64_kernel, d64, 64, 3, decode_by_waves)
PK_MIXED_STEP_KERNEL(mixed_step_few_kernel, few128, 128, 2, decode_by_waves)
PK_MIXED_STEP_KERNEL(mixed_step64_few_kernel, few64, 64, 2, decode_by_waves)
PK_MIXED_STEP_KERNEL(mixed_step_few_group_kernel, few128, 128, 2, decode_by_workgroup)
PK_MIXED_STEP_KERNEL(mixed_step64_few_group_kernel, few64, 64, 2, decode_by_workgroup)
PK_MIXED_STEP_KERNEL(mixed_step_group_kernel, d128, 128, 2, decode_by_workgroup)
PK_MIXED_STEP_KERNEL(mixed_step64_group_kernel, d64, 64, 3, decode_by_workgroup)
#undef PK_MIXED_STEP_KERNEL

}  // namespace

// bf16, d = 128 or 64.  Returns a hipError_t as int.
int launch_mixed_step_bf16(const PrefillArgs& args, const DecodeArgs& decode_args, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    PrefillArgs pa = args;
    DecodeArgs da = decode_args;
    da.heads_per_kv = pa.Hq / pa.Hkv;
    da.by_r = FastDiv::by(static_cast<uint32_t>(da.heads_per_kv));
    const int r = pa.heads_per_kv = da.heads_per_kv >> (2 - pa.row_shift);  // workgroups per (query tile, KV head)
    pa.by_r = FastDiv::by(static_cast<uint32_t>(r));
    pa.by_hkv = FastDiv::by(static_cast<uint32_t>(pa.Hkv));
    const int64_t pairs = static_cast<int64_t>(pa.n_tiles) * pa.Hkv;
    const int64_t n_prefill = (pairs + 7) / 8 * 8 * r;                      // as in the prefill launch (XCD map)
    const int64_t units = static_cast<int64_t>(da.n_items) * da.Hkv;
    const int64_t n_decode = da.arrived ? units : (units + 3) / 4;
    const int64_t P = n_prefill / 8, D = (n_decode + 7) / 8;
    const int64_t grid = (P + D) * 8;
    if (grid > 0x7FFFFFFF) return static_cast<int>(hipErrorInvalidValue);
    const MixedOrder m = MixedOrder::of(static_cast<int>(n_prefill), P, D);
    if (pa.d != da.d || (pa.d != 128 && pa.d != 64)) return static_cast<int>(hipErrorInvalidValue);
    if (grid > 0) {
        const dim3 wgs(static_cast<unsigned>(grid));
        if (pa.light) {
            if (pa.d == 128 && da.arrived) hipLaunchKernelGGL(mixed_step_few_group_kernel, wgs, dim3(256), 0, st, pa, da, m);
            else if (pa.d == 128) hipLaunchKernelGGL(mixed_step_few_kernel, wgs, dim3(256), 0, st, pa, da, m);
            else if (da.arrived) hipLaunchKernelGGL(mixed_step64_few_group_kernel, wgs, dim3(256), 0, st, pa, da, m);
            else hipLaunchKernelGGL(mixed_step64_few_kernel, wgs, dim3(256), 0, st, pa, da, m);
        } else if (pa.d == 128 && da.arrived) hipLaunchKernelGGL(mixed_step_group_kernel, wgs, dim3(256), 0, st, pa, da, m);
        else if (pa.d == 128) hipLaunchKernelGGL(mixed_step_kernel, wgs, dim3(256), 0, st, pa, da, m);
        else if (da.arrived) hipLaunchKernelGGL(mixed_step64_group_kernel, wgs, dim3(256), 0, st, pa, da, m);
        else hipLaunchKernelGGL(mixed_step64_kernel, wgs, dim3(256), 0, st, pa, da, m);
    }
    int e = static_cast<int>(hipGetLastError());
    if (e == 0) e = launch_prefill_merge_bf16(pa, stream);
    if (e != 0) return e;
    return da.arrived ? 0 : launch_decode_merge_bf16(da, stream);
}

}  // namespace pk
