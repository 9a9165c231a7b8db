// Packed decode attention (Sec. 3.2): one query row per request over the
// group-contiguous buffer, split-KV partials and a log-sum-exp merge.
//
// A work item is a run of buffer tokens [tok_begin, tok_end) of one segment
// (a shared prefix or a private suffix) together with the requests whose
// queries attend to it: one request for a suffix, all members of the
// (sub-)family for a prefix -- the prefix is streamed from HBM once and used
// for every member's rows.  One wave handles (work item, KV head) -- or, in batches
// without shared prefixes, a workgroup that merges in the same launch --: the query
// rows of up to 32/r requests x r heads sit on the N side of 16x16x32 bf16
// MFMAs, the buffer tiles are already in MFMA operand order, so every load is
// a fully coalesced 16-byte-per-lane read straight into the operand
// registers (no LDS).  HBM-bound: 4*D bytes per token and KV head.
#include <mutex>

#include "../../include/packinfer.h"
#include "common.hip.h"
#include "decode_body.hip.h"
#include "kernels.h"

namespace pk {
namespace {

// Work items with at most 16 query rows: one column tile, two register sets (204 registers for D = 128).
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void decode_bf16_kernel(DecodeArgs a) {
    const int item = a.by_hkv(blockIdx.x), kvh = blockIdx.x - item * a.Hkv;
    decode_body<D, 1, 2>(a, item, kvh);
}

// Batches with shared prefixes: the first n_wide work items carry 17..32 query rows (two column
// tiles) and have registers for one set.  Both kinds run in ONE launch so that the short prefix pass and
// the suffix pass fill the chip together.
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void decode_bf16_mixed_kernel(DecodeArgs a) {
    const int item = a.by_hkv(blockIdx.x), kvh = blockIdx.x - item * a.Hkv;
    if (item < a.n_wide) decode_body<D, 2, 1>(a, item, kvh);
    else decode_body<D, 1, 2>(a, item, kvh);
}

// Batches whose items carry up to 16 rows of one request each (DecodeArgs::arrived; the schedule builder's choice): one launch.
template <int D>
__global__ __launch_bounds__(64 * kGroupWaves, 2) void decode_bf16_group_kernel(DecodeArgs a) {
    __shared__ __align__(16) unsigned char lds[kGroupLds<D>];
    const int item = a.by_hkv(blockIdx.x), kvh = blockIdx.x - item * a.Hkv;
    decode_group_body<D>(a, item, kvh, lds);
}

// out[i, h, :] = sum_j exp(lse_j - lse) o_j over the request's partial slots (consecutive).
// Workgroup = (request, 256 / D heads): a lane owns four columns of one head and a wave's load is 1 KiB of one
// slot.  Wave w takes slots w, w + WAVES, ... in batches of kBatch, weighted against the batch's own
// maximum (an earlier sum is rescaled), so that the partial results and their lse are requested together
// instead of one after the other; with more than one wave the sums meet in LDS.  Requests with a single
// work item were written by the decode kernel and are skipped.
constexpr int kBatch = 8;

template <int D, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void decode_merge_kernel(DecodeArgs a) {
    constexpr int HPW = 256 / D;                   // heads per workgroup
    __shared__ floatx4 red_acc[WAVES][64];
    __shared__ float red_m[WAVES][64], red_tot[WAVES][64];
    const int i = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = WAVES > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int p0 = a.req_part_start[i], p1 = a.req_part_start[i + 1];
    if (p1 <= p0) return;
    const int h = blockIdx.y * HPW + lane * 4 / D, col = lane * 4 % D;
    const int hr = h < a.Hq ? h : a.Hq - 1;        // (lanes beyond the last head repeat it and store nothing)
    const float* lse_base = a.part_lse + hr;
    const float* o_base = a.part_o + static_cast<int64_t>(hr) * D + col;
    const int64_t o_stride = static_cast<int64_t>(a.Hq) * D;
    float m = -INFINITY, tot = 0.f;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int p = p0 + wave; p < p1; p += kBatch * WAVES) {
        float lse[kBatch];
        floatx4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int q = p + WAVES * u;
            lse[u] = q < p1 ? lse_base[static_cast<int64_t>(q) * a.Hq] : -INFINITY;
            v[u] = q < p1 ? *reinterpret_cast<const floatx4*>(o_base + q * o_stride) : floatx4{0.f, 0.f, 0.f, 0.f};
        }
        float m_new = m;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) m_new = fmaxf(m_new, lse[u]);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = expf(m - m_use);
        tot *= alpha;
        acc *= alpha;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float w = expf(lse[u] - m_use);
            tot += w;
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fmaf(w, v[u][c], acc[c]);
        }
        m = m_new;
    }
    if constexpr (WAVES > 1) {
        red_acc[wave][lane] = acc;
        red_m[wave][lane] = m;
        red_tot[wave][lane] = tot;
        __syncthreads();
        if (wave != 0) return;
        float mx = m;
#pragma unroll
        for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, red_m[w][lane]);
        const float m_use = mx == -INFINITY ? 0.f : mx;
        tot = 0.f;
        acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = expf(red_m[w][lane] - m_use);
            tot = fmaf(f, red_tot[w][lane], tot);
            const floatx4 x = red_acc[w][lane];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fmaf(f, x[c], acc[c]);
        }
    }
    if (h >= a.Hq) return;
    const float inv = tot > 0.f ? 1.f / tot : 0.f;
    const int64_t dst = (static_cast<int64_t>(i) * a.Hq + h) * D + col;
    if (a.out_f32)
        *reinterpret_cast<float4*>(static_cast<float*>(a.out) + dst) = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    else
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + dst) =
            make_uint2(pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv));
}

// One wave takes up to two batches: with 16 partial results a request, four waves that meet in LDS take as
// long (72.7 and 72.5 us for 16 families of 8, 69.8 and 69.4 us for a tree of 128) and occupy four times the
// wave slots.  The kernel is bound by its three dependent round trips to memory (slot range, partial results,
// output); one column pair per lane, one head per workgroup and the maximum before the sum took
// four: decode and merge 12.2 -> 11.4 us for four requests, 72.3 -> 69.4 us for that tree.
constexpr int kOneWaveParts = 2 * kBatch;
// Few long sequences leave hundreds of partial results to a workgroup: with sixteen waves instead of four, decode
// and merge of 3 sequences of up to 65536 tokens and one KV head 25.7 -> 18.9 us, of 2 17.2 -> 12.6 us, of one with
// eight KV heads 22.2 -> 21.1 us.
constexpr int kFourWaveParts = 2 * 4 * kBatch;

template <int D>
void launch_merge(const DecodeArgs& a, hipStream_t st) {
    if (a.n > 0 && a.max_parts > 0) {
        const dim3 mgrid(static_cast<unsigned>(a.n), static_cast<unsigned>((a.Hq + 256 / D - 1) / (256 / D)));
        if (a.max_parts <= kOneWaveParts) hipLaunchKernelGGL((decode_merge_kernel<D, 1>), mgrid, dim3(64), 0, st, a);
        else if (a.max_parts <= kFourWaveParts) hipLaunchKernelGGL((decode_merge_kernel<D, 4>), mgrid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((decode_merge_kernel<D, 16>), mgrid, dim3(1024), 0, st, a);
    }
}

template <int D>
int launch_d(const DecodeArgs& a, hipStream_t st) {
    if (a.n_items > 0) {
        // The KV head is the fastest index.  Workgroup numbers go round-robin over the eight XCDs, so that (with
        // eight KV heads) an XCD streams the tiles of one head, an eighth of the buffer, instead of touching
        // all of it: 200 requests with D = 64 83.4 -> 76.2 us, a tree of 128 69.0 -> 63.1 us, 16 families of 8
        // 72.4 -> 68.5 us, 256 requests of 32..32768 tokens 213.9 -> 205.5 us.
        const int64_t waves = static_cast<int64_t>(a.n_items) * a.Hkv;
        if (waves > 0x7FFFFFFF) return static_cast<int>(hipErrorInvalidValue);
        const dim3 grid(static_cast<unsigned>(waves));
        if (a.arrived) {
            hipLaunchKernelGGL(decode_bf16_group_kernel<D>, grid, dim3(64 * kGroupWaves), 0, st, a);
            return static_cast<int>(hipGetLastError());
        }
        if (a.n_wide > 0) hipLaunchKernelGGL(decode_bf16_mixed_kernel<D>, grid, dim3(64), 0, st, a);
        else hipLaunchKernelGGL(decode_bf16_kernel<D>, grid, dim3(64), 0, st, a);
    }
    launch_merge<D>(a, st);
    return static_cast<int>(hipGetLastError());
}

}  // namespace

// Scratch of pk_packed_decode_attn_static (plan tables + split-KV partials) for callers that
// cannot allocate.  In host code the array's name is only a handle for hipGetSymbolAddress: the
// device address differs per GPU and is looked up once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[PK_STATIC_SCRATCH_BYTES];

int static_scratch_address(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mutex;
    static void* address[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_cast<int>(e);
    if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> lock(mutex);
    if (!address[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return static_cast<int>(e);
        if (!p) return static_cast<int>(hipErrorInvalidSymbol);
        address[dev] = p;
    }
    *ptr = address[dev];
    return 0;
}

int launch_decode_merge_bf16(const DecodeArgs& a, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.d == 128) launch_merge<128>(a, st);
    else if (a.d == 64) launch_merge<64>(a, st);
    else return static_cast<int>(hipErrorInvalidValue);
    return static_cast<int>(hipGetLastError());
}

int launch_decode_bf16(const DecodeArgs& args, void* stream) {
    DecodeArgs a = args;
    a.heads_per_kv = a.Hq / a.Hkv;
    a.by_r = FastDiv::by(static_cast<uint32_t>(a.heads_per_kv));
    a.by_hkv = FastDiv::by(static_cast<uint32_t>(a.Hkv));
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (a.d == 128) return launch_d<128>(a, st);
    if (a.d == 64) return launch_d<64>(a, st);
    return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace pk
