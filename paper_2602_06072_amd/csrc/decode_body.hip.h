// Device code of the packed decode work item (Sec. 3.2), shared by the decode kernels and by the
// fused mixed-step kernel: one wave handles (work item, KV head), or the waves of a workgroup together.
#pragma once
#include <type_traits>

#include "arrival.h"
#include "common.hip.h"
#include "kernels.h"

namespace pk {
namespace {

constexpr int kNonTemporal = 2;                // cache policy of a buffer load

// maximum over the four lane groups of 16: rows 0/1 and 2/3 change places, then the halves of the wave
__device__ __forceinline__ float max_over_lane_groups(float x) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// SETS: register sets for tiles.  Rolling in each: the K part of the set's next tile is requested as soon as
// the scores of its present one are done and the V part as soon as P.V is done, so that all but one of
// the 2 * SETS half tiles are always in flight.  Every request is unconditional (past the last tile its
// descriptor is empty: zeros, no memory traffic): behind a condition the compiler waits for everything
// outstanding at the next use, since it has to take the smaller count of the two paths, and tiles are
// fetched and processed in turns.  Measured with and without the condition (and with permlane swaps for the
// LDS look-ups of the maximum): 256 requests of 32..32768 tokens 206.0 -> 201.6 us, four requests 12.1 ->
// 11.5, a tree of 128 63.1 -> 61.0, 16 families of 8 66.2 -> 64.9, 200 requests with D = 64 73.8 -> 73.2.
// The first tile is requested before the look-up of the requests (the other order: 65.6 and 74.1 us).
//
// What a wave has of a work item: lane (n, g) holds columns 16 t + 4 g .. + 3 of its query row 16 c + n.
template <int D, int NT>
struct ItemRows {
    int req[NT], hq[NT], slot[NT];             // request, query head and partial slot (-1: the item writes the output)
    bool ok[NT];                               // a request's row
    floatx4 o[NT][D / 16];                     // sum of p v, relative to m
    float m[NT], l[NT];                        // maximum (exp2 domain); sum of p
};

// Tiles first, first + STRIDE, ... of the item
template <int D, int NT, int SETS, int STRIDE>
__device__ __forceinline__ void decode_tiles(const DecodeArgs& a, const int item, const int kvh, const int first, ItemRows<D, NT>& rows) {
    constexpr int KS = D / 32;                 // K steps per 16-key sub-tile
    constexpr int VT = D / 16;                 // V column blocks
    constexpr int NK = 2 * KS;                 // 16-byte chunks per lane of a tile's K part
    constexpr int TILE_BYTES = 2 * 32 * D * 2; // K part + V part
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;   // (one wave per work item and KV head)
    const int r = a.heads_per_kv;
    const int32_t* it = a.items + 8 * static_cast<int64_t>(item);
    // the last item of a suffix also covers the tokens appended since the plan was made
    const int tok_begin = it[0], tok_end = it[1] + (it[4] ? a.grown : 0), mem_first = it[2], n_mem = it[3];
    const int64_t n_tiles = a.buf_tokens / 32;
    const unsigned char* base = static_cast<const unsigned char*>(a.kv_buf) + static_cast<int64_t>(kvh) * n_tiles * TILE_BYTES;
    const int lane16 = lane * 16;              // this lane's offset into a 1-KiB piece
    const int b0 = tok_begin / 32 + first, b1 = (tok_end + 31) / 32;

    u32x4 k0[NK], v0[VT], k1[SETS > 1 ? NK : 1], v1[SETS > 1 ? VT : 1];
    auto load = [&](auto& regs, int piece0, auto count, int b) {
        const __amdgpu_buffer_rsrc_t tile = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char*>(base + static_cast<int64_t>(b) * TILE_BYTES), 0, b < b1 ? TILE_BYTES : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < decltype(count)::value; ++i)
            regs[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(tile, lane16, (piece0 + i) * 1024, kNonTemporal));
    };
    auto load_k = [&](auto& kr, int b) { load(kr, 0, std::integral_constant<int, NK>{}, b); };
    auto load_v = [&](auto& vr, int b) { load(vr, NK, std::integral_constant<int, VT>{}, b); };
    load_k(k0, b0);
    __builtin_amdgcn_sched_barrier(0);
    load_v(v0, b0);
    __builtin_amdgcn_sched_barrier(0);

    // rows without a request repeat the last one (their column of the MFMAs is nobody else's) and store nothing
    int (&req_of)[NT] = rows.req, (&hq_of)[NT] = rows.hq, (&slot_of)[NT] = rows.slot;
    bool (&ok)[NT] = rows.ok;
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        const int mi = a.by_r(c * 16 + n), mc = min(mi, n_mem - 1);
        ok[c] = mi < n_mem;
        req_of[c] = a.members[mem_first + mc];
        slot_of[c] = a.member_slot[mem_first + mc];
        hq_of[c] = kvh * r + (c * 16 + n) - mi * r;
    }

    // query operand (B side): lane (n, g) holds Q[row n][32s + 8g .. +8]
    bf16x8 qf[NT][KS];
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int s = 0; s < KS; ++s)
            qf[c][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(
                static_cast<const uint16_t*>(a.q) + (static_cast<int64_t>(req_of[c]) * a.Hq + hq_of[c]) * D + 32 * s + 8 * g));

    floatx4 (&o)[NT][VT] = rows.o;
    float (&m)[NT] = rows.m, (&l)[NT] = rows.l;
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        m[c] = -INFINITY; l[c] = 0.f;
#pragma unroll
        for (int t = 0; t < VT; ++t) o[c][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const float sl2 = a.scale * kLog2e;

    // scores and probabilities of tile b for column tile c: leaves P (bf16, B operand) and the
    // factor alpha for what has been accumulated so far
    auto scores = [&](const auto& kraw, int b, int c, bf16x8& pf, float& alpha) {
        const bool edge = (b * 32 < tok_begin) || (b * 32 + 32 > tok_end);
        floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kraw[s]), qf[c][s], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kraw[KS + s]), qf[c][s], s1, 0, 0, 0);
        }
        // lane (n, g) now holds scores of row n against keys 32b + 16u + 4g + j
        float x[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) { x[j] = s0[j] * sl2; x[4 + j] = s1[j] * sl2; }
        if (edge) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int key = b * 32 + (j < 4 ? 4 * g + j : 16 + 4 * g + (j - 4));
                if (key < tok_begin || key >= tok_end) x[j] = -INFINITY;
            }
        }
        float mx = x[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) mx = fmaxf(mx, x[j]);
        mx = max_over_lane_groups(mx);
        const float m_new = fmaxf(m[c], mx);
        const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
        alpha = __builtin_amdgcn_exp2f(m[c] - m_use);      // 0 on the first tile
        float ps = 0.f;
        uint32_t pw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            floatx2 pp;
            pp[0] = __builtin_amdgcn_exp2f(x[2 * j] - m_use);
            pp[1] = __builtin_amdgcn_exp2f(x[2 * j + 1] - m_use);
            ps += pp[0] + pp[1];
            pw[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
        }
        l[c] = l[c] * alpha + ps;
        m[c] = m_new;
        pf = __builtin_bit_cast(bf16x8, u32x4{pw[0], pw[1], pw[2], pw[3]});
    };
    auto pv = [&](const auto& vraw, int c, const bf16x8& pf, float alpha) {
#pragma unroll
        for (int t = 0; t < VT; ++t) {
            floatx4 acc = o[c][t];
            acc[0] *= alpha; acc[1] *= alpha; acc[2] *= alpha; acc[3] *= alpha;
            o[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vraw[t]), pf, acc, 0, 0, 0);
        }
    };
    // one tile, and the requests for the one that replaces it (the barriers keep them here: hoisted, they
    // need registers of their own)
    auto step = [&](auto& kr, auto& vr, int b, auto fetch) {
        bf16x8 pf[NT];
        float alpha[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) scores(kr, b, c, pf[c], alpha[c]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(fetch)::value) load_k(kr, b + SETS * STRIDE);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NT; ++c) pv(vr, c, pf[c], alpha[c]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(fetch)::value) load_v(vr, b + SETS * STRIDE);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Q came last: it is waited for here, so that inside the loop only the tiles are
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SETS == 1) {
        __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0)
        for (int b = b0; b < b1; b += STRIDE) step(k0, v0, b, std::true_type{});
    } else {
        load_k(k1, b0 + STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        load_v(v1, b0 + STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0F70 | ((NK + VT) & 0xF) | ((NK + VT) >> 4 << 14));   // vmcnt: the second set alone
        int b = b0;
        for (; b + STRIDE < b1; b += 2 * STRIDE) {
            step(k0, v0, b, std::true_type{});
            step(k1, v1, b + STRIDE, std::true_type{});
        }
        if (b < b1) step(k0, v0, b, std::false_type{});
    }

#pragma unroll
    for (int c = 0; c < NT; ++c) {
        l[c] += __shfl_xor(l[c], 16, 64);
        l[c] += __shfl_xor(l[c], 32, 64);
    }
}

// Four columns of a row of the output.
template <int D>
__device__ __forceinline__ void store_columns(const DecodeArgs& a, const int64_t dst, const floatx4 x) {
    if (a.out_f32)
        *reinterpret_cast<float4*>(static_cast<float*>(a.out) + dst) = make_float4(x[0], x[1], x[2], x[3]);
    else
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + dst) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
}
__device__ __forceinline__ float row_lse(const float m, const float l) { return l > 0.f ? (m + log2f(l)) * kLn2 : -INFINITY; }

// one wave for the whole item
template <int D, int NT, int SETS>
__device__ __forceinline__ void decode_body(const DecodeArgs& a, const int item, const int kvh) {
    ItemRows<D, NT> r;
    decode_tiles<D, NT, SETS, 1>(a, item, kvh, 0, r);
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        if (!r.ok[c]) continue;
        const float inv = r.l[c] > 0.f ? 1.f / r.l[c] : 0.f;
        // (which of the two is asked once per row: once per store it is 110 instructions and 14 branches more, 2 to 3 % of a launch of 10 us)
        if (r.slot[c] < 0) {                       // the only work item of this request: write the final output
            const int64_t dst = (static_cast<int64_t>(r.req[c]) * a.Hq + r.hq[c]) * D + 4 * g;
#pragma unroll
            for (int t = 0; t < D / 16; ++t) store_columns<D>(a, dst + 16 * t, r.o[c][t] * inv);
            continue;
        }
        const int64_t row = static_cast<int64_t>(r.slot[c]) * a.Hq + r.hq[c];
        float* po = a.part_o + row * D + 4 * g;
#pragma unroll
        for (int t = 0; t < D / 16; ++t) {
            const floatx4 x = r.o[c][t] * inv;
            *reinterpret_cast<float4*>(po + 16 * t) = make_float4(x[0], x[1], x[2], x[3]);
        }
        if (g == 0) a.part_lse[row] = row_lse(r.m[c], r.l[c]);
    }
}

// Partial results that another workgroup of the same launch reads: written through to memory, and read past whatever an L2 has
// of an earlier launch (relaxed atomics at device scope).  The order between them and the count comes from instructions and not from
// the memory model's: gfx950 counts a device-scope store as done (vmcnt) when it has been written through, so a wave that waits for its
// stores before the barrier in front of the count has published them; a release would also write back the whole L2.
__device__ __forceinline__ void publish(float* p, const floatx4 x) {
    uint64_t* q = reinterpret_cast<uint64_t*>(p);
    __hip_atomic_store(q, __builtin_bit_cast(uint64_t, floatx2{x[0], x[1]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, __builtin_bit_cast(uint64_t, floatx2{x[2], x[3]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
struct DeviceCount {
    uint32_t* x;
    __device__ __forceinline__ uint32_t next(const uint32_t limit) const {
        return __builtin_amdgcn_atomic_inc32(x, limit, __ATOMIC_RELAXED, "agent");
    }
};
__device__ __forceinline__ floatx4 read_published(const float* p) {
    const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
    const floatx2 a = __builtin_bit_cast(floatx2, __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const floatx2 b = __builtin_bit_cast(floatx2, __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return floatx4{a[0], a[1], b[0], b[1]};
}

// A batch in one launch: a workgroup takes a work item of one request, its waves the item's tiles in turns, and
// puts their results together in LDS; the workgroup that is the last to finish an item of a (request, KV head) merges
// the partial results of all of them, in the order of their slots whichever workgroup it is.  Nobody waits for another workgroup.
// Short batches are bound by latency: a launch, two to four round trips for tables, Q and the first tiles, the tiles, and
// for split requests a write, a count and a read at the memory side (about 2 us) in place of a second launch (4 to 5 us).
// Long ones are bound by HBM; there four waves to an item leave fewer items, starts, ends and partial results: 480 rows of up to
// 65536 tokens 2.86 -> 2.59 ms (6.9 TB/s), 256 requests of 32..32768 201 -> 194 us, one request of 500 tokens 8.9 -> 6.3 us,
// four of 300..3000 10.2 -> 9.6 us.  With eight waves to an item the one request takes 6.8 us; with
// batches of 16 partial results in the merge instead of 8 the four take 10.4 us, with 4 9.9.
// `lds`: kGroupLds<D> bytes; a.arrived: a count per (request, KV head), zero between launches (arrival.h).
constexpr int kGroupWaves = 4;
template <int D> constexpr int kGroupLds = kGroupWaves * 16 * (D + 4 + 2) * 4 + 16;
template <int D>
__device__ __forceinline__ void decode_group_body(const DecodeArgs& a, const int item, const int kvh, unsigned char* lds) {
    constexpr int WAVES = kGroupWaves, PITCH = D + 4;          // (16 bytes more: the 16 rows of a lane group on different banks)
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    float* po = reinterpret_cast<float*>(lds);                 // [WAVES][16][PITCH]
    float* pm = po + WAVES * 16 * PITCH;                       // [WAVES][16]: maxima, then sums
    float* pl = pm + WAVES * 16;
    int* last = reinterpret_cast<int*>(pl + WAVES * 16);
    {
        ItemRows<D, 1> r;
        decode_tiles<D, 1, 2, WAVES>(a, item, kvh, wave, r);
#pragma unroll
        for (int t = 0; t < D / 16; ++t) *reinterpret_cast<floatx4*>(po + (wave * 16 + n) * PITCH + 16 * t + 4 * g) = r.o[0][t];
        if (g == 0) { pm[wave * 16 + n] = r.m[0]; pl[wave * 16 + n] = r.l[0]; }
    }
    const int mem = a.items[8 * static_cast<int64_t>(item) + 2];
    const int req = a.members[mem], slot = a.member_slot[mem];
    __syncthreads();
    const int heads = a.heads_per_kv, hq0 = kvh * heads;
    for (int x = threadIdx.x; x < heads * (D / 4); x += 64 * WAVES) {
        const int row = x / (D / 4), col = 4 * (x % (D / 4));
        float mx = pm[row];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, pm[w * 16 + row]);
        const float m_use = mx == -INFINITY ? 0.f : mx;
        float l = 0.f;
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = __builtin_amdgcn_exp2f(pm[w * 16 + row] - m_use);
            const floatx4 v = *reinterpret_cast<const floatx4*>(po + (w * 16 + row) * PITCH + col);
            l = fmaf(f, pl[w * 16 + row], l);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(f, v[e], o[e]);
        }
        o *= l > 0.f ? 1.f / l : 0.f;
        if (slot < 0) {
            store_columns<D>(a, (static_cast<int64_t>(req) * a.Hq + hq0 + row) * D + col, o);
        } else {
            publish(a.part_o + (static_cast<int64_t>(slot) * a.Hq + hq0 + row) * D + col, o);
            if (col == 0)
                __hip_atomic_store(a.part_lse + static_cast<int64_t>(slot) * a.Hq + hq0 + row,
                                   row_lse(mx, l), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (slot < 0) return;
    const int p0 = a.req_part_start[req], p1 = a.req_part_start[req + 1];
    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wave's partial results are in memory
    __syncthreads();
    if (threadIdx.x == 0) {
        const DeviceCount count{reinterpret_cast<uint32_t*>(a.arrived) + static_cast<int64_t>(req) * a.Hkv + kvh};
        *last = arrives_last(count, static_cast<uint32_t>(p1 - p0));
    }
    __syncthreads();
    if (*last == 0) return;
    // out[req, h, :] = sum_j exp(lse_j - lse) o_j over the request's slots, in batches as in decode_merge_kernel
    constexpr int BATCH = 8;
    for (int x = threadIdx.x; x < heads * (D / 4); x += 64 * WAVES) {
        const int row = x / (D / 4), col = 4 * (x % (D / 4));
        const float* lse_base = a.part_lse + hq0 + row;
        const float* o_base = a.part_o + static_cast<int64_t>(hq0 + row) * D + col;
        float m = -INFINITY, tot = 0.f;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int p = p0; p < p1; p += BATCH) {
            float lse[BATCH];
            floatx4 v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int q = min(p + u, p1 - 1);
                lse[u] = __hip_atomic_load(lse_base + static_cast<int64_t>(q) * a.Hq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                v[u] = read_published(o_base + static_cast<int64_t>(q) * a.Hq * D);
            }
            float m_new = m;
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                if (p + u >= p1) lse[u] = -INFINITY;
                m_new = fmaxf(m_new, lse[u]);
            }
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = expf(m - m_use);
            tot *= alpha;
            acc *= alpha;
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const float w = expf(lse[u] - m_use);
                tot += w;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = fmaf(w, v[u][e], acc[e]);
            }
            m = m_new;
        }
        store_columns<D>(a, (static_cast<int64_t>(req) * a.Hq + hq0 + row) * D + col, acc * (tot > 0.f ? 1.f / tot : 0.f));
    }
}

}  // namespace
}  // namespace pk
