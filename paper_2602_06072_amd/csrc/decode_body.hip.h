// Device code of the packed decode work item (Sec. 3.2), shared by the decode kernels and by the
// fused mixed-step kernel: one wave handles (work item, KV head).
#pragma once
#include <type_traits>

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
template <int D, int NT, int SETS>
__device__ __forceinline__ void decode_body(const DecodeArgs& a, const int item, const int kvh) {
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
    const int b0 = tok_begin / 32, b1 = (tok_end + 31) / 32;

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
    int req_of[NT], hq_of[NT], slot_of[NT];
    bool ok[NT];
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

    floatx4 o[NT][VT];
    float m[NT], l[NT];
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
        if constexpr (decltype(fetch)::value) load_k(kr, b + SETS);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NT; ++c) pv(vr, c, pf[c], alpha[c]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(fetch)::value) load_v(vr, b + SETS);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Q came last: it is waited for here, so that inside the loop only the tiles are
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SETS == 1) {
        __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0)
        for (int b = b0; b < b1; ++b) step(k0, v0, b, std::true_type{});
    } else {
        load_k(k1, b0 + 1);
        __builtin_amdgcn_sched_barrier(0);
        load_v(v1, b0 + 1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0F70 | ((NK + VT) & 0xF) | ((NK + VT) >> 4 << 14));   // vmcnt: the second set alone
        int b = b0;
        for (; b + 1 < b1; b += 2) {
            step(k0, v0, b, std::true_type{});
            step(k1, v1, b + 1, std::true_type{});
        }
        if (b < b1) step(k0, v0, b, std::false_type{});
    }

#pragma unroll
    for (int c = 0; c < NT; ++c) {
        float lt = l[c];
        lt += __shfl_xor(lt, 16, 64);
        lt += __shfl_xor(lt, 32, 64);
        if (!ok[c]) continue;
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        if (slot_of[c] < 0) {
            // the only work item of this request: write the final output
            const int64_t dst = (static_cast<int64_t>(req_of[c]) * a.Hq + hq_of[c]) * D;
#pragma unroll
            for (int t = 0; t < VT; ++t) {
                const float x0 = o[c][t][0] * inv, x1 = o[c][t][1] * inv, x2 = o[c][t][2] * inv, x3 = o[c][t][3] * inv;
                if (a.out_f32)
                    *reinterpret_cast<float4*>(static_cast<float*>(a.out) + dst + 16 * t + 4 * g) = make_float4(x0, x1, x2, x3);
                else
                    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + dst + 16 * t + 4 * g) =
                        make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
            }
            continue;
        }
        const int slot = slot_of[c];
        float* po = a.part_o + (static_cast<int64_t>(slot) * a.Hq + hq_of[c]) * D;
#pragma unroll
        for (int t = 0; t < VT; ++t) {
            float4 w = make_float4(o[c][t][0] * inv, o[c][t][1] * inv, o[c][t][2] * inv, o[c][t][3] * inv);
            *reinterpret_cast<float4*>(po + 16 * t + 4 * g) = w;
        }
        if (g == 0)
            a.part_lse[static_cast<int64_t>(slot) * a.Hq + hq_of[c]] =
                lt > 0.f ? (m[c] + log2f(lt)) * kLn2 : -INFINITY;
    }
}

}  // namespace
}  // namespace pk
