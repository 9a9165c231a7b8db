// Host-callable launchers of the gfx950 kernels.  Every launcher enqueues on
// `stream` and returns the hipError_t of the launch as int (0 = success).
// All pointers are device pointers.
#pragma once
#include <cstdint>

#include "arrival.h"

namespace pk {

// Copies `bytes` (a multiple of 16) from pinned host memory to device memory, then stores `stamp` to the
// pinned host word `done`.  Weak: the host code also links without any kernels (null then), and copies by command.
__attribute__((weak)) int launch_upload(const void* src, void* dst, int64_t bytes, uint32_t* done, uint32_t stamp, void* stream);

struct ReorgArgs {
    const void* k_pages; const void* v_pages;       // [num_blocks][page][Hkv][d]
    const int32_t* block_table; int32_t max_blocks; int32_t page_size; int64_t num_blocks;
    const int32_t* seg; int32_t n_seg;              // [n_seg][4]
    const int32_t* blk_first;                       // [n_tiles]
    void* kv_buf; int64_t buf_tokens; int Hkv; int d;
};
int launch_reorg_bf16(const ReorgArgs& a, void* stream);
int launch_reorg_f32(const ReorgArgs& a, void* stream);

struct AppendArgs {
    const void* k_new; const void* v_new;           // [n][Hkv][d]
    void* kv_buf; const int32_t* req_seg;           // [n][4]: prefix_off, L_P, suffix_off, L_Q (absolute tokens)
    int64_t buf_tokens; int32_t n; int32_t step; int Hkv; int d;
};
int launch_append_bf16(const AppendArgs& a, void* stream);
int launch_append_f32(const AppendArgs& a, void* stream);

// Division of 0 <= x < 2^31 by a launch constant as a multiplication: x / d = x * mul >> (31 + shift), exact
// because mul = ceil(2^(31 + shift) / d) with 2^shift >= d.  (A division by a kernel argument is a
// sequence of some forty dependent instructions that every workgroup runs before it knows its work.)
struct FastDiv {
    uint32_t mul, shift;
    static FastDiv by(uint32_t d) {
        uint32_t s = 0;
        while ((1u << s) < d) ++s;
        return {static_cast<uint32_t>(((uint64_t{1} << (31 + s)) + d - 1) / d), s};
    }
    PK_HOST_DEVICE int operator()(int x) const {
        return static_cast<int>(static_cast<uint64_t>(static_cast<uint32_t>(x)) * mul >> (31 + shift));
    }
};

struct DecodeArgs {
    const void* q; const void* kv_buf; void* out;
    const int32_t* items; int32_t n_items; int32_t n_wide;   // the first n_wide items have > 16 query rows
    const int32_t* members; const int32_t* member_slot;
    const int32_t* req_part_start;
    const int32_t* req_seg;
    const int32_t* chain_start; const int32_t* chain;   // per request: (offset, tokens) of its shared segments
    float* part_o; float* part_lse;
    int64_t buf_tokens; int32_t n; int Hq; int Hkv; int d; float scale; int out_f32;
    int32_t grown;                                  // tokens appended to every suffix since the plan was made
    int32_t max_parts;                              // most partial results of one request
    int32_t* arrived;                               // not null: a workgroup per (work item, KV head), which counts itself in here ([n][Hkv])
    int heads_per_kv; FastDiv by_r, by_hkv;         // set by the bf16 launches: Hq / Hkv, divisions by it and by Hkv
};
int launch_decode_bf16(const DecodeArgs& a, void* stream);
int launch_decode_merge_bf16(const DecodeArgs& a, void* stream);   // the LSE merge alone
// Device address of the library's fixed scratch array on the current device (looked up once per
// device); returns a hipError_t as int.
int static_scratch_address(void** ptr);
int launch_decode_f32(const DecodeArgs& a, void* stream);

struct PrefillArgs {
    const void* q; const void* k; const void* v; void* out;
    const int32_t* tiles; int32_t n_tiles;
    const int32_t* run_first; const int32_t* runs;   // rows of a tile beyond its first run of consecutive rows
    const int32_t* kvtiles;
    const int32_t* q_start; const int32_t* kv_start; int32_t n;
    int64_t total_q_rows; int64_t total_kv_rows;
    int Hq; int Hkv; int d; float scale; int out_f32;
    int pipeline;                                   // 0: K/V tiles copied straight into LDS; 1: staged through registers
    int eight;                                      // pipeline 0: workgroups of eight waves
    int row_shift;                                  // a query tile has 32 << row_shift rows; a workgroup's waves take them 32 at a time, for as many heads as there are waves
    int light;                                      // pipeline 0: a launch of little work, prefill_few_body.hip.h
    int through;                                    // of those: the output is written through the L2
    // lists cut into pieces (light launches): `tiles` are the pieces then, and what they leave in `part` is put together by a second launch
    float* part;
    const int32_t* merges; int32_t n_merges;        // [n_merges][4] first slot, pieces, Q row of tile row 0, rows of a tile whose list is cut
    int heads_per_kv; FastDiv by_r, by_hkv;         // set by the launches of pipeline 0: workgroups per (query tile, KV head), divisions by it and by Hkv
};
#if defined(__HIPCC__)
// Row `local` (0..127) of query tile `tile`: its Q row (-1: padding) and its key range [lo, hi).
// d4..d7 are words 4..7 of the tile's descriptor (rows | runs << 16; Q row, lo, hi of tile row 0).
// A run is a stretch of consecutive rows of one request: inside it the Q row and hi advance by one
// per row.  Tiles of one run (nearly all) need nothing but the descriptor.
__device__ __forceinline__ void prefill_tile_row(const PrefillArgs& a, int tile, int d4, int d5, int d6, int d7,
                                                 int local, int& qrow, int& lo, int& hi) {
    const int n_rows = d4 & 0xFFFF, n_runs = d4 >> 16;
    int begin = 0, q0 = d5, l0 = d6, h0 = d7;
    if (n_runs > 1) {                               // uniform: a packed tile that holds several requests
        const int32_t* rp = a.runs + 4 * static_cast<int64_t>(a.run_first[tile]);
        for (int r = 1; r < n_runs; ++r, rp += 4) {
            const int rb = rp[0];
            if (local >= rb) { begin = rb; q0 = rp[1]; l0 = rp[2]; h0 = rp[3]; }
        }
    }
    const bool valid = local < n_rows;
    qrow = valid ? q0 + (local - begin) : -1;
    lo = valid ? l0 : 0;
    hi = valid ? h0 + (local - begin) : 0;
}
#endif
int launch_prefill_bf16(const PrefillArgs& a, void* stream);
int launch_prefill_f32(const PrefillArgs& a, void* stream);
int launch_prefill_merge_bf16(const PrefillArgs& a, void* stream);   // nothing where no list is cut; heads_per_kv and the divisions set
// prefill tiles and decode work items of one step in one launch (bf16, d = 128), then the LSE merge
int launch_mixed_step_bf16(const PrefillArgs& pa, const DecodeArgs& da, void* stream);

struct PagedDecodeArgs {
    const void* q; const void* k_pages; const void* v_pages; void* out;
    const int32_t* block_table; int32_t max_blocks; int32_t page_size; int64_t num_blocks;
    const int32_t* kv_start;                        // [n+1] cumulative kv_lens
    float* part_o; float* part_lse;
    int32_t n; int32_t n_splits; int32_t split_tokens;
    int Hq; int Hkv; int d; float scale; int out_f32;
};
int launch_padded_decode_bf16(const PagedDecodeArgs& a, void* stream);

}  // namespace pk
