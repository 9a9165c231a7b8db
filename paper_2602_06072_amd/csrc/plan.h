// Internal structures of the packing plan and of its device tables.
// Host-side only; the device kernels see the tables as plain int32 arrays.
#pragma once
#include <cstddef>
#include <cstdint>
#include <exception>
#include <new>
#include <string>
#include <vector>

#include "../../include/packinfer.h"

namespace pk {

// ---- tile shapes shared by the schedule builder and the kernels -----------
constexpr int kPrefillBM = 128;     // query rows per workgroup tile (4 waves x 32)
constexpr int kPrefillBN = 64;      // keys per K/V tile
constexpr int kDecodeBlock = PK_KV_BLOCK;   // tokens per buffer tile
constexpr int kDecodeMaxRows = 32;  // query rows (members x heads-per-KV-head) per work item
constexpr int kTileDescWords = 16;  // int32 words per query-tile descriptor of the prefill schedules (one 64-byte scalar load)

struct Member {                     // O_g[i] of Alg. 1 Part 2, offsets relative to the group base
    int32_t req, prefix_off, lp, suffix_off, lq;   // prefix_off / lp: the innermost shared segment (suffix_off / 0: none)
    int32_t node = -1;              // index of that segment in Group::nodes
    int32_t shared = 0;             // tokens of the request that lie in shared segments (its suffix starts there)
};

struct Node {                       // a shared segment of the group's prefix forest (Sec. 3.2, Eq. 5)
    int32_t id = 0;                 // the caller's node number (tree plans) or a running number
    int32_t off = 0, len = 0;       // where it lies in the group buffer
    int32_t parent = -1;            // index in Group::nodes; parents come first
    int32_t start = 0;              // logical token position of its first token inside a request
    std::vector<int32_t> reqs;      // the requests below it, ascending
};

struct Group {
    int64_t load = 0;               // L(S_g): unique KV tokens
    int64_t buf_tokens = 0;         // M(S_g) incl. headroom
    int64_t buf_base = 0;           // token offset of B_g inside the buffer
    std::vector<Member> members;    // layout order
    std::vector<Node> nodes;        // layout order (a one-level family is one node)
};

// One array inside the workspace.
struct TableRef {
    size_t offset = 0;              // bytes from the workspace base
    size_t count = 0;               // int32 elements
};

// Host image of everything that is copied to the device for one head shape.
struct DeviceTables {
    int Hq = 0, Hkv = 0, d = 0, dtype = -1;
    std::vector<int32_t> host;      // concatenated tables (each 64-int aligned)
    // common
    TableRef q_start, kv_start;     // [n+1] caller-order cumulative rows
    // re-layout
    TableRef reorg_seg;             // [nseg][4] dst0, ntok, req, src0 (sorted by dst0)
    TableRef reorg_blk_first;       // [NB] first segment that may overlap tile b
    int32_t n_reorg_seg = 0;
    // decode
    struct DecodeSched {
        TableRef items;             // [n_items][8]
        TableRef members;           // request ids of the work items' rows
        TableRef member_slot;       // partial slot of each (item, member), -1: the item writes the output
        TableRef req_part_start;    // [n+1] first slot of each request (slots of a request are consecutive)
        TableRef arrived;           // group: [n][Hkv] zeros, how many of its items have finished
        int32_t n_items = 0, n_members = 0, n_wide = 0, n_parts = 0, split_tokens = 0;   // (shared segments may have a split of their own)
        int32_t max_parts = 0;      // most partial results of one request
        bool group = false;         // a workgroup of several waves per (work item, KV head), not a wave
        bool chosen = false;        // group, or shared segments with a split of their own:
        int32_t wave_items = 0, wave_members = 0, wave_parts = 0;   // work items, their members and partial results with a wave each and one split
    } dec;
    TableRef dec_req_seg;           // [n][4] absolute prefix_off, L_P, suffix_off, L_Q (innermost shared segment)
    TableRef dec_chain_start;       // [n+1] first entry of each request in dec_chain
    TableRef dec_chain;             // (absolute offset, tokens) of a request's shared segments, outermost first
    int32_t pad_split_tokens = 0, pad_n_splits = 0;   // padded decode comparison: uniform splits
    // prefill (packed and padded schedules share one format)
    struct PrefillSched {
        TableRef tiles;             // [n_tiles][16] kv_first, n_kv, leading / trailing skipped key tiles per 32 rows (4 x 8 bits each),
                                    // rows | runs << 16, then Q row, lo, hi of tile row 0 (the first run), then k_start and
                                    // info of the first three key tiles, then the end of the keys that the tile sees (INT32_MAX: the
                                    // list says it)
        TableRef run_first;         // [n_tiles] first entry of the tile's further runs
        TableRef runs;              // (first tile row, its Q row, lo, its hi) of the runs after a tile's first
        TableRef kvtiles;           // [n_kv_total][2] k_start, n | codes << 8 (2 bits per 32 rows: 0 skip, 1 masked, 2 unmasked); with
                                    // row_shift < 2 a list per request, which its query tiles share (all codes 2)
        // lists cut into pieces (split_lists): what the launch works on instead of `tiles`
        TableRef pieces;            // [n_pieces][16] descriptors of the pieces, and in the last word the slot of their partial results + 1 (0: a whole list)
        TableRef merges;            // [n_merges][4] first slot, pieces, Q row of tile row 0, rows of every tile whose list is cut
        TableRef piece_kvtiles;     // their key-tile lists
        int32_t n_pieces = 0, n_merges = 0, piece_shift = 2;      // (piece_shift: their row_shift)
        double whole_us = 0;                                      // estimate of the launch with whole lists
        int32_t n_tiles = 0;
        int64_t issued_pairs = 0;
        int32_t n_query_tiles = 0;  // packed: of 128 rows, whatever row_shift is
        int row_shift = 2;          // rows of a query tile: 32 << row_shift
        bool eight = false;         // workgroups of eight waves, twice the heads (the prefill launch, d = 128)
        bool light = false;         // a launch of little work: prefill_few_body.hip.h (the schedule builder's choice)
    } packed, padded;
    int num_cus = 0;                // of the device the schedules are built for
    struct Copy {                   // of a schedule into the workspace that the plan is bound to
        bool made = false;
        uint64_t capture = 0;       // the stream capture that it is part of (0: none); it has not run and counts inside that capture only
    };
    // packed prefill schedule of a decode plan (one query row per request): built on first use like the padded one, uploaded behind the tables
    std::vector<int32_t> host_packed;
    bool packed_built = false;
    Copy packed_copy;
    size_t packed_offset = 0;
    // padded prefill schedule: built on first use, uploaded behind the partial results
    std::vector<int32_t> host_padded;
    bool padded_built = false;
    Copy padded_copy;
    size_t padded_offset = 0;
    // partial results (floats) live after the tables
    size_t tables_bytes = 0;
    size_t partial_offset = 0;      // bytes
    size_t partial_bytes = 0;
    size_t prefill_part_bytes = 0;  // of them, partial results of pieces of key-tile lists
    size_t total_bytes = 0;
    size_t decode_only_bytes = 0;   // what decides whether a plan may use the fixed scratch: its tables and the packed decode partials, dec.chosen: as they would
                                    // be with a wave per work item and one split.  The tables of its packed prefill count, though they are never copied there:
                                    // which plans are admitted does not depend on when these tables are made
    bool group_over_scratch = false;    // those of dec.chosen do not fit the static scratch, the others would
};

}  // namespace pk

struct pk_plan {
    int32_t n = 0;
    int64_t token_budget = 0;
    int32_t headroom = 0;
    bool decode_only = false;       // every q_len == 1
    bool tree = false;              // made by pk_pack_plan_tree (nested shared segments)
    std::vector<int32_t> kv_lens, q_lens, prefix_lens;   // prefix_lens: 0 if no family
    std::vector<pk::Group> groups;
    int64_t buf_tokens = 0;         // whole buffer, multiple of PK_KV_BLOCK
    int64_t unique_tokens = 0;
    int64_t unmasked_pairs = 0;
    std::vector<int32_t> words;     // canonical serialisation
    int32_t tune_decode_split = 0;  // pk_plan_tune: 0 = chosen by the schedule builder
    int32_t tune_prefill_pipeline = 0;   // 1: the register-staged prefill kernel (pk_plan_tune)
    // binding state: a cache of what was last built / uploaded for this plan, also filled by the
    // size query on a const plan (calls on one plan are serialised by the caller)
    mutable pk::DeviceTables tables;
    mutable void* bound_ws = nullptr;
    mutable size_t bound_bytes = 0;
    uint64_t bound_stamp = 0;       // stamp of the bind that wrote bound_ws (0: none)
    uint64_t bound_capture = 0;     // the stream capture that its copy is part of, as in DeviceTables::Copy
};

namespace pk {

void set_error(const std::string& msg);

// Exception barrier of the C ABI: nothing may unwind through an extern "C" entry point.  Host
// containers can throw (std::bad_alloc, std::length_error); the entry point then reports an
// error code and a message like any other failure.
template <class R, class F>
R guarded(R on_alloc, R on_other, const char* who, F&& body) noexcept {
    try {
        return body();
    } catch (const std::bad_alloc&) {
        try { set_error(std::string(who) + ": out of host memory"); } catch (...) {}
        return on_alloc;
    } catch (const std::exception& e) {
        try { set_error(std::string(who) + ": " + e.what()); } catch (...) {}
        return on_other;
    } catch (...) {
        try { set_error(std::string(who) + ": unknown failure"); } catch (...) {}
        return on_other;
    }
}

// schedule.cpp
void build_tables(const pk_plan& plan, int Hq, int Hkv, int d, int dtype, int num_cus, DeviceTables& out);
void build_prefill_padded(const pk_plan& plan, DeviceTables& t);
void build_prefill_of_decode(const pk_plan& plan, DeviceTables& t);    // the packed schedule of a decode plan
size_t kv_buf_bytes(const pk_plan& plan, int Hkv, int d, int dtype);

}  // namespace pk
