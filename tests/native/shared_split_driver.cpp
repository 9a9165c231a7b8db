// Test infrastructure: decode tables of random batches with shared segments (trees and families, headroom, several head shapes).  Every request is covered once,
// every item by one request's or one segment's tokens, its slots follow one another, and what a plan needs of the fixed scratch is what it needs with one split for all
// segments.  Built with g++, no device code; the kernel launchers are never reached.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../include/packinfer.h"
#include "../../paper_2602_06072_amd/csrc/kernels.h"
#include "../../paper_2602_06072_amd/csrc/plan.h"

namespace pk {
int launch_reorg_bf16(const ReorgArgs&, void*) { std::abort(); }
int launch_reorg_f32(const ReorgArgs&, void*) { std::abort(); }
int launch_append_bf16(const AppendArgs&, void*) { std::abort(); }
int launch_append_f32(const AppendArgs&, void*) { std::abort(); }
int launch_decode_bf16(const DecodeArgs&, void*) { std::abort(); }
int launch_decode_f32(const DecodeArgs&, void*) { std::abort(); }
int launch_decode_merge_bf16(const DecodeArgs&, void*) { std::abort(); }
int static_scratch_address(void**) { return 1; }
int launch_prefill_bf16(const PrefillArgs&, void*) { std::abort(); }
int launch_prefill_f32(const PrefillArgs&, void*) { std::abort(); }
int launch_mixed_step_bf16(const PrefillArgs&, const DecodeArgs&, void*) { std::abort(); }
int launch_padded_decode_bf16(const PagedDecodeArgs&, void*) { std::abort(); }
}  // namespace pk

int main() {
    std::mt19937 rng(5);
    auto upto = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
    const int heads[][3] = {{32, 8, 128}, {16, 2, 128}, {16, 16, 128}, {64, 8, 128}, {8, 8, 64}, {4, 1, 128}, {28, 4, 128}, {6, 3, 64}, {32, 1, 128}};
    int longer = 0, shorter = 0;
    for (int round = 0; round < 600; ++round) {
        const int n = upto(2, round % 3 ? 60 : 400), families = upto(1, n / 2), most = 1 << upto(4, 12);
        const bool tree = rng() % 2;
        std::vector<int32_t> parent, len, node, kv, q(static_cast<size_t>(n), 1);
        if (tree) { parent.push_back(-1); len.push_back(upto(1, most)); }
        for (int k = 0; k < families; ++k) { parent.push_back(tree ? 0 : -1); len.push_back(upto(1, most)); }
        const int own = 1 << upto(0, 9), headroom = rng() % 2 ? 8 : 0;
        for (int i = 0; i < n; ++i) {
            const int k = (i < families ? i : upto(0, families - 1)) + tree;       // (every node has a request)
            node.push_back(k);
            kv.push_back(len[static_cast<size_t>(k)] + (tree ? len[0] : 0) + upto(headroom ? 0 : 1, own));
        }
        pk_plan* plan = nullptr;
        if (pk_pack_plan_tree(kv.data(), q.data(), n, parent.data(), len.data(), static_cast<int32_t>(len.size()), node.data(), 8192, headroom, &plan) != PK_OK) return 1;
        const int* h = heads[round % 9];
        pk::build_tables(*plan, h[0], h[1], h[2], PK_BF16, 256, plan->tables);
        const pk::DeviceTables t = plan->tables;
        const pk::DeviceTables::DecodeSched& s = t.dec;
        if (s.chosen && !s.group) (s.n_items < s.wave_items ? longer : shorter) += 1;
        auto table = [&](const pk::TableRef& r) { return t.host.data() + r.offset / sizeof(int32_t); };
        const int32_t *item = table(s.items), *member = table(s.members), *slot = table(s.member_slot), *start = table(s.req_part_start);
        std::vector<int64_t> tokens(static_cast<size_t>(n), 0);
        std::vector<int32_t> pieces(static_cast<size_t>(n), 0), seen(static_cast<size_t>(s.n_parts), 0);
        int max_parts = 0;
        for (int x = 0; x < s.n_items; ++x, item += 8) {
            if (item[3] * (h[0] / h[1]) > 32 && item[3] > 1) return 2;
            if ((x < s.n_wide) != (item[3] * (h[0] / h[1]) > 16)) return 3;
            for (int y = item[2]; y < item[2] + item[3]; ++y) {
                tokens[static_cast<size_t>(member[y])] += item[1] - item[0];
                ++pieces[static_cast<size_t>(member[y])];
                if (slot[y] >= 0) {
                    if (slot[y] < start[member[y]] || slot[y] >= start[member[y] + 1]) return 4;
                    ++seen[static_cast<size_t>(slot[y])];
                }
            }
        }
        for (int i = 0; i < n; ++i) {
            const int parts = start[i + 1] - start[i];
            max_parts = parts > max_parts ? parts : max_parts;
            if (tokens[static_cast<size_t>(i)] != kv[static_cast<size_t>(i)] || parts != (pieces[static_cast<size_t>(i)] > 1 ? pieces[static_cast<size_t>(i)] : 0)) return 5;
        }
        for (const int32_t c : seen)
            if (c != 1) return 6;
        if (max_parts != s.max_parts || s.group) return 7;
        // one split for all (the knob): the same need, its tables where the plan's own would not fit
        if (pk_plan_tune(plan, PK_TUNE_DECODE_SPLIT, s.split_tokens) != PK_OK) return 8;
        pk::build_tables(*plan, h[0], h[1], h[2], PK_BF16, 256, plan->tables);
        if (plan->tables.decode_only_bytes != t.decode_only_bytes || plan->tables.dec.chosen) return 9;
        if (t.decode_only_bytes <= PK_STATIC_SCRATCH_BYTES && t.partial_offset + static_cast<size_t>(s.n_parts) * h[0] * (static_cast<size_t>(h[2]) + 1) * 4 > PK_STATIC_SCRATCH_BYTES) return 10;
        pk_plan_destroy(plan);
    }
    std::printf("%d %d\n", longer, shorter);
    return longer >= 10 && shorter >= 10 ? 0 : 11;
}
