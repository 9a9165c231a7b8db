// Test infrastructure: prints the pieces that the packed prefill's key-tile lists are cut into, one line per batch.  Reads lines "Hq Hkv d n q_len.. kv_len..";
// prints "row_shift piece_shift part_bytes | whole tiles (16 words each) | pieces (16 words each) | merges (4 words each) | key-tile list of the pieces".
// Built with g++, no device code; the kernel launchers are never reached.
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <sstream>
#include <string>
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
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        int Hq, Hkv, d, n;
        if (!(in >> Hq >> Hkv >> d >> n) || n <= 0) return 2;
        std::vector<int32_t> q(static_cast<size_t>(n)), kv(static_cast<size_t>(n));
        for (auto& x : q) in >> x;
        for (auto& x : kv) in >> x;
        pk_plan* plan = nullptr;
        if (!in || pk_pack_plan(kv.data(), q.data(), nullptr, nullptr, n, 16384, 0, &plan) != PK_OK) return 3;
        pk::build_tables(*plan, Hq, Hkv, d, PK_BF16, 256, plan->tables);
        const pk::DeviceTables& t = plan->tables;
        const pk::DeviceTables::PrefillSched& s = t.packed;
        if (t.total_bytes < t.partial_offset + t.prefill_part_bytes) return 4;
        auto print = [&](const pk::TableRef& r, bool any) {
            std::printf(" |");
            const int32_t* w = t.host.data() + r.offset / sizeof(int32_t);
            for (size_t x = 0; any && x < r.count; ++x) std::printf(" %d", w[x]);
        };
        const bool cut = s.n_merges > 0;
        std::printf("%d %d %zu", s.row_shift, s.piece_shift, t.prefill_part_bytes);
        print(s.tiles, true);
        print(s.pieces, cut);
        print(s.merges, cut);
        print(s.piece_kvtiles, cut);
        std::printf("\n");
        pk_plan_destroy(plan);
    }
    return 0;
}
