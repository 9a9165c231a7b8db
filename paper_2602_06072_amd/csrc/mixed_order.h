// In which order the prefill and decode workgroups of a mixed step are launched.
//
// They are dealt in sets of eight (every workgroup keeps its XCD), and the sets in cycles: up to kRun prefill sets, kRun decode sets, and what is left of the
// cycle's share of the prefill sets; the last cycle goes on to the end with what is left of either kind.  Spread over the launch, the decode runs load the memory system evenly;
// alternating one by one until the decode work is gone they saturate it for the first quarter of the
// launch, and the prefill tiles of that stretch wait (spread 1.3 % faster for 32 chunks and 480 rows of a 70B-shaped layer, small steps
// unchanged).  Workgroups go to the compute units of an XCD one per unit before any unit gets its second: runs of 32 sets, one workgroup for every unit, put one of each kind on a unit in
// launches of one round.  Runs of 4 / 8 / 16 / 32 / 64 sets: 32 chunks and 480 rows 11.97 / 11.90 / 11.64 / 11.75 / 12.04 ms, 8 chunks and 200 rows with 32/8 heads 1339 / 1339 /
// 1331 / 1334 / 1358 us, 16 prompts of 30 to 300 rows beside 60 decode rows with 16/2 heads 31.0 / 29.4 / 29.6 / 26.8 / 33.3.
// No set is padding: where runs were filled up with workgroups that end at once, the first decode workgroups of a small step met its few prefill workgroups on the same units
// while others stayed idle.  us, filled up / now: 3 short prompts with 16/2 heads beside 3 decode rows 12.2 / 10.8, 2 with 32/8 beside 4 10.1 / 8.4, 1 with 16/2 beside 46
// 10.2 / 8.8; 72 drawn steps 1.02 times as fast in the geometric mean, between 0.95 and 1.2.
#pragma once
#include <cstdint>

#include "kernels.h"

namespace pk {

struct MixedOrder {
    static constexpr int kRun = 32;     // sets
    int n_prefill;                      // prefill workgroups
    int prefill, decode;                // sets of a cycle
    int lead, last_lead;                // of them, prefill sets in front of the decode sets (in the last cycle)
    int last, last_decode;              // number of the last cycle, and its decode sets
    FastDiv by_cycle;

    // P prefill and D decode sets (fewer than 2^28 together)
    static MixedOrder of(int n_prefill, int64_t P, int64_t D) {
        MixedOrder m{};
        m.n_prefill = n_prefill;
        m.decode = kRun;
        if (P >= D) {                   // the decode runs spread over the prefill sets
            m.last = D > 0 ? static_cast<int>((D + kRun - 1) / kRun) - 1 : 0;
            m.prefill = static_cast<int>(P / (m.last + 1));
            m.lead = m.last_lead = m.prefill < kRun ? m.prefill : kRun;
        } else {                        // in turns, and what is left of decode
            m.last = P > 0 ? static_cast<int>((P + kRun - 1) / kRun) - 1 : 0;
            m.prefill = m.lead = kRun;
            m.last_lead = static_cast<int>(P - static_cast<int64_t>(m.last) * kRun);
        }
        m.last_decode = static_cast<int>(D - static_cast<int64_t>(m.last) * kRun);
        m.by_cycle = FastDiv::by(static_cast<uint32_t>(m.prefill + m.decode));
        return m;
    }
    // set `y` of the launch: its number among its kind
    PK_HOST_DEVICE int set_of(const int y, bool& is_decode) const {
        const int q = by_cycle(y), c = q < last ? q : last, r = y - c * (prefill + decode);
        const int p = c == last ? last_lead : lead, d = c == last ? last_decode : decode;
        is_decode = r >= p && r - p < d;      // (prefill first: the heaviest tiles start at once)
        return is_decode ? c * decode + r - p : c * prefill + (r < p ? r : r - d);
    }
};

}  // namespace pk
