// Test infrastructure: every set of workgroups of a mixed step comes once in the launch, whatever the numbers of both kinds.
#include <cstdio>
#include <vector>

#include "mixed_order.h"

static bool covers(int64_t P, int64_t D) {
    const pk::MixedOrder m = pk::MixedOrder::of(static_cast<int>(8 * P), P, D);
    std::vector<char> seen(static_cast<size_t>(P + D), 0);
    for (int y = 0; y < P + D; ++y) {
        bool decode = false;
        const int x = m.set_of(y, decode);
        if (x < 0 || x >= (decode ? D : P)) return false;
        char& s = seen[static_cast<size_t>(decode ? P + x : x)];
        if (s || (y == 0 && decode && P > 0)) return false;       // (the heaviest prefill tiles start first)
        s = 1;
    }
    return true;
}

int main() {
    const int edges[] = {0, 1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 700, 1023, 1024, 20001};
    for (int P = 0; P < 140; ++P)
        for (int D = 0; D < 140; ++D)
            if (!covers(P, D)) { std::printf("%d prefill sets, %d decode sets\n", P, D); return 1; }
    for (int P : edges)
        for (int D : edges)
            if (!covers(P, D)) { std::printf("%d prefill sets, %d decode sets\n", P, D); return 1; }
    return 0;
}
