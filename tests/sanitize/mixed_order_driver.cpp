// Lists the blocks of mixed launches for tests/test_mixed_order.py: reads
// "prefills decodes round" lines, checks that the order ends and that each
// tile of both kinds is some block's exactly once, and prints per line the
// blocks, those without a tile, and the later prefill blocks (those after the
// first round) of each of the four places in a row of 4 x 8 blocks.
#include <cstdio>
#include <vector>

#include "../../paper_2607_04206_amd/csrc/mixed_order.h"

using namespace sangam;

int main() {
    long long p, d, round;
    while (std::scanf("%lld %lld %lld", &p, &d, &round) == 3) {
        MixedOrder m;
        const int64_t blocks = mixed_order(&m, p, d, round);
        std::vector<unsigned char> seen[2] = {std::vector<unsigned char>(size_t(p)), std::vector<unsigned char>(size_t(d))};
        int64_t empty = 0, bad = 0, place[4] = {0, 0, 0, 0};
        for (int64_t b = 0; b < blocks; ++b) {
            const MixedBlock x = mixed_block(m, uint32_t(b));
            if (x.index < 0) {
                ++empty;
                continue;
            }
            bad += seen[x.decode][size_t(x.index)]++ != 0;
            if (!x.decode && b >= m.first_prefill) ++place[b / 8 % 4];
        }
        for (const auto& v : seen)
            for (unsigned char c : v) bad += c != 1;
        std::printf("%lld %lld %lld %lld %lld %lld %lld\n", (long long)blocks, (long long)empty, (long long)bad, (long long)place[0],
                    (long long)place[1], (long long)place[2], (long long)place[3]);
    }
    return 0;
}
