// The block order of csrc/bl_internal.h on the host, for tests/test_dealt_blocks.py:
// reads lines "groups parts first step" and prints the launch's blocks, then
// "bid group part" of every step-th block from the first on, -1 -1 for one without
// a task.
#include <cstdio>

#include "../../paper_2602_07400_amd/csrc/bl_internal.h"

int main()
{
    long long groups, parts, first, step;
    while (std::scanf("%lld %lld %lld %lld", &groups, &parts, &first, &step) == 4) {
        const int64_t blocks = bl::dealt_blocks(groups, parts);
        std::printf("blocks %lld\n", (long long)blocks);
        for (int64_t b = first; b < blocks; b += step) {
            int g = -1, p = -1;
            if (!bl::dealt_task((int)b, (int)groups, (int)parts, g, p))
                g = p = -1;
            std::printf("%lld %d %d\n", (long long)b, g, p);
        }
    }
    return 0;
}
