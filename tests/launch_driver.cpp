// stride_blocks (csrc/launch.h): every launch has fewer than 2^32 threads, at
// least one workgroup, and a thread an item while the device is not full.
#include <cstdio>

#include "launch.h"

int main()
{
    const uint64_t sizes[] = {0, 1, 255, 256, 257, (1ull << 24) - 1, 1ull << 24, (1ull << 24) + 1,
                              (1ull << 32) - 1, 1ull << 32, (1ull << 32) + 1, 1ull << 40, ~0ull >> 8};
    for (unsigned threads : {64u, 256u, 1024u})
        for (uint64_t items : sizes) {
            const uint64_t b = dfpr::stride_blocks(items, threads);
            if (b < 1 || b * threads >= (1ull << 32) || (items <= (1ull << 22) && b * threads < items)) {
                std::printf("items %llu threads %u: %llu workgroups\n", (unsigned long long)items, threads,
                            (unsigned long long)b);
                return 1;
            }
        }
    std::printf("ok\n");
    return 0;
}
