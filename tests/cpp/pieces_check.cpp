// The pieces that a launch over many items is cut into (csrc/pieces.h), on the
// CPU: for every item count they cover each item once, in order, and no piece
// has more threads than a launch takes.  Prints "ok" when every check holds.
#include <stdio.h>

#include "pieces.h"

int main()
{
    const uint32_t counts[] = {0u, 1u, 255u, 256u, 257u, 131073u, (1u << 28) + 5u, (1u << 29) - 1u, 1u << 29, (1u << 29) + 1u,
                               (1u << 30) - 1u, 1u << 30, (1u << 30) + 12345u, 1u << 31, 0xFFFFFFE0u, 0xFFFFFFFFu};
    // items per 256-thread block of the actuation and free-space kernels
    for (uint32_t per_block : {1u, 4u, 16u, 32u, 64u, 256u})
        for (uint32_t n : counts) {
            uint64_t next = 0;
            bool good = true;
            habmi::in_pieces(n, per_block, 256u, [&](uint32_t first, uint32_t count, uint32_t blocks) {
                good = good && first == next && count > 0 && (uint64_t)blocks * per_block >= count &&
                       (uint64_t)(blocks - 1) * per_block < count && (uint64_t)blocks * 256u <= (1ull << 31);
                next += count;
            });
            if (!good || next != n) {
                fprintf(stderr, "%u items, %u to a block\n", n, per_block);
                return 1;
            }
        }
    puts("ok");
    return 0;
}
