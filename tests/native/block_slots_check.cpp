// Host-only check of the rule that keeps finalize inside its arrays: whatever
// number of classes the numbering finds, every array position it makes from a
// block id lies below nb + 1, and ids below nb are their own positions.
// Numbers the classes as the kernels do (ids in order, sizes and edge counts by
// id, then an exclusive scan of the counts over nb blocks) on checked arrays.
// Prints "ok <cases>"; any position out of range ends the program.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "bsim_internal.h"

int main() {
    int cases = 0;
    for (uint32_t nb : {0u, 1u, 2u, 63u, 64u, 2048u}) {
        for (uint32_t found : {0u, 1u, 2u, 62u, 63u, 64u, 65u, 2047u, 2048u, 2049u, 5000u}) {
            std::vector<uint32_t> sizes(nb + 1), edges(nb + 1), start(nb + 1);
            for (uint32_t id = 0; id < found; id++) {
                const uint32_t b = bsim::block_slot(id, nb);
                if (id < nb && b != id) return std::printf("id %u of %u moved to %u\n", id, nb, b), 1;
                sizes.at(b)++;
                edges.at(b) += 3;
            }
            uint32_t run = 0;
            for (uint32_t b = 0; b < nb; b++) start[b] = run, run += edges[b];
            // an edge's place: its block's start and the claim within the block
            if (nb)
                for (uint32_t id = 0; id < found; id++)
                    if (start.at(bsim::block_slot(id, nb)) + edges.at(bsim::block_slot(id, nb)) > 3 * found)
                        return std::printf("edges past the end\n"), 1;
            cases++;
        }
    }
    // a name that was never numbered (any word) is inside as well
    for (uint32_t id : {0u, 7u, 0x7FFFFFFFu, 0xFFFFFFFFu})
        for (uint32_t nb : {0u, 1u, 9u, 0xFFFFFFFEu}) {
            if (bsim::block_slot(id, nb) > (nb ? nb - 1 : 0u)) return std::printf("%u of %u\n", id, nb), 1;
            cases++;
        }
    std::printf("ok %d\n", cases);
    return 0;
}
