// Prints, for `count` chains read from stdin, the wavefronts per workgroup of the
// batched cluster flip and how often each chain's next step is opened by it and
// by the batched Metropolis pass: count kTT / 64, then count times two numbers.
#include <stdio.h>

#include <vector>

#include "cvf_internal.h"

int main()
{
    unsigned count;
    while (scanf("%u", &count) == 1) {
        printf("%u %u", count, cvf::kTT / 64);
        for (uint32_t waves : {cvf::kSwWaves, cvf::kMetWaves}) {
            std::vector<int> opened(count, 0);
            for (uint32_t b = 0; b < cvf::open_blocks(count, waves); ++b)
                for (uint32_t w = 0; w < waves; ++w)
                    if (cvf::open_chain(b, w, waves) < count) ++opened[cvf::open_chain(b, w, waves)];
            for (int n : opened) printf(" %d", n);
        }
        printf("\n");
    }
    return 0;
}
