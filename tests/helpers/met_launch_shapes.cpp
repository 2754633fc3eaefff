// Prints the launch of the Metropolis colour kernels as a chain takes it, for
// every L read from stdin: L quad rows row_blocks through
#include <stdio.h>

#include "met_launch.h"

int main()
{
    unsigned L;
    while (scanf("%u", &L) == 1) {
        const cvf::MetShape m = cvf::met_launch(L);
        printf("%u %u %u %u %d\n", L, m.quad, m.rows, m.row_blocks, cvf::met_through(L) ? 1 : 0);
    }
    return 0;
}
