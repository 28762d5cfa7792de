// Prints, for each "n k" on stdin, the dynamic LDS of the operator kernels, the
// words of a quad as a power of two, and whether a block fits a compute unit.
#include <cstdio>

#include "internal.h"

int main()
{
    int n, k;
    while (std::scanf("%d %d", &n, &k) == 2) {
        int32_t log_q = 0;
        const size_t bytes = gapa::ga_op_lds_layout(n, k, &log_q);
        std::printf("%zu %d %d\n", bytes, log_q, bytes + gapa::kOpStaticLds <= gapa::kOpLdsMax);
    }
}
