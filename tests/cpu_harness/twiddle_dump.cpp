// twiddle_dump.cpp -- the transforms' twiddles (fft_twiddles of ch_route.h, test
// infrastructure).  stdin: lengths; stdout: per length "re im" of every m < n.
#include <cstdio>

#include "../../paper_2105_01865_amd/csrc/ch_route.h"

int main()
{
    int n;
    while (scanf("%d", &n) == 1)
        for (double v : chp::fft_twiddles(n)) printf("%.17g\n", v);
    return 0;
}
