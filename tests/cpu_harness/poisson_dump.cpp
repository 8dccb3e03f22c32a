// poisson_dump.cpp -- which transforms a pressure solve takes, the radices of
// their lines and the spectrum's row pitch (ch_route.h, test infrastructure).
//
// stdin:  lines "nx ny nz walls precision" (0 FP64, 1 FP32)
// stdout: per line "own pitch", then per axis "passes r0 r1 ..."
#include <cstdio>

#include "../../paper_2105_01865_amd/csrc/ch_route.h"

int main()
{
    int n[3], walls, prec;
    while (scanf("%d %d %d %d %d", n, n + 1, n + 2, &walls, &prec) == 5) {
        chk::FftLine line[3] = {};
        const bool own = chp::own_lines(n, walls != 0, prec, line);
        printf("%d %d", own ? 1 : 0, chp::spectrum_pitch(n[0], n[1], n[2], walls != 0, own));
        for (int d = 0; d < 3; ++d) {
            printf(" %d", line[d].passes);
            for (int p = 0; p < line[d].passes; ++p) printf(" %d", line[d].radix[p]);
        }
        printf("\n");
    }
    return 0;
}
