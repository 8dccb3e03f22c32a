// axes_dump.cpp -- the box that drops are labelled on (drop_axes of ch_route.h,
// test infrastructure).  stdin: lines "nx ny nz bcx bcy bcz"; stdout: the same six
// numbers of the folded box.
#include <cstdio>

#include "../../paper_2105_01865_amd/csrc/ch_route.h"

int main()
{
    int n[3], b[3], m[3], c[3];
    while (scanf("%d %d %d %d %d %d", n, n + 1, n + 2, b, b + 1, b + 2) == 6) {
        chp::drop_axes(n, b, m, c);
        printf("%d %d %d %d %d %d\n", m[0], m[1], m[2], c[0], c[1], c[2]);
    }
    return 0;
}
