// Prints atom_ranges for each request on stdin: n G and the n work estimates.
#include <cstdio>

#include "gpr_layout.h"

int main()
{
    int n, G;
    while (std::scanf("%d %d", &n, &G) == 2) {
        std::vector<double> w(n);
        for (double &x : w)
            if (std::scanf("%lf", &x) != 1) return 1;
        const gpr::AtomRanges a = gpr::atom_ranges(w, n, (n + 1 + 63) / 64 * 64, G);
        std::printf("%d %d", a.G, a.lmax);
        for (int g = 0; g <= a.G; ++g) std::printf(" %d", a.bnd[g]);
        std::printf("\n");
    }
    return 0;
}
