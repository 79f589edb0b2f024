// Prints, for each request on stdin (n and the n masses), heavy and the atoms' classes (1: light).
#include <cstdio>

#include "gpr_layout.h"

int main()
{
    int n;
    while (std::scanf("%d", &n) == 1) {
        std::vector<double> m(n);
        for (double &x : m)
            if (std::scanf("%lf", &x) != 1) return 1;
        const gpr::MarginRule r = gpr::margin_rule(m.data(), n);
        std::printf("%.17g", r.heavy);
        for (double x : m) std::printf(" %d", (float)(1.0 / x) > r.im_light ? 1 : 0);
        std::printf("\n");
    }
    return 0;
}
