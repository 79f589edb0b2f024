// gpr_layout.h -- host-side rules that lay a replica out over workgroups.  Plain C++, so that a test
// can compile it by itself.
#pragma once
#include <algorithm>
#include <cmath>
#include <vector>

namespace gpr {

constexpr int MAX_G = 32;

// atom ranges of the workgroups of one replica
struct AtomRanges {
    int G;                // workgroups per replica (1, 2, 4, ... MAX_G)
    int lmax;             // LDS length of the per-group arrays: the largest range, rounded up to 16
    int bnd[MAX_G + 1];   // group g owns atoms [bnd[g], bnd[g + 1]); every bnd[g] < n is a multiple of 16
};

// Ranges for G workgroups: contiguous, starting at multiples of 16 (so that every wave of the pair
// loop covers 16 atoms of one group), with boundaries placed where the running sum of the per-atom
// work estimate crosses g/G of the total.  No range is empty: the position exchange has a group
// overwrite its words of two steps before once every other group's words of the last step are
// there, and a group without atoms writes none, so nobody would wait for it to read.  Each group
// gets a block of 16 atoms at least, and a replica of fewer blocks than G runs on fewer groups, the
// next power of two down.
inline AtomRanges atom_ranges(const std::vector<double> &work, int n, int np, int G)
{
    const int nblk = (n + 15) / 16;
    while (G > nblk) G /= 2;
    AtomRanges a{};
    a.G = G;
    a.bnd[G] = n;
    if (G == 1) {
        a.lmax = np;
        return a;
    }
    std::vector<double> cum(n + 1, 0.0);
    for (int i = 0; i < n; ++i) cum[i + 1] = cum[i] + work[i];
    for (int g = 1; g < G; ++g) {
        const double target = cum[n] * g / G;
        const int at = (int)(std::lower_bound(cum.begin(), cum.end(), target) - cum.begin());
        const int lo = std::min(at / 16 * 16, n), hi = std::min(n, lo + 16);
        const int b = (target - cum[lo] <= cum[hi] - target) ? lo : hi;
        a.bnd[g] = std::min(std::max(b, a.bnd[g - 1] + 16), 16 * (nblk - (G - g)));
    }
    int lmax = 16;
    for (int g = 0; g < G; ++g) lmax = std::max(lmax, a.bnd[g + 1] - a.bnd[g]);
    a.lmax = (lmax + 15) / 16 * 16;
    return a;
}

// Pair-list margins by mass: an atom of less than four times the lightest's mass (light: 1/m above
// im_light) may move half the skin between builds, any other one `heavy` times that, in proportion
// to how much slower the lightest of them is, times 1.35 (measured on masses of 1 and 12 to 16: with
// 1.7, 2.2 and 3.0, 20-step launches take 2 % less, 1,000-step launches 1 to 3 % more and plain
// steps 4 to 6 % more).
struct MarginRule {
    float im_light;       // 0: every atom is light
    double heavy;
};
inline MarginRule margin_rule(const double *mass, int n)
{
    double mmin = mass[0], mheavy = INFINITY;
    for (int i = 0; i < n; ++i) mmin = std::min(mmin, mass[i]);
    for (int i = 0; i < n; ++i)
        if (mass[i] >= 4.0 * mmin) mheavy = std::min(mheavy, mass[i]);
    if (!std::isfinite(mheavy)) return {0.f, 1.0};
    return {(float)(1.0 / mheavy), std::min(1.0, 1.35 * std::sqrt(mmin / mheavy))};
}

} // namespace gpr
