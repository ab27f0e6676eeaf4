// smc_gmm_split.hpp -- how the mixture kernels spread a population over the
// chip: waves of a workgroup and lanes of a particle (host code only, so that
// the rule can be checked without a GPU).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace smc {

constexpr int GMM_MAXW = 8;  // waves per particle tile

// How a mixture kernel spreads a particle's data: W waves of a workgroup and,
// within a wave, 2^lsl neighbouring lanes (a wave then holds 64 >> lsl
// particles).
struct GmmSplit {
    int W, lsl;
};
// `setup`: a kernel's work besides the data, in data points (three proposals
// and decisions; the prior draws; the constants of the likelihood alone).
constexpr double GMM_SETUP_STEP = 60.0, GMM_SETUP_INIT = 30.0, GMM_SETUP_LOGLIK = 12.0;

// Waves per 64-particle tile: enough waves overall to fill the GPU, at most
// GMM_MAXW, and no more than the data can feed (>= 32 points per wave).
inline int gmm_waves(int64_t n, int64_t nd)
{
    const int64_t tiles = (n + 63) / 64;
    int W = 1;
    while (W < GMM_MAXW && tiles * W < 8192 && nd >= (int64_t)(2 * W) * 32)
        W *= 2;
    return W;
}

// The split with the least modelled time, in units of one data point's terms.
// A lane's chain is `setup` (what a launch does besides its data, overlapped
// by the waves sharing the SIMD to three quarters) plus its points, which the
// SIMD's waves share at about 85 % of issue; compute units take workgroups in
// whole turns.  The model puts the line where the measurements have it
// (random-walk step, K = 4, 1000 points; setup 60, us):
//   particles   8 waves x 64   best sliced            taken
//   64          101            18 (4 waves x 1)       the same
//   1000        102            26 (4 waves x 4)       the same
//   4000        105            46 (4 waves x 16)      the same
//   12000       111            102 (4 waves x 16)     the same
//   16384       116            117 (4 waves x 64)     8 waves x 64
//   20000       197            153 (4 waves x 16)     the same
//   40000       283            256 (4 waves x 32)     the same
// and K = 6 with the gradient, 1000 vectors, 10^4 points: 633 -> 57 us.
// A single component takes three to five instructions a point, and a point
// of a lane's own costs it a load besides: it counts 2.5 times (value of 10^4
// points, us: 4096 vectors 22 sliced against 25, 8192 39 / 25, 16384 77 / 25).
// Above 2^17 particles the turns are many and the split no longer matters.
inline GmmSplit gmm_split(int64_t n, int64_t nd, int K, double setup)
{
    constexpr int CUS = 256, SIMDS = 4;
    const auto cost = [&](const GmmSplit &sp) {
        const int64_t per = 64 >> sp.lsl, wgs = (n + per - 1) / per;
        const int64_t turns = (wgs + CUS - 1) / CUS;
        const double w = std::max(1.0, (double)turns * sp.W / SIMDS);  // waves of a SIMD
        const double points = (double)nd / ((double)sp.W * (1 << sp.lsl)) *
                              (K == 1 && sp.lsl > 0 ? 2.5 : 1.0);
        return setup * (1.0 + 0.25 * (w - 1.0)) + points * (0.15 + 0.85 * w);
    };
    GmmSplit best{gmm_waves(n, nd), 0};
    if (n > (1 << 17))
        return best;
    double t = 0.97 * cost(best);
    for (int lsl = 0; lsl <= 6 && (int64_t)4 << lsl <= nd; ++lsl) {
        const GmmSplit sp{4, lsl};
        const double c = cost(sp);
        if (c < t) {
            t = c;
            best = sp;
        }
    }
    return best;
}

}  // namespace smc
