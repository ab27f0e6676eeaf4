// The mixture kernels' split rule for lines of "n nd K setup" on standard
// input (setup: step, init or loglik): "W lsl" each.
#include <cstdio>
#include <cstring>

#include "../../paper_1306_5583_amd/csrc/smc_gmm_split.hpp"

int main()
{
    long long n, nd;
    int K;
    char what[16];
    while (std::scanf("%lld %lld %d %15s", &n, &nd, &K, what) == 4) {
        const double setup = !std::strcmp(what, "step")   ? smc::GMM_SETUP_STEP
                             : !std::strcmp(what, "init") ? smc::GMM_SETUP_INIT
                                                          : smc::GMM_SETUP_LOGLIK;
        const smc::GmmSplit s = smc::gmm_split(n, nd, K, setup);
        std::printf("%d %d\n", s.W, s.lsl);
    }
}
