// Host-only driver of the plan construction code: which plans run their rows in
// pairs, by the length of their deconvolution series.  Built and run by
// tests/test_host_series.py.
#include <cstdio>
#include <string>

#include "plan_host.hpp"

int main() {
    struct Case {
        int n;
        phi_dtype dtype;
        bool gaussian;
        double tol;
        bool pairs;
    };
    const Case cases[] = {
        // padded side 2048, FP32: up to 12 terms
        {512, PHI_F32, false, 1e-7, false},  {514, PHI_F32, false, 1e-7, true},  {1024, PHI_F32, false, 1e-7, true},
        {1024, PHI_F32, false, 1e-2, true},  {514, PHI_F32, true, 1e-7, true},   {600, PHI_F32, true, 1e-7, false},
        {700, PHI_F32, true, 1e-7, false},   {800, PHI_F32, true, 1e-6, false},  {700, PHI_F32, true, 1e-6, true},
        // longer rows, and FP64 from padded side 4096: up to 32
        {1500, PHI_F32, true, 1e-7, true},   {4096, PHI_F32, false, 1e-7, true}, {1024, PHI_F64, false, 1e-12, false},
        {1026, PHI_F64, false, 1e-12, true}, {2048, PHI_F64, false, 1e-12, true}, {1026, PHI_F64, true, 1e-12, true},
        {2048, PHI_F64, false, 1e-15, false},
    };
    int failures = 0;
    for (const Case& c : cases) {
        phi_params p;
        phi::fill_defaults(&p, c.n, 16.0 / c.n, c.dtype);
        p.n_r = 16;
        p.n_theta = 32;
        p.tol = c.tol;
        if (c.gaussian) p.flags = PHI_KERNEL_GAUSSIAN;
        phi::HostPlan hp;
        std::string err;
        if (phi::build_host_plan(&p, &hp, &err) != PHI_OK) {
            std::printf("plan n=%d failed: %s\n", c.n, err.c_str());
            ++failures;
            continue;
        }
        const int most = hp.log_fine == 11 ? 12 : 32;
        const bool ok = (hp.pair_taps > 0) == c.pairs && hp.pair_taps <= most &&
                        hp.delta.size() == (hp.pair_taps ? hp.pair_taps + 1u : 0u);
        std::printf("n=%d f%d %s tol=%g: %d terms: %s\n", c.n, c.dtype == PHI_F32 ? 32 : 64, c.gaussian ? "gaussian" : "es",
                    c.tol, hp.pair_taps, ok ? "ok" : "NOT AS THE RULE SAYS");
        failures += ok ? 0 : 1;
    }
    return failures ? 1 : 0;
}
