// Host-only driver of the plan construction code: the tiles of the half-plane
// node set fit the workspace sized for the tiles of all nodes, n_sub E^2 entries
// with E = bin + w - 1, whichever node kernel the set is laid out for.  Built and
// run by tests/test_host_tiles.py.
#include <algorithm>
#include <cstdio>
#include <string>

#include "plan_host.hpp"

int main() {
    struct Case {
        int n, n_r, n_theta, pad, bin, sub_nodes;
        double tol;
        phi_dtype dtype;
    };
    const Case cases[] = {
        {2394, 128, 256, 2, 0, 0, 1e-7, PHI_F32}, {2412, 64, 128, 2, 0, 0, 1e-4, PHI_F32},
        {1156, 128, 256, 4, 0, 0, 1e-4, PHI_F64}, {64, 256, 512, 2, 0, 8, 1e-2, PHI_F64},
        {64, 64, 128, 2, 0, 0, 1e-12, PHI_F64},   {8, 6, 10, 2, 0, 0, 1e-12, PHI_F64},
        {100, 33, 50, 2, 8, 24, 1e-7, PHI_F32},   {128, 24, 48, 2, 16, 8, 1e-6, PHI_F32},
        {64, 1, 2, 2, 0, 0, 0.1, PHI_F32},
    };
    int failures = 0;
    for (const Case& c : cases) {
        phi_params p;
        phi::fill_defaults(&p, c.n, 16.0 / c.n, c.dtype);
        p.n_r = c.n_r;
        p.n_theta = c.n_theta;
        p.pad = c.pad;
        p.bin = c.bin;
        p.sub_nodes = c.sub_nodes;
        p.tol = c.tol;
        phi::HostPlan hp;
        std::string err;
        if (phi::build_host_plan(&p, &hp, &err) != PHI_OK) {
            std::printf("plan n=%d failed: %s\n", c.n, err.c_str());
            ++failures;
            continue;
        }
        const long long tile = static_cast<long long>(hp.tile) * hp.tile;
        const long long last = *std::max_element(hp.half.contrib.begin(), hp.half.contrib.end());
        const bool ok = hp.half.n_sub <= hp.n_sub && last < hp.half.n_sub * tile;
        std::printf("n=%d tile=%d subproblems %d, half plane %d, last tile entry %lld of %lld: %s\n", c.n, hp.tile,
                    hp.n_sub, hp.half.n_sub, last, hp.n_sub * tile, ok ? "ok" : "TOO LARGE");
        failures += ok ? 0 : 1;
    }
    return failures ? 1 : 0;
}
