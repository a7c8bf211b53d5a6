// Records the launches of the packed-FP16 half-sweep of several lattices instead of making them (host code
// only, no GPU): for each line of block shapes "bx by bz bt ..." on stdin, one line with workgroups,
// threads per workgroup and bytes of LDS of every launch.  Every lattice is 4 blocks long in each direction.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, lds, ...) \
    std::printf("%u %u %zu ", dim3(grid).x, dim3(block).x, (size_t)(lds))
#define hipGetLastError() hipSuccess

#include "dd_sap_fp16.hip"

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::vector<dd::SapLat> lat;
        int b[4];
        while (in >> b[0] >> b[1] >> b[2] >> b[3]) {
            dd::Geom g{};
            g.bvol = 1;
            for (int mu = 0; mu < 4; ++mu) {
                g.b[mu] = b[mu];
                g.NB[mu] = 4;
                g.L[mu] = 4 * b[mu];
                g.bvol *= b[mu];
            }
            g.nblk = 256;
            g.V = 256LL * g.bvol;
            lat.push_back(dd::sap_lat(g, dd::SapArgs{}));
        }
        const hipError_t e = dd::launch_sap_half_pk_multi(nullptr, lat.data(), (int)lat.size(), 0, 0);
        std::printf("%s\n", e == hipSuccess ? "" : "refused");
    }
}
