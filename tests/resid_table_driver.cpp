// Splits residual jobs into launches as the solvers do, with the launches recorded instead of made (host code
// only, no GPU).  Input: one line per set of lattices, their numbers of sites; output: for every launch
// "owner held : first+count ..." -- the lattice whose array of partial sums it uses, how many that array
// holds, and every entry's range in it -- or "refused".
#include "dd_ops.cpp"

#include <algorithm>
#include <cstdio>
#include <iostream>
#include <sstream>

static std::vector<dd_ctx> ctx;

namespace dd {
int resid_grid(const Geom &g) { return (int)((g.V + BLAS_WG - 1) / BLAS_WG); }
hipError_t launch_resid64(hipStream_t, const ResidTab &t, int, double *partials)
{
    for (size_t k = 0; k < ctx.size(); ++k)
        if (ctx[k].partials == partials)
            std::printf("%zu %d :", k, std::max(MAX_PARTIALS, resid_grid(ctx[k].g)));
    for (int k = 0; k < t.n; ++k) std::printf(" %lld+%d", t.e[k].poff, t.e[k].nwg);
    std::printf(" ; ");
    return hipSuccess;
}
hipError_t launch_finalize_multi(hipStream_t, const MultiBlasTab &, const int *, const double *, int, double *)
{
    return hipSuccess;
}
}  // namespace dd

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::vector<long long> sites;
        for (long long v; in >> v;) sites.push_back(v);
        ctx.clear();
        ctx.resize(sites.size());
        std::vector<ddh::ResidJob> jobs;
        for (size_t k = 0; k < sites.size(); ++k) {
            ctx[k].g.V = sites[k];
            for (int mu = 0; mu < 4; ++mu) ctx[k].g.b[mu] = 4;
            ctx[k].partials = (double *)(uintptr_t)(4096 * (k + 1));  // a tag, never followed
            jobs.push_back({&ctx[k], nullptr, nullptr, nullptr, (int)k});
        }
        const hipError_t e = ddh::resid_table(&ctx[0], nullptr, jobs, false, nullptr);
        std::printf("%s\n", e == hipSuccess ? "" : "refused");
    }
}
