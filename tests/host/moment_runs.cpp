// Host check of the runs that the moment projection sums (no GPU): every
// grouped point is marked (sign bit) exactly where its displacement's x or y
// component differs from the point before in its chunk; chunk starts and
// padding are not.  Exit status 0 (ok), 1 (builder error), 2 (a mark is wrong).
#include <cmath>
#include <cstdio>

#include "hub_internal.h"

int main() {
    const double cell[3] = {5.0, 6.0, 7.0};
    const int ngrid[3] = {11, 12, 13};
    std::vector<SiteDef> sites(3);
    const double at[3][3] = {{0.1, 0.2, 6.9}, {2.5, 2.6, 3.0}, {4.0, 1.0, 1.0}}, rc[3] = {3.1, 2.4, 0.9};
    for (int i = 0; i < 3; ++i) {
        for (int a = 0; a < 3; ++a) sites[i].R[a] = at[i][a];
        sites[i].l = i;
        sites[i].zeta = 1.3;
        sites[i].rc = rc[i];
        sites[i].species = i;
        sites[i].ueff_fixed = sites[i].zeta_dn = NAN;
    }
    long marked = 0, points = 0;
    for (int chunk : {64, 512}) {
        HostTables T;
        if (hub_build_host(cell, ngrid, sites, chunk, T) != HUB_OK || !T.grouped.ok) return 1;
        const GroupTables& G = T.grouped;
        if (G.run_gidx.size() != G.gidx.size()) return std::puts("size"), 2;
        for (const HubChunk& C : G.chunks)
            for (int e = 0; e < C.ne; ++e) {
                const size_t i = static_cast<size_t>(C.e0) + e;
                const double* d = &G.d0[3 * i];
                const bool run = e > 0 && e < C.nreal && (d[0] != d[-3] || d[1] != d[-2]);
                if ((G.run_gidx[i] < 0) != run || (G.run_gidx[i] & INT32_MAX) != G.gidx[i]) return std::puts("mark"), 2;
                marked += run;
                points += e < C.nreal;
            }
    }
    // runs of several points exist, and more than one a chunk
    return marked > 0 && 2 * marked < points ? 0 : 2;
}
