// Host check of the image-summed list's size limits (no GPU): a cell with 20
// functions on its points; the list is built up to exactly its own size and
// declined, with nothing left in it, for one byte less or one k-point more.
// Exit status 0 (ok), 1 (builder error), 2 (a check failed, named on stdout).
#include <cmath>
#include <cstdio>

#include "hub_internal.h"

int main() {
    const double cell[3] = {4.0, 4.0, 4.0};
    const int ngrid[3] = {9, 8, 10};
    std::vector<SiteDef> sites(3);
    const double at[3][3] = {{0.0, 0.0, 0.0}, {2.0, 2.0, 2.0}, {1.0, 3.0, 0.5}}, rc[3] = {3.9, 3.5, 2.0};
    const int l[3] = {3, 3, 2};
    for (int i = 0; i < 3; ++i) {
        for (int a = 0; a < 3; ++a) sites[i].R[a] = at[i][a];
        sites[i].l = l[i];
        sites[i].zeta = 1.3;
        sites[i].rc = rc[i];
        sites[i].species = i;
        sites[i].ueff_fixed = sites[i].zeta_dn = NAN;
    }
    for (int chunk : {64, 128, 512}) {
        HostTables T;
        if (hub_build_host(cell, ngrid, sites, chunk, T) != HUB_OK) return 1;
        const int64_t G = 9 * 8 * 10;
        BlochTables B;
        if (!hub_build_bloch(T, G, chunk, B, 3)) return std::puts("no limit: declined"), 2;
        const int64_t size = B.wlen * 3 * 8;
        BlochTables C;
        if (!hub_build_bloch(T, G, chunk, C, 3, size) || C.wlen != B.wlen || C.gidx != B.gidx)
            return std::puts("declined at its size"), 2;
        for (int t = 0; t < 2; ++t) {
            BlochTables D = B;
            if (t == 0 ? hub_build_bloch(T, G, chunk, D, 3, size - 1) : hub_build_bloch(T, G, chunk, D, 4, size))
                return std::puts("built past the limit"), 2;
            if (!D.chunks.empty() || !D.gidx.empty() || !D.cval.empty()) return std::puts("left in the list"), 2;
        }
    }
    return 0;
}
