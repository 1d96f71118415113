// Host check of the Bloch-summed work list built by the library's sphere
// builder (no GPU): reads a system and complex states for one k-point, checks
// every index against its buffer, that every covered grid point appears once
// per pass and every cover once in all, and writes
// c[j][s] = dV sum_entries (sum_covers exp(i k.T) phi) psi[g][s], the sum the
// projection kernel evaluates, for comparison with the oracle's projections.
//
// Input (binary, native endianness): cell[3] f64, ngrid[3] i32, nsites i32,
// per site {R[3] f64, l i32, zeta f64, rc f64, species i32}, k_red[3] f64,
// nstates i32, psi[G][nstates] complex f64.  Output: c as complex f64.
// Exit status 0 (ok), 1 (bad input or builder error), 2 (a check failed).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <vector>

#include "hub_internal.h"

namespace {
template <typename T>
bool get(FILE* f, T* p, size_t n) { return std::fread(p, sizeof(T), n, f) == n; }
}  // namespace

int main(int argc, char** argv) {
    if (argc != 3) return 1;
    FILE* f = std::fopen(argv[1], "rb");
    if (!f) return 1;
    double cell[3], k[3];
    int ngrid[3], ns = 0, S = 0;
    bool ok = get(f, cell, 3) && get(f, ngrid, 3) && get(f, &ns, 1) && ns > 0;
    std::vector<SiteDef> sites(ok ? ns : 0);
    for (auto& s : sites) {
        ok = ok && get(f, s.R, 3) && get(f, &s.l, 1) && get(f, &s.zeta, 1) && get(f, &s.rc, 1) && get(f, &s.species, 1);
        s.ueff_fixed = s.zeta_dn = NAN;
    }
    ok = ok && get(f, k, 3) && get(f, &S, 1) && S > 0;
    const long G = static_cast<long>(ngrid[0]) * ngrid[1] * ngrid[2];
    std::vector<std::complex<double>> psi(ok ? G * S : 0);
    ok = ok && get(f, psi.data(), psi.size());
    std::fclose(f);
    if (!ok) return 1;
    HostTables T;
    if (hub_build_host(cell, ngrid, sites, 128, T) != HUB_OK) return 1;
    BlochTables B;
    hub_build_bloch(T, G, 128, B);

    const long nimg = static_cast<long>(T.images.size() / 3);
    long bad = 0, w = 0, rows = 0, covers = 0, points = 0;
    bad += B.cptr.size() != B.gidx.size() + 1 || B.f_orb.size() != B.chunks.size() * HUB_GF_MAX;
    bad += B.pass_ptr.empty() || B.pass_ptr.back() != static_cast<int>(B.chunks.size());
    for (const SiteSphere& sp : T.spheres) covers += static_cast<long>(sp.g.size());
    const double dV = cell[0] / ngrid[0] * cell[1] / ngrid[1] * cell[2] / ngrid[2];
    std::vector<std::complex<double>> part;
    std::vector<int> row_orb;
    for (size_t p = 0; p + 1 < B.pass_ptr.size() && !bad; ++p) {
        std::vector<char> seen(G, 0);
        for (int ci = B.pass_ptr[p]; ci < B.pass_ptr[p + 1] && !bad; ++ci) {
            const HubChunk& C = B.chunks[ci];
            bad += C.layer != static_cast<int>(p) || C.L < 1 || C.L > HUB_GF_MAX || C.ne % HUB_ENTRY_ALIGN ||
                   C.nreal < 1 || C.nreal > C.ne || C.phi0 != w || C.part0 != rows || C.e0 < 0 ||
                   C.e0 + static_cast<size_t>(C.ne) > B.gidx.size();
            if (bad) break;
            part.resize((rows + C.L) * S);
            for (int q = 0; q < HUB_GF_MAX; ++q) bad += (q < C.L) != (B.f_orb[ci * HUB_GF_MAX + q] >= 0);
            for (int q = 0; q < C.L; ++q) row_orb.push_back(B.f_orb[ci * HUB_GF_MAX + q]);
            for (int e = 0; e < C.ne; ++e) {
                const int g = B.gidx[C.e0 + e];
                bad += g < 0 || g >= G;
                if (bad) break;
                if (e < C.nreal) {
                    bad += seen[g]++;
                    ++points;
                } else {
                    bad += g != B.gidx[C.e0 + C.nreal - 1] || B.cptr[C.e0 + e] != B.cptr[C.e0 + e + 1];
                }
                for (int c = B.cptr[C.e0 + e]; c < B.cptr[C.e0 + e + 1]; ++c) {
                    const int f0 = B.cfun[c] & 255, L = B.cfun[c] >> 8;
                    bad += f0 + L > C.L || B.cimg[c] < 0 || B.cimg[c] >= nimg ||
                           B.coff[c] + L > static_cast<long>(B.cval.size());
                    if (bad) break;
                    const int32_t* im = &T.images[3 * B.cimg[c]];
                    const double a = 2.0 * M_PI * (k[0] * im[0] + k[1] * im[1] + k[2] * im[2]);
                    const std::complex<double> ph(std::cos(a), std::sin(a));
                    for (int m = 0; m < L; ++m)
                        for (int s = 0; s < S; ++s)
                            part[(rows + f0 + m) * S + s] += dV * ph * B.cval[B.coff[c] + m] * psi[static_cast<long>(g) * S + s];
                    --covers;
                }
            }
            rows += C.L;
            w += static_cast<long>(C.ne) * hub_bloch_row(C.L);
        }
        for (long g = 0; p == 0 && g < G; ++g) {
            bool any = false;
            for (const SiteSphere& sp : T.spheres) any = any || std::binary_search(sp.g.begin(), sp.g.end(), g);
            bad += any != (seen[g] != 0);
        }
    }
    bad += covers != 0 || rows != B.part_rows || w != B.wlen;
    bad += B.red_ptr.size() != static_cast<size_t>(T.J) + 1 || B.red_row.size() != static_cast<size_t>(rows);
    std::vector<std::complex<double>> c(static_cast<size_t>(T.J) * S);
    for (int j = 0; j < T.J && !bad; ++j)
        for (int t = B.red_ptr[j]; t < B.red_ptr[j + 1]; ++t) {
            const int r = B.red_row[t];
            bad += r < 0 || r >= rows || row_orb[r] != j;
            if (bad) break;
            for (int s = 0; s < S; ++s) c[static_cast<size_t>(j) * S + s] += part[static_cast<size_t>(r) * S + s];
        }
    std::printf("passes %zu chunks %zu points %ld bad %ld\n", B.pass_ptr.size() - 1, B.chunks.size(), points, bad);
    if (bad) return 2;
    FILE* o = std::fopen(argv[2], "wb");
    if (!o) return 1;
    const bool wrote = std::fwrite(c.data(), sizeof(c[0]), c.size(), o) == c.size();
    std::fclose(o);
    return wrote ? 0 : 1;
}
