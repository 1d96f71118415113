// Host check of the Coulomb tensors' work list (no GPU): builds the spheres
// and the plan of every site, checks every slot and plane index against its
// buffer, and sums the work items in plain loops as the kernels do (planes
// x' <= x, the plane x' = x with half weight, tensor = S + S^T), for
// comparison with the oracle's direct double sum.
//
// Input (binary, native endianness): cell[3] f64, ngrid[3] i32, nsites i32,
// per site {R[3] f64, l i32, zeta f64, rc f64, species i32}.  Output: per
// site L^4 f64.
// Exit status 0 (ok), 1 (bad input or builder error), 2 (an index out of
// range, or a point in no slot or in two).
#include <cmath>
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
    double cell[3];
    int ngrid[3], ns = 0;
    bool ok = get(f, cell, 3) && get(f, ngrid, 3) && get(f, &ns, 1) && ns > 0;
    std::vector<SiteDef> sites(ok ? ns : 0);
    for (auto& s : sites) {
        ok = ok && get(f, s.R, 3) && get(f, &s.l, 1) && get(f, &s.zeta, 1) && get(f, &s.rc, 1) && get(f, &s.species, 1);
        s.ueff_fixed = s.zeta_dn = NAN;
    }
    std::fclose(f);
    if (!ok) return 1;
    HostTables T;
    if (hub_build_host(cell, ngrid, sites, 64, T) != HUB_OK) return 1;
    std::vector<int> which;
    for (int s = ns - 1; s >= 0; --s) which.push_back(s);              // any order
    CoulombPlan P;
    hub_coulomb_plan(T, which, P);

    double h[3];
    for (int i = 0; i < 3; ++i) h[i] = cell[i] / ngrid[i];
    const double g0 = hub_g0_cell_average(h), dV = h[0] * h[1] * h[2];
    long bad = P.sites.size() != which.size() || P.item_ptr.size() != which.size() + 1;
    std::vector<std::vector<double>> tensors(ns);
    int64_t slots = 0, rho0 = 0, part0 = 0;
    for (size_t i = 0; i < P.sites.size() && !bad; ++i) {
        const CoulombSite& S = P.sites[i];
        const SiteSphere& sp = T.spheres[which[i]];
        const int np = S.L * (S.L + 1) / 2;
        bad += S.index != which[i] || S.L != T.site_L[which[i]] || S.npad < np || S.npad % 16 || S.slot0 != slots;
        bad += S.rho0 != rho0 || S.part0 != part0 || S.nitems != P.item_ptr[i + 1] - P.item_ptr[i];
        const HubInt2* pl = &P.planes[S.plane0];
        int64_t n = 0;
        for (int x = 0; x < S.n[0]; ++x) {
            bad += pl[x].x != n;
            n += (pl[x].y + 15) / 16 * 16;
        }
        // the densities by slot, from the per-site work list as the kernel reads it
        std::vector<double> rho(n * np, 0.0);
        std::vector<int> pos(3 * n, 0), hit(n, 0);
        for (int t = S.chunk0; t < S.chunk1; ++t) {
            const HubChunk& C = T.chunks[T.site_chunk_ids[t]];
            const int32_t* im = &T.images[3 * C.img];
            for (int e = 0; e < C.nreal; ++e) {
                const int g = T.gidx[C.e0 + e];
                const int c[3] = {g / (ngrid[1] * ngrid[2]), g / ngrid[2] % ngrid[1], g % ngrid[2]};
                int r[3];
                for (int k = 0; k < 3; ++k) {
                    r[k] = c[k] + im[k] * ngrid[k] - S.lo[k];
                    bad += r[k] < 0 || r[k] >= S.n[k];
                }
                if (bad) break;
                const HubInt2 ln = P.lines[S.line0 + r[0] * S.n[1] + r[1]];
                const int64_t slot = ln.x + (r[2] - ln.y);
                bad += slot < pl[r[0]].x || slot >= pl[r[0]].x + pl[r[0]].y;
                if (bad) break;
                ++hit[slot];
                for (int k = 0; k < 3; ++k) pos[3 * slot + k] = r[k];
                const double* p = &T.phi[C.phi0 + static_cast<int64_t>(e) * S.L];
                for (int a = 0, q = 0; a < S.L; ++a)
                    for (int b = a; b < S.L; ++b) rho[slot * np + q++] = p[a] * p[b];
            }
        }
        for (int x = 0; x < S.n[0]; ++x)
            for (int s = 0; s < (pl[x].y + 15) / 16 * 16; ++s) bad += hit[pl[x].x + s] != (s < pl[x].y);
        bad += n > 0 && static_cast<int64_t>(sp.g.size()) > n;
        std::vector<double> sum(np * np, 0.0), W(np);
        for (int k = P.item_ptr[i]; k < P.item_ptr[i + 1] && !bad; ++k) {
            const CoulombItem& it = P.items[k];
            bad += it.site != static_cast<int>(i) || it.part != k - P.item_ptr[i] || it.nblk < 1 ||
                   it.nblk > HUB_COUL_MAXBLK || it.x < 0 || it.x >= S.n[0] || it.x0 < 0 || it.x1 > it.x || it.s0 % 16 ||
                   it.s1 % 16 || it.s0 >= it.s1 || it.slot < pl[it.x].x ||
                   it.slot + 16 * it.nblk > pl[it.x].x + (pl[it.x].y + 15) / 16 * 16;
            if (bad) break;
            int walked = 0;
            for (int x = it.x0; x <= it.x1; ++x) {
                const int a = std::max(pl[x].x, it.s0), b = std::min(pl[x].x + (pl[x].y + 15) / 16 * 16, it.s1);
                walked += std::max(0, b - a);
                for (int t = it.slot; t < it.slot + 16 * it.nblk; ++t) {
                    std::fill(W.begin(), W.end(), 0.0);
                    for (int s = a; s < b; ++s) {
                        double r2 = 0.0;
                        for (int c = 0; c < 3; ++c) {
                            const double d = (c == 0 ? it.x - x : pos[3 * t + c] - pos[3 * s + c]) * h[c];
                            r2 += d * d;
                        }
                        const double K = (it.x == x ? 0.5 : 1.0) * (r2 > 0.0 ? 1.0 / std::sqrt(r2) : g0);
                        for (int q = 0; q < np; ++q) W[q] += K * rho[static_cast<int64_t>(s) * np + q];
                    }
                    for (int p = 0; p < np; ++p)
                        for (int q = 0; q < np; ++q) sum[p * np + q] += rho[static_cast<int64_t>(t) * np + p] * W[q];
                }
            }
            bad += walked != it.s1 - it.s0;
        }
        if (bad) break;
        std::vector<double>& X = tensors[which[i]];
        const int L = S.L;
        X.assign(static_cast<size_t>(L) * L * L * L, 0.0);
        for (int a = 0, p = 0; a < L; ++a)
            for (int b = a; b < L; ++b, ++p)
                for (int c = 0, q = 0; c < L; ++c)
                    for (int d = c; d < L; ++d, ++q) {
                        const double v = dV * dV * (sum[p * np + q] + sum[q * np + p]);
                        for (auto [u, w] : {std::pair{a, b}, std::pair{b, a}})
                            for (auto [y, z] : {std::pair{c, d}, std::pair{d, c}}) X[((u * L + w) * L + y) * L + z] = v;
                    }
        slots += n;
        rho0 += n * S.npad;
        part0 += static_cast<int64_t>(S.nitems) * S.npad * S.npad;
    }
    bad += slots != P.slots || rho0 != P.rho || part0 != P.part;
    std::printf("sites %zu slots %ld items %zu bad %ld\n", P.sites.size(), static_cast<long>(slots), P.items.size(), bad);
    if (bad) return 2;
    FILE* o = std::fopen(argv[2], "wb");
    if (!o) return 1;
    bool wrote = true;
    for (const auto& X : tensors) wrote = wrote && std::fwrite(X.data(), sizeof(double), X.size(), o) == X.size();
    std::fclose(o);
    return wrote ? 0 : 1;
}
