// On-site Coulomb tensors, evaluated on the real-space grid (Sec. III: the
// integrals are computed from the orbitals on the grid; App. B gives the
// (m m'|m'' m''') notation):
//
//   (ab|cd) = dV^2 sum_{p, p'} rho_ab(p) K(p - p') rho_cd(p'),
//   rho_ab = phi_a phi_b,  K(r) = 1/|r| (r != 0),  K(0) = G0,
//
// over a site's unfolded sphere points (free-space, single-centre).  G0 is
// the average of 1/r over one grid cell.  This is the direct O(P^2) double
// sum of every site in one launch per pair-density width:
//
//   k_coul_rho:  the pair densities of the points, sorted into planes of
//                constant x (each padded to a multiple of 16 points with
//                zero densities), and each point's (y, z) as byte offsets
//                into a plane of the kernel;
//   k_coul_pair: partial sums S_ij = sum_p rho_i(p) W_j(p), W_j(p) =
//                sum_p' K(p - p') rho_j(p'), over one work item (up to 256
//                points of one plane against a range of source points);
//   k_coul_sum:  adds a site's items in order and writes the L^4 tensor.
//
// K depends on |dx|, |dy|, |dz| only, so a pair of planes needs one |dy| x
// |dz| plane of it: a work-group computes that plane once per source plane
// and every pair reads it from LDS.  The rest is a contraction on the FP64 matrix instructions: W (16 points x 16 densities)
// += K (16 x 4) rho (4 x 16), and S += rho^T W on the same layout (the output
// registers of one product are the operand of the next).  K is symmetric, so
// only the planes x' <= x are summed, the plane x' = x with half weight, and
// the tensor is S + S^T.
//
// Bound: FP64 issue.  The matrix products reach 71 TF/s here, and every vector
// instruction, FP64 or not, holds them up, which is why K is read and not
// evaluated per pair and why a pair block costs two vector instructions
// (|dy|, |dz| as one offset) per product.  Measured: one d shell of 17 152
// points 125 us (7.7 ms with a lane per point that evaluated K for every pair
// on 34 work-groups), 64 p/d/f shells of 746 830 points 4.9 ms (385 ms).

#include "ksmall.h"

namespace {

typedef double hub_d4 __attribute__((ext_vector_type(4)));

// Densities of one site, a thread per entry of the per-site work list.
__global__ void __launch_bounds__(256) k_coul_rho(const CoulombArgs a) {
    const CoulombSite S = a.sites[blockIdx.y];
    const HubChunk* __restrict__ chunks = a.chunks;
    // grid.x walks the site's chunks
    for (int ci = S.chunk0 + blockIdx.x; ci < S.chunk1; ci += gridDim.x) {
        const HubChunk C = chunks[a.chunk_ids[ci]];
        const int32_t* im = a.images + 3 * C.img;
        for (int t = threadIdx.x; t < C.nreal; t += blockDim.x) {
            const int e = C.e0 + t;
            const int g = a.gidx[e];
            const int gx = g / (a.ngrid[1] * a.ngrid[2]), gr = g - gx * (a.ngrid[1] * a.ngrid[2]);
            const int gy = gr / a.ngrid[2], gz = gr - gy * a.ngrid[2];
            const int x = gx + im[0] * a.ngrid[0] - S.lo[0];
            const int y = gy + im[1] * a.ngrid[1] - S.lo[1];
            const int z = gz + im[2] * a.ngrid[2] - S.lo[2];
            const HubInt2 ln = a.lines[S.line0 + x * S.n[1] + y];
            const int64_t slot = S.slot0 + ln.x + (z - ln.y);
            a.yz[slot] = HubInt2{y * S.n[2] * 8, z * 8};
            double ph[7];
            const double* p = a.phi + C.phi0 + static_cast<int64_t>(t) * S.L;
#pragma unroll
            for (int m = 0; m < 7; ++m) ph[m] = m < S.L ? p[m] : 0.0;
            double* r = a.rho + S.rho0 + (slot - S.slot0) * S.npad;
            int k = 0;
#pragma unroll
            for (int i = 0; i < 7; ++i)
#pragma unroll
                for (int j = i; j < 7; ++j)
                    if (j < S.L) r[k++] = ph[i] * ph[j];
            for (; k < S.npad; ++k) r[k] = 0.0;
        }
    }
}

// Zero densities in the padding slots of every plane of the launch's sites.
__global__ void __launch_bounds__(64) k_coul_pad(const CoulombArgs a) {
    const CoulombSite S = a.sites[blockIdx.y];
    for (int x = blockIdx.x; x < S.n[0]; x += gridDim.x) {
        const HubInt2 pl = a.planes[S.plane0 + x];                      // first slot, points
        const int npad = ((pl.y + 15) / 16 * 16 - pl.y);
        for (int o = threadIdx.x; o < npad * S.npad; o += 64)
            a.rho[S.rho0 + static_cast<int64_t>(pl.x + pl.y) * S.npad + o] = 0.0;
        for (int o = threadIdx.x; o < npad; o += 64) a.yz[S.slot0 + pl.x + pl.y + o] = HubInt2{0, 0};
    }
}

// |a - b| + c in one instruction (from the plain expression the compiler makes
// six where it can share a sum; vector instructions hold up the products).
__device__ __forceinline__ unsigned sad(unsigned a, unsigned b, unsigned c) {
    unsigned d;
    asm("v_sad_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Kernel value at byte offset o: an LDS address (the offset counts from 0 of
// the work-group's LDS), or from Kg in device memory.
typedef __attribute__((address_space(3))) double lds_double;
template <bool LDSK>
__device__ __forceinline__ double kernel_at(const double* __restrict__ Kg, unsigned o) {
    if constexpr (LDSK) return *reinterpret_cast<const lds_double*>(o);
    else return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(Kg) + o);
}

__device__ __forceinline__ double coul_kernel(const CoulombArgs& a, int dx, int dy, int dz) {
    const double x = static_cast<double>(dx) * a.h[0];
    const double y = static_cast<double>(dy) * a.h[1];
    const double z = static_cast<double>(dz) * a.h[2];
    const double r2 = x * x + y * y + z * z;
    const double K = r2 > 0.0 ? rsqrt(r2) : a.g0;
    return dx == 0 ? 0.5 * K : K;                                    // x' = x is counted from both sides
}

// Kernel planes of one site in global memory, for spheres whose planes do not
// fit in the work-group's LDS.
__global__ void __launch_bounds__(256) k_coul_table(const CoulombArgs a, const CoulombSite S) {
    const int64_t n = static_cast<int64_t>(S.n[0]) * S.n[1] * S.n[2];
    for (int64_t o = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; o < n;
         o += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        const int dz = static_cast<int>(o % S.n[2]);
        const int64_t r = o / S.n[2];
        a.ktab[o] = coul_kernel(a, static_cast<int>(r / S.n[1]), static_cast<int>(r % S.n[1]), dz);
    }
}

// One work item for MB target blocks of 16 points per wave.  Operand layouts
// of the 16x16x4 product (lane l): A[l % 16][l / 16], B[l / 16][l % 16],
// D[l / 16 + 4 r][l % 16] in register r.  A wave past the item's last block
// repeats it and leaves it out of its sum.
template <int MB, int NT, bool LDSK>
__device__ __forceinline__ void pair_item(const CoulombArgs& a, const CoulombSite& S, const CoulombItem& it,
                                          double* lds) {
    constexpr int NP = 16 * NT;
    const double* __restrict__ rho = a.rho + S.rho0;
    const HubInt2* __restrict__ yz = a.yz + S.slot0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, i16 = lane & 15, k4 = lane >> 4;
    const int b0 = wave * MB;
    HubInt2 tgt[MB];
#pragma unroll
    for (int t = 0; t < MB; ++t) tgt[t] = yz[it.slot + 16 * min(b0 + t, it.nblk - 1) + i16];
    hub_d4 acc[MB][NT];
#pragma unroll
    for (int t = 0; t < MB; ++t)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[t][n] = hub_d4{0.0, 0.0, 0.0, 0.0};
    const int nyz = S.n[1] * S.n[2];
    for (int xs = it.x0; xs <= it.x1; ++xs) {
        const HubInt2 pl = a.planes[S.plane0 + xs];
        const int s0 = max(pl.x, it.s0), s1 = min(pl.x + (pl.y + 15) / 16 * 16, it.s1);
        const int dx = it.x - xs;
        const double* __restrict__ Kg = nullptr;
        const unsigned base = LDSK ? static_cast<unsigned>(reinterpret_cast<uintptr_t>((lds_double*)lds)) : 0u;
        if constexpr (LDSK) {
            __syncthreads();
            for (int o = threadIdx.x; o < nyz; o += 256) {
                const int dy = o / S.n[2];
                lds[o] = coul_kernel(a, dx, dy, o - dy * S.n[2]);
            }
            __syncthreads();
        } else {
            Kg = a.ktab + static_cast<int64_t>(dx) * nyz;
        }
        if (s0 >= s1) continue;
        // acc += K rho, 16 sources at a time (the plane's slots are multiples
        // of 16); the densities and offsets of the next 16 are loaded while
        // the current ones are contracted, into the other of two buffers.
        // Uniform addresses and constant lane offsets: vector instructions
        // and FP64 products do not issue together.
        struct Src {
            double r[4][NT];
            HubInt2 c[4];
        };
        auto load = [&](int s, Src& x) {
            const double* __restrict__ rs = rho + static_cast<int64_t>(s) * NP;
            const HubInt2* __restrict__ cs = yz + s;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x.c[u] = cs[4 * u + k4];
#pragma unroll
                for (int n = 0; n < NT; ++n) x.r[u][n] = rs[4 * u * NP + 16 * n + (k4 * NP + i16)];
            }
        };
        auto contract = [&](const Src& x, Src& y, int next) {
            double K[4][MB];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < MB; ++t)
                    K[u][t] = kernel_at<LDSK>(Kg, sad(tgt[t].x, x.c[u].x, sad(tgt[t].y, x.c[u].y, base)));
            load(next, y);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < MB; ++t)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[t][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(K[u][t], x.r[u][n], acc[t][n], 0, 0, 0);
        };
        Src sa, sb;
        load(s0, sa);
        int s = s0;
        for (; s + 32 <= s1; s += 32) {
            contract(sa, sb, s + 16);
            contract(sb, sa, s + 32 < s1 ? s + 32 : s0);
        }
        if (s < s1) contract(sa, sb, s0);
    }
    // S += rho^T W of the wave's points
    hub_d4 T[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) T[i][j] = hub_d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < MB; ++t) {
        if (b0 + t >= it.nblk) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t sl = it.slot + 16 * (b0 + t) + 4 * r + k4;
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const double x = rho[sl * NP + 16 * i + i16];
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    T[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, acc[t][j][r], T[i][j], 0, 0, 0);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                lds[((wave * NP) + 16 * i + k4 + 4 * r) * NP + 16 * j + i16] = T[i][j][r];
    __syncthreads();
    // the waves in order, and S + S^T (the same number for (i, j) and (j, i))
    double* __restrict__ out = a.part + S.part0 + static_cast<int64_t>(it.part) * (NP * NP);
    for (int o = threadIdx.x; o < NP * NP; o += 256) {
        const int q = (o % NP) * NP + o / NP;
        const double x = ((lds[o] + lds[NP * NP + o]) + lds[2 * NP * NP + o]) + lds[3 * NP * NP + o];
        const double y = ((lds[q] + lds[NP * NP + q]) + lds[2 * NP * NP + q]) + lds[3 * NP * NP + q];
        out[o] = x + y;
    }
}

// One work item per work-group of four waves; each wave takes a quarter of
// the item's target blocks, and all waves walk the same sources.
// At least two waves per SIMD: with at most 256 registers the products keep
// their sums in vector registers (with more, the compiler moves every sum to
// accumulation registers and back each 16 sources).
template <int NT, bool LDSK>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_coul_pair(const CoulombArgs a, const CoulombItem* __restrict__ items) {
    extern __shared__ double lds[];
    const CoulombItem it = items[blockIdx.x];
    const CoulombSite S = a.sites[it.site];
    switch ((it.nblk + 3) / 4) {
    case 1: pair_item<1, NT, LDSK>(a, S, it, lds); break;
    case 2: pair_item<2, NT, LDSK>(a, S, it, lds); break;
    case 3: pair_item<3, NT, LDSK>(a, S, it, lds); break;
    default: pair_item<4, NT, LDSK>(a, S, it, lds); break;
    }
}

// Tensor rows of pair i = blockIdx.x of site blockIdx.y: the site's items in
// NS interleaved slices, each summed in order, then the slices in order.
__global__ void __launch_bounds__(1024) k_coul_sum(const CoulombArgs a) {
    __shared__ double red[1024];
    const CoulombSite S = a.sites[blockIdx.y];
    const int i = blockIdx.x, L = S.L, np = L * (L + 1) / 2, NP = S.npad;
    if (i >= np) return;
    const int NS = 1024 / NP;
    const int j = threadIdx.x % NP, sl = threadIdx.x / NP;
    const double* __restrict__ p = a.part + S.part0;
    double s = 0.0;
    for (int b = sl; b < S.nitems; b += 8 * NS) {
        double u[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            u[k] = p[static_cast<int64_t>(b + k * NS < S.nitems ? b + k * NS : b) * (NP * NP) + i * NP + j];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 8; ++k) s += b + k * NS < S.nitems ? u[k] : 0.0;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (sl != 0 || j >= np) return;
    double t = 0.0;
    for (int k = 0; k < NS; ++k) t += red[k * NP + j];
    const double v = a.dV * a.dV * t;
    // pair index i -> (A <= B), j -> (C <= D)
    int A = 0, B = 0, C = 0, D = 0;
    for (int x = 0, q = 0; x < L; ++x)
        for (int y = x; y < L; ++y, ++q) {
            if (q == i) { A = x; B = y; }
            if (q == j) { C = x; D = y; }
        }
    auto at = [L](int w, int x, int y, int z) { return ((w * L + x) * L + y) * L + z; };
    double* __restrict__ o = a.tensor + static_cast<int64_t>(S.index) * 2401;
    o[at(A, B, C, D)] = v;
    o[at(B, A, C, D)] = v;
    o[at(A, B, D, C)] = v;
    o[at(B, A, D, C)] = v;
}

template <int NT, bool LDSK>
hipError_t launch_pair(const CoulombArgs& a, const CoulombItem* items, int nitems, size_t lds, hipStream_t st) {
    if (nitems > 0)
        hipLaunchKernelGGL((k_coul_pair<NT, LDSK>), dim3(nitems), dim3(256), lds, st, a, items);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_coulomb_prepare(const CoulombArgs& a, int nsites, int maxplanes, hipStream_t st) {
    if (nsites <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_coul_rho, dim3(64, nsites), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_coul_pad, dim3(maxplanes, nsites), dim3(64), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_coulomb_table(const CoulombArgs& a, const CoulombSite& S, hipStream_t st) {
    hipLaunchKernelGGL(k_coul_table, dim3(1024), dim3(256), 0, st, a, S);
    return hipGetLastError();
}

hipError_t launch_coulomb_pair(const CoulombArgs& a, const CoulombItem* items, int nitems, int npad, int plane,
                               hipStream_t st) {
    const size_t red = static_cast<size_t>(4) * npad * npad * sizeof(double);
    if (a.ktab) {
        return npad == 16 ? launch_pair<1, false>(a, items, nitems, red, st)
                          : launch_pair<2, false>(a, items, nitems, red, st);
    }
    const size_t k = static_cast<size_t>(plane) * sizeof(double);
    if (k > HUB_COUL_LDS) return hipErrorInvalidValue;
    const size_t lds = k > red ? k : red;
    return npad == 16 ? launch_pair<1, true>(a, items, nitems, lds, st)
                      : launch_pair<2, true>(a, items, nitems, lds, st);
}

hipError_t launch_coulomb_sum(const CoulombArgs& a, int nsites, int maxpair, hipStream_t st) {
    if (nsites <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_coul_sum, dim3(maxpair, nsites), dim3(1024), 0, st, a);
    return hipGetLastError();
}
