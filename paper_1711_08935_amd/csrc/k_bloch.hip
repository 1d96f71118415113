// Projection and apply over the Bloch-summed work list (BlochTables): complex
// states whose grid points carry more (orbital, image) functions than one
// pass of the grouped list takes.  With W_f(e) = sum_T exp(i k.T) phi_f the
// sum over the images of function f at entry e,
//   part[q][row][col] = sum_e W_f(e) psi_q[g_e][col],
//   hpsi_q[g_e][col] += sum_f conj(W_f(e)) B_f(col),
//   B = alpha scale V c (Eq. pot_V_U), the image phases being in W.
// W depends on the k-point only and is built once per context.
//
// Every row is read (and written) once per pass, mostly once in all, instead
// of once per 16 (orbital, image) functions, and a function costs four FP64
// multiply-adds per column whatever its images (two per image before).  The
// contractions run on the FP64 matrix instructions with the real and
// imaginary parts as separate rows: the operands come from vector loads in
// lane order, where 32 scalar values per entry would not fit the scalar
// registers.  Bound: FP64 matrix rate and HBM about equally (110 592 points, 16
// functions, 16 sets of 64 FP32 columns: 0.18 ms of products, 0.22 ms of rows
// and tables for the projection).  Measured there against the grouped list's
// five passes (76 functions): projection 0.31 ms (0.76), reduction 0.020
// (0.099), apply 0.43 (1.39).  31 functions in FP64, 16 sets of 45 columns:
// 0.37 and 0.52 ms (0.56 and 0.95).  Where few points need a second pass or rows
// are short the passes win (use_bloch, hub_api.hip).

#include "kbloch.h"

namespace {

typedef double hub_d4 __attribute__((ext_vector_type(4)));

// Tables W of one k-point (blockIdx.y) and chunk (blockIdx.x): row e holds the
// real parts of its 8 or 16 functions, then the imaginary parts.
__global__ void __launch_bounds__(256) k_bloch_table(const BlochTableArgs a) {
    const HubChunk C = a.chunks[blockIdx.x];
    const int k = blockIdx.y;
    const int half = C.L > 8 ? 16 : 8;
    double* __restrict__ W = a.W + k * a.wlen + C.phi0;
    for (int o = threadIdx.x; o < C.ne * half; o += blockDim.x) {
        const int e = o / half, f = o - e * half;
        double wr = 0.0, wi = 0.0;
        for (int c = a.cptr[C.e0 + e]; c < a.cptr[C.e0 + e + 1]; ++c) {
            const int f0 = a.cfun[c] & 255, L = a.cfun[c] >> 8;
            if (f < f0 || f >= f0 + L) continue;
            const double v = a.cval[a.coff[c] + f - f0];
            const double* ph = a.phase + (static_cast<int64_t>(k) * a.nimg + a.cimg[c]) * 2;
            wr = fma(ph[0], v, wr);
            wi = fma(ph[1], v, wi);
        }
        W[static_cast<int64_t>(e) * 2 * half + f] = wr;
        W[static_cast<int64_t>(e) * 2 * half + half + f] = wi;
    }
}

// 16-entry blocks [first, last) of part idx of the parts that share a chunk's
// n entries, whole pairs of blocks.
__device__ __forceinline__ void block_range(int n, int parts, int idx, int& first, int& last) {
    const int pairs = n / 32, per = (pairs + parts - 1) / parts;
    first = 2 * idx * per;
    last = 2 * (pairs < (idx + 1) * per ? pairs : (idx + 1) * per);
}

// One wave per (chunk, 16 NJ columns of one set); lane l holds columns l % 16
// (and l % 16 + 16) of the tile.  Operands of the 16x16x4 product: A[l % 16][l / 16]
// = W rows (mt = 0: real parts of functions l % 16, mt = 1: imaginary parts;
// MT = 1: real parts of 8 functions, then imaginary parts), B[l / 16][l % 16]
// = state values, D[l / 16 + 4 r][l % 16].  The rows and tables of the next 16
// entries are loaded while the current ones are contracted, their grid
// indexes one block earlier.
template <typename T, int MT, int NJ>
__device__ __forceinline__ void project_tile(const BlochArgs& a, const HubChunk& C, int q, int c0, int part_of,
                                             const int32_t* __restrict__ gidx, const double* __restrict__ W,
                                             double* __restrict__ part) {
    constexpr int RL = 16 * MT;
    const int lane = threadIdx.x, i16 = lane & 15, g4 = lane >> 4;
    const T* __restrict__ psi_q = static_cast<const T*>(a.psi) + static_cast<int64_t>(q) * a.qstride;
    const int32_t* __restrict__ gi = gidx + C.e0 + g4;
    const double* __restrict__ w0 = W + C.phi0 + g4 * RL + i16;
    const int64_t stride = a.ld * 2;
    int64_t cofs[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = c0 + 16 * j + i16;
        cofs[j] = 2 * static_cast<int64_t>(col < a.ncol ? col : 0);
    }
    struct Blk {
        T x[4][NJ][2];
        double w[4][MT];
    };
    auto index = [&](int b, int (&g)[4]) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) g[kb] = gi[16 * b + 4 * kb];
    };
    auto load = [&](int b, const int (&g)[4], Blk& B) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) load_row_stream<T, 2>(psi_q + g[kb] * stride + cofs[j], B.x[kb][j]);
#pragma unroll
            for (int m = 0; m < MT; ++m) B.w[kb][m] = w0[(16 * b + 4 * kb) * RL + 16 * m];
        }
    };
    hub_d4 acc[MT][NJ][2];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[m][j][0] = acc[m][j][1] = hub_d4{0.0, 0.0, 0.0, 0.0};
    auto contract = [&](const Blk& B) {
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const double x = static_cast<double>(B.x[kb][j][p]);
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m][j][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(B.w[kb][m], x, acc[m][j][p], 0, 0, 0);
                }
    };
    // whole pairs of blocks (C.ne is a multiple of 32); the block past the last
    // re-reads the last one
    int first, nb;
    block_range(C.ne, a.split, part_of, first, nb);
    Blk A, B;
    int ga[4], gb[4];
    if (first < nb) {
        index(first, ga);
        index(first + 1, gb);
        load(first, ga, A);
    }
    for (int b = first; b < nb; b += 2) {
        load(b + 1, gb, B);
        const int n0 = b + 2 < nb ? b + 2 : nb - 1, n1 = b + 3 < nb ? b + 3 : nb - 1;
        index(n0, ga);
        __builtin_amdgcn_sched_barrier(0);
        contract(A);
        load(n0, ga, A);
        index(n1, gb);
        __builtin_amdgcn_sched_barrier(0);
        contract(B);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = c0 + 16 * j + i16;
        if (col >= a.ncol) continue;
#pragma unroll
        for (int r = 0; r < 2 * MT; ++r) {
            const int f = g4 + 4 * r;
            if (f >= C.L) continue;
            hub_d2 z;
            if constexpr (MT == 2) {
                z[0] = acc[0][j][0][r] - acc[1][j][1][r];
                z[1] = acc[0][j][1][r] + acc[1][j][0][r];
            } else {
                z[0] = acc[0][j][0][r] - acc[0][j][1][r + 2];
                z[1] = acc[0][j][1][r] + acc[0][j][0][r + 2];
            }
            *reinterpret_cast<hub_d2*>(
                part + ((static_cast<int64_t>(q) * a.prows + static_cast<int64_t>(C.part0 + f) * a.split + part_of) *
                            a.ncol + col) * 2) = z;
        }
    }
}

template <typename T, int NJ>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_bloch_project(const BlochArgs a, const int32_t* __restrict__ gidx, const double* __restrict__ W,
                double* __restrict__ part) {
    const HubSlot slot = hub_slot(a.tiles);
    if (slot.chunk >= a.nchunks) return;
    const HubChunk C = a.chunks[a.chunk0 + slot.chunk];
    const int tps = (a.ncol + 16 * NJ - 1) / (16 * NJ);
    const int tile = slot.tile / a.split, part_of = slot.tile - tile * a.split;
    const int q = tile / tps, c0 = (tile - q * tps) * (16 * NJ);
    const int k = a.spinor ? a.q0 + q : (a.q0 + q) / a.nspin;
    const double* __restrict__ Wk = W + k * a.wlen;
    if (C.L > 8) project_tile<T, 2, NJ>(a, C, q, c0, part_of, gidx, Wk, part);
    else project_tile<T, 1, NJ>(a, C, q, c0, part_of, gidx, Wk, part);
}

// Coefficients of one work-group (one wave): z[f][i] = alpha scale sum_b V_ab c_b
// of the chunk's function f (orbital a of its site) and column c0 + i, as
// coefficient() of the grouped apply forms them.  The projections of the
// chunk's orbitals and the rows of V of its functions are staged in LDS, every
// load of the two in flight together, so that the wave waits twice (for the
// functions' records and for these) however many functions it has.  From a
// buffer that a launch of its own filled, the apply took as long on full
// launches (110 592 points, 16 sets of 64 columns: 454 us, 456 here) and longer
// on small ones (13 824 points, 16 sets of 13 columns: 24.3 us, 20.4 here).
template <bool SPINOR, int NF, int NC>
struct CoefLds {
    static constexpr int NV = SPINOR ? 4 : 1;        // blocks of n that a site's columns use
    hub_d2 c[NF][NC];                                // the projections, then the coefficients z
    hub_d2 V[NV][NF][HUB_LMAX];
};

template <bool SPINOR, int NF, int NC>
__device__ __forceinline__ void bloch_coefficients(const ApplyArgs& a, const HubFun* __restrict__ fun, int nf, int q,
                                                   int c0, CoefLds<SPINOR, NF, NC>& lds) {
    using Lds = CoefLds<SPINOR, NF, NC>;
    constexpr int STEP = 64 / NC, NT = NF / STEP;                    // functions at once; per lane
    constexpr int VT = (Lds::NV * NF * 8 + 63) / 64;                 // rows of V, eight slots a function
    const int lane = threadIdx.x, i = lane % NC, h = lane / NC;
    const int col = c0 + i, colc = col < a.ncol ? col : 0;
    const double* __restrict__ cq = a.c + static_cast<int64_t>(q) * a.J * a.ncol * 2;
    hub_d2 x[NT], v[VT];
    double U[VT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int f = h + STEP * t;
        const HubFun F = fun[f < nf ? f : 0];
        x[t] = *reinterpret_cast<const hub_d2*>(cq + (static_cast<int64_t>(F.o0 + F.m) * a.ncol + colc) * 2);
    }
#pragma unroll
    for (int t = 0; t < VT; ++t) {
        const int o = lane + 64 * t, b = o & 7, f = (o >> 3) % NF, blk = (o >> 3) / NF;
        const HubFun F = fun[f < nf ? f : 0];
        const int ch = SPINOR ? blk : (a.q0 + q) % a.nspin;
        v[t] = *reinterpret_cast<const hub_d2*>(
            a.n + ((static_cast<int64_t>(F.site) * a.nblk + ch) * 49 + (b < F.L ? b : 0) * 7 + F.m) * 2);
        U[t] = a.ueff[F.site];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < NT; ++t) lds.c[h + STEP * t][i] = x[t];
#pragma unroll
    for (int t = 0; t < VT; ++t) {
        // V_ab = U (delta_ab / 2 - n_ba); spinors: block 2 sigma' + sigma of n
        // gives V^{sigma sigma'}
        const int o = lane + 64 * t, b = o & 7, f = (o >> 3) % NF, blk = (o >> 3) / NF;
        const HubFun F = fun[f < nf ? f : 0];
        const bool diag = F.m == b && (!SPINOR || blk == 0 || blk == 3);
        hub_d2 w;
        w[0] = SPINOR ? U[t] * (diag ? 0.5 : 0.0) - U[t] * v[t][0] : U[t] * ((diag ? 0.5 : 0.0) - v[t][0]);
        w[1] = -U[t] * v[t][1];
        if (b < HUB_LMAX) lds.V[blk][f][b] = w;
    }
    __syncthreads();
    double sc = a.alpha;
    if (a.colscale != nullptr && col < a.ncol)
        sc *= a.colscale[static_cast<int64_t>(q) * a.nstates + (SPINOR ? col >> 1 : col)];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int f = h + STEP * t;
        const HubFun F = fun[f < nf ? f : 0];
        const int f0 = f - F.m;                                      // the site's first function
        double br = 0.0, bi = 0.0;
#pragma unroll
        for (int s = 0; s < (SPINOR ? 2 : 1); ++s) {
            // spinor columns 2 s + sigma; tiles start at even columns
            const int blk = SPINOR ? 2 * s + (i & 1) : 0, is = SPINOR ? (i & ~1) + s : i;
#pragma unroll
            for (int b = 0; b < HUB_LMAX; ++b) {
                if (b >= F.L || f >= nf) break;
                const hub_d2 w = lds.V[blk][f][b], y = lds.c[f0 + b][is];
                br = fma(w[0], y[0], fma(-w[1], y[1], br));
                bi = fma(w[0], y[1], fma(w[1], y[0], bi));
            }
        }
        x[t] = hub_d2{br * sc, bi * sc};
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) lds.c[h + STEP * t][i] = x[t];
    __syncthreads();
}

// The same tile in the apply: A[l % 16][.] = W of point l % 16 of a 16-point
// block, the functions' parts split over the lane groups in the order of the
// table row (lane group l / 16 takes RL / 4 consecutive values), B = the
// coefficients in that order, the sum starts at hpsi.
template <typename T, bool SPINOR, int MT, int NJ>
__device__ __forceinline__ void apply_tile(const BlochArgs& a, const ApplyArgs& u, const HubChunk& C,
                                           const HubFun* __restrict__ fun, int q, int c0, int first, int nb,
                                           const int32_t* __restrict__ gidx, const double* __restrict__ W,
                                           T* __restrict__ hpsi, CoefLds<SPINOR, 8 * MT, 16 * NJ>& lds) {
    constexpr int RL = 16 * MT, KB = RL / 4;
    const int lane = threadIdx.x, i16 = lane & 15, g4 = lane >> 4;
    T* __restrict__ h_q = hpsi + static_cast<int64_t>(q) * a.qstride;
    const int64_t stride = a.ld * 2;
    bool ok[NJ];
    int64_t cofs[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = c0 + 16 * j + i16;
        ok[j] = col < a.ncol;
        cofs[j] = 2 * static_cast<int64_t>(ok[j] ? col : 0);
    }
    bloch_coefficients<SPINOR, 8 * MT, 16 * NJ>(u, fun, C.L, q, c0, lds);
    // conj(W) B = (Wr Br + Wi Bi) + i (Wr Bi - Wi Br)
    double bf[KB][NJ][2];
    const bool imag = g4 >> 1;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int f = KB * (g4 & 1) + kb;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const hub_d2 z = lds.c[f][16 * j + i16];
            const bool use = f < C.L && ok[j];
            bf[kb][j][0] = use ? (imag ? z[1] : z[0]) : 0.0;
            bf[kb][j][1] = use ? (imag ? -z[0] : z[1]) : 0.0;
        }
    }
    const int32_t* __restrict__ gi = gidx + C.e0 + g4;
    const double* __restrict__ w0 = W + C.phi0 + i16 * RL + g4 * KB;
    struct Blk {
        T x[4][NJ][2];
        double w[KB];
    };
    auto index = [&](int b, int (&g)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) g[r] = gi[16 * b + 4 * r];
    };
    auto load = [&](int b, const int (&g)[4], Blk& B) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < NJ; ++j) load_row<T, 2>(h_q + g[r] * stride + cofs[j], B.x[r][j]);
#pragma unroll
        for (int kb = 0; kb < KB; kb += 2) {
            const hub_d2 z = *reinterpret_cast<const hub_d2*>(w0 + 16 * b * RL + kb);
            B.w[kb] = z[0];
            B.w[kb + 1] = z[1];
        }
    };
    auto update = [&](int b, const int (&g)[4], const Blk& B) {
        hub_d4 acc[NJ][2];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[j][p][r] = static_cast<double>(B.x[r][j][p]);
            }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    acc[j][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(B.w[kb], bf[kb][j][p], acc[j][p], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // padding entries repeat the last point
            if (16 * b + 4 * r + g4 >= C.nreal) continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (!ok[j]) continue;
                const T out[2] = {static_cast<T>(acc[j][0][r]), static_cast<T>(acc[j][1][r])};
                store_row<T, 2>(h_q + g[r] * stride + cofs[j], out);
            }
        }
    };
    Blk A, B;
    int ga[4], gb[4], gn[4];
    index(first, ga);
    index(first + 1, gb);
    load(first, ga, A);
    for (int b = first; b < nb; b += 2) {
        load(b + 1, gb, B);
        const int n0 = b + 2 < nb ? b + 2 : nb - 1, n1 = b + 3 < nb ? b + 3 : nb - 1;
        index(n0, gn);
        __builtin_amdgcn_sched_barrier(0);
        update(b, ga, A);
#pragma unroll
        for (int r = 0; r < 4; ++r) ga[r] = gn[r];
        // the block past the last re-reads the last one, whose copy is not used
        load(n0, ga, A);
        index(n1, gn);
        __builtin_amdgcn_sched_barrier(0);
        update(b + 1, gb, B);
#pragma unroll
        for (int r = 0; r < 4; ++r) gb[r] = gn[r];
    }
}

template <typename T, bool SPINOR, int NJ>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_bloch_apply(const BlochArgs a, const ApplyArgs u, const int32_t* __restrict__ gidx, const double* __restrict__ W,
              T* __restrict__ hpsi) {
    __shared__ union Lds {
        CoefLds<SPINOR, 16, 16 * NJ> wide;
        CoefLds<SPINOR, 8, 16 * NJ> narrow;
        __device__ Lds() {}
    } lds;
    const HubSlot slot = hub_slot(a.tiles);
    if (slot.chunk >= a.nchunks) return;
    const int ci = a.chunk0 + slot.chunk;
    const HubChunk C = a.chunks[ci];
    const int tps = (a.ncol + 16 * NJ - 1) / (16 * NJ);
    const int tile = slot.tile / a.split, part_of = slot.tile - tile * a.split;
    int first, nb;
    block_range(C.ne, a.split, part_of, first, nb);
    if (first >= nb) return;
    const int q = tile / tps, c0 = (tile - q * tps) * (16 * NJ);
    const int k = a.spinor ? a.q0 + q : (a.q0 + q) / a.nspin;
    const double* __restrict__ Wk = W + k * a.wlen;
    const HubFun* __restrict__ fun = a.fun + ci * HUB_GF_MAX;
    if (C.L > 8) apply_tile<T, SPINOR, 2, NJ>(a, u, C, fun, q, c0, first, nb, gidx, Wk, hpsi, lds.wide);
    else apply_tile<T, SPINOR, 1, NJ>(a, u, C, fun, q, c0, first, nb, gidx, Wk, hpsi, lds.narrow);
}

}  // namespace

hipError_t launch_bloch_table(const BlochTableArgs& a, int nchunks, int nk, hipStream_t st) {
    hipLaunchKernelGGL(k_bloch_table, dim3(nchunks, nk), dim3(256), 0, st, a);
    return hipGetLastError();
}

// 32 columns per wave unless that leaves more lanes idle than 16 (13 FP64
// columns of six sets: 38 us, 51 with 32)
int bloch_nj(int ncol) { return (ncol + 31) / 32 * 2 == (ncol + 15) / 16 ? 2 : 1; }

namespace {

template <typename T, int NJ>
hipError_t project_t(const BlochArgs& a, hipStream_t st) {
    BlochArgs b = a;
    b.tiles = a.nq * ((a.ncol + 16 * NJ - 1) / (16 * NJ)) * a.split;
    hipLaunchKernelGGL((k_bloch_project<T, NJ>), dim3(static_cast<unsigned>(hub_slot_grid(a.nchunks, b.tiles))), dim3(64),
                       0, st, b, b.gidx, b.W, b.part);
    return hipGetLastError();
}

template <typename T, bool SPINOR, int NJ>
hipError_t apply_t(const BlochArgs& a, const ApplyArgs& u, hipStream_t st) {
    BlochArgs b = a;
    b.tiles = a.nq * ((a.ncol + 16 * NJ - 1) / (16 * NJ)) * a.split;
    hipLaunchKernelGGL((k_bloch_apply<T, SPINOR, NJ>), dim3(static_cast<unsigned>(hub_slot_grid(a.nchunks, b.tiles))),
                       dim3(64), 0, st, b, u, b.gidx, b.W, static_cast<T*>(u.hpsi));
    return hipGetLastError();
}

template <typename T, int NJ>
hipError_t apply_s(const BlochArgs& a, const ApplyArgs& u, hipStream_t st) {
    return a.spinor ? apply_t<T, true, NJ>(a, u, st) : apply_t<T, false, NJ>(a, u, st);
}

}  // namespace

hipError_t launch_bloch_project(const BlochArgs& a, int prec, hipStream_t st) {
    if (bloch_nj(a.ncol) == 2) return prec == HUB_F64 ? project_t<double, 2>(a, st) : project_t<float, 2>(a, st);
    return prec == HUB_F64 ? project_t<double, 1>(a, st) : project_t<float, 1>(a, st);
}

hipError_t launch_bloch_apply(const BlochArgs& a, const ApplyArgs& u, int prec, hipStream_t st) {
    if (bloch_nj(a.ncol) == 2) return prec == HUB_F64 ? apply_s<double, 2>(a, u, st) : apply_s<float, 2>(a, u, st);
    return prec == HUB_F64 ? apply_s<double, 1>(a, u, st) : apply_s<float, 1>(a, u, st);
}
