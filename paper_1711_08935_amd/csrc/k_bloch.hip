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
// (0.099), apply 0.43 (1.39).  It wins from two passes on: 31 functions in
// FP64, 16 sets of 45 columns 0.37 and 0.52 ms (0.56 and 0.95).

#include "k_apply.h"
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

// B[q][j][col] = alpha scale sum_b V_ab c_b of every orbital j, a lane per
// column (a.phase: ones).
template <bool SPINOR>
__global__ void __launch_bounds__(64) k_bloch_coef(const ApplyArgs a, const int32_t* __restrict__ orb_site,
                                                   double* __restrict__ B) {
    const int col = blockIdx.x * 64 + threadIdx.x, j = blockIdx.y, q = blockIdx.z;
    if (col >= a.ncol) return;
    const int site = orb_site[j], o0 = a.site_orb0[site];
    const HubFun F{site, o0, a.site_L[site], j - o0, 0, -1, {0, 0}};
    double b[2];
    coefficient<true, SPINOR, 1>(a, F, q, col, b);
    double* o = B + ((static_cast<int64_t>(q) * a.J + j) * a.ncol + col) * 2;
    o[0] = b[0];
    o[1] = b[1];
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

// The same tile in the apply: A[l % 16][.] = W of point l % 16 of a 16-point
// block, the functions' parts split over the lane groups in the order of the
// table row (lane group l / 16 takes RL / 4 consecutive values), B = the
// coefficients in that order, the sum starts at hpsi.
template <typename T, int MT, int NJ>
__device__ __forceinline__ void apply_tile(const BlochArgs& a, const HubChunk& C, const int32_t* __restrict__ orb,
                                           int q, int c0, int part_of, const int32_t* __restrict__ gidx,
                                           const double* __restrict__ W, const double* __restrict__ Bc,
                                           T* __restrict__ hpsi) {
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
    // conj(W) B = (Wr Br + Wi Bi) + i (Wr Bi - Wi Br)
    double bf[KB][NJ][2];
    const bool imag = g4 >> 1;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int f = KB * (g4 & 1) + kb;
        const int o = f < C.L ? orb[f] : -1;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const hub_d2 z = *reinterpret_cast<const hub_d2*>(
                Bc + (static_cast<int64_t>(q) * a.J + (o < 0 ? 0 : o)) * a.ncol * 2 + cofs[j]);
            const bool use = o >= 0 && ok[j];
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
    int first, nb;
    block_range(C.ne, a.split, part_of, first, nb);
    if (first >= nb) return;
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

template <typename T, int NJ>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_bloch_apply(const BlochArgs a, const int32_t* __restrict__ gidx, const double* __restrict__ W,
              const double* __restrict__ Bc, T* __restrict__ hpsi) {
    const HubSlot slot = hub_slot(a.tiles);
    if (slot.chunk >= a.nchunks) return;
    const int ci = a.chunk0 + slot.chunk;
    const HubChunk C = a.chunks[ci];
    const int tps = (a.ncol + 16 * NJ - 1) / (16 * NJ);
    const int tile = slot.tile / a.split, part_of = slot.tile - tile * a.split;
    const int q = tile / tps, c0 = (tile - q * tps) * (16 * NJ);
    const int k = a.spinor ? a.q0 + q : (a.q0 + q) / a.nspin;
    const double* __restrict__ Wk = W + k * a.wlen;
    const int32_t* __restrict__ orb = a.f_orb + ci * HUB_GF_MAX;
    if (C.L > 8) apply_tile<T, 2, NJ>(a, C, orb, q, c0, part_of, gidx, Wk, Bc, hpsi);
    else apply_tile<T, 1, NJ>(a, C, orb, q, c0, part_of, gidx, Wk, Bc, hpsi);
}

}  // namespace

hipError_t launch_bloch_table(const BlochTableArgs& a, int nchunks, int nk, hipStream_t st) {
    hipLaunchKernelGGL(k_bloch_table, dim3(nchunks, nk), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_bloch_coef(const ApplyArgs& a, int nq, const int32_t* orb_site, double* B, hipStream_t st) {
    const dim3 grid((a.ncol + 63) / 64, a.J, nq);
    if (a.spinor) hipLaunchKernelGGL(k_bloch_coef<true>, grid, dim3(64), 0, st, a, orb_site, B);
    else hipLaunchKernelGGL(k_bloch_coef<false>, grid, dim3(64), 0, st, a, orb_site, B);
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

template <typename T, int NJ>
hipError_t apply_t(const BlochArgs& a, const double* B, void* hpsi, hipStream_t st) {
    BlochArgs b = a;
    b.tiles = a.nq * ((a.ncol + 16 * NJ - 1) / (16 * NJ)) * a.split;
    hipLaunchKernelGGL((k_bloch_apply<T, NJ>), dim3(static_cast<unsigned>(hub_slot_grid(a.nchunks, b.tiles))), dim3(64), 0,
                       st, b, b.gidx, b.W, B, static_cast<T*>(hpsi));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bloch_project(const BlochArgs& a, int prec, hipStream_t st) {
    if (bloch_nj(a.ncol) == 2) return prec == HUB_F64 ? project_t<double, 2>(a, st) : project_t<float, 2>(a, st);
    return prec == HUB_F64 ? project_t<double, 1>(a, st) : project_t<float, 1>(a, st);
}

hipError_t launch_bloch_apply(const BlochArgs& a, int prec, const double* B, void* hpsi, hipStream_t st) {
    if (bloch_nj(a.ncol) == 2) return prec == HUB_F64 ? apply_t<double, 2>(a, B, hpsi, st) : apply_t<float, 2>(a, B, hpsi, st);
    return prec == HUB_F64 ? apply_t<double, 1>(a, B, hpsi, st) : apply_t<float, 1>(a, B, hpsi, st);
}
