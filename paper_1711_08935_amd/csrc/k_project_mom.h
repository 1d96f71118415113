// Projection of complex states on the grouped work list's orbitals and on
// their position moments about the site centres, in one pass over the state
// rows: the projections c and the moments rho_{a,i} of the DFT+U current of
// the velocity gauge (Sec. V).
//
// For a grouped chunk every point carries the same covers (site, image), so
// the displacement of a point from the centre of cover k is its displacement
// d0 from the chunk's first cover plus a constant offset D_k.  The kernel
// sums, per function f and column,
//   acc_0 = sum_e phi_f(e) x(e),   acc_i = sum_e phi_f(e) d0_i(e) x(e)
// (x the state value at the entry's point, rotated by the grid-point phase
// under a field) and writes acc_0 and acc_i + D_k(f),i acc_0, the moment
// about the function's own site, into four planes of the workspace; the
// grouped reduction then applies dV and the Bloch phases to all four.
//
// The entries of a chunk are in grid order, z fastest, so they come in runs
// that share d0's x and y components (7.7 entries on average for the d and p
// shells of a rocksalt cell on a 48^3 grid).  Within a run the kernel sums
// run = sum phi x and the z moment only, 4 FP64 FMAs per function and entry
// instead of 8, and adds run, d0_x run and d0_y run at the run's end: the
// same products, factored, so the rounding errors are no larger.
//
// Work mapping: a 1-D grid of four-wave work-groups over (item, group of four
// column tiles) (hub_slot); a wave takes at most MOM_NFW of the chunk's
// functions, and the waves that share a tile's rows are in one work-group, so
// that a state row comes from HBM once.  An item is (chunk, sub): the
// work-group's tiles are divided into hub_mom_waves(L) subs.  Each lane owns
// one complex column of one state set (64 columns per wave).  The host orders
// the items by their cost (FP64 instructions per wave), longest first, so
// that short items fill the end of the launch.
//
// What bounds it: the reads of the uniform data (orbital values, d0_z and,
// under a field, the phase) through the scalar cache, whose latency the
// contraction of MOM_PF entries hides, beside the state rows from HBM.  Rocksalt
// cell, 48^3, 4 shells, 64 columns x 16 sets, FP32 states: 298 us under a
// field and 274 without, against 345 and 331 for one-wave work-groups of up
// to 8 functions and eight FMAs per function and entry (three waves per SIMD).
// The FP64 issue alone is 145 us, the rows 200.

#pragma once

#include "kcommon.h"

namespace {

// Functions per wave: 5, the shells of a d site; 5 x 5 x 2 FP64 accumulators
// leave four waves per SIMD.  With 8 (two waves) the same sums took longer
// than the former kernel (project stage 455 us), and 5 in one-wave
// work-groups read the rows of an 8-function chunk from HBM twice (389).
constexpr int MOM_NFW = HUB_MOM_NFW;
static_assert(4 * MOM_NFW >= HUB_GF_MAX, "four waves cover a chunk's functions");
constexpr int MOM_WAVES = 4;
// Rows per batch (2: 303 us), and entries whose uniform data is read at once:
// with 1 the scalar cache's latency shows (424 us under a field), and 4 do
// not fit the scalar registers.
constexpr int MOM_U = 4;
constexpr int MOM_PF = 2;
// grid points with the sign bit set start a new run
constexpr uint32_t MOM_POINT = 0x7fffffffu;

template <typename T, int NFW, bool GAUGE>
__device__ __forceinline__ void mom_body(const ProjArgs& a, const HubChunk& C, int ci, int f0, int q, int col,
                                         bool active, const int32_t* __restrict__ gidx,
                                         const double* __restrict__ tab, const double* __restrict__ d0,
                                         const double* __restrict__ fdel, const double* __restrict__ pg,
                                         double* __restrict__ part) {
    constexpr int U = MOM_U;
    const int NF = C.L;
    const int colc = active ? col : 0;
    const T* __restrict__ psi_q = reinterpret_cast<const T*>(a.psi) + static_cast<int64_t>(q) * a.qstride;
    const int32_t* __restrict__ gi = gidx + C.e0;
    const double* __restrict__ tb = tab + C.phi0 + f0;          // entry e: tb[e * NF + f]
    const double* __restrict__ dp = d0 + 3 * static_cast<int64_t>(C.e0);
    const uint32_t rowstride = static_cast<uint32_t>(a.ld * 2);   // elements (checked at launch)

    double acc[4][NFW][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f = 0; f < NFW; ++f) acc[i][f][0] = acc[i][f][1] = 0.0;
    double run[NFW][2];   // the current run's sums of phi x
    double rx = 0.0, ry = 0.0;   // its displacement
#pragma unroll
    for (int f = 0; f < NFW; ++f) run[f][0] = run[f][1] = 0.0;

    // per-entry uniform data: the orbital values of the wave's functions, the
    // z displacement and the grid point's phase
    struct Ent {
        double w[NFW];
        double dz;
        double ph[2];
    };
    // read at 32-bit byte offsets from the chunk's table and displacement
    // rows (a chunk's are far below 4 GiB), advanced entry by entry; the
    // offsets stop at the last entry, so the read after it repeats it
    const uint32_t wstep = static_cast<uint32_t>(NF) * sizeof(double);
    const uint32_t wlast = static_cast<uint32_t>(C.ne - 1) * wstep;
    const uint32_t dlast = static_cast<uint32_t>(C.ne - 1) * (3 * sizeof(double));
    uint32_t wnext = 0, dnext = 0;
    auto read_next = [&](Ent& x, int g) {
        const char* __restrict__ wb = reinterpret_cast<const char*>(tb) + wnext;
        const char* __restrict__ db = reinterpret_cast<const char*>(dp) + dnext;
#pragma unroll
        for (int f = 0; f < NFW; ++f) x.w[f] = *reinterpret_cast<const double*>(wb + f * sizeof(double));
        x.dz = *reinterpret_cast<const double*>(db + 2 * sizeof(double));
        if constexpr (GAUGE) {
            const char* __restrict__ pb = reinterpret_cast<const char*>(pg) +
                                          (static_cast<uint32_t>(g) & MOM_POINT) * static_cast<uint32_t>(2 * sizeof(double));
            x.ph[0] = *reinterpret_cast<const double*>(pb);
            x.ph[1] = *reinterpret_cast<const double*>(pb + sizeof(double));
        }
        wnext = min(wnext + wstep, wlast);
        dnext = min(dnext + static_cast<uint32_t>(3 * sizeof(double)), dlast);
    };
    // grid points of batch b (read one batch before their rows are loaded)
    auto read_idx = [&](int b, int (&g)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) g[u] = gi[b * U + u];
    };
    auto load_batch = [&](const int (&g)[U], T (&r)[U][2]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            load_row_stream<T, 2>(psi_q + static_cast<uint64_t>(static_cast<uint32_t>(g[u]) & MOM_POINT) * rowstride + 2 * colc,
                                  r[u]);
    };
    auto fma_entry = [&](const Ent& x, const T (&r)[2]) {
        double v0 = static_cast<double>(r[0]), v1 = static_cast<double>(r[1]);
        if constexpr (GAUGE) {
            const double t0 = v0 * x.ph[0] - v1 * x.ph[1];
            v1 = v0 * x.ph[1] + v1 * x.ph[0];
            v0 = t0;
        }
        const double z0 = x.dz * v0, z1 = x.dz * v1;
#pragma unroll
        for (int f = 0; f < NFW; ++f) {
            run[f][0] = fma(x.w[f], v0, run[f][0]);
            run[f][1] = fma(x.w[f], v1, run[f][1]);
            acc[3][f][0] = fma(x.w[f], z0, acc[3][f][0]);
            acc[3][f][1] = fma(x.w[f], z1, acc[3][f][1]);
        }
    };
    // end of a run whose entries have the displacement (dx, dy, .)
    auto end_run = [&](double dx, double dy) {
#pragma unroll
        for (int f = 0; f < NFW; ++f)
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                acc[0][f][z] += run[f][z];
                acc[1][f][z] = fma(dx, run[f][z], acc[1][f][z]);
                acc[2][f][z] = fma(dy, run[f][z], acc[2][f][z]);
                run[f][z] = 0.0;
            }
    };
    // Contract a batch (grid points g, those of the next batch gn) MOM_PF entries
    // at a time; the uniform data of the next MOM_PF entries is read while the
    // current ones are contracted (the scheduling barriers keep those reads
    // from being hoisted together).  The entries after the last re-read the
    // last one's table row.
    uint32_t dcur = 0;   // byte offset of the entry's displacement
    auto fma_batch = [&](Ent (&cur)[MOM_PF], const T (&r)[U][2], const int (&g)[U], const int (&gn)[U]) {
#pragma unroll
        for (int u = 0; u < U; u += MOM_PF) {
            Ent nx[MOM_PF];
#pragma unroll
            for (int p = 0; p < MOM_PF; ++p)
                read_next(nx[p], u + MOM_PF + p < U ? g[(u + MOM_PF + p) % U] : gn[(u + MOM_PF + p) % U]);
#pragma unroll
            for (int p = 0; p < MOM_PF; ++p) {
                if (g[u + p] < 0) {
                    end_run(rx, ry);
                    rx = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(dp) + dcur);
                    ry = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(dp) + dcur + sizeof(double));
                }
                dcur += 3 * sizeof(double);
                fma_entry(cur[p], r[u + p]);
                // the sums are done here, not after the next run's end (whose
                // branch the orbital values would otherwise outlive)
#pragma unroll
                for (int f = 0; f < NFW; ++f) {
                    asm volatile("" : "+v"(run[f][0]), "+v"(run[f][1]));
                    asm volatile("" : "+v"(acc[3][f][0]), "+v"(acc[3][f][1]));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < MOM_PF; ++p) cur[p] = nx[p];
        }
    };
    // Two row buffers; the grid points of a batch are read one batch ahead
    // of its row loads, and the batches past the last re-read the last one.
    const int nbt = C.ne / U;
    if (nbt > 0) {
        T ra[U][2], rb[U][2];
        int ga[U], gb[U], gc[U];
        Ent cur[MOM_PF];
        read_idx(0, ga);
#pragma unroll
        for (int p = 0; p < MOM_PF; ++p) read_next(cur[p], ga[p]);
        rx = dp[0];
        ry = dp[1];
        load_batch(ga, ra);
        read_idx(nbt > 1 ? 1 : 0, gb);
        int b = 0;
        for (; b + 2 <= nbt; b += 2) {
            load_batch(gb, rb);
            read_idx(b + 2 < nbt ? b + 2 : nbt - 1, gc);
            __builtin_amdgcn_sched_barrier(0);
            fma_batch(cur, ra, ga, gb);
#pragma unroll
            for (int u = 0; u < U; ++u) ga[u] = gc[u];
            load_batch(ga, ra);
            read_idx(b + 3 < nbt ? b + 3 : nbt - 1, gc);
            __builtin_amdgcn_sched_barrier(0);
            fma_batch(cur, rb, gb, ga);
#pragma unroll
            for (int u = 0; u < U; ++u) gb[u] = gc[u];
        }
        if (b < nbt) fma_batch(cur, ra, ga, gb);
        end_run(rx, ry);
    }
    if (!active) return;
    const double* __restrict__ del = fdel + (static_cast<int64_t>(ci) * HUB_GF_MAX + f0) * 3;
#pragma unroll
    for (int f = 0; f < NFW; ++f) {
        const int64_t o = ((static_cast<int64_t>(q) * a.prows + C.part0 + f0 + f) * a.ncol + col) * 2;
        part[o] = acc[0][f][0];
        part[o + 1] = acc[0][f][1];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double D = del[3 * f + i];
            part[(i + 1) * a.pplane + o] = fma(D, acc[0][f][0], acc[i + 1][f][0]);
            part[(i + 1) * a.pplane + o + 1] = fma(D, acc[0][f][1], acc[i + 1][f][1]);
        }
    }
}

template <typename T, bool GAUGE>
__global__ void __launch_bounds__(MOM_WAVES * HUB_WAVE)
k_project_mom(const ProjArgs a, const int32_t* __restrict__ gidx, const double* __restrict__ tab,
              const double* __restrict__ d0, const double* __restrict__ fdel, const double* __restrict__ pg,
              double* __restrict__ part) {
    const HubSlot slot = hub_slot(a.tiles);
    if (slot.chunk >= a.nchunks) return;
    const int item = a.chunk_list[slot.chunk];
    const int ci = item >> 2, sub = item & 3;
    const HubChunk C = a.chunks[ci];
    const int lane = threadIdx.x & (HUB_WAVE - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / HUB_WAVE);
    const int wide = hub_mom_waves(C.L);                    // waves that share a tile
    const int h = w & (wide - 1);
    const int tile = MOM_WAVES * slot.tile + sub * (MOM_WAVES / wide) + w / wide;
    const int tps = (a.ncol + HUB_WAVE - 1) / HUB_WAVE;     // column tiles per state set
    if (h >= hub_mom_parts(C.L) || tile >= a.nq * tps) return;
    const int f0 = hub_mom_first(C.L, h);
    const int nfw = hub_mom_first(C.L, h + 1) - f0;
    const int q = tile / tps;
    const int col = (tile - q * tps) * HUB_WAVE + lane;
    const bool active = col < a.ncol;
#define HUB_MCASE(n) \
    case n: mom_body<T, n, GAUGE>(a, C, ci, f0, q, col, active, gidx, tab, d0, fdel, pg, part); break;
    static_assert(MOM_NFW == 5, "the cases below cover 1..5 functions");
    switch (nfw) {
        HUB_MCASE(1) HUB_MCASE(2) HUB_MCASE(3) HUB_MCASE(4) HUB_MCASE(5)
    default: break;
    }
#undef HUB_MCASE
}

// Launch over nitems work items of grouped chunks (every pass, functions
// <= 16 per chunk) of complex states of storage type T.
template <typename T>
hipError_t launch_project_mom_prec(const ProjArgs& a, int nitems, int nq, hipStream_t st) {
    if (nitems <= 0 || nq <= 0 || a.ncol <= 0) return hipSuccess;
    if (a.ncplx != 2 || !a.d0 || !a.fdel || !a.mgidx || a.ld < 0 || a.ld * 2 > static_cast<int64_t>(UINT32_MAX))
        return hipErrorInvalidValue;
    ProjArgs b = a;
    b.nchunks = nitems;
    b.nq = nq;
    b.tiles = static_cast<int>((static_cast<int64_t>(nq) * ((a.ncol + HUB_WAVE - 1) / HUB_WAVE) + MOM_WAVES - 1) /
                               MOM_WAVES);
    const dim3 grid(static_cast<unsigned>(hub_slot_grid(nitems, b.tiles)));
    if (a.pg)
        hipLaunchKernelGGL((k_project_mom<T, true>), grid, dim3(MOM_WAVES * HUB_WAVE), 0, st, b, b.mgidx, b.tab,
                           b.d0, b.fdel, b.pg, b.part);
    else
        hipLaunchKernelGGL((k_project_mom<T, false>), grid, dim3(MOM_WAVES * HUB_WAVE), 0, st, b, b.mgidx, b.tab,
                           b.d0, b.fdel, b.pg, b.part);
    return hipGetLastError();
}

}  // namespace
