// Launch arguments of the kernels over Bloch-summed orbitals (k_bloch.hip).
#pragma once

#include "kcommon.h"

struct BlochTableArgs {
    const HubChunk* chunks;
    const int32_t *cptr, *cimg, *cfun;       // covers per entry (BlochTables)
    const int64_t* coff;
    const double* cval;
    const double* phase;                     // [nk][nimg] (re, im) of exp(i k.T)
    int nimg;
    int64_t wlen;
    double* W;                               // [nk][wlen]
};

struct BlochArgs {
    const void* psi;                         // projection: states
    int64_t ld, qstride;                     // as in ProjArgs
    int ncol, nq, q0, nspin, spinor, J;
    const HubChunk* chunks;
    int chunk0, nchunks;                     // the launch's chunks
    int tiles;                               // (set, columns) tiles times split (set by the launcher)
    int split;                               // work-groups that share a chunk's entries in one tile
    const int32_t* gidx;
    const HubFun* fun;                       // [chunk][HUB_GF_MAX] functions (image unused)
    const double* W;
    int64_t wlen;
    double* part;                            // projection: [nq][prows][ncol] complex, row r split + s
    int64_t prows;
};

// 16-column blocks per wave (1 or 2) for ncol columns.
int bloch_nj(int ncol);
hipError_t launch_bloch_table(const BlochTableArgs& a, int nchunks, int nk, hipStream_t st);
hipError_t launch_bloch_project(const BlochArgs& a, int prec, hipStream_t st);
// u: the states, projections, occupations and scales of the apply (the chunk
// fields, phases and sink are not used).
hipError_t launch_bloch_apply(const BlochArgs& a, const ApplyArgs& u, int prec, hipStream_t st);
