// Internal declarations shared by the host builder, the C-ABI layer and the
// HIP kernels of the Hubbard library.  Not part of the public ABI.
#pragma once

#include <cstdint>
#include <vector>

#include "hub.h"

// One work-list chunk: a run of sphere entries of one site inside one apply
// layer, all with the same lattice image (so one Bloch phase serves the whole
// chunk).  Within a layer no two entries share a grid point, so chunks of the
// same layer can be applied concurrently without atomics.
struct HubChunk {
    int32_t site;
    int32_t layer;
    int32_t e0;      // first entry
    int32_t ne;      // entries, padded to a multiple of HUB_ENTRY_ALIGN
    int32_t L;       // orbitals of the site (2l+1)
    int32_t orb0;    // global index j of the site's first orbital
    int32_t part0;   // first row of this chunk in the projection workspace
    int32_t species;
    int64_t phi0;    // offset of the chunk's orbital values (entries * L)
    int32_t img;     // lattice image shared by every entry of the chunk
    int32_t nreal;   // real entries; entries nreal..ne-1 repeat the last grid
                     // point with zero orbital values
};

// Chunk entry lists are padded to a multiple of this many entries, so that
// every wave's share (1, 2 or 4 waves per work-group) holds whole batches of
// the kernels' entry loops (at most 8 entries).
#define HUB_ENTRY_ALIGN 32

struct SiteDef {
    double R[3];
    int l;
    double zeta;
    double rc;
    int species;
    double ueff_fixed;   // NaN: ACBN0
    double zeta_dn;      // spin-down exponent of spinor orbitals; NaN: zeta
};

struct alignas(8) HubInt2 {
    int32_t x, y;
};

// Host copy of one site's sphere, points sorted by (g, image).
struct SiteSphere {
    int32_t lo[3] = {}, n[3] = {};           // lowest unfolded coordinates and extents of the points
    std::vector<HubInt2> lines;              // [n[0]][n[1]] (points, lowest z - lo[2]) along z; no gaps
    std::vector<int32_t> g;      // folded grid index
    std::vector<int32_t> img3;   // lattice image (3 per point)
    std::vector<int32_t> ijk;    // unfolded integer coordinates (3 per point)
    std::vector<double> phi;     // [p][m]
    std::vector<double> grad;    // [p][m][3]
    std::vector<double> phi_dn;  // [p][m], spin-down orbitals (spin-dependent contexts)
    std::vector<double> grad_dn; // [p][m][3], their gradients
};

// One function of a grouped chunk as the apply reads it: orbital m (first
// orbital o0, L orbitals) of a site, seen through a lattice image; spin: the
// component whose orbital it is (spin-dependent orbitals), else -1.
struct alignas(32) HubFun {
    int32_t site, o0, L, m, img, spin, pad[2];
};

// Largest number of functions (orbitals of all covering sites) a grouped
// chunk may carry; the covers of a point with more are split over passes
// of at most this many functions each.
#define HUB_GF_MAX 16

// Work list grouped by cover signature: every grid point covered by any
// sphere appears in one grouped chunk per pass, together with its
// (site, image) covers in a fixed slot order, so the projection reads each
// state row once per pass and the apply writes it once per pass.  The
// chunk's functions are the concatenated orbitals of its slots; a point with
// more than HUB_GF_MAX functions has its slots split over several passes.
struct GroupTables {
    bool ok = false;
    int nfmax = 0;                           // most functions covering one grid point
    int npass = 1;                           // apply passes (chunk.layer): points with more
                                             // than HUB_GF_MAX functions are split over passes
    std::vector<HubChunk> chunks;            // L = number of functions, e0/ne over points
    std::vector<int32_t> gidx;               // per point
    std::vector<double> tab;                 // per point, L values (slot-major)
    // position moments (velocity-gauge current): per point (in gidx order)
    // the displacement of its unfolded position from the centre of the site
    // of its chunk's first cover, d0[point][3]; per chunk and function the
    // offset from that displacement to the one about the function's own
    // site, fdel[chunk][HUB_GF_MAX][3] (constant over a chunk's points)
    std::vector<double> d0;
    std::vector<double> fdel;
    // gidx, with the sign bit set on points that start a new run: d0's x or y
    // component differs from the point before in the chunk
    std::vector<int32_t> run_gidx;
    std::vector<int32_t> f_orb;              // per chunk HUB_GF_MAX: global orbital j of function f
    std::vector<int32_t> f_img;              // per chunk HUB_GF_MAX: lattice image of function f
    std::vector<int32_t> red_ptr;            // CSR orbital j -> workspace rows
    std::vector<int32_t> red_row, red_img;
    int64_t part_rows = 0;
};

struct HostTables {
    int nsites = 0, J = 0, nlayers = 0, nspecies = 0;
    std::vector<int32_t> site_L, site_orb0, site_species;
    std::vector<HubChunk> chunks;            // sorted by (layer, site)
    std::vector<int32_t> gidx, img;          // per entry
    std::vector<double> phi;                 // per entry, L values
    std::vector<double> gphi;                // per entry, 3L values [m][i]
    std::vector<double> mphi;                // per entry, 3L values [m][i]: (r_p - R)_i phi_m
    // Spin-dependent orbitals (some site has a spin-down exponent): per
    // entry 2L values [sigma][m], the orbital of each spin component (sites
    // without one repeat their orbital); the grouped list then carries 2L
    // functions per cover as well.
    bool spindep = false;
    std::vector<double> phi2;
    std::vector<double> gphi_dn, mphi_dn;    // per entry, 3L values [m][i] of the spin-down orbitals
    std::vector<int32_t> images;             // unique lattice images, 3 per image
    std::vector<int32_t> site_chunk_ptr;     // CSR site -> chunk ids
    std::vector<int32_t> site_chunk_ids;
    std::vector<int32_t> layer_chunk_ptr;    // chunks of layer l: [ptr[l], ptr[l+1])
    std::vector<int32_t> layer_site_ptr;     // chunk range of (layer, site): [l*nsites+s]
    std::vector<int32_t> species_orb_ptr;    // CSR species -> orbital j
    std::vector<int32_t> species_orb_ids;
    std::vector<int32_t> orb_site;           // j -> site
    int64_t part_rows = 0;                   // sum of L over chunks
    int64_t nentries = 0;
    std::vector<SiteSphere> spheres;
    GroupTables grouped;
};

// Work list of the state-gradient force form (Sec. IV): <phi|D_i psi>, D_i
// the 4th-order central difference along axis i, equals by summation by
// parts -dV sum over the dilated sphere (every unfolded point within two
// steps of a sphere point along an axis) of exp(i k.T) (D_i phi)(p)
// psi(g(p)), with phi zero outside the sphere.  The table holds D_i phi, so
// the projection machinery of the orbital gradients computes
// d = dV sum exp(i k.T) (D phi) psi = -<phi|D psi> and the force contraction
// is shared.  Chunks are per (site, image) as in one layer of the layered
// list; the projection needs no layers.
struct StencilTables {
    std::vector<HubChunk> chunks;            // site-major, then image, g ascending
    std::vector<int32_t> gidx;               // per entry
    std::vector<double> tab;                 // per entry, 3L values [m][i]
    std::vector<double> tab_dn;              // the same for the spin-down orbitals (spin-dependent contexts)
    std::vector<int32_t> site_chunk_ptr;     // CSR site -> chunk ids
    std::vector<int32_t> site_chunk_ids;
    int64_t part_rows = 0;                   // sum of L over chunks
    int64_t nentries = 0;                    // real (unpadded) entries
};

// Host builder (sphere.cpp).  Returns HUB_OK or a negative status.
int hub_build_host(const double cell[3], const int ngrid[3], const std::vector<SiteDef>& sites,
                   int chunk_entries, HostTables& out);

// Work list of the Coulomb tensors (k_coulomb.hip): each site's sphere points
// sorted into planes of constant x, in a plane by (y, z), every plane padded
// to a multiple of 16 slots.  Slots count from the site's first one.
struct CoulombSite {
    int32_t index;           // site of the context
    int32_t L, npad;         // orbitals; pair densities L (L + 1) / 2 padded to 16 or 32
    int32_t n[3], lo[3];     // extents and lowest unfolded coordinates of its points
    int32_t chunk0, chunk1;  // its chunks in site_chunk_ids
    int32_t line0;           // lines[line0 + x * n[1] + y] = (first slot, lowest z)
    int32_t plane0;          // planes[plane0 + x] = (first slot, points)
    int32_t nitems;
    int64_t slot0;           // first slot in the launch's point arrays
    int64_t rho0, part0;     // first double of its densities and of its items' sums
};
// Targets: nblk blocks of 16 slots of plane x from slot on; sources: slots
// [s0, s1) of the planes x0..x1 <= x.
struct CoulombItem {
    int32_t site;            // position in the plan's sites
    int32_t x, slot, nblk, x0, x1, s0, s1;
    int32_t part;            // position among the site's items
};
struct CoulombPlan {
    std::vector<CoulombSite> sites;
    std::vector<CoulombItem> items;          // site by site
    std::vector<HubInt2> lines, planes;
    std::vector<int32_t> item_ptr;           // items of sites[i]: [item_ptr[i], item_ptr[i + 1])
    int64_t slots = 0, rho = 0, part = 0;    // points, densities and partial sums (doubles)
};
// Least 16 x 16 x 4 products per wave that a work item is split to.
#define HUB_COUL_MINCOST 512
#define HUB_COUL_MAXBLK 16                   // target blocks per work item, four per wave
// LDS for a plane of the kernel (|dy| x |dz| doubles); larger planes are read
// from a table in device memory.
#define HUB_COUL_LDS 65536

// Work list of Bloch-summed orbitals (complex states whose points carry more
// than HUB_GF_MAX (orbital, image) functions, where the grouped list needs
// several passes): for one k-point the images of a site's orbital at a grid
// point enter only through W_j(g) = sum_T exp(i k.T) phi_j(r_g + T), so a
// point carries one complex function per orbital of its covering sites.
// Chunks hold points of one set of covering sites, split over passes of at
// most HUB_GF_MAX functions as in the grouped list.
struct BlochTables {
    std::vector<HubChunk> chunks;            // L functions, layer = pass, phi0: first double of the chunk
                                             // in one k-point's table (rows of hub_bloch_row(L) doubles)
    std::vector<int32_t> gidx;               // per entry
    std::vector<int32_t> f_orb;              // per chunk HUB_GF_MAX: orbital j of function f, or -1
    std::vector<int32_t> red_ptr, red_row;   // CSR orbital j -> workspace rows
    std::vector<int32_t> pass_ptr;           // chunks of pass p: [pass_ptr[p], pass_ptr[p + 1])
    int64_t part_rows = 0, wlen = 0;         // workspace rows; doubles of one k-point's table
    // covers of each entry (CSR), from which the device builds the tables
    std::vector<int32_t> cptr, cimg, cfun;   // cfun: first function | L << 8
    std::vector<int64_t> coff;               // first value in cval
    std::vector<double> cval;
};
// doubles per entry: the real, then the imaginary parts of 8 or 16 functions
inline int hub_bloch_row(int nf) { return nf > 8 ? 32 : 16; }
// False, and out empty, where the tables of nk k-points would take more than
// wlimit bytes or an index would pass 32 bits; counted before the tables of the
// entries are filled.
bool hub_build_bloch(const HostTables& T, int64_t G, int chunk_entries, BlochTables& out, int nk = 1,
                     int64_t wlimit = INT64_MAX);

// Plan for the sites which[0..] of the context (sphere.cpp).
void hub_coulomb_plan(const HostTables& T, const std::vector<int>& which, CoulombPlan& out);

// Closed-form average of 1/|r| over one grid cell centred at the origin.
double hub_g0_cell_average(const double h[3]);

// Dilated-sphere tables of the state-gradient force form from the spheres of
// ``T`` (sphere.cpp).  Every image it needs is in T.images (hub_build_host
// registers the images of the points two steps past each sphere point).
int hub_build_stencil(const double cell[3], const int ngrid[3], const std::vector<SiteDef>& sites,
                      const HostTables& T, int chunk_entries, StencilTables& out);
