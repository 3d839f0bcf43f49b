// Internal declarations of the elastic operator library (device parameter
// block, workspace layout, kernel launchers).  Not part of the public ABI.
//
// Volume layout.  Every wavefield and material array is stored padded:
// row pitch px >= nx + 2 (a multiple of 32 elements), py = ny + 2 rows per
// plane, and nz + 4 planes of which the first and last two are guards.
// Cell (i, j, k) sits at element (k + 2) * px * py + j * px + i.  The
// padding of a wavefield is zero and is never written, so a stencil tap that
// leaves the grid (by at most two cells along one axis) reads zero -- the
// zero extension of the fields -- without a bounds check: a tap at i = -1 or
// -2 lands in the padding columns at the end of the previous row, a tap at
// j = -1, -2 in the padding rows at the end of the previous plane, and taps
// beyond the upper faces in the padding of the same row or plane.  Material
// maps hold, in their +x, +y, +z padding, the value of the nearest cell, so
// the staggered averages at the last index replicate it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <exception>
#include <memory>
#include <new>
#include <utility>
#include <vector>

#include "el.h"

namespace el {

// Wavefield array ids (same order as el_plan_field).
enum Field { U1 = 0, U2, U3, S11, S22, S33, S23, S13, S12, NFIELD };

// Padded volume geometry (elements).
struct Vol {
    int nx, ny, nz;
    int px, py;              // row pitch, rows per plane
    long long plane;         // px * py
    long long total;         // plane * (nz + 4)
    long long origin;        // element of cell (0,0,0): 2 * plane
};
Vol make_vol(int nx, int ny, int nz);

// Record the detail of a failure for el_last_error() and return the status.
el_status set_error(el_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

// Ends an entry point of the ABI that allocates host memory, as a function-try-block: no exception
// crosses the interface.
#define EL_CATCH                                                              \
    catch (const std::bad_alloc &) {                                          \
        return el::set_error(EL_ENOMEM, "host memory ran out");               \
    } catch (const std::exception &e) {                                       \
        return el::set_error(EL_EDEVICE, "unexpected failure: %s", e.what()); \
    }

constexpr int kNoPml = -8;

// A plan's arrays and constants, passed to the kernels by value.  The arrays lie in the plan's
// workspace at equal distances, so a base address and a few strides say where each one is (in
// units of 256 bytes, which fit 32 bits): a stencil kernel loads this struct once, with a few
// wide scalar loads, and forms addresses with scalar arithmetic.  With a pointer per array the
// loops spent their time on scalar loads that each waited for the one before.
template <typename T>
struct Dev {
    char *ws;                // workspace
    unsigned vstr;           // volume arrays (9 fields, 4 maps): stride, the first at offset 0
    unsigned moff[3], mstr[3];   // memory variables of each axis: first of six, stride
    unsigned coff[3], cstr[3];   // C-PML coefficients of each axis: first of four, stride
    unsigned incoff;         // increment blocks
    int nx, ny, nz;
    unsigned sy, sz;         // byte strides of +y and +z (the +x stride is sizeof(T))
    int P;                   // C-PML cells per face, kNoPml = none (then no cell is in or near a layer)
    int high[3], xw;         // boundary-slab storage (below)
    T dt, inv_dx;

    __host__ __device__ T *at(unsigned off256) const { return reinterpret_cast<T *>(ws + ((unsigned long long)off256 << 8)); }
    __host__ __device__ T *f(int id) const { return at((unsigned)id * vstr); }    // wavefields (padded)
    // cell maps (padded, edge-replicated)
    __host__ __device__ T *lam() const { return f(NFIELD); }
    __host__ __device__ T *mu() const { return f(NFIELD + 1); }
    __host__ __device__ T *rho() const { return f(NFIELD + 2); }
    __host__ __device__ T *alpha() const { return f(NFIELD + 3); }
    // boundary-slab memory variables of axis j: mem(j, i) = phi^{ij} (u^i point),
    // mem(j, 3 + i) = psi^{ij} (sigma^{ij} point)
    __host__ __device__ T *mem(int j, int q) const { return at(moff[j] + (unsigned)q * mstr[j]); }
    // C-PML a and b along x (0) and y (1), h = 0 integer / 1 half positions; along z the pairs (a, b)
    __host__ __device__ T *pa(int j, int h) const { return at(coff[j] + 2u * (unsigned)h * cstr[j]); }
    __host__ __device__ T *pb(int j, int h) const { return at(coff[j] + (2u * (unsigned)h + 1u) * cstr[j]); }
    __host__ __device__ T *zab(int h) const { return at(coff[2] + 2u * (unsigned)h * cstr[2]); }
    // adjoint increments Theta^T y of one trace row: for every entry of the block list, 64 elements
    // (lanes) per plane of each of its sub-tiles with scatter points, zero off the points
    __host__ __device__ T *inc() const { return at(incoff); }
    __host__ __device__ int hi(int a) const { return (a == 0 ? nx : (a == 1 ? ny : nz)) - 1 - P; }   // first index of the high slab
    __host__ __device__ int W() const { return P > 0 ? 2 * (P + 7) : 0; }   // slab planes per axis
    __host__ __device__ int px() const { return (int)(sy / sizeof(T)); }    // row pitch (elements)
    __host__ __device__ long long plane() const { return (long long)(sz / sizeof(T)); }
};

// Boundary-slab storage of the C-PML memory variables.  Along each axis the variables live on
// two extended ranges of planes: the low range covers coordinates -2 .. P+4 and the high
// range hi-4 .. n+1 (hi = n-1-P), stored at slab coordinates 0 .. P+6 and P+7 .. 2P+13, so
// W = 2 (P + 7) planes in all.  Cells of the layer (c <= P or c >= hi) own their value; the
// extra planes let a 4-tap difference centred on any cell within two planes of a layer read
// its taps without tests, and hold zeros (the adjoint keeps its memory variables multiplied
// by the layer coefficient a, which vanishes outside the layer).  Where the two ranges would
// overlap (n <= 2P + 9, fewer than ten planes between the layers) one range -2 .. n+1 holds them
// all at slab coordinates c + 2 (n + 4 < W); d.high is the slab coordinate of cell 0 in the
// range that a cell near the high layer uses.
// Is a cell in a layer?  Does its 4-tap stencil along the axis reach one?  The slab coordinate of a
// cell of which either is true.
__host__ __device__ inline bool in_layer(int c, int P, int hi) { return c <= P || c >= hi; }
__host__ __device__ inline bool near_layer(int c, int P, int hi) { return c <= P + 2 || c >= hi - 2; }
__host__ __device__ inline int slab_coord(int c, int P, int high) { return c <= P + 2 ? c + 2 : c + high; }
// Element order: axis x as [side][k][j][s'] with s' the coordinate within the side's
// d.xw = P + 7 planes (a tile's rows of one side are contiguous; the two sides are touched by
// different tiles; a single range is one side of d.xw = W planes), axis y as [k][s][i], axis z
// as [s][j][i].
template <typename T>
__device__ inline unsigned slab_byte(const Dev<T> &d, int axis, int s, int i, int j, int k) {
    unsigned e;
    if (axis == 0) {
        const int side = s >= d.xw ? 1 : 0;
        e = (((unsigned)side * d.nz + k) * d.ny + j) * d.xw + (s - side * d.xw);
    } else {
        e = axis == 1 ? ((unsigned)k * d.W() + s) * d.nx + i : ((unsigned)s * d.ny + j) * d.nx + i;
    }
    return e * (unsigned)sizeof(T);
}
// Column tiles of the stencil passes: kTileX x kTileY cells in x-y, a chunk of zc planes in z.
// A tile is four sub-tiles of kWaveX x kWaveY columns, one wavefront wide: sub-tile s covers
// columns (s & 1) kWaveX .. and rows (s >> 1) kWaveY .. of the tile.
constexpr int kTileX = 64;
constexpr int kTileY = 4;
constexpr int kWaveX = 32;
constexpr int kWaveY = 2;
// An entry of the block list: planes of a tile column and what its block does there.
// A general entry (kBlkGen) updates one sub-tile (kBlkSubShift), a wavefront per velocity
// component or per kind of stress.  A fluid entry updates the fluid sub-tiles set in the four bits
// from kBlkMaskShift, a wavefront each; those also set from kBlkUniShift have uniform lambda, rho and alpha (k_classify), taken
// from a per-tile table instead of the maps.  The general update differences s22 only along y and
// s33 only along z, with taps reaching two cells into a neighbouring tile, so a fluid tile stores
// s22 only on two-row bands along the y faces (bits 0, 1 from kBlkEdgeShift: lower, upper) and
// s33 only on two-plane bands along the z faces (bits 2, 3) it shares with tiles that are not
// fluid; kBlkKeep: the fluid sub-tiles of a tile that is not fluid store both everywhere.
// Of these planes, the sub-tiles set in the four bits from kBlkIncShift hold scatter points: the
// first one's increments (Dev::inc) begin at plane slot, the next one's z1 - z0 planes on.
// kBlkFirst marks the first of the entries that cover the same planes of a tile, kBlkFast the (only)
// entry of fluid ones.
// An entry is one 64-byte line, read with one scalar load: what a block needs before its first
// vector load.
template <typename T>
struct alignas(64) BlockEnt {
    int bx, by, z0, z1;      // tile along x and y, planes
    unsigned flags;          // 0: padding block
    int slot;                // first plane of the tile's increments (kWaveX kWaveY elements each)
    unsigned fluid[kWaveY];  // kBlkGen: fluid columns of the sub-tile's rows
    unsigned uniform[kWaveY];// those of the tile's reference medium (k_classify)
    T lam, rho, alpha;       // a uniform tile's medium, a general tile's reference medium (k_classify)
};
constexpr unsigned kBlkGen = 1u << 0;
constexpr int kBlkSubShift = 1;
constexpr int kBlkMaskShift = 4;
constexpr int kBlkUniShift = 8;
constexpr int kBlkEdgeShift = 12;
constexpr unsigned kBlkKeep = 1u << 16;
constexpr unsigned kBlkFirst = 1u << 17;
constexpr unsigned kBlkFast = 1u << 18;
constexpr int kBlkIncShift = 20;
constexpr int kZBlock = 4, kZDeep = 8;   // planes per block: usually, at most (block_planes)
constexpr long long kFewBlocks = 5120, kManyBlocks = 10240;   // see block_planes
struct Tiles {
    int ntx, nty, nzc, zc;   // tiles along x and y, z chunks, planes per chunk
    int nz, zb;              // planes, planes per block (block_list chooses its own)
    int shortest() const { return zb < 3 ? 2 : zb - 1; }   // planes of a block, unless its run has fewer; s33's bands have two
    static int longest(int zb) { return 3 * zb - 4; }   // planes of a block at most (zb > 2): 2 shortest() + zb - 2
    bool bands() const { return nty >= 8 && nz >= 8 * kZBlock; }            // see piece_xcd
    bool boxes(int nx, int ny) const { return bands() && nty <= 24 && (long long)nx * ny * nz <= 1 << 20; }
    int run() const { return (int)(((long long)ntx * nty * ((nz + kZBlock - 1) / kZBlock) + 511) / 512); }
    int ntiles;              // ntx * nty * nzc
    int cap;                 // entries per XCD at most
    int per;                 // entries per XCD: the grid has 8 * per blocks
    bool once;               // the state outgrows the Infinity Cache (kStreamBytes)
    const void *order;       // device: the block list (BlockEnt<T>); entry b is block b's, on XCD b % 8
};
Tiles make_tiles(int nx, int ny, int nz);
// XCD (0..7) that processes a piece of tile row by from plane z on; blocks run on XCD blockIdx % 8.
int piece_xcd(const Tiles &t, int by, int z, long long index);
// The block list, padded to 8 * per entries: the entries of XCD x at x, x + 8, x + 16, ..., in
// z-major order.  fast: per tile, 1 if it is fluid (null: every tile takes the general update).
// lanes: per tile and row, its fluid columns; then, per tile and row, those of the tile's
// reference medium; med: per tile, lambda, rho, alpha, 0 (k_classify).  points: i, j, k of the
// scatter points.
template <typename T>
struct BlockList {
    std::unique_ptr<BlockEnt<T>[]> entries;
    bool fits = true;        // false: an XCD's entries outgrow their room, and there is no list
    int per = 0;
    bool once = false;       // Tiles::once
    long long planes = 0;    // increment planes of kWaveX x kWaveY elements
    std::vector<int> pos;    // each point's element in them
};
template <typename T>
BlockList<T> block_list(const Tiles &t, int nx, int ny, int npml, const unsigned char *fast, const unsigned char *uni,
                        const unsigned long long *lanes, const T *med, const std::vector<int> &points);
// Faces of fluid tile q shared with tiles that are not fluid: bits 0, 1 along y, 2, 3 along z
// (lower, upper); 0 unless q is a fluid tile.
unsigned tile_edges(const Tiles &t, const unsigned char *fast, int q);

// Relaxation mechanisms of the frequency-dependent absorption (el_relaxation): after every
// velocity pass the tiles holding a velocity point with beta > 0 apply the pointwise
// sub-update R (forward) or R^T (adjoint) to u and the memory variables zeta_l.
template <typename T>
struct Relax {
    int L;                   // mechanisms (0: none)
    T w[EL_MAX_MECH];        // weights
    T c[EL_MAX_MECH];        // exp(-omega_l dt)
    const T *ar;             // strength alpha_r, a padded cell map (edge-replicated like the others)
    const unsigned char *flag;   // per tile: 1 if some velocity point of it has beta > 0 (set-up)
    int *count;              // per tile: its (cell, component) velocity points with beta > 0 (set-up)
    long long *off;          // per tile: index of its first point in pts (set-up)
    // the velocity points with beta > 0, tile by tile, within a tile by component, then plane,
    // row, column: the padded element index with the component in bits 30-31, beta, and the
    // memory variables [l][point]
    unsigned *pts;
    T *beta;
    T *zeta;
    long long npts;
};

constexpr unsigned kRelaxElemMask = (1u << 30) - 1;

// Receiver tables (cell offsets are padded element indices).
struct Rec {
    int nrec;
    const long long *idx;    // [L][8] corner elements
    const double *w;         // [L][8] trilinear weights
    const unsigned char *fl; // [L][8] 1 where the corner lies in a fluid tile: trace is 3 s11
    // grid-point-major transpose for the deterministic scatter
    int npts;
    const long long *pt;     // [npts] touched elements
    const int *ptc;          // [npts][3] their i, j, k
    const int *row;          // [npts + 1] offsets into ent_rec / ent_w
    const int *ent_rec;      // receiver of each entry
    const double *ent_w;     // weight of each entry
    const int *pos;          // [npts] element of each point in the increment blocks (Dev::inc)
};

// Receiver gather: p_hat_m[l] = -sum_c w_lc (s11 + s22 + s33)[c]  (Sec. 3, eq. interpgrid), in
// double.  One wavefront serves 8 receivers; lane = 8 * receiver + corner, reduced over 8
// lanes.  On a fluid tile s22 = s33 = s11 (the lean stress loop stores s11 alone there), and
// the trace is taken as 3 s11, the same double as the sum of the three equal terms.
template <typename T>
__device__ __forceinline__ double trace_at(const Dev<T> &d, const Rec &r, int e) {
    const long long q = r.idx[e];
    const double s11 = (double)d.f(S11)[q];
    return r.fl[e] ? 3.0 * s11 : s11 + (double)d.f(S22)[q] + (double)d.f(S33)[q];
}
// The receivers of gather block gb (256 threads: 4 wavefronts, 32 receivers) into out[].
template <typename T>
__device__ __forceinline__ void gather_block(const Dev<T> &d, const Rec &r, double *out, int gb) {
    const int lane = threadIdx.x & 63;
    const int wave = (gb * 256 + (int)threadIdx.x) >> 6;
    const int l = wave * 8 + (lane >> 3);
    const int c = lane & 7;
    double v = 0.0;
    if (l < r.nrec) v = r.w[8 * l + c] * trace_at(d, r, 8 * l + c);
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    if (l < r.nrec && c == 0) out[l] = -v;
}
inline int gather_blocks(int nrec) { return ((nrec + 7) / 8 + 3) / 4; }

// Theta^T y at point t of the grid-point-major table for the trace row y (entries summed in a
// fixed order): with the adjoint stress kept as w = C s it adds 3 lambda + 2 mu times this value
// to w11, w22 and w33.
template <typename T>
__device__ __forceinline__ T scatter_value(const Rec &r, const double *y, int t) {
    double acc = 0.0;
    for (int e = r.row[t]; e < r.row[t + 1]; ++e) acc += r.ent_w[e] * y[r.ent_rec[e]];
    return T(-acc);
}
// The increments of scatter block sb (256 points) into the plan's increment blocks, where the
// adjoint stress pass that follows picks them up.
template <typename T>
__device__ __forceinline__ void scatter_block(const Dev<T> &d, const Rec &r, const double *y, int sb) {
    const int t = sb * 256 + (int)threadIdx.x;
    if (t < r.npts) d.inc()[r.pos[t]] = scatter_value<T>(r, y, t);
}
inline int scatter_blocks(int npts) { return (npts + 255) / 256; }

// Arguments of a stencil launch over the tiles of G plans of one precision (G = 1: a plan's
// own passes; G = kGroupMax: the grouped passes of el_group).  Member q owns blocks first[q] .. first[q+1]-1; each
// first[q] is a multiple of 8, so that the member's block b - first[q] runs on XCD
// (b - first[q]) % 8 as its tile order assumes.  Entries past the last member repeat the
// total block count (or lie beyond every block).  row[q]: the trace row that member's gather
// blocks write (forward velocity launch) or its scatter blocks read (adjoint velocity launch), or
// null.
constexpr int kGroupMax = 4;
template <typename T, int G>
struct Grp {
    Dev<T> d[G];
    Tiles tl[G];
    Rec r[G];
    double *row[G];
    int first[G + 1];
    int n;
};
template <typename T, int G>
__device__ __forceinline__ int member_of(const Grp<T, G> &g) {
    int q = 0;
    if (G == 1) {
        asm("" : "+s"(q));
        return q;
    }
#pragma unroll
    for (int k = 1; k < G; ++k) q += (int)blockIdx.x >= g.first[k] ? 1 : 0;
    return q;
}

// Workspace layout (byte offsets), computed identically for sizing and binding.
struct Layout {
    size_t vol[NFIELD + 4];  // wavefields, then the maps lam, mu, rho, alpha: equal strides from 0
    size_t mem[3][6];        // equal strides along each axis
    size_t coef[3][4];       // C-PML a, b at integer, then at half positions: equal strides along each axis (z: pairs
                             // (a, b) over both arrays of a position)
    size_t rec_idx, rec_w, csr_pt, csr_ptc, csr_row, csr_rec, csr_w;
    size_t rec_fl[2], csr_pos[2], inc[2];   // without, with the fluid update (as tile_order)
    long long inc_planes;    // room of each inc, in planes of kWaveX x kWaveY elements
    size_t stats;            // media statistics (16 doubles)
    size_t counter;          // device step counter of captured step graphs
    size_t tile_order[2];    // block lists of the stencil passes (8 * cap entries)
    size_t tile_flags;       // per tile: 1 if the fluid update applies; then per tile: 1 if uniform
    size_t tile_media;       // per tile: lambda, rho, alpha, 0 (elements of the plan's precision)
    size_t tile_lanes;       // per tile and row: 64-bit masks of fluid columns, then of uniform ones
    size_t partial;          // reduction partials
    size_t energy;           // modified energy: kinetic part of each wavefront of the velocity blocks,
                             // sums of those, and potential part of each block
    size_t relax_map;        // alpha_r (padded cell map), with relaxation mechanisms only
    size_t relax_flag;       // per tile: relaxation applies
    size_t relax_count;      // per tile: velocity points with beta > 0 (int)
    size_t relax_off;        // per tile: first point of the tile in the point list (long long)
    size_t relax_pts;        // point list: element index and component (unsigned), at most 3 per cell
    size_t relax_beta;       // beta of each point
    size_t relax_zeta;       // memory variables of the relaxation mechanisms (Relax::zeta)
    size_t total;
};

constexpr int kDotBlocks = 1024;
constexpr int kStats = 8;   // media statistics (launch_media_stats)

bool layout(const el_grid &g, int nrec, Layout *L);

// Launchers (return hipError_t of the launch).
template <typename T> hipError_t launch_convert_maps(const Dev<T> &d, const float *lam, const float *mu,
                                                     const float *rho, const float *alpha, hipStream_t s);
hipError_t launch_media_stats(const float *lam, const float *mu, const float *rho, const float *alpha,
                              long long n, double dt, double *stats, double *partial, hipStream_t s);
template <typename T> hipError_t launch_zero_state(const Dev<T> &d, hipStream_t s);
template <typename T> hipError_t launch_classify(const Dev<T> &d, const Tiles &tl, unsigned char *fast,
                                                 unsigned char *uni, T *med, unsigned long long *lanes,
                                                 hipStream_t s);
template <typename T> hipError_t launch_inject(const Dev<T> &d, const T *p0, hipStream_t s);
// The forward velocity launch can also gather a trace row (grow != null) from the stresses it
// reads and does not write: extra blocks after the tiles' run gather_block.
// epart != null: the launch also writes the kinetic part of the modified energy, one double per
// wavefront of every block (4 per block, 8 * per blocks); launch_energy_pot writes the potential
// part, one double per block; launch_energy_final sums the wavefronts' parts in groups into
// kin_block (one double per 64 blocks), then everything into *out.
// ctr != null (captured step graphs): a device step counter.  The velocity launch gathers row
// *ctr of the traces at grow and the stress launch then advances the counter; the adjoint
// velocity launch scatters row *ctr - 1 of the traces at y and the adjoint stress launch then
// steps the counter back.
template <typename T> hipError_t launch_velocity(const Dev<T> &d, const Tiles &tl, hipStream_t s,
                                                 const Rec *r = nullptr, double *grow = nullptr,
                                                 double *epart = nullptr, int *ctr = nullptr);
template <typename T> hipError_t launch_energy_pot(const Dev<T> &d, const Tiles &tl, double *epart, hipStream_t s);
hipError_t launch_energy_final(const double *kin, double *kin_block, const double *pot, int nb, double *out,
                               hipStream_t s);
template <typename T> hipError_t launch_stress(const Dev<T> &d, const Tiles &tl, hipStream_t s, int *ctr = nullptr);
template <typename T> hipError_t launch_gather(const Dev<T> &d, const Rec &r, double *trace_row, hipStream_t s);
// The adjoint velocity launch can also form the increments Theta^T y of a trace row (r and y
// non-null) in extra blocks after the tiles'; the adjoint stress launch adds them to the cells it
// has updated.
template <typename T> hipError_t launch_adj_velocity(const Dev<T> &d, const Tiles &tl, hipStream_t s,
                                                     const Rec *r = nullptr, const double *y = nullptr,
                                                     int *ctr = nullptr);
template <typename T> hipError_t launch_adj_stress(const Dev<T> &d, const Tiles &tl, hipStream_t s, int *ctr = nullptr);
// Theta^T y of the first row, into the zero state.
template <typename T> hipError_t launch_scatter(const Dev<T> &d, const Rec &r, const double *y, hipStream_t s);
template <typename T> hipError_t launch_zero_inc(const Dev<T> &d, long long n, hipStream_t s);
// Grouped passes (el_group): pass 0 velocity (with the gather blocks of members whose row is
// set), 1 stress, 2 adjoint velocity (with the scatter blocks of members whose row is set), 3
// adjoint stress; g.first from the members' 8 * per blocks plus gather or scatter blocks.
template <typename T> hipError_t launch_group_pass(const Grp<T, kGroupMax> &g, int pass, hipStream_t s);
template <typename T> hipError_t launch_extract(const Dev<T> &d, T *p, hipStream_t s);
template <typename T> hipError_t launch_fluid_fill(const Dev<T> &d, const Tiles &tl, hipStream_t s);
hipError_t launch_eir(const double *h, int nh, const double *in, double *out, int M, int L, int transpose,
                      hipStream_t s);
template <typename T> hipError_t launch_dot(const T *a, const T *b, long long n, double *partial, double *out,
                                            hipStream_t s);
hipError_t launch_set_counter(int *ctr, int v, hipStream_t s);
// Relaxation: statistics of the strength map (stats[0] min, [1] non-finite count, [2] max
// over the cells within `margin` of a face), its padded copy, the per-tile flags, the
// memory variables' reset, and the pointwise sub-update (ADJ: its transpose).
hipError_t launch_relax_stats(const float *ar, int nx, int ny, int nz, int margin, double *stats, double *partial,
                              hipStream_t s);
template <typename T> hipError_t launch_relax_setup(const Dev<T> &d, const Tiles &tl, const float *ar_cells,
                                                    const Relax<T> &r, hipStream_t s);
template <typename T> hipError_t launch_relax_compact(const Dev<T> &d, const Tiles &tl, const Relax<T> &r,
                                                      hipStream_t s);
template <typename T> hipError_t launch_relax_zero(const Tiles &tl, const Relax<T> &r, hipStream_t s);
template <typename T> hipError_t launch_relax(const Dev<T> &d, const Tiles &tl, const Relax<T> &r, bool adjoint,
                                              hipStream_t s);

}  // namespace el

// Host state of a plan (the opaque el_plan of the ABI).
struct el_plan_ {
    el_grid g;
    int nrec;
    long long N;
    el::Layout L;
    char *ws;
    int device;
    el::Dev<float> df;
    el::Dev<double> dd;
    el::Relax<float> rf;               // relaxation mechanisms (L = 0: none)
    el::Relax<double> rd;
    long long relax_tiles = 0;         // tiles the relaxation sub-update visits
    long long relax_cells = 0;         // and their cells
    long long relax_points = 0;        // (cell, component) velocity points with beta > 0
    el::Rec rec;
    el::Tiles tiles;
    std::vector<unsigned char> fast;   // per tile: the fluid update applies (host copy)
    std::vector<unsigned char> uni;    // per tile: fluid with uniform lambda, rho, alpha (host copy)
    std::vector<unsigned long long> lanes;   // per tile and row: its fluid columns, then those of its
                                             // reference medium (host copy)
    std::vector<char> med;             // per tile: lambda, rho, alpha, 0 (host copy, of the plan's precision)
    long long column_cells = 0;        // cells of fluid columns in such tiles
    long long uniform_cells = 0;       // cells of uniform fluid tiles
    long long fast_tiles = 0, fast_cells = 0;
    long long fast_layer_cells = 0;    // sum over axes of fluid-tile cells in that axis's C-PML layers
    long long fast_skipped = 0;        // s22 and s33 stores a fluid stress pass leaves out
    std::vector<int> rec_tile;         // [L][8] tile of each receiver corner (host)
    std::vector<int> points;           // i, j, k of the scatter points (host)
    bool once[2] = {};                 // Tiles::once and
    int per[2] = {};                   // Tiles::per of the tables without, with the fluid update (0: not made yet)
    bool fluid_path = true;            // use the fluid update where it applies
    hipEvent_t done;
    double cmax;
    // benchmark instrumentation: per kernel kind, event pairs and how many are in use
    int timing_every = 0;              // bracket the launches of steps m with m % timing_every == 0
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[EL_K_COUNT];
    size_t used[EL_K_COUNT] = {};
};

// The plan's relaxation parameters in the plan's precision.
template <typename T> inline el::Relax<T> &plan_relax(el_plan_ *p);
template <> inline el::Relax<float> &plan_relax<float>(el_plan_ *p) { return p->rf; }
template <> inline el::Relax<double> &plan_relax<double>(el_plan_ *p) { return p->rd; }

// What a plan's passes take under its present fluid-update setting.  An operation that is enqueued
// in parts (el_exec, el_group) keeps the copy it began with: el_plan_fluid_path may change the
// setting in between, and the rest of the operation must still read the stresses (and only those)
// that its earlier passes stored.
template <typename T>
struct Passes {
    el::Dev<T> d;
    el::Tiles tiles;
    el::Rec rec;
    bool fill;               // some tiles are fluid: k_fluid_fill ends the operation
};
template <typename T> inline el::Dev<T> &plan_dev(el_plan_ *p);
template <> inline el::Dev<float> &plan_dev<float>(el_plan_ *p) { return p->df; }
template <> inline el::Dev<double> &plan_dev<double>(el_plan_ *p) { return p->dd; }
template <typename T> inline Passes<T> plan_passes(el_plan_ *p) {
    return Passes<T>{plan_dev<T>(p), p->tiles, p->rec, p->fluid_path && p->fast_tiles > 0};
}
// Both precisions' places for such a copy; one is used.
struct PassesOf {
    Passes<float> f;
    Passes<double> d;
};
template <typename T> inline Passes<T> &passes(PassesOf &o);
template <> inline Passes<float> &passes<float>(PassesOf &o) { return o.f; }
template <> inline Passes<double> &passes<double>(PassesOf &o) { return o.d; }
