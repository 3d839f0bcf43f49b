// Host side of the C ABI declared in include/el.h: validation, workspace
// layout, C-PML profiles, receiver tables and the time loops of H and H^T.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <vector>

#include "el_impl.h"

using namespace el;

namespace {

thread_local char g_err[512];

#define fail el::set_error

el_status hip_fail(hipError_t e, const char *what) {
    return fail(EL_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr, what)                        \
    do {                                           \
        hipError_t e_ = (expr);                    \
        if (e_ != hipSuccess) return hip_fail(e_, what); \
    } while (0)

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// 4th-order staggered 3-D stability bound: c dt/dx <= 1 / (sqrt(3) (9/8 + 1/24)).
const double kCflMax = 6.0 / (7.0 * std::sqrt(3.0));

// Receivers may sit up to this many cells outside [0, n-1] (rounding of x/dx); they are clamped onto the box.
const double kRecSlack = 1e-9;

}  // namespace

namespace el {

el_status set_error(el_status st, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

Vol make_vol(int nx, int ny, int nz) {
    Vol v;
    v.nx = nx;
    v.ny = ny;
    v.nz = nz;
    v.px = (nx + 2 + 31) / 32 * 32;
    v.py = ny + 2;
    v.plane = (long long)v.px * v.py;
    v.total = v.plane * (nz + 4);
    v.origin = 2 * v.plane;
    return v;
}

bool layout(const el_grid &g, int nrec, Layout *L) {
    const size_t es = g.precision == EL_F64 ? 8 : 4;
    const size_t N = (size_t)make_vol(g.nx, g.ny, g.nz).total;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align256(bytes);
        return o;
    };
    for (int f = 0; f < NFIELD + 4; ++f) L->vol[f] = take(N * es);
    const int P = g.npml;
    const size_t W = P > 0 ? 2 * (size_t)(P + 7) : 0;
    const size_t ns[3] = {W * g.ny * g.nz, (size_t)g.nx * W * g.nz, (size_t)g.nx * g.ny * W};
    const int n[3] = {g.nx, g.ny, g.nz};
    for (int a = 0; a < 3; ++a)
        for (int q = 0; q < 6; ++q) L->mem[a][q] = P > 0 ? take(ns[a] * es) : 0;
    for (int a = 0; a < 3; ++a)
        for (int q = 0; q < 4; ++q) L->coef[a][q] = take(n[a] * es);
    const size_t E = 8 * (size_t)std::max(nrec, 1);
    L->rec_idx = take(E * 8);
    L->rec_w = take(E * 8);
    for (size_t &o : L->rec_fl) o = take(E);
    L->csr_pt = take(E * 8);
    L->csr_ptc = take(E * 3 * 4);
    L->csr_row = take((E + 1) * 4);
    L->csr_rec = take(E * 4);
    L->csr_w = take(E * 8);
    L->stats = take(16 * 8);
    L->counter = take(256);
    {
        const Tiles t = make_tiles(g.nx, g.ny, g.nz);
        // increments: the planes of a sub-tile's piece with points (as deep as block_planes may make it
        // here), at most every plane there is
        const size_t every = (size_t)4 * t.ntx * t.nty * g.nz;
        const size_t planes = std::min(E * Tiles::longest(every >= kManyBlocks * kZDeep ? kZDeep : kZBlock), every);
        L->inc_planes = (long long)planes;
        for (size_t &o : L->csr_pos) o = take(E * 4);
        for (size_t &o : L->inc) o = take(planes * kWaveX * kWaveY * es);
        for (size_t &o : L->tile_order) o = take((size_t)8 * t.cap * sizeof(BlockEnt<double>));
        L->tile_flags = take(2 * (size_t)t.ntiles);
        L->tile_media = take((size_t)4 * t.ntiles * es);
        L->tile_lanes = take((size_t)2 * kTileY * t.ntiles * 8);
        L->energy = take(((size_t)(4 + 1) * 8 * t.cap + (size_t)8 * t.cap / 64 + 1) * sizeof(double));
        const int nm = g.relax.nmech;
        L->relax_map = nm > 0 ? take(N * es) : 0;
        L->relax_flag = nm > 0 ? take((size_t)t.ntiles) : 0;
        L->relax_count = nm > 0 ? take((size_t)t.ntiles * sizeof(int)) : 0;
        const size_t cap = (size_t)t.ntiles * 3 * t.zc * kTileX * kTileY;   // points at most
        L->relax_off = nm > 0 ? take((size_t)t.ntiles * sizeof(long long)) : 0;
        L->relax_pts = nm > 0 ? take(cap * sizeof(unsigned)) : 0;
        L->relax_beta = nm > 0 ? take(cap * es) : 0;
        L->relax_zeta = nm > 0 ? take(cap * nm * es) : 0;
    }
    L->partial = take(kStats * kDotBlocks * 8);
    L->total = off;
    return true;
}

// Tiles of kTileX x kTileY columns by chunks of chunk_planes() planes: kZChunk where that makes
// kMinTiles tiles, else fewer, down to two.  The chunk decides which cells next to a solid run the
// general update, whose sums round differently from the fluid update's.  How many planes a block
// updates is another matter (block_planes): the blocks of block_list() cover any run of planes
// over which a tile column's chunks ask for the same update.
constexpr int kZChunk = 6;
constexpr long long kMinTiles = 4096;
constexpr int kMaxTiles = (1 << 24) - 1;   // (arrays below 4 GiB keep under it)
// The Infinity Cache: a state of less is still there when the next pass reads it (ld_own).  By the
// bytes that a step touches the hint loses 17 to 24% at 126 to 188 MiB (shells of 160^3 and, in double
// precision, 144^3), 7% at 228 (solid 152^3), and gains 5% at 248 (shell of 208^3) and 4% at 263 (solid
// 160^3).
constexpr long long kStreamBytes = 256ll << 20;
int chunk_planes(int nx, int ny, int nz) {
    const long long cols = (long long)((nx + kTileX - 1) / kTileX) * ((ny + kTileY - 1) / kTileY);
    int zc = kZChunk;
    while (zc > 2 && cols * ((nz + zc - 1) / zc) < kMinTiles) --zc;
    return std::min(zc, nz);
}
Tiles make_tiles(int nx, int ny, int nz) {
    Tiles t;
    t.ntx = (nx + kTileX - 1) / kTileX;
    t.nty = (ny + kTileY - 1) / kTileY;
    t.zc = chunk_planes(nx, ny, nz);
    t.zb = kZBlock;
    t.nz = nz;
    t.nzc = (nz + t.zc - 1) / t.zc;
    t.ntiles = t.ntx * t.nty * t.nzc;
    t.order = nullptr;
    t.per = t.cap = 0;
    t.once = false;
    // an XCD's entries at most: four per piece.  The pieces of a tile column are at least two planes
    // apart but for a last one; with blocks of kZBlock at least and runs of kZChunk planes (every
    // plane of a tile column is in an entry, so block_planes counts cols nz planes or more) a run of
    // D planes has at most (D + 1) / 3, seven in 18 planes
    const bool deep = t.zc == kZChunk && (long long)t.ntx * t.nty * nz >= kFewBlocks * kZBlock;
    long long cnt[8] = {}, all = 0;
    for (int z0 = 0, z1 = 0; z0 < nz; z0 = z1) {
        for (z1 = z0 + 1; z1 < nz && z1 * 8 / nz == z0 * 8 / nz; ++z1) {}
        const int n = 4 * t.ntx * (deep ? 7 * (z1 - z0) / 18 + 2 : (z1 - z0 + 1) / 2 + 1);
        for (int by = 0; by < t.nty; ++by) cnt[piece_xcd(t, by, z0, 0)] += n;
        all += (long long)n * t.nty;
    }
    t.cap = (int)*std::max_element(cnt, cnt + 8);
    if (!t.bands()) t.cap = (int)((all + 7) / 8 + 4 * t.run());
    // a box of equal cost held at most the entries of a band's bound in 800 lists of random media; where
    // the media ask for more than a quarter above, block_list takes the bands
    if (t.boxes(nx, ny)) t.cap += t.cap / 4;
    return t;
}

// XCD of a piece of a tile column.  With at least eight tile rows and eight pieces along z, the
// rows and the planes are cut into eight bands each and region (y band, z band) goes to XCD
// (y band + z band) mod 8: a Latin square, so every XCD holds one region of every y band and of
// every z band (the same share of the C-PML layers of y and z; every region spans the x extent)
// and a region's neighbouring tiles share one L2.  Smaller grids deal runs of pieces (index: the
// piece's number in z-major order) round-robin.
//
// Where those regions are slivers, y bands of at most three tile rows on a grid of at most a
// million cells, each XCD takes one box of equal cost instead (cut_regions): its surface is smaller,
// so fewer taps miss its L2.  Measured (us per forward / adjoint step, bands and boxes): skull
// medium 48^3 12.2/12.5 and 11.7/12.1, 64^3 14.1/15.5 and 13.3/14.8, 96^3 26.8/29.5 and 26.6/29.1,
// 112^3 36.2/39.9 and 36.4/40.5, 128^3 41.8/46.6 and 42.7/47.8, 192^3 116.9/125.7 and 123.1/133.2,
// 288^3 365/385 and 387/408; soft tissue 64^3 11.0/11.0 and 10.6/10.9, 96^3 17.4/17.8 and
// 16.8/17.5, 128^3 31.4/33.2 and 32.4/34.0, 208^3 138/144 and 144/151.  On large grids the bands
// win: every XCD is at the same planes at the same time, and carries the same mix of updates.
int piece_xcd(const Tiles &t, int by, int z, long long index) {
    if (t.bands()) return (by * 8 / t.nty + z * 8 / t.nz) % 8;
    return (int)(index / t.run() % 8);
}

unsigned tile_edges(const Tiles &t, const unsigned char *fast, int q) {
    if (!fast || !fast[q]) return 0;
    const int b[2] = {(q / t.ntx) % t.nty, q / t.ntx / t.nty};
    const int nb[2] = {t.nty, t.nzc};
    const int step[2] = {t.ntx, t.ntx * t.nty};
    unsigned edges = 0;
    for (int a = 0; a < 2; ++a) {   // y, z
        if (b[a] > 0 && !fast[q - step[a]]) edges |= 1u << (2 * a);
        if (b[a] + 1 < nb[a] && !fast[q + step[a]]) edges |= 1u << (2 * a + 1);
    }
    return edges;
}

// What the regions are cut by: the cost of a sub-tile's general update, of the layers of an axis
// (both in units of a fluid sub-tile), and how uneven a cut may be.
constexpr double kGeneralCost = 2.0, kLayerCost = 0.3, kEvenCut = 0.02;
// The sub-tiles of a tile: those with columns in the grid, of these those whose columns are all fluid
// and those whose columns are all uniform; per sub-tile and row, its fluid and uniform columns (of a
// tile that is not fluid).
struct Subs {
    unsigned in = 0, fluid = 0, same = 0;
    unsigned cols[4][kWaveY] = {}, uniform[4][kWaveY] = {};
    int entries() const { return __builtin_popcount(in & ~fluid) + (fluid ? 1 : 0); }
};
Subs subs_of(const Tiles &t, int nx, int ny, const unsigned char *fast, const unsigned long long *lanes, int bx, int by, int q) {
    Subs u;
    u.in = (nx - bx * kTileX > kWaveX ? 3u : 1u) * (ny - by * kTileY > kWaveY ? 5u : 1u);
    if (!fast) return u;
    if (fast[q]) {
        u.fluid = u.same = u.in;
        return u;
    }
    const unsigned long long *fl = lanes + (size_t)kTileY * q, *un = lanes + (size_t)kTileY * (t.ntiles + (size_t)q);
    if (!(fl[0] | fl[1] | fl[2] | fl[3])) return u;   // no fluid column: most tiles of a solid
    for (int s = 0; s < 4; ++s) {
        if (!(u.in >> s & 1u)) continue;
        const int x0 = bx * kTileX + (s & 1) * kWaveX, y0 = by * kTileY + (s >> 1) * kWaveY;
        const unsigned valid = nx - x0 >= kWaveX ? ~0u : (1u << (nx - x0)) - 1;
        bool all = true, same = true;
        for (int r = 0; r < kWaveY && y0 + r < ny; ++r) {
            const int row = (s >> 1) * kWaveY + r;
            u.cols[s][r] = (unsigned)(fl[row] >> ((s & 1) * kWaveX)) & valid;
            u.uniform[s][r] = (unsigned)(un[row] >> ((s & 1) * kWaveX)) & valid;
            all = all && u.cols[s][r] == valid;
            same = same && u.uniform[s][r] == valid;
        }
        if (all) u.fluid |= 1u << s;
        if (all && same) u.same |= 1u << s;
    }
    return u;
}
static_assert(kTileX == 2 * kWaveX && kTileY == 2 * kWaveY && kTileY == 4, "four sub-tiles of two rows");

// Planes per block.  A long column of planes reads fewer halo planes, a short one gives more
// wavefronts and a shorter chain of planes per wavefront: kZBlock, two where that leaves few blocks,
// kZDeep on large grids that are mostly solid, whose six stresses cost more halo.
// Measured (us per forward / adjoint step, blocks of 2, 3 and 4 planes; blocks of 4 planes there
// are): skull medium 64^3 (900) 13.5/14.8, 14.6/15.4, 16.7/17.3; 96^3 (2800)
// 26.6/29.6, 27.4/29.4, 32.9/35.1; 128^3 (5000) 42.3/47.2, 43.2/47.8, 44.4/48.5; 136^3 (6700)
// 47.3/51.8, 48.9/52.2, 48.0/51.5; 152^3 (8700) 60.3/70.3, 56.4/61.9, 56.1/59.5; 192^3 124/140, 118/130,
// 116/124; 384^3 818/915, 785/842, 771/811 (6 planes 773/808); soft tissue 112^3 24.0/25.9,
// 25.9/27.5, 24.4/25.9; 144^3 (3888) 41.6/44.1, 42.8/44.8, 43.2/44.8; all solid 48^3 13.0/13.4,
// 13.4/13.7, 15.0/15.1; 80^3 (3200) 26.3/28.3, 25.9/27.6, 26.6/27.6; 112^3 (6272) 50.2/56.7,
// 50.0/53.9, 48.5/52.6; 128^3 skull in double precision 77.5/92.3, 79.2/93.8, 79.6/95.1.
// Mostly solid, 4, 6, 8 and 12 planes: 157 x 131 x 109 (5500 blocks of 8) 65.2/70.5, 68.2/72.8,
// 67.6/73.6, 76.4/80.3; 203 x 187 x 150 (14288) 210/232, 211/232, 209/232, 214/235; 256^3 550/598,
// 541/587, 544/587, 547/591; 320^3 1028/1108, 1007/1082, 1006/1079, 1004/1077; 384^3 1725/1851,
// 1691/1805, 1680/1790, 1680/1785; 192^3 in double precision (13824) 531/599, 521/586, 518/582, 525/584.
int block_planes(const Tiles &t, int nx, int ny, int P, const unsigned char *fast, const unsigned char *uni,
                 const unsigned long long *lanes, long long *touched) {
    long long planes = 0;        // over the entries
    long long subs = 0, general = 0;   // sub-tiles
    // elements of the state that a time step touches, by kind of sub-tile: all nine fields and four maps
    // (general), u, s11 and three maps (fluid) or none of the maps (uniform); of every layer that a cell
    // is in, the six memory variables of its axis (general) or the two diagonal ones
    long long state = 0;
    auto layers = [P](int c0, int c1, int n) {
        return P <= 0 ? 0ll : (long long)std::max(0, std::min(c1, P + 1) - c0) + std::max(0, c1 - std::max(c0, n - 1 - P));
    };
    int q = 0;
    for (int bz = 0; bz < t.nzc; ++bz) {
        const int z0 = bz * t.zc, z1 = std::min(z0 + t.zc, t.nz), depth = z1 - z0;
        for (int by = 0; by < t.nty; ++by)
            for (int bx = 0; bx < t.ntx; ++bx, ++q) {
                auto add = [&](int x0, int w, int y0, int h, int arrays, int memory) {
                    w = std::min(w, nx - x0);
                    h = std::min(h, ny - y0);
                    state += (long long)w * h * depth * arrays +
                             memory * (layers(x0, x0 + w, nx) * h * depth + layers(y0, y0 + h, ny) * w * depth + layers(z0, z1, t.nz) * w * h);
                };
                if (fast && fast[q]) {
                    planes += depth;
                    subs += 4;
                    add(bx * kTileX, kTileX, by * kTileY, kTileY, uni[q] ? 4 : 7, 2);
                    continue;
                }
                const Subs u = subs_of(t, nx, ny, fast, lanes, bx, by, q);
                planes += u.entries() * depth;
                subs += __builtin_popcount(u.in);
                general += __builtin_popcount(u.in & ~u.fluid);
                if (!u.fluid) add(bx * kTileX, kTileX, by * kTileY, kTileY, NFIELD + 4, 6);
                for (int s = 0; u.fluid && s < 4; ++s)
                    if (u.in >> s & 1u) {
                        const bool fl = u.fluid >> s & 1u;
                        add(bx * kTileX + (s & 1) * kWaveX, kWaveX, by * kTileY + (s >> 1) * kWaveY, kWaveY,
                            !fl ? NFIELD + 4 : (u.same >> s & 1u ? 4 : 7), fl ? 2 : 6);
                    }
            }
    }
    *touched = state;
    if (planes < kFewBlocks * kZBlock) return 2;
    return 4 * general >= 3 * subs && planes >= kManyBlocks * kZDeep ? kZDeep : kZBlock;
}

// Regions of equal cost, one per XCD: boxes of tile columns and planes, by cutting the grid, then
// each part, at the point of its longest axis that halves its cost; another axis where that one's
// whole tiles (columns of cells) would leave the halves uneven.
struct Region {
    int b[3], e[3];   // tiles along x and y, planes
};
void cut_regions(const Tiles &t, const std::vector<float> &cost, Region box, int parts, Region *out) {
    if (parts == 1) {
        *out = box;
        return;
    }
    std::vector<double> along[3];
    for (int a = 0; a < 3; ++a) along[a].assign(box.e[a] - box.b[a], 0.0);
    for (int z = box.b[2]; z < box.e[2];) {
        const int bz = z / t.zc, z1 = std::min((bz + 1) * t.zc, box.e[2]);
        double plane = 0;
        for (int by = box.b[1]; by < box.e[1]; ++by) {
            const float *row = &cost[((size_t)bz * t.nty + by) * t.ntx];
            double sum = 0;
            for (int bx = box.b[0]; bx < box.e[0]; ++bx) {
                along[0][bx - box.b[0]] += row[bx] * (z1 - z);
                sum += row[bx];
            }
            along[1][by - box.b[1]] += sum * (z1 - z);
            plane += sum;
        }
        for (; z < z1; ++z) along[2][z - box.b[2]] = plane;
    }
    double total = 0;
    for (double c : along[0]) total += c;
    const int unit[3] = {kTileX, kTileY, 1};
    int axis = -1, at = 0;
    double best = 0;
    for (int a = 2; a >= 0; --a) {
        const int n = box.e[a] - box.b[a];
        if (n < 2) continue;
        double left = 0, off = 1;
        int cut = 1;
        for (int c = 1; c < n; ++c) {
            left += along[a][c - 1];
            const double o = std::fabs(left / total - 0.5);
            if (o < off) {
                off = o;
                cut = c;
            }
        }
        const double score = off <= kEvenCut ? (double)n * unit[a] : -off;
        if (axis < 0 || score > best) {
            axis = a;
            at = cut;
            best = score;
        }
    }
    if (axis < 0) {   // one tile of one plane: nothing to share out
        out[0] = box;
        for (int q = 1; q < parts; ++q) out[q] = Region{{0, 0, 0}, {0, 0, 0}};
        return;
    }
    Region lo = box, hi = box;
    lo.e[axis] = hi.b[axis] = box.b[axis] + at;
    cut_regions(t, cost, lo, parts / 2, out);
    cut_regions(t, cost, hi, parts / 2, out + parts / 2);
}
// Cost of a tile's chunk per plane, in sub-tiles of the fluid update.
std::vector<float> chunk_costs(const Tiles &t, int nx, int ny, int P, const unsigned char *fast,
                               const unsigned long long *lanes) {
    std::vector<float> cost(t.ntiles);
    auto layers = [P](int c0, int c1, int n) { return P <= 0 ? 0 : std::max(0, std::min(c1, P) - c0) + std::max(0, c1 - std::max(c0, n - P)); };
    int q = 0;
    for (int bz = 0; bz < t.nzc; ++bz) {
        const int z0 = bz * t.zc, z1 = std::min(z0 + t.zc, t.nz);
        const float lz = (float)kLayerCost * layers(z0, z1, t.nz) / (float)(z1 - z0);
        for (int by = 0; by < t.nty; ++by) {
            const int y0 = by * kTileY, y1 = std::min(y0 + kTileY, ny);
            const float ly = (float)kLayerCost * layers(y0, y1, ny) / (float)(y1 - y0);
            for (int bx = 0; bx < t.ntx; ++bx, ++q) {
                const int x0 = bx * kTileX, x1 = std::min(x0 + kTileX, nx);
                const Subs u = subs_of(t, nx, ny, fast, lanes, bx, by, q);
                const float c = __builtin_popcount(u.fluid) + (float)kGeneralCost * __builtin_popcount(u.in & ~u.fluid);
                cost[q] = c * (1.f + lz + ly + (float)kLayerCost * layers(x0, x1, nx) / (float)(x1 - x0));
            }
        }
    }
    return cost;
}

// Do chunks q and q + step of a tile column (one above the other) ask for the same update?
template <typename T>
bool same_update(const Tiles &t, const unsigned char *fast, const unsigned char *uni, const unsigned long long *lanes,
                 const T *med, int q) {
    const int r = q + t.ntx * t.nty;
    if (!fast) return true;
    const bool med_same = med[4 * (size_t)q] == med[4 * (size_t)r] && med[4 * (size_t)q + 1] == med[4 * (size_t)r + 1] &&
                          med[4 * (size_t)q + 2] == med[4 * (size_t)r + 2];
    if (fast[q] != fast[r]) return false;
    if (fast[q])
        return uni[q] == uni[r] && (!uni[q] || med_same) && (tile_edges(t, fast, q) & 3) == (tile_edges(t, fast, r) & 3);
    const unsigned long long *fq = lanes + (size_t)kTileY * q, *fr = lanes + (size_t)kTileY * r;
    const size_t un = (size_t)kTileY * t.ntiles;   // the uniform columns' masks
    unsigned long long any = 0;
    for (int w = 0; w < kTileY; ++w) {
        if (fq[w] != fr[w] || fq[un + w] != fr[un + w]) return false;
        any |= fq[un + w];
    }
    return !any || med_same;
}

template <typename T>
BlockList<T> cut_list(const Tiles &tiles, int nx, int ny, int npml, const unsigned char *fast, const unsigned char *uni,
                      const unsigned long long *lanes, const T *med, const std::vector<int> &points, bool boxed) {
    Tiles t = tiles;
    long long touched = 0;
    t.zb = block_planes(t, nx, ny, npml, fast, uni, lanes, &touched);
    BlockList<T> out;
    out.once = touched * (long long)sizeof(T) > kStreamBytes;
    // room for cap entries per XCD (an entry costs its 64 bytes only once it is written)
    out.entries.reset(new BlockEnt<T>[8 * (size_t)t.cap]);
    BlockEnt<T> *order = out.entries.get();
    size_t count[8] = {};
    // per tile column: its run of chunks that ask for the same update, and the next plane to cover
    struct Run {
        int z0, z1, next;
    };
    std::vector<Run> runs((size_t)t.ntx * t.nty, Run{0, 0, 0});
    const int step = t.ntx * t.nty;
    Region region[8] = {};
    if (boxed) cut_regions(t, chunk_costs(t, nx, ny, npml, fast, lanes), Region{{0, 0, 0}, {t.ntx, t.nty, t.nz}}, 8, region);
    auto xcd_of = [&](int bx, int by, int z, long long index) {
        if (boxed)
            for (int x = 0; x < 8; ++x) {
                const Region &g = region[x];
                if (bx >= g.b[0] && bx < g.e[0] && by >= g.b[1] && by < g.e[1] && z >= g.b[2] && z < g.e[2]) return x;
            }
        return piece_xcd(t, by, z, index);
    };
    // with scatter points: the pieces (entries at first, first + 8, ..., n of them; their sub-tiles
    // with points; the first one's first increment plane), and per column and plane, 1 + the number
    // of the piece that begins there
    struct Piece {
        size_t first;
        int n, z0, z1;
        unsigned with;
        int slot;
    };
    std::vector<Piece> piece;
    std::vector<int> begins(points.empty() ? 0 : (size_t)step * t.nz, 0);
    long long pieces = 0;
    for (int z = 0; z < t.nz; ++z)
        for (int by = 0; by < t.nty; ++by)
            for (int bx = 0; bx < t.ntx; ++bx) {
                Run &run = runs[by * t.ntx + bx];
                if (run.next != z) continue;
                const int bz = z / t.zc, q = bz * step + by * t.ntx + bx;
                if (run.z1 == z) {   // the next run (runs end with a chunk)
                    int e = q;
                    while (e + step < t.ntiles && same_update(t, fast, uni, lanes, med, e)) e += step;
                    run = {z, std::min((e / step + 1) * t.zc, t.nz), z};
                }
                // a piece of it: to the next multiple of zb, where all columns are cut, if that
                // leaves neither piece under the shortest (the last of a long run has two planes at
                // least: a deep one would come last on its XCD and the others wait for it)
                int cut = (z + t.shortest() + t.zb - 1) / t.zb * t.zb;
                if (run.z1 - cut < (z == run.z0 ? t.shortest() : 2)) cut = run.z1;
                run.next = cut;
                const int x = xcd_of(bx, by, z, pieces++);
                const size_t first = count[x];
                BlockEnt<T> e = {bx, by, z, cut, 0, -1, {}, {}, med[4 * (size_t)q], med[4 * (size_t)q + 1], med[4 * (size_t)q + 2]};
                const Subs u = subs_of(t, nx, ny, fast, lanes, bx, by, q);
                auto put = [&](unsigned flags) {
                    e.flags = flags | (count[x] == first ? kBlkFirst : 0u);
                    if (count[x] < (size_t)t.cap) order[8 * count[x] + x] = e;
                    ++count[x];
                };
                if (fast && fast[q]) {
                    unsigned edges = tile_edges(t, fast, q) & 3u;
                    if (e.z0 == run.z0) edges |= tile_edges(t, fast, q) & 4u;
                    if (e.z1 == run.z1) edges |= tile_edges(t, fast, q + ((run.z1 - 1) / t.zc - bz) * step) & 8u;
                    put(kBlkFast | u.in << kBlkMaskShift | (uni[q] ? u.in << kBlkUniShift : 0u) | edges << kBlkEdgeShift);
                } else {
                    for (int s = 0; s < 4; ++s) {
                        if (!((u.in & ~u.fluid) >> s & 1u)) continue;
                        for (int r = 0; r < kWaveY; ++r) {
                            e.fluid[r] = u.cols[s][r];
                            e.uniform[r] = u.uniform[s][r];
                        }
                        put(kBlkGen | (unsigned)s << kBlkSubShift);
                    }
                    if (u.fluid) put(kBlkKeep | u.fluid << kBlkMaskShift | u.same << kBlkUniShift);
                }
                if (points.empty()) continue;
                piece.push_back({8 * first + x, (int)(count[x] - first), z, cut, 0u, 0});
                begins[(size_t)z * step + by * t.ntx + bx] = (int)piece.size();
            }
    const size_t per = *std::max_element(count, count + 8);
    out.fits = per <= (size_t)t.cap;
    if (!out.fits) return out;
    // increments: the planes of every sub-tile's piece with points, one after the other; a point's
    // element there (plane, then lane)
    const size_t np = points.size() / 3;
    std::vector<int> of(np);
    for (size_t p = 0; p < np; ++p) {
        const int i = points[3 * p], j = points[3 * p + 1];
        size_t at = (size_t)points[3 * p + 2] * step + j / kTileY * t.ntx + i / kTileX;
        while (!begins[at]) at -= step;
        of[p] = begins[at] - 1;
        piece[of[p]].with |= 1u << (2 * (j % kTileY / kWaveY) + i % kTileX / kWaveX);
    }
    for (Piece &p : piece) {
        if (!p.with) continue;
        p.slot = (int)out.planes;
        out.planes += __builtin_popcount(p.with) * (p.z1 - p.z0);
        for (int n = 0; n < p.n; ++n) {
            order[p.first + 8 * (size_t)n].slot = p.slot;
            order[p.first + 8 * (size_t)n].flags |= p.with << kBlkIncShift;
        }
    }
    out.pos.resize(np);
    for (size_t q = 0; q < np; ++q) {
        const int i = points[3 * q], j = points[3 * q + 1], k = points[3 * q + 2];
        const Piece &p = piece[of[q]];
        const int sub = 2 * (j % kTileY / kWaveY) + i % kTileX / kWaveX;
        const int plane = p.slot + __builtin_popcount(p.with & ((1u << sub) - 1u)) * (p.z1 - p.z0) + k - p.z0;
        out.pos[q] = (plane * kWaveY + j % kWaveY) * kWaveX + i % kWaveX;
    }
    out.per = (int)per;
    for (int x = 0; x < 8; ++x)
        for (size_t e = count[x]; e < per; ++e) order[8 * e + x] = BlockEnt<T>{};
    return out;
}
template <typename T>
BlockList<T> block_list(const Tiles &t, int nx, int ny, int npml, const unsigned char *fast, const unsigned char *uni,
                        const unsigned long long *lanes, const T *med, const std::vector<int> &points) {
    const bool boxed = t.boxes(nx, ny);
    BlockList<T> out = cut_list(t, nx, ny, npml, fast, uni, lanes, med, points, boxed);
    if (boxed && !out.fits) out = cut_list(t, nx, ny, npml, fast, uni, lanes, med, points, false);
    return out;
}
template BlockList<float> block_list<float>(const Tiles &, int, int, int, const unsigned char *, const unsigned char *,
                                            const unsigned long long *, const float *, const std::vector<int> &);
template BlockList<double> block_list<double>(const Tiles &, int, int, int, const unsigned char *, const unsigned char *,
                                              const unsigned long long *, const double *, const std::vector<int> &);

}  // namespace el

extern "C" {

const char *el_version(void) { return "elastic-pact-mi355x 0.1.0 (gfx950)"; }

const char *el_status_string(el_status s) {
    switch (s) {
        case EL_OK: return "EL_OK";
        case EL_EINVAL: return "EL_EINVAL";
        case EL_EUNSTABLE: return "EL_EUNSTABLE";
        case EL_ERANGE: return "EL_ERANGE";
        case EL_ENOMEM: return "EL_ENOMEM";
        case EL_EDEVICE: return "EL_EDEVICE";
        case EL_EBUSY: return "EL_EBUSY";
        default: return "EL_UNKNOWN";
    }
}

const char *el_last_error(void) { return g_err; }

el_status el_grid_check(const el_grid *g, const double *rec, int32_t nrec) {
    if (!g) return fail(EL_EINVAL, "grid is NULL");
    if (g->nx < 4 || g->ny < 4 || g->nz < 4)
        return fail(EL_EINVAL, "grid %dx%dx%d: every axis needs at least 4 cells", g->nx, g->ny, g->nz);
    if (!(g->dx > 0) || !std::isfinite(g->dx)) return fail(EL_EINVAL, "dx must be positive and finite");
    if (!(g->dt > 0) || !std::isfinite(g->dt)) return fail(EL_EINVAL, "dt must be positive and finite");
    if (g->nsteps < 1) return fail(EL_EINVAL, "nsteps must be >= 1");
    if (g->npml < 0) return fail(EL_EINVAL, "npml must be >= 0");
    const int n[3] = {g->nx, g->ny, g->nz};
    for (int a = 0; a < 3; ++a)
        if (g->npml > 0 && n[a] < 2 * g->npml + 2)
            return fail(EL_EINVAL, "axis %d has %d cells, fewer than 2*npml+2 = %d", a, n[a], 2 * g->npml + 2);
    if (g->precision != EL_F32 && g->precision != EL_F64) return fail(EL_EINVAL, "precision must be EL_F32 or EL_F64");
    {
        const long long es = g->precision == EL_F64 ? 8 : 4;
        const long long bytes = make_vol(g->nx, g->ny, g->nz).total * es;
        if (bytes >= (1LL << 32))
            return fail(EL_EINVAL, "grid %dx%dx%d: one padded volume array needs %lld bytes; the kernels address at most 4 GiB per array",
                        g->nx, g->ny, g->nz, bytes);
        // the C-PML memory variables of axis a live on W = 2 (P + 7) planes of that axis
        // (slab_byte forms 32-bit byte offsets into them as well)
        if (g->npml > 0) {
            const long long W = 2LL * (g->npml + 7);
            const long long slab[3] = {W * g->ny * g->nz, W * g->nx * g->nz, W * g->nx * g->ny};
            for (int a = 0; a < 3; ++a)
                if (slab[a] * es >= (1LL << 32))
                    return fail(EL_EINVAL,
                                "grid %dx%dx%d, npml %d: a C-PML memory-variable array of axis %d needs %lld bytes; "
                                "the kernels address at most 4 GiB per array",
                                g->nx, g->ny, g->nz, g->npml, a, slab[a] * es);
        }
        const int zc = chunk_planes(g->nx, g->ny, g->nz);
        const long long tiles = (long long)((g->nx + kTileX - 1) / kTileX) * ((g->ny + kTileY - 1) / kTileY) *
                                ((g->nz + zc - 1) / zc);
        if (tiles > kMaxTiles)
            return fail(EL_EINVAL, "grid %dx%dx%d: %lld stencil tiles, at most %d", g->nx, g->ny, g->nz, tiles, kMaxTiles);
    }
    {
        const el_relaxation &rx = g->relax;
        if (rx.nmech < 0 || rx.nmech > EL_MAX_MECH)
            return fail(EL_EINVAL, "relax.nmech = %d outside 0..%d", rx.nmech, EL_MAX_MECH);
        for (int l = 0; l < rx.nmech; ++l)
            if (!(rx.omega[l] > 0) || !std::isfinite(rx.omega[l]) || !(rx.weight[l] >= 0) || !std::isfinite(rx.weight[l]))
                return fail(EL_EINVAL, "relaxation mechanism %d: omega must be > 0 and weight >= 0, both finite", l);
    }
    if (nrec < 0) return fail(EL_EINVAL, "nrec must be >= 0");
    if (nrec > (1 << 26)) return fail(EL_EINVAL, "too many receivers");
    if (nrec > 0 && !rec) return fail(EL_EINVAL, "rec_xyz is NULL");
    for (int l = 0; l < nrec; ++l)
        for (int a = 0; a < 3; ++a) {
            const double x = rec[3 * l + a] / g->dx;
            if (!(x >= -kRecSlack && x <= (double)(n[a] - 1) + kRecSlack))
                return fail(EL_ERANGE, "receiver %d axis %d at %.6g cells is outside [0, %d]", l, a, x, n[a] - 1);
        }
    return EL_OK;
}

el_status el_plan_bytes(const el_grid *g, int32_t nrec, size_t *bytes) {
    el_status st = el_grid_check(g, nullptr, 0);
    if (st != EL_OK) return st;
    if (nrec < 0) return fail(EL_EINVAL, "nrec must be >= 0");
    if (!bytes) return fail(EL_EINVAL, "bytes is NULL");
    Layout L;
    layout(*g, nrec, &L);
    *bytes = L.total;
    return EL_OK;
}

}  // extern "C"

namespace {

// C-PML profile of one axis (Appendix A.1-A.2, kappa = 1): with xi the depth into
// the layer over its thickness, measured from planes P and n-1-P and clamped to
// [0, 1], d = d0 xi^npow, beta = pi f0 (1 - xi), b = exp(-(d + beta) dt),
// a = d / (d + beta) (b - 1); a = 0 where xi = 0.
void pml_axis(const el_grid &g, int n, double d0, double f0, double npow, int half, std::vector<double> &a,
              std::vector<double> &b) {
    a.assign(n, 0.0);
    b.assign(n, 1.0);
    const int P = g.npml;
    for (int i = 0; i < n; ++i) {
        const double x = i + 0.5 * half;
        double depth = 0.0;
        if (x < P) depth = P - x;
        if (x > n - 1 - P) depth = x - (n - 1 - P);
        double xi = depth / P;
        if (xi > 1.0) xi = 1.0;
        if (xi > 0.0) {
            const double d = d0 * std::pow(xi, npow);
            const double beta = M_PI * f0 * (1.0 - xi);
            b[i] = std::exp(-(d + beta) * g.dt);
            a[i] = d / (d + beta) * (b[i] - 1.0);
        } else {
            b[i] = std::exp(-(M_PI * f0) * g.dt);
        }
    }
}

template <typename T>
void bind(Dev<T> &d, el_plan_ *p) {
    const el_grid &g = p->g;
    char *ws = p->ws;
    const Vol v = make_vol(g.nx, g.ny, g.nz);
    d.nx = g.nx;
    d.ny = g.ny;
    d.nz = g.nz;
    d.P = g.npml > 0 ? g.npml : kNoPml;
    d.sy = (unsigned)(v.px * sizeof(T));
    d.sz = (unsigned)(v.plane * sizeof(T));
    d.dt = T(g.dt);
    d.inv_dx = T(1.0 / g.dx);
    d.ws = ws;
    auto u256 = [](size_t off) { return (unsigned)(off >> 8); };
    const Layout &L = p->L;
    d.vstr = u256(L.vol[1] - L.vol[0]);
    d.incoff = u256(L.inc[1]);
    const int n[3] = {g.nx, g.ny, g.nz};
    for (int a = 0; a < 3; ++a) {
        const bool single = n[a] <= 2 * g.npml + 9;   // (npml = 0: not used)
        d.high[a] = single ? 2 : (g.npml + 7) - (n[a] - 1 - g.npml - 4);
        if (a == 0) d.xw = single ? d.W() : g.npml + 7;
        d.moff[a] = u256(L.mem[a][0]);
        d.mstr[a] = u256(L.mem[a][1] - L.mem[a][0]);
        d.coff[a] = u256(L.coef[a][0]);
        d.cstr[a] = u256(L.coef[a][1] - L.coef[a][0]);
    }
}

// Relaxation parameters in the plan's precision: weights, c_l = exp(-omega_l dt), buffers.
template <typename T>
void bind_relax(Relax<T> &r, el_plan_ *p) {
    const el_relaxation &rx = p->g.relax;
    r = Relax<T>{};
    r.L = rx.nmech;
    for (int l = 0; l < rx.nmech; ++l) {
        r.w[l] = T(rx.weight[l]);
        r.c[l] = T(std::exp(-rx.omega[l] * p->g.dt));
    }
    if (rx.nmech > 0) {
        r.ar = reinterpret_cast<T *>(p->ws + p->L.relax_map);
        r.flag = reinterpret_cast<unsigned char *>(p->ws + p->L.relax_flag);
        r.count = reinterpret_cast<int *>(p->ws + p->L.relax_count);
        r.off = reinterpret_cast<long long *>(p->ws + p->L.relax_off);
        r.pts = reinterpret_cast<unsigned *>(p->ws + p->L.relax_pts);
        r.beta = reinterpret_cast<T *>(p->ws + p->L.relax_beta);
        r.zeta = reinterpret_cast<T *>(p->ws + p->L.relax_zeta);
    }
}

template <typename T>
el_status upload_pml(el_plan_ *p, Dev<T> &d, hipStream_t s) {
    const el_grid &g = p->g;
    const double R = g.pml_R > 0 ? g.pml_R : 1e-3;
    const double npow = g.pml_npower > 0 ? g.pml_npower : 2.0;
    const double f0 = g.pml_f0 > 0 ? g.pml_f0 : 1500.0 / (8.0 * g.dx);
    const double d0 = g.npml > 0 ? -(npow + 1.0) * p->cmax * std::log(R) / (2.0 * g.npml * g.dx) : 0.0;
    const int n[3] = {g.nx, g.ny, g.nz};
    std::vector<double> a, b;
    for (int ax = 0; ax < 3; ++ax)
        for (int h = 0; h < 2; ++h) {
            if (g.npml > 0) {
                pml_axis(g, n[ax], d0, f0, npow, h, a, b);
            } else {
                a.assign(n[ax], 0.0);
                b.assign(n[ax], 1.0);
            }
            std::vector<T> at(a.begin(), a.end()), bt(b.begin(), b.end()), ab;
            if (ax == 2) {
                for (int k = 0; k < n[2]; ++k) {
                    ab.push_back(at[k]);
                    ab.push_back(bt[k]);
                }
                HIP_TRY(hipMemcpyAsync(d.zab(h), ab.data(), ab.size() * sizeof(T), hipMemcpyHostToDevice, s), "copy PML a, b");
            } else {
                HIP_TRY(hipMemcpyAsync(d.pa(ax, h), at.data(), n[ax] * sizeof(T), hipMemcpyHostToDevice, s), "copy PML a");
                HIP_TRY(hipMemcpyAsync(d.pb(ax, h), bt.data(), n[ax] * sizeof(T), hipMemcpyHostToDevice, s), "copy PML b");
            }
            HIP_TRY(hipStreamSynchronize(s), "PML upload");
        }
    return EL_OK;
}

// Trilinear weights on the normal-stress grid (Sec. 3, eq. interpgrid): base index
// floor(x/dx) clamped to n-2, fraction x/dx - base; corner c = (c&1, c>>1&1, c>>2&1).
el_status upload_receivers(el_plan_ *p, const double *rec, hipStream_t s) {
    const el_grid &g = p->g;
    const int L = p->nrec;
    const int n[3] = {g.nx, g.ny, g.nz};
    const Vol v = make_vol(g.nx, g.ny, g.nz);
    std::vector<long long> idx(8 * (size_t)L);
    std::vector<int> cidx(3 * 8 * (size_t)L);
    std::vector<double> w(8 * (size_t)L);
    p->rec_tile.assign(8 * (size_t)L, 0);
    for (int l = 0; l < L; ++l) {
        int b[3];
        double f[3];
        for (int a = 0; a < 3; ++a) {
            const double x = std::min(std::max(rec[3 * l + a] / g.dx, 0.0), (double)(n[a] - 1));
            int bb = (int)std::floor(x);
            if (bb > n[a] - 2) bb = n[a] - 2;
            b[a] = bb;
            f[a] = x - bb;
        }
        for (int c = 0; c < 8; ++c) {
            const int ox = c & 1, oy = (c >> 1) & 1, oz = (c >> 2) & 1;
            idx[8 * l + c] = v.origin + (long long)(b[2] + oz) * v.plane + (long long)(b[1] + oy) * v.px + (b[0] + ox);
            cidx[3 * (8 * l + c) + 0] = b[0] + ox;
            cidx[3 * (8 * l + c) + 1] = b[1] + oy;
            cidx[3 * (8 * l + c) + 2] = b[2] + oz;
            w[8 * l + c] = (ox ? f[0] : 1 - f[0]) * (oy ? f[1] : 1 - f[1]) * (oz ? f[2] : 1 - f[2]);
            const Tiles &t = p->tiles;
            p->rec_tile[8 * l + c] = ((b[2] + oz) / t.zc * t.nty + (b[1] + oy) / kTileY) * t.ntx + (b[0] + ox) / kTileX;
        }
    }
    // grid-point-major transpose: entries sorted by (cell, receiver, corner)
    std::vector<int> order(8 * (size_t)L);
    for (size_t e = 0; e < order.size(); ++e) order[e] = (int)e;
    std::sort(order.begin(), order.end(), [&](int x, int y) { return idx[x] != idx[y] ? idx[x] < idx[y] : x < y; });
    std::vector<long long> pt;
    std::vector<int> ptc, row, erec;
    std::vector<double> ew;
    for (size_t e = 0; e < order.size(); ++e) {
        const int o = order[e];
        if (pt.empty() || pt.back() != idx[o]) {
            pt.push_back(idx[o]);
            for (int a = 0; a < 3; ++a) ptc.push_back(cidx[3 * o + a]);
            row.push_back((int)e);
        }
        erec.push_back(o / 8);
        ew.push_back(w[o]);
    }
    row.push_back((int)order.size());
    char *ws = p->ws;
    Rec &r = p->rec;
    r.nrec = L;
    r.idx = reinterpret_cast<long long *>(ws + p->L.rec_idx);
    r.w = reinterpret_cast<double *>(ws + p->L.rec_w);
    r.npts = (int)pt.size();
    r.pt = reinterpret_cast<long long *>(ws + p->L.csr_pt);
    r.ptc = reinterpret_cast<int *>(ws + p->L.csr_ptc);
    r.row = reinterpret_cast<int *>(ws + p->L.csr_row);
    r.ent_rec = reinterpret_cast<int *>(ws + p->L.csr_rec);
    r.ent_w = reinterpret_cast<double *>(ws + p->L.csr_w);
    if (L > 0) {
        HIP_TRY(hipMemcpyAsync((void *)r.idx, idx.data(), idx.size() * 8, hipMemcpyHostToDevice, s), "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.w, w.data(), w.size() * 8, hipMemcpyHostToDevice, s), "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.pt, pt.data(), pt.size() * 8, hipMemcpyHostToDevice, s), "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.ptc, ptc.data(), ptc.size() * 4, hipMemcpyHostToDevice, s), "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.row, row.data(), row.size() * 4, hipMemcpyHostToDevice, s), "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.ent_rec, erec.data(), erec.size() * 4, hipMemcpyHostToDevice, s),
                "copy receivers");
        HIP_TRY(hipMemcpyAsync((void *)r.ent_w, ew.data(), ew.size() * 8, hipMemcpyHostToDevice, s), "copy receivers");
    }
    HIP_TRY(hipStreamSynchronize(s), "receiver upload");
    p->points = std::move(ptc);
    return EL_OK;
}

// The block list, the receiver corners' fluid flags and the points' places in the increments, with
// the fluid tiles when the fluid update is on and without them otherwise.  Each setting has
// tables of its own, made when it is first asked for, so a launch captured under one stays whole.
// The plan takes them once they are complete: a failure leaves it as it was.
template <typename T>
el_status set_tables_t(el_plan p, Dev<T> &d, bool fluid, hipStream_t s) {
    const int on = fluid ? 1 : 0;
    const unsigned char *fast = on ? p->fast.data() : nullptr;
    char *ws = p->ws;
    Dev<T> nd = d;
    nd.incoff = (unsigned)(p->L.inc[on] >> 8);
    if (p->per[on] == 0 && p->tiles.ntiles > 0) {
        const BlockList<T> list = block_list<T>(p->tiles, p->g.nx, p->g.ny, p->g.npml, fast, p->uni.data(), p->lanes.data(),
                                                reinterpret_cast<const T *>(p->med.data()), p->points);
        if (!list.fits) return fail(EL_EINVAL, "the block list needs more than %d entries per XCD", p->tiles.cap);
        if (list.planes > p->L.inc_planes)
            return fail(EL_EINVAL, "the receivers need %lld planes of increments, room for %lld", list.planes, p->L.inc_planes);
        std::vector<unsigned char> fl(p->rec_tile.size(), 0);
        for (size_t e = 0; e < fl.size(); ++e) fl[e] = fast && fast[p->rec_tile[e]] ? 1 : 0;
        HIP_TRY(hipMemcpyAsync(ws + p->L.tile_order[on], list.entries.get(), 8 * (size_t)list.per * sizeof(BlockEnt<T>),
                               hipMemcpyHostToDevice, s), "block list");
        HIP_TRY(launch_zero_inc(nd, list.planes * kWaveX * kWaveY, s), "increments");
        if (!fl.empty()) {
            HIP_TRY(hipMemcpyAsync(ws + p->L.rec_fl[on], fl.data(), fl.size(), hipMemcpyHostToDevice, s), "receiver flags");
            HIP_TRY(hipMemcpyAsync(ws + p->L.csr_pos[on], list.pos.data(), list.pos.size() * 4, hipMemcpyHostToDevice, s),
                    "increments");
        }
        HIP_TRY(hipStreamSynchronize(s), "block list");
        p->once[on] = list.once;
        p->per[on] = list.per;
    }
    d = nd;
    p->rec.fl = reinterpret_cast<unsigned char *>(ws + p->L.rec_fl[on]);
    p->rec.pos = reinterpret_cast<int *>(ws + p->L.csr_pos[on]);
    p->tiles.order = ws + p->L.tile_order[on];
    p->tiles.once = p->once[on];
    p->tiles.per = p->per[on];
    p->fluid_path = fluid;
    return EL_OK;
}

el_status set_tables(el_plan p, bool fluid, hipStream_t s) {
    return p->g.precision == EL_F64 ? set_tables_t(p, p->dd, fluid, s) : set_tables_t(p, p->df, fluid, s);
}

el_status check_plan(el_plan p) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
    if (dev != p->device) return fail(EL_EINVAL, "current device %d is not the plan's device %d", dev, p->device);
    return EL_OK;
}

// Launch one kernel of time step m, bracketed by an event pair when timing samples that step.
template <typename F>
hipError_t timed(el_plan p, int kind, int m, hipStream_t s, F launch) {
    if (p->timing_every <= 0 || m % p->timing_every != 0) return launch();
    auto &v = p->ev[kind];
    if (p->used[kind] == v.size()) {
        v.emplace_back(nullptr, nullptr);
        hipError_t e = hipEventCreate(&v.back().first);
        if (e == hipSuccess) e = hipEventCreate(&v.back().second);
        if (e != hipSuccess) {
            if (v.back().first) (void)hipEventDestroy(v.back().first);
            v.pop_back();
            return e;
        }
    }
    auto &pr = v[p->used[kind]++];
    hipError_t e = hipEventRecord(pr.first, s);
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    return hipEventRecord(pr.second, s);
}

// energy != null: also the modified energy E_{m-1} = (kinetic + potential) / 2 of every
// `every`-th level m - 1, formed during update m (the velocity pass, which turns u_{m-3/2}
// into u_{m-1/2} while sigma_{m-1} stays in place) into energy[(m - 1) / every].
template <typename T>
el_status run_forward(el_plan p, Dev<T> &d, const T *p0, double *traces, hipStream_t s, int every = 0,
                      double *energy = nullptr) {
    const int M = p->g.nsteps, L = p->nrec;
    const int nb = 8 * p->tiles.per;
    double *ekin = reinterpret_cast<double *>(p->ws + p->L.energy);   // per wavefront
    double *epot = ekin + (size_t)nb * 4;                              // per block
    double *ekb = epot + nb;                                           // per 64 blocks
    const Relax<T> &rx = plan_relax<T>(p);
    HIP_TRY(launch_zero_state(d, s), "zero state");
    HIP_TRY(launch_relax_zero(p->tiles, rx, s), "relaxation state");
    HIP_TRY(launch_inject(d, p0, s), "inject");
    // trace row m-1 is gathered by extra blocks of velocity pass m (which reads those stresses
    // and writes none); the last row by a gather launch of its own
    for (int m = 1; m < M; ++m) {
        double *row = traces + (size_t)(m - 1) * L;
        const bool en = energy && (m - 1) % every == 0;
        if (en) HIP_TRY(launch_energy_pot(d, p->tiles, epot, s), "potential energy");
        HIP_TRY(timed(p, EL_K_VELOCITY, m, s,
                      [&] { return launch_velocity(d, p->tiles, s, &p->rec, row, en ? ekin : nullptr); }),
                "velocity pass");
        if (en) HIP_TRY(launch_energy_final(ekin, ekb, epot, nb, energy + (m - 1) / every, s), "energy");
        if (rx.L > 0)
            HIP_TRY(timed(p, EL_K_RELAX, m, s, [&] { return launch_relax(d, p->tiles, rx, false, s); }), "relaxation");
        HIP_TRY(timed(p, EL_K_STRESS, m, s, [&] { return launch_stress(d, p->tiles, s); }), "stress pass");
    }
    HIP_TRY(timed(p, EL_K_GATHER, M - 1, s, [&] { return launch_gather(d, p->rec, traces + (size_t)(M - 1) * L, s); }),
            "gather");
    if (p->fluid_path && p->fast_tiles > 0) HIP_TRY(launch_fluid_fill(d, p->tiles, s), "fluid fill");
    return EL_OK;
}

template <typename T>
el_status run_adjoint(el_plan p, Dev<T> &d, const double *y, T *out, hipStream_t s) {
    const int M = p->g.nsteps, L = p->nrec;
    const Relax<T> &rx = plan_relax<T>(p);
    HIP_TRY(launch_zero_state(d, s), "zero state");
    HIP_TRY(launch_relax_zero(p->tiles, rx, s), "relaxation state");
    HIP_TRY(timed(p, EL_K_SCATTER, M - 1, s, [&] { return launch_scatter(d, p->rec, y + (size_t)(M - 1) * L, s); }),
            "scatter");
    for (int m = M - 1; m >= 1; --m) {
        // the adjoint velocity launch also forms the increments Theta^T y of row m-1, which the
        // adjoint stress launch adds
        HIP_TRY(timed(p, EL_K_ADJ_VELOCITY, m, s,
                      [&] { return launch_adj_velocity(d, p->tiles, s, &p->rec, y + (size_t)(m - 1) * L); }),
                "adjoint velocity pass");
        // the transposed relaxation sits between the transposed stress and velocity updates of
        // the step (the forward applies R between its velocity and stress updates)
        if (rx.L > 0)
            HIP_TRY(timed(p, EL_K_RELAX, m, s, [&] { return launch_relax(d, p->tiles, rx, true, s); }), "relaxation");
        HIP_TRY(timed(p, EL_K_ADJ_STRESS, m, s, [&] { return launch_adj_stress(d, p->tiles, s); }), "adjoint stress pass");
    }
    if (p->fluid_path && p->fast_tiles > 0) HIP_TRY(launch_fluid_fill(d, p->tiles, s), "fluid fill");
    HIP_TRY(launch_extract(d, out, s), "extract");
    return EL_OK;
}

}  // namespace

extern "C" {

el_status el_plan_create(el_plan *out, const el_grid *grid, const float *lam, const float *mu, const float *rho,
                         const float *alpha, const float *alpha_r, const double *rec, int32_t nrec, void *workspace,
                         size_t workspace_bytes, void *stream) try {
    if (!out) return fail(EL_EINVAL, "out is NULL");
    *out = nullptr;
    el_status st = el_grid_check(grid, rec, nrec);
    if (st != EL_OK) return st;
    if (!lam || !mu || !rho || !alpha) return fail(EL_EINVAL, "a material map is NULL");
    if (grid->relax.nmech > 0 && !alpha_r) return fail(EL_EINVAL, "alpha_r is NULL with relaxation mechanisms");
    if (!workspace) return fail(EL_EINVAL, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return fail(EL_EINVAL, "workspace is not 256-byte aligned");
    Layout L;
    layout(*grid, nrec, &L);
    if (workspace_bytes < L.total)
        return fail(EL_ENOMEM, "workspace has %zu bytes, the plan needs %zu", workspace_bytes, L.total);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev), "hipGetDevice");

    std::unique_ptr<el_plan_, el_status (*)(el_plan)> own(new el_plan_(), el_plan_destroy);   // until it is whole
    el_plan_ *p = own.get();
    p->g = *grid;
    p->nrec = nrec;
    p->N = (long long)grid->nx * grid->ny * grid->nz;
    p->L = L;
    p->ws = static_cast<char *>(workspace);
    p->device = dev;
    p->tiles = make_tiles(grid->nx, grid->ny, grid->nz);
    // media checks on the device, in double
    double *stats = reinterpret_cast<double *>(p->ws + L.stats);
    double *partial = reinterpret_cast<double *>(p->ws + L.partial);
    hipError_t e = launch_media_stats(lam, mu, rho, alpha, p->N, grid->dt, stats, partial, s);
    if (e != hipSuccess) return hip_fail(e, "media statistics");
    double hs[kStats];
    e = hipMemcpyAsync(hs, stats, sizeof hs, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "media statistics");
    if (hs[6] > 0) return fail(EL_EINVAL, "%.0f non-finite material values", hs[6]);
    if (!(hs[1] > 0)) return fail(EL_EINVAL, "rho must be > 0 (min %.6g)", hs[1]);
    if (hs[2] < 0) return fail(EL_EINVAL, "mu must be >= 0 (min %.6g)", hs[2]);
    if (!(hs[3] > 0)) return fail(EL_EINVAL, "lambda + 2 mu must be > 0 (min %.6g)", hs[3]);
    // a positive bulk modulus (Sec. 2.1): the adjoint state w = C s divides by 3 lambda + 2 mu
    if (!(hs[7] > 0)) return fail(EL_EINVAL, "3 lambda + 2 mu must be > 0 (min %.6g)", hs[7]);
    if (hs[5] < 0 || hs[4] >= 1.0)
        return fail(EL_EUNSTABLE, "dt*alpha must lie in [0, 1) (range %.6g .. %.6g)", hs[5], hs[4]);
    p->cmax = std::sqrt(hs[0]);
    const double cfl = p->cmax * grid->dt / grid->dx;
    if (cfl > kCflMax)
        return fail(EL_EUNSTABLE, "CFL c_max dt/dx = %.6g exceeds the 4th-order staggered limit %.6g", cfl, kCflMax);
    if (grid->relax.nmech > 0) {
        // alpha_r: finite, >= 0, and zero within npml + 2 cells of a face
        const int margin = grid->npml > 0 ? grid->npml + 2 : 0;
        e = launch_relax_stats(alpha_r, grid->nx, grid->ny, grid->nz, margin, stats + 8, partial, s);
        double rs[3] = {0, 0, 0};
        if (e == hipSuccess) e = hipMemcpyAsync(rs, stats + 8, sizeof rs, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "relaxation strength statistics");
        if (rs[1] > 0) return fail(EL_EINVAL, "%.0f non-finite alpha_r values", rs[1]);
        if (rs[0] < 0) return fail(EL_EINVAL, "alpha_r must be >= 0 (min %.6g)", rs[0]);
        if (rs[2] > 0)
            return fail(EL_EINVAL, "alpha_r must be 0 within npml + 2 = %d cells of a face (max there %.6g)", margin, rs[2]);
    }

    e = hipEventCreateWithFlags(&p->done, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "event");
    if (grid->precision == EL_F64) {
        bind(p->dd, p);
        bind_relax(p->rd, p);
        e = launch_convert_maps(p->dd, lam, mu, rho, alpha, s);
        if (e == hipSuccess && p->rd.L > 0) e = launch_relax_setup(p->dd, p->tiles, alpha_r, p->rd, s);
        if (e != hipSuccess) return hip_fail(e, "copy maps");
        st = upload_pml(p, p->dd, s);
    } else {
        bind(p->df, p);
        bind_relax(p->rf, p);
        e = launch_convert_maps(p->df, lam, mu, rho, alpha, s);
        if (e == hipSuccess && p->rf.L > 0) e = launch_relax_setup(p->df, p->tiles, alpha_r, p->rf, s);
        if (e != hipSuccess) return hip_fail(e, "copy maps");
        st = upload_pml(p, p->df, s);
    }
    if (st != EL_OK) return st;
    if (grid->relax.nmech > 0 && p->tiles.ntiles > 0) {
        std::vector<unsigned char> rflag(p->tiles.ntiles, 0);
        std::vector<int> rcount(p->tiles.ntiles, 0);
        e = hipMemcpyAsync(rflag.data(), p->ws + L.relax_flag, rflag.size(), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(rcount.data(), p->ws + L.relax_count, rcount.size() * sizeof(int), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "relaxation tiles");
        const Tiles &t = p->tiles;
        // the point list: the points of tile q start at roff[q] (tiles in index order)
        std::vector<long long> roff(t.ntiles, 0);
        long long npts = 0;
        for (int q = 0; q < t.ntiles; ++q) {
            roff[q] = npts;
            if (!rflag[q]) continue;
            const int bx = q % t.ntx, r = q / t.ntx, by = r % t.nty, bz = r / t.nty;
            p->relax_tiles += 1;
            p->relax_points += rcount[q];
            npts += rcount[q];
            p->relax_cells += (long long)std::min(kTileX, grid->nx - bx * kTileX) * std::min(kTileY, grid->ny - by * kTileY) *
                              std::min(t.zc, grid->nz - bz * t.zc);
        }
        // a point keeps its element index in 30 bits
        const long long elements = (long long)(grid->precision == EL_F64 ? p->dd.plane() : p->df.plane()) * (grid->nz + 4);
        if (elements > (long long)kRelaxElemMask + 1)
            return fail(EL_EINVAL, "relaxation needs a padded grid of at most 2^30 elements (%lld)", elements);
        e = hipMemcpyAsync(p->ws + L.relax_off, roff.data(), roff.size() * sizeof(long long), hipMemcpyHostToDevice, s);
        p->rf.npts = p->rd.npts = npts;
        if (e == hipSuccess)
            e = grid->precision == EL_F64 ? launch_relax_compact(p->dd, t, p->rd, s) : launch_relax_compact(p->df, t, p->rf, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "relaxation point list");
    }
    st = upload_receivers(p, rec, s);
    if (st != EL_OK) return st;
    {
        // fluid tiles (el_kernels.hip, k_classify), then the order table
        unsigned char *flags = reinterpret_cast<unsigned char *>(p->ws + L.tile_flags);
        unsigned char *uflags = flags + p->tiles.ntiles;
        unsigned long long *lanes = reinterpret_cast<unsigned long long *>(p->ws + L.tile_lanes);
        void *media = p->ws + L.tile_media;
        e = grid->precision == EL_F64
                ? launch_classify(p->dd, p->tiles, flags, uflags, static_cast<double *>(media), lanes, s)
                : launch_classify(p->df, p->tiles, flags, uflags, static_cast<float *>(media), lanes, s);
        p->med.assign(4 * (size_t)p->tiles.ntiles * (grid->precision == EL_F64 ? 8 : 4), 0);
        if (e == hipSuccess) e = hipMemcpyAsync(p->med.data(), media, p->med.size(), hipMemcpyDeviceToHost, s);
        p->fast.assign(p->tiles.ntiles, 0);
        p->uni.assign(p->tiles.ntiles, 0);
        p->lanes.assign((size_t)2 * kTileY * p->tiles.ntiles, 0);
        std::vector<unsigned long long> &hl = p->lanes;
        if (e == hipSuccess && p->tiles.ntiles > 0)
            e = hipMemcpyAsync(hl.data(), lanes, hl.size() * 8, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess && p->tiles.ntiles > 0)
            e = hipMemcpyAsync(p->fast.data(), flags, p->fast.size(), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess && p->tiles.ntiles > 0)
            e = hipMemcpyAsync(p->uni.data(), uflags, p->uni.size(), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return hip_fail(e, "fluid tiles");
        const Tiles &t = p->tiles;
        const int P = grid->npml;
        const int n[3] = {grid->nx, grid->ny, grid->nz};
        // cells c of [c0, c1) in the layers of an axis of n cells (depth > 0: c < P or c > n-1-P)
        auto in_layers = [P](int c0, int c1, int nn) {
            if (P <= 0) return 0;
            const int lo = std::max(0, std::min(c1, P) - c0);
            const int hi = std::max(0, c1 - std::max(c0, nn - P));
            return lo + hi;
        };
        // the columns of a tile row before column c
        auto below = [](int c) { return c <= 0 ? 0ull : (c >= 64 ? ~0ull : (1ull << c) - 1ull); };
        for (int q = 0; q < t.ntiles; ++q) {
            if (!p->fast[q]) {
                // fluid columns of a general tile: all their cells take the fluid update
                const int bx = q % t.ntx, r = q / t.ntx, by = r % t.nty, bz = r / t.nty;
                const int z0 = bz * t.zc, dep = std::min(t.zc, n[2] - z0);
                for (int row = 0; row < kTileY; ++row) {
                    const unsigned long long m = hl[(size_t)kTileY * q + row];
                    if (!m) continue;
                    const unsigned long long um = hl[(size_t)kTileY * ((size_t)t.ntiles + q) + row];
                    p->uniform_cells += (long long)__builtin_popcountll(um) * dep;
                    const int x0 = bx * kTileX, j = by * kTileY + row;
                    const long long cols = __builtin_popcountll(m);
                    const long long xcols = P <= 0 ? 0
                                                   : __builtin_popcountll(m & below(P - x0)) +
                                                         __builtin_popcountll(m & ~below(n[0] - P - x0));
                    p->column_cells += cols * dep;
                    p->fast_layer_cells += (xcols + cols * in_layers(j, j + 1, n[1])) * dep + cols * in_layers(z0, z0 + dep, n[2]);
                }
                continue;
            }
            const int bx = q % t.ntx, r = q / t.ntx, by = r % t.nty, bz = r / t.nty;
            const int c0[3] = {bx * kTileX, by * kTileY, bz * t.zc};
            const int w[3] = {std::min(kTileX, n[0] - c0[0]), std::min(kTileY, n[1] - c0[1]), std::min(t.zc, n[2] - c0[2])};
            p->fast_tiles += 1;
            p->fast_cells += (long long)w[0] * w[1] * w[2];
            if (p->uni[q]) p->uniform_cells += (long long)w[0] * w[1] * w[2];
            for (int a = 0; a < 3; ++a)
                p->fast_layer_cells += (long long)in_layers(c0[a], c0[a] + w[a], n[a]) * w[(a + 1) % 3] * w[(a + 2) % 3];
            // s22 (s33) is stored only on two-cell bands along y (z) faces next to general tiles
            const int edges = (int)tile_edges(t, p->fast.data(), q);
            for (int a = 1; a < 3; ++a) {
                const int lo = (edges >> (2 * (a - 1))) & 1, hi = (edges >> (2 * (a - 1) + 1)) & 1;
                p->fast_skipped += (long long)std::max(0, w[a] - 2 * lo - 2 * hi) * w[(a + 1) % 3] * w[(a + 2) % 3];
            }
        }
        st = set_tables(p, true, s);
        if (st != EL_OK) return st;
    }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "plan set-up");
    e = hipEventRecord(p->done, s);
    if (e != hipSuccess) return hip_fail(e, "event");
    *out = own.release();
    return EL_OK;
} EL_CATCH

el_status el_plan_destroy(el_plan p) {
    if (!p) return EL_OK;
    if (p->done) (void)hipEventDestroy(p->done);
    for (auto &v : p->ev)
        for (auto &pr : v) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
    delete p;
    return EL_OK;
}

el_status el_plan_timing(el_plan p, int32_t every) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    if (every < 0) return fail(EL_EINVAL, "every must be >= 0");
    p->timing_every = every;
    return EL_OK;
}

el_status el_plan_kernel_time(el_plan p, int32_t kind, int64_t *launches, double *total_ms) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    if (kind < 0 || kind >= EL_K_COUNT) return fail(EL_EINVAL, "kernel kind %d outside 0..%d", kind, EL_K_COUNT - 1);
    double ms = 0.0;
    const size_t n = p->used[kind];
    for (size_t q = 0; q < n; ++q) {
        auto &pr = p->ev[kind][q];
        HIP_TRY(hipEventSynchronize(pr.second), "wait for timing event");
        float t = 0.f;
        HIP_TRY(hipEventElapsedTime(&t, pr.first, pr.second), "elapsed time");
        ms += t;
    }
    p->used[kind] = 0;
    if (launches) *launches = (int64_t)n;
    if (total_ms) *total_ms = ms;
    return EL_OK;
}

el_status el_forward(el_plan p, const void *p0, double *traces, void *stream) try {
    el_status st = check_plan(p);
    if (st != EL_OK) return st;
    if (!p0 || (!traces && p->nrec > 0)) return fail(EL_EINVAL, "p0 or traces is NULL");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamWaitEvent(s, p->done, 0), "order after the previous operation");
    st = p->g.precision == EL_F64 ? run_forward(p, p->dd, static_cast<const double *>(p0), traces, s)
                                  : run_forward(p, p->df, static_cast<const float *>(p0), traces, s);
    if (st != EL_OK) return st;
    HIP_TRY(hipEventRecord(p->done, s), "record completion");
    return EL_OK;
} EL_CATCH

el_status el_forward_energy(el_plan p, const void *p0, double *traces, int32_t every, double *energy, void *stream) try {
    el_status st = check_plan(p);
    if (st != EL_OK) return st;
    if (!p0 || (!traces && p->nrec > 0)) return fail(EL_EINVAL, "p0 or traces is NULL");
    if (every < 1) return fail(EL_EINVAL, "every must be >= 1");
    if (!energy && p->g.nsteps > 1) return fail(EL_EINVAL, "energy is NULL");
    if (p->g.relax.nmech > 0)
        return fail(EL_EINVAL, "the modified energy is not defined with relaxation mechanisms (their memory variables "
                               "hold energy it does not count)");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamWaitEvent(s, p->done, 0), "order after the previous operation");
    st = p->g.precision == EL_F64
             ? run_forward(p, p->dd, static_cast<const double *>(p0), traces, s, every, energy)
             : run_forward(p, p->df, static_cast<const float *>(p0), traces, s, every, energy);
    if (st != EL_OK) return st;
    HIP_TRY(hipEventRecord(p->done, s), "record completion");
    return EL_OK;
} EL_CATCH

el_status el_adjoint(el_plan p, const double *y, void *p_adj, void *stream) try {
    el_status st = check_plan(p);
    if (st != EL_OK) return st;
    if ((!y && p->nrec > 0) || !p_adj) return fail(EL_EINVAL, "y or p_adj is NULL");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamWaitEvent(s, p->done, 0), "order after the previous operation");
    st = p->g.precision == EL_F64 ? run_adjoint(p, p->dd, y, static_cast<double *>(p_adj), s)
                                  : run_adjoint(p, p->df, y, static_cast<float *>(p_adj), s);
    if (st != EL_OK) return st;
    HIP_TRY(hipEventRecord(p->done, s), "record completion");
    return EL_OK;
} EL_CATCH

el_status el_eir_apply(const double *h, int32_t nh, const double *in, double *out, int32_t nsteps, int32_t nrec,
                       int32_t transpose, void *stream) {
    if (!h || !in || !out) return fail(EL_EINVAL, "h, in or out is NULL");
    if (nh < 1) return fail(EL_EINVAL, "nh must be >= 1");
    if (nsteps < 1 || nrec < 0) return fail(EL_EINVAL, "nsteps must be >= 1 and nrec >= 0");
    if (transpose != 0 && transpose != 1) return fail(EL_EINVAL, "transpose must be 0 or 1");
    const char *a0 = reinterpret_cast<const char *>(in), *b0 = reinterpret_cast<const char *>(out);
    const size_t bytes = (size_t)nsteps * nrec * sizeof(double);
    if (bytes > 0 && a0 < b0 + bytes && b0 < a0 + bytes) return fail(EL_EINVAL, "in and out overlap");
    if ((size_t)nsteps * (size_t)nrec > (size_t)INT32_MAX * 64) return fail(EL_EINVAL, "traces too large");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    HIP_TRY(launch_eir(h, nh, in, out, nsteps, nrec, transpose, s), "transducer response");
    return EL_OK;
}

el_status el_dot_f64(el_plan p, int32_t space, const void *a, const void *b, double *out, void *stream) {
    el_status st = check_plan(p);
    if (st != EL_OK) return st;
    if (!a || !b || !out) return fail(EL_EINVAL, "a, b or out is NULL");
    if (space != 0 && space != 1) return fail(EL_EINVAL, "space must be 0 (N) or 1 (LM)");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    HIP_TRY(hipStreamWaitEvent(s, p->done, 0), "order after the previous operation");
    double *partial = reinterpret_cast<double *>(p->ws + p->L.partial);
    hipError_t e;
    if (space == 1)
        e = launch_dot(static_cast<const double *>(a), static_cast<const double *>(b),
                       (long long)p->g.nsteps * p->nrec, partial, out, s);
    else if (p->g.precision == EL_F64)
        e = launch_dot(static_cast<const double *>(a), static_cast<const double *>(b), p->N, partial, out, s);
    else
        e = launch_dot(static_cast<const float *>(a), static_cast<const float *>(b), p->N, partial, out, s);
    if (e != hipSuccess) return hip_fail(e, "dot");
    HIP_TRY(hipEventRecord(p->done, s), "record completion");
    return EL_OK;
}

el_status el_plan_field(el_plan p, int32_t id, void **ptr, size_t *count) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    if (id < 0 || id >= NFIELD) return fail(EL_EINVAL, "field id %d outside 0..8", id);
    if (!ptr || !count) return fail(EL_EINVAL, "ptr or count is NULL");
    *ptr = p->ws + p->L.vol[id];
    *count = (size_t)make_vol(p->g.nx, p->g.ny, p->g.nz).total;
    return EL_OK;
}

el_status el_plan_layout(el_plan p, int64_t *row_pitch, int64_t *plane_pitch, int64_t *origin) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    const Vol v = make_vol(p->g.nx, p->g.ny, p->g.nz);
    if (row_pitch) *row_pitch = v.px;
    if (plane_pitch) *plane_pitch = v.plane;
    if (origin) *origin = v.origin;
    return EL_OK;
}

el_status el_plan_fluid_path(el_plan p, int32_t enable, el_fluid_stats *stats) try {
    el_status st = check_plan(p);
    if (st != EL_OK) return st;
    if (enable != -1 && enable != 0 && enable != 1) return fail(EL_EINVAL, "enable must be -1, 0 or 1");
    if (enable >= 0 && (enable != 0) != p->fluid_path) {
        HIP_TRY(hipEventSynchronize(p->done), "wait for the plan's previous operation");
        st = set_tables(p, enable != 0, nullptr);
        if (st != EL_OK) return st;
    }
    if (stats) {
        *stats = el_fluid_stats{};
        if (p->fluid_path) {
            stats->tiles = p->fast_tiles;
            stats->cells = p->fast_cells + p->column_cells;
            stats->column_cells = p->column_cells;
            stats->layer_cells = p->fast_layer_cells;
            stats->skipped_stores = p->fast_skipped;
            stats->uniform_cells = p->uniform_cells;
        }
    }
    return EL_OK;
} EL_CATCH

el_status el_plan_relaxation(el_plan p, int64_t *tiles, int64_t *cells, int64_t *points) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    if (tiles) *tiles = p->relax_tiles;
    if (cells) *cells = p->relax_cells;
    if (points) *points = p->relax_points;
    return EL_OK;
}

el_status el_plan_sizes(el_plan p, int64_t *ncells, int32_t *nrec, int32_t *nsteps) {
    if (!p) return fail(EL_EINVAL, "plan is NULL");
    if (ncells) *ncells = p->N;
    if (nrec) *nrec = p->nrec;
    if (nsteps) *nsteps = p->g.nsteps;
    return EL_OK;
}

}  // extern "C"
