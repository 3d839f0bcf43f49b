// Checks of the stencil passes' block list on the host, called from test_block_list.py: the list is
// made by the library's own block_list() from media classified here cell by cell, and walked as the
// kernels walk it.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <string>

#include "el_impl.h"

using namespace el;

namespace el {
int block_planes(const Tiles &t, int nx, int ny, int P, const unsigned char *fast, const unsigned char *uni,
                 const unsigned long long *lanes, long long *touched);
}

namespace {

std::string g_msg;
int bad(const char *what, int a = 0, int b = 0, int c = 0) {
    char buf[200];
    snprintf(buf, sizeof buf, "%s (%d, %d, %d)", what, a, b, c);
    g_msg = buf;
    return 1;
}

struct Grid3 {
    int nx, ny, nz;
    const unsigned char *solid, *medium;   // cell maps, x fastest
    size_t at(int i, int j, int k) const { return ((size_t)k * ny + j) * nx + i; }
    // cells within two of column (i, j), planes [z0, z1), clipped to the grid
    template <typename F>
    bool all(int i0, int i1, int j0, int j1, int z0, int z1, F f) const {
        for (int k = std::max(z0 - 2, 0); k < std::min(z1 + 2, nz); ++k)
            for (int j = std::max(j0 - 2, 0); j < std::min(j1 + 2, ny); ++j)
                for (int i = std::max(i0 - 2, 0); i < std::min(i1 + 2, nx); ++i)
                    if (!f(at(i, j, k))) return false;
        return true;
    }
};

}  // namespace

extern "C" {

const char *check_message() { return g_msg.c_str(); }

// out: planes per block, entries per XCD, room per XCD, general sub-tiles' share in per mille, whether
// the passes stream, elements that a step touches in thousands.
// room > 0 replaces the room per XCD; then 2 is returned if the list does not fit it.
int check_blocks(int nx, int ny, int nz, int npml, const unsigned char *solid, const unsigned char *medium, int fluid,
                 const int *points, int npoints, int nrec, int room, int *out) {
    const Grid3 g{nx, ny, nz, solid, medium};
    Tiles t = make_tiles(nx, ny, nz);
    if (room > 0) t.cap = room;
    std::vector<unsigned char> fast(t.ntiles, 0), uni(t.ntiles, 0);
    std::vector<unsigned long long> lanes((size_t)2 * kTileY * t.ntiles, 0);
    std::vector<float> med((size_t)4 * t.ntiles, 0.f);
    for (int q = 0; q < t.ntiles; ++q) {
        const int bx = q % t.ntx, by = q / t.ntx % t.nty, bz = q / t.ntx / t.nty;
        const int x0 = bx * kTileX, y0 = by * kTileY, z0 = bz * t.zc;
        const int x1 = std::min(x0 + kTileX, nx), y1 = std::min(y0 + kTileY, ny), z1 = std::min(z0 + t.zc, nz);
        auto liquid = [&](size_t e) { return !solid[e]; };
        fast[q] = g.all(x0, x1, y0, y1, z0, z1, liquid);
        unsigned char ref = medium[g.at(std::max(x0 - 2, 0), std::max(y0 - 2, 0), std::max(z0 - 2, 0))];
        auto same = [&](size_t e) { return medium[e] == ref; };
        uni[q] = fast[q] && g.all(x0, x1, y0, y1, z0, z1, same);
        bool found = fast[q];
        for (int r = 0; r < kTileY && y0 + r < ny; ++r)
            for (int c = 0; x0 + c < x1; ++c) {
                if (!g.all(x0 + c, x0 + c + 1, y0 + r, y0 + r + 1, z0, z1, liquid)) continue;
                if (!found) ref = medium[g.at(x0 + c, y0 + r, z0)];
                found = true;
                lanes[(size_t)kTileY * q + r] |= 1ull << c;
                if (g.all(x0 + c, x0 + c + 1, y0 + r, y0 + r + 1, z0, z1, same))
                    lanes[(size_t)kTileY * (t.ntiles + q) + r] |= 1ull << c;
            }
        med[4 * (size_t)q] = ref;
    }
    const unsigned char *f = fluid ? fast.data() : nullptr;
    const std::vector<int> pts(points, points + 3 * (size_t)npoints);
    long long touched = 0;
    out[0] = block_planes(t, nx, ny, npml, f, uni.data(), lanes.data(), &touched);
    const BlockList<float> list = block_list<float>(t, nx, ny, npml, f, uni.data(), lanes.data(), med.data(), pts);
    out[2] = t.cap;
    if (!list.fits) return 2;
    out[1] = list.per;
    if (list.per > t.cap) return bad("more entries than room", list.per, t.cap);
    el_grid gr{};
    gr.nx = nx;
    gr.ny = ny;
    gr.nz = nz;
    gr.dx = 1;
    gr.dt = 1;
    gr.nsteps = 2;
    gr.npml = npml;
    Layout L;
    layout(gr, nrec, &L);
    if (list.planes > L.inc_planes) return bad("more increment planes than room", (int)list.planes, (int)L.inc_planes);

    // planes of every sub-tile: covered once, by the update its columns ask for
    const size_t cols = (size_t)t.ntx * t.nty;
    std::vector<unsigned char> seen(cols * 4 * nz, 0), put33(cols * nz, 0);
    std::vector<int> where(cols * 4 * nz, -1);   // the plane's increments (64 elements each), -1: none
    long long general = 0, subs = 0;
    for (int e = 0; e < 8 * list.per; ++e) {
        const BlockEnt<float> &b = list.entries[e];
        if (!b.flags) continue;
        if (b.z0 < 0 || b.z1 > nz || b.z0 >= b.z1) return bad("planes of an entry", b.z0, b.z1, nz);
        const bool gen = (b.flags & kBlkGen) != 0;
        const unsigned mask = gen ? 1u << (b.flags >> kBlkSubShift & 3) : b.flags >> kBlkMaskShift & 15;
        const unsigned unis = b.flags >> kBlkUniShift & 15, with = b.flags >> kBlkIncShift & 15;
        const size_t col = (size_t)b.by * t.ntx + b.bx;
        for (int k = b.z0; k < b.z1; ++k) {
            const int q = (k / t.zc) * (int)cols + (int)col;
            const bool tile = f && f[q];
            if (tile != ((b.flags & kBlkFast) != 0)) return bad("kind of a tile", b.bx, b.by, k);
            if (tile && ((b.flags >> kBlkEdgeShift ^ tile_edges(t, f, q)) & 3)) return bad("y faces", b.bx, b.by, k);
            if (!gen) {
                const unsigned ed = b.flags >> kBlkEdgeShift;
                const bool keep = (b.flags & kBlkKeep) != 0;
                put33[col * nz + k] |= keep || ((ed & 4) && k < b.z0 + 2) || ((ed & 8) && k >= b.z1 - 2);
            }
            for (int s = 0; s < 4; ++s) {
                if (!(mask >> s & 1)) continue;
                if (seen[(col * 4 + s) * nz + k]++) return bad("covered twice", b.bx, b.by, k);
                const int before = __builtin_popcount(with & ((1u << s) - 1));
                where[(col * 4 + s) * nz + k] = with >> s & 1 ? b.slot + before * (b.z1 - b.z0) + k - b.z0 : -1;
                general += gen;
                ++subs;
                bool all = true, same = true;
                const int x0 = b.bx * kTileX + (s & 1) * kWaveX, y0 = b.by * kTileY + (s >> 1) * kWaveY;
                for (int r = 0; r < kWaveY && y0 + r < ny; ++r) {
                    const unsigned valid = nx - x0 >= kWaveX ? ~0u : (1u << (nx - x0)) - 1;
                    const size_t row = (size_t)kTileY * q + (s >> 1) * kWaveY + r;
                    const unsigned fl = f && !tile ? (unsigned)(lanes[row] >> (s & 1) * kWaveX) & valid : 0;
                    const unsigned ul = f && !tile ? (unsigned)(lanes[(size_t)kTileY * t.ntiles + row] >> (s & 1) * kWaveX) & valid : 0;
                    if (gen && (b.fluid[r] != fl || b.uniform[r] != ul)) return bad("columns", b.bx, b.by, k);
                    if (gen && ul && b.lam != med[4 * (size_t)q]) return bad("reference medium", b.bx, b.by, k);
                    all = all && fl == valid;
                    same = same && ul == valid;
                }
                const bool u = unis >> s & 1;
                if (!gen && !(tile || all)) return bad("fluid update of a sub-tile that is not", b.bx, b.by, k);
                if (gen && all) return bad("general update of a fluid sub-tile", b.bx, b.by, k);
                if (!gen && u != (tile ? uni[q] != 0 : same)) return bad("uniform media", b.bx, b.by, k);
                if (!gen && u && b.lam != med[4 * (size_t)q]) return bad("medium", b.bx, b.by, k);
                if (!gen && !tile && !(b.flags & kBlkKeep)) return bad("stores of a fluid sub-tile", b.bx, b.by, k);
            }
        }
    }
    for (size_t col = 0; col < cols; ++col)
        for (int s = 0; s < 4; ++s) {
            const bool in = (int)(col % t.ntx) * kTileX + (s & 1) * kWaveX < nx && (int)(col / t.ntx) * kTileY + (s >> 1) * kWaveY < ny;
            for (int k = 0; k < nz; ++k)
                if ((seen[(col * 4 + s) * nz + k] != 0) != in) return bad("not covered", (int)col, s, k);
        }
    // s33 on the planes of fluid tiles that a general tile's taps reach
    if (f)
        for (size_t col = 0; col < cols; ++col)
            for (int k = 0; k < nz; ++k) {
                if (!fast[(size_t)(k / t.zc) * cols + col]) continue;
                bool read = false;
                for (int m = std::max(k - 2, 0); m <= std::min(k + 2, nz - 1); ++m) read = read || !fast[(size_t)(m / t.zc) * cols + col];
                if (read && !put33[col * nz + k]) return bad("s33 not stored", (int)col, 0, k);
            }
    // every point's increment lies where its cell's stress update reads it, and nowhere else
    std::vector<int> pos = list.pos;
    if ((int)pos.size() != npoints) return bad("points");
    for (int p = 0; p < npoints; ++p) {
        const int i = points[3 * p], j = points[3 * p + 1], k = points[3 * p + 2];
        const size_t col = (size_t)(j / kTileY) * t.ntx + i / kTileX;
        const int s = 2 * (j % kTileY / kWaveY) + i % kTileX / kWaveX;
        const int plane = where[(col * 4 + s) * nz + k];
        if (plane < 0 || plane >= list.planes) return bad("no increments at a point", i, j, k);
        if (pos[p] != plane * 64 + (j % kWaveY) * kWaveX + i % kWaveX) return bad("increment of a point", i, j, k);
    }
    std::sort(pos.begin(), pos.end());
    if (std::adjacent_find(pos.begin(), pos.end()) != pos.end()) return bad("two points share an increment");
    std::vector<int> planes;
    for (int w : where)
        if (w >= 0) planes.push_back(w);
    std::sort(planes.begin(), planes.end());
    if (std::adjacent_find(planes.begin(), planes.end()) != planes.end()) return bad("two planes share increments");
    out[4] = list.once;
    out[5] = (int)(touched / 1000);
    out[3] = subs ? (int)(1000 * general / subs) : 0;
    return 0;
}

}  // extern "C"
