// Stencil passes of the forward operator H and of its adjoint H^T (gfx950).
//
// One time step is two passes.  Both operators use the same two shapes:
//
//  velocity-shaped  out^c = J_c out^c + k_c sum_a D_a[In_ca]          (c = component, a = axis)
//  stress-shaped    out   = out + C Eps[In]                          (C = Voigt stiffness)
//
// Forward (Appendix, Discrete formulation; Sec. 2.2 eq. it):
//   velocity: In_ca = sigma^{ca}, k_c = dt / rho_c; the C-PML memory variable
//             phi^{ca} <- b_a phi^{ca} + a_a D_a sigma^{ca} is formed at the output
//             point and added to the sum.
//   stress:   In_ca = u^c, C scaled by dt; psi^{ca} <- b_a psi^{ca} + a_a D_a u^c
//             is added to each strain term.
// Adjoint, in the variables r = Q^{-1} q (velocity adjoint over the staggered
// density) and w = C s (stiffness times stress adjoint).  One adjoint step
// applies the transposes of the four forward sub-updates in reverse order,
// with the diagonal factors J, B, B~ of each step deferred to the next one:
//   velocity: In_ca = dt w_(ca) + a_a psi~^{ca}, k_c = -1 / rho_c, then
//             phi~^{ca} <- b_a phi~^{ca} + dt chi_a r^c at the output point;
//   stress:   In_ca = dt r^c + a_a phi~^{ca}, C scaled by -1, then
//             psi~^{ca} <- b_a psi~^{ca} + dt w_(ca) at the output point.
// The adjoint stores its memory variables multiplied by the layer coefficient,
// g = a psi~ and g = a phi~ (b and a are diagonal, so g <- b g + a dt w).
// These follow from Psi^T = -dt Div C, Phi^T = -dt Eps Q^{-1} and the
// zero-extended identity Dp^T = -Dm between the two difference types.  The
// difference of In is evaluated as dt D[w] (or dt D[r]) plus, only where a
// tap reaches a C-PML slab of that axis, D[g] on the extended slab planes.
//
// Tiling: tiles of 64 x 4 columns and a few planes, each four sub-tiles of 32 x 2 columns, one
// wavefront wide; a wavefront marches along z through its sub-tile's planes.  Inputs
// differentiated along z sit in four-deep register queues; taps along x and y are read from
// memory, where the neighbouring wavefronts and tiles keep them in L1/L2.  There is no LDS and
// no barrier.  The padded volume layout (see el_impl.h) makes every tap a plain load: addresses
// are a 32-bit byte offset, shared by all fields, from the field's base address.  What a block
// does stands in a list (block_list, on the host) that gives every XCD (block id mod 8)
// contiguous regions of tile columns' pieces spread over the volume, so every XCD holds the same share of the
// C-PML layers and a region's neighbouring tiles share one L2.
//
// Fluid sub-tiles: where mu = 0 on the columns and within two cells of them (k_classify),
// s22 = s33 = s11 and the shear stresses are zero on every tap, so both passes run a lean loop
// that differences s11 alone and carries only the diagonal memory variables, a wavefront per
// sub-tile.  s22 and s33 are read only by the general loops, which difference s22 along y and
// s33 along z with taps reaching two cells into a neighbouring tile, so a fluid tile stores s22
// only on two-row bands along y faces and s33 only on two-plane bands along z faces shared with
// tiles that are not fluid, s11 everywhere; k_fluid_fill restores s22 = s33 = s11 on fluid tiles
// at the end of an operation.  Fluid sub-tiles of uniform media take lambda, rho and alpha from
// the block's list entry.
//
// General sub-tiles: a wavefront per velocity component, and per kind of stress (the normal
// stresses, each shear stress).  The components share no arithmetic and few taps, so the split
// costs few loads; it leaves each wavefront 40 to 70 registers instead of 96 (7 or 8 wavefronts
// per SIMD instead of 5) and one batch of loads per plane, memory variables and adjoint taps
// included, where one wavefront for all of them had to load each layer axis after the other.
// On grids that leave the device a few wavefronts per SIMD that chain was the time; on larger
// ones the wavefronts in flight were.  Fluid lanes of a mixed sub-tile mask off the loads they do
// not need.  The results are those of the general loops.
//
// What the time went to on a small grid was seen from the clock at each wavefront's start, first
// load and end: chains of scalar loads (an address per array from the kernel arguments, the list
// entry, the tile's masks and medium), each waiting for the one before, took as long as the
// planes.  So the arrays' addresses are formed from one base and a few strides (Dev), an entry is
// one 64-byte line, and the layer coefficients are loaded without a branch.  A wavefront's
// scalar registers limit how many fit, too: at most 80 for 8 per SIMD, 96 for 7.
//
// Measured (MI355X, us per forward and adjoint step together, with a wavefront per sub-tile and now;
// "adjoint": that step alone): skull medium 64^3 42.1 to 27.7, 96^3 adjoint 41.9 to 29.6, 128^3
// 101.9 to 89.4, 128^3 in double precision 197 to 169, 256^3 636 to 540, 384^3 1640 to 1583;
// all solid 157 x 131 x 109 141 to 137, 203 x 187 x 150 549 to 442, 256^3 1188 to 1132, 320^3 2106 to
// 2086, 384^3 3474 to 3471 (without layers 2953 to 3039).  On the largest grids the split itself
// loses: a sub-tile's halo is no longer shared in L1 with the tile's other sub-tiles, the passes ask
// L2 for 10 to 13% more lines (384^3, TCC_REQ) and the lines in flight bound them.  Blocks of two or
// four sub-tiles share the halo and lose more, waiting for 8 or 16 free wavefronts (384^3 solid
// 1801/1911 to 1882/2064 and 2076/2557 us); ld_own makes up for it.
#include "el_impl.h"

namespace el {

constexpr int TX = kTileX;
constexpr int TY = kTileY;
constexpr int NT = TX * TY;

template <typename T>
__device__ __forceinline__ T ldb(const T *base, unsigned off) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}
template <typename T>
__device__ __forceinline__ void stb(T *base, unsigned off, T v) {
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + off) = v;
}

// Cells of a wavefront: kWaveX columns of kWaveY rows (32 x 2), one 128-byte line of each of
// two rows per load, as coalesced as a 64 x 1 row, while a wavefront that meets a solid region
// holds half as many fluid columns that must run the general update with it (the shell of the
// skull medium crosses most 64-wide rows of the tiles it touches).
static_assert(TX == 2 * kWaveX && TY == 2 * kWaveY && kWaveX * kWaveY == 64, "a tile is four sub-tiles of one wavefront");

// p as an address of memory no kernel in flight writes: uniform loads from it are scalar ones.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *constant(const T *p) {
    return (const __attribute__((address_space(4))) T *)(unsigned long long)p;
}
// This block's list entry: its first cell, its planes, and the rest of BlockEnt.
template <typename T>
struct Block {
    int x0, y0, z0, z1, slot;
    unsigned fl, fluid[2], uniform[2];
    T lam, rho, alpha;
};
template <typename T>
__device__ __forceinline__ bool block_of(const Tiles &tl, Block<T> &b, int bid) {
    const auto *e = constant(static_cast<const BlockEnt<T> *>(tl.order)) + bid;
    b.x0 = e->bx * TX;
    b.y0 = e->by * TY;
    b.z0 = e->z0;
    b.z1 = e->z1;
    b.fl = e->flags;
    b.slot = e->slot;
#pragma unroll
    for (int r = 0; r < kWaveY; ++r) {
        b.fluid[r] = e->fluid[r];
        b.uniform[r] = e->uniform[r];
    }
    b.lam = e->lam;
    b.rho = e->rho;
    b.alpha = e->alpha;
    return b.fl != 0;
}
// Wavefront number within the block, as a scalar.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
// Column and row within the tile of this thread's cell in sub-tile sub.
__device__ __forceinline__ int sub_col(int sub) { return (sub & 1) * kWaveX + ((int)threadIdx.x & (kWaveX - 1)); }
__device__ __forceinline__ int sub_row(int sub) { return (sub >> 1) * kWaveY + (((int)threadIdx.x & 63) / kWaveX); }

// Lanes of a general sub-tile with fluid columns.  fl: this lane's column is fluid; ul: its
// lambda, rho and alpha are the tile's reference medium (in the per-tile table).
template <typename T>
__device__ __forceinline__ void fluid_lanes(const Block<T> &b, bool &fl, bool &ul) {
    const unsigned lane = threadIdx.x & 63u, col = lane & (kWaveX - 1);
    fl = (((lane < kWaveX ? b.fluid[0] : b.fluid[1]) >> col) & 1u) != 0;
    ul = (((lane < kWaveX ? b.uniform[0] : b.uniform[1]) >> col) & 1u) != 0;
}

// Reciprocal: the hardware v_rcp_f32 (within 1 ulp) in single precision, the correctly
// rounded quotient in double precision.  Both give +inf for +0 and 0 for +inf.
template <typename T>
__device__ __forceinline__ T rcp(T x);
template <>
__device__ __forceinline__ float rcp<float>(float x) {
    return __builtin_amdgcn_rcpf(x);
}
template <>
__device__ __forceinline__ double rcp<double>(double x) {
    return 1.0 / x;
}

// Harmonic mean of four non-negative moduli given their reciprocals (Sec. 2.2: the shear
// modulus at an edge point); zero when any modulus is zero, whose reciprocal is +inf.
template <typename T>
__device__ __forceinline__ T harmonic4r(T r0, T r1, T r2, T r3) {
    return T(4) * rcp(r0 + r1 + r2 + r3);
}

// The updates below say themselves which products are fused into an addition (fma), and nothing
// else is: a cell's value is the same to the last bit whichever wavefront, block or precision
// variant computes it, and stays so when a loop is split in another way.
#pragma clang fp contract(off)

// Each plane of a column is processed as: every load of the plane (taps, old values, media,
// memory variables), one scheduling fence (so they are in flight together: one memory round
// trip per plane), the arithmetic and the stores.

// An array's address, kept in scalar registers for the whole column (left to itself the
// compiler forms it again on every plane).
template <typename T> using Arr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ Arr<T> held(T *p) {
    Arr<T> a = (Arr<T>)p;
    asm("" : "+s"(a));
    return a;
}
// Load and store at a lane's byte offset, and a load at a constant distance from it (an
// immediate of the load).
template <typename T>
__device__ __forceinline__ T ldb(Arr<T> base, unsigned off) {
    return *(Arr<T>)((Arr<char>)base + off);
}
template <typename T>
__device__ __forceinline__ void stb(Arr<T> base, unsigned off, T v) {
    *(Arr<T>)((Arr<char>)base + off) = v;
}
template <typename T>
__device__ __forceinline__ T ldi(Arr<T> base, unsigned off, int elements) {
    return *((Arr<T>)((Arr<char>)base + off) + elements);
}
// The same for an old and a new value of a field, which one lane reads and writes and no other reads
// in this pass.  ONCE: with a hint that it need not stay in the caches, so that it does not take the
// place of taps there.
//
// Where the state outgrows the Infinity Cache that is what the general update gains from: with
// several wavefronts per sub-tile its taps ask L2 for 10 to 13% more lines than one wavefront for all
// of a sub-tile did, and L1 holds fewer of them.  Where the state fits the next pass reads the value
// from that cache, and the hint costs more than it gives.  Measured (us per forward / adjoint step,
// without and with it): all solid 128^3 66.9/74.3 and 81.3/86.9, 152^3 118/134 and 127/141, 160^3
// 156/166 and 150/160, 192^3 262/286 and 251/268, 320^3 1066/1136 and 1038/1109, 384^3 1801/1911 and
// 1753/1865; a thin shell in water 160^3 64/66 and 77/81, 192^3 110/120 and 118/123, 208^3 157/171
// and 152/159, 256^3 278/290 and 266/283; in double precision solid 112^3 95/112 and 130/146, 128^3
// 181/207 and 178/198, shell 144^3 100/116 and 123/137, 160^3 162/185 and 166/180.  See
// kStreamBytes for the line.
template <typename T, bool ONCE>
__device__ __forceinline__ T ld_own(Arr<T> base, unsigned off) {
    Arr<T> a = (Arr<T>)((Arr<char>)base + off);
    return ONCE ? __builtin_nontemporal_load(a) : *a;
}
template <typename T, bool ONCE>
__device__ __forceinline__ void st_own(Arr<T> base, unsigned off, T v) {
    Arr<T> a = (Arr<T>)((Arr<char>)base + off);
    if (ONCE) __builtin_nontemporal_store(v, a);
    else *a = v;
}
// The four samples from t0 to t0 + 3 cells along axis A.
template <typename T, int A>
__device__ __forceinline__ void taps(Arr<T> f, unsigned o, int t0, unsigned st, T (&v)[4]) {
#pragma unroll
    for (int n = 0; n < 4; ++n) v[n] = A == 0 ? ldi<T>(f, o, t0 + n) : ldb<T>(f, o + (unsigned)(t0 + n) * st);
}
// 4th-order staggered difference (Sec. 2.2, eq. derivative) from consecutive samples: Dp, the
// value at i + 1/2, from i-1 .. i+2; Dm, the value at i, from i-2 .. i+1.  Without the 1/dx.
template <typename T>
__device__ __forceinline__ T diff4(const T (&v)[4]) {
    return fma(v[2] - v[1], T(9) / T(8), T(-1) / T(24) * (v[3] - v[0]));
}
// Adjoint: a main difference (times dt) plus, where a tap reaches a layer, that of the memory
// variable.
template <typename T>
__device__ __forceinline__ T add_near(bool on, T d, const T (&near)[4], T h) {
    return on ? fma(diff4(near), h, d) : d;
}
// Voigt field of sigma^{ca}.
__host__ __device__ constexpr int sig(int c, int a) {
    return c == a ? S11 + c : (c + a == 3 ? S23 : (c + a == 2 ? S13 : S12));
}
// f(std::integral_constant<int, A>) for A = 0, 1, 2.
template <typename F>
__device__ __forceinline__ void axes(F f) {
    f(std::integral_constant<int, 0>());
    f(std::integral_constant<int, 1>());
    f(std::integral_constant<int, 2>());
}

// Where a column lies in the C-PML slabs: the byte offset of the cell's slab point in the x and y
// slab arrays at the current plane, its offset within a plane of the z slab arrays, and whether
// the cell has a value there (own) or taps that reach a layer (near, adjoint); along z the same of
// the current plane.
template <typename T, bool ADJ>
struct Slab {
    bool own[3], near[3];
    unsigned off[2], zoff;
    int sz;                  // slab coordinate of the current plane
    unsigned step[2];        // x and y: to the next plane
    unsigned st[3];          // between slab coordinates
    int P, hiz, highz;
    // onx, ony: this lane takes part along x (y); along z it is the caller's to say
    __device__ __forceinline__ Slab(const Dev<T> &d, int i, int j, int z0, bool onx, bool ony) {
        P = d.P;
        hiz = d.hi(2);
        highz = d.high[2];
        const int cell[2] = {i, j};
        st[0] = sizeof(T);
        st[1] = st[0] * (unsigned)d.nx;
        st[2] = st[1] * (unsigned)d.ny;
        step[0] = st[0] * (unsigned)d.ny * (unsigned)d.xw;
        step[1] = st[1] * (unsigned)d.W();
        zoff = ((unsigned)j * (unsigned)d.nx + (unsigned)i) * st[0];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const int c = cell[a], h = d.hi(a);
            const bool on = a == 0 ? onx : ony;
            own[a] = on && in_layer(c, P, h);
            near[a] = on && near_layer(c, P, h);
            off[a] = slab_byte(d, a, slab_coord(c, P, d.high[a]), i, j, z0);
        }
        plane(z0);
    }
    __device__ __forceinline__ void plane(int k) {
        own[2] = in_layer(k, P, hiz);
        near[2] = near_layer(k, P, hiz);
        sz = slab_coord(k, P, highz);
    }
    __device__ __forceinline__ void next(int k) {
        off[0] += step[0];
        off[1] += step[1];
        plane(k);
    }
    // own value of m along axis A, into v (left as it is where the cell has none, or off; on: along z)
    template <int A>
    __device__ __forceinline__ void ld(Arr<T> m, bool on, T &v) const {
        if (A == 2) {
            if (own[2] && on) v = ldb<T>(m, zoff + (unsigned)sz * st[2]);
        } else if (own[A]) {
            v = ldb<T>(m, off[A]);
        }
    }
    template <int A>
    __device__ __forceinline__ void put(Arr<T> m, T v) const {
        stb<T>(m, A == 2 ? zoff + (unsigned)sz * st[2] : off[A], v);
    }
    // four taps of m along axis A from t0 (-1: Dp, -2: Dm), into v (left as it is where none
    // reaches a layer, or off)
    template <int A>
    __device__ __forceinline__ void ld4(Arr<T> m, bool on, int t0, T (&v)[4]) const {
        if (!near[A] || (A == 2 && !on)) return;
        if (A == 2) {
#pragma unroll
            for (int n = 0; n < 4; ++n) v[n] = ldb<T>(m, zoff + (unsigned)(sz + t0 + n) * st[2]);
        } else {
            taps<T, A>(m, off[A], t0, st[A], v);
        }
    }
};
// Layer coefficients of a column along x and y (a = 0 off the layers); along z per plane.
template <typename T>
__device__ __forceinline__ void ld_coef(const Dev<T> &d, int i, int j, int hx, int hy, T (&pa)[3], T (&pb)[3]) {
    const unsigned oi = (unsigned)i * (unsigned)sizeof(T), oj = (unsigned)j * (unsigned)sizeof(T);
    pa[0] = ldb<T>(held(d.pa(0, hx)), oi);
    pb[0] = ldb<T>(held(d.pb(0, hx)), oi);
    pa[1] = ldb<T>(held(d.pa(1, hy)), oj);
    pb[1] = ldb<T>(held(d.pb(1, hy)), oj);
    pa[2] = pb[2] = T(0);
}
// Addresses of a role's memory variables along the three axes.
template <typename T, bool ADJ, typename FO, typename FN>
__device__ __forceinline__ void hold_mem(FO fo, FN fn, Arr<T> (&mo)[3], Arr<T> (&mn)[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        mo[a] = held(fo(a));
        mn[a] = ADJ ? held(fn(a)) : nullptr;
    }
}

// ------------------------------------------------------------------------
// velocity-shaped pass.  In_ca lives in field sigma^{ca} (forward) or w_(ca) (adjoint);
// Dp where a == c, Dm elsewhere.
// ------------------------------------------------------------------------
// Fluid columns.  UNI: uniform media, whose rho and alpha come from the per-tile table instead
// of the maps (the same values, so the same results).
//
// s22 = s33 = s11 and the shear stresses are zero on every tap, so the three nonzero
// differences are those of s11 along x, y and z.  Of the C-PML memory variables only the
// diagonal ones (phi^{cc}; in the adjoint a psi~^{cc} and a phi~^{cc}) act on fluid cells: the
// others stay zero or meet only zero moduli.
//
// EN (forward only): also accumulate into kin the kinetic part sum_c rho_c u_old^c u_new^c of
// the modified energy (Sec. 2.2), with the staggered density of the update itself.
template <typename T, bool ADJ, bool UNI, bool EN>
__device__ __forceinline__ void fluid_vel(const Dev<T> &d, int i, int j, int z0, int z1, unsigned o, T rho_t,
                                          T alp_t, double &kin) {
    const T h = d.inv_dx, dt = d.dt;
    const unsigned st[3] = {(unsigned)sizeof(T), d.sy, d.sz};
    Slab<T, ADJ> sl(d, i, j, z0, true, true);
    Arr<T> s11 = held(d.f(S11));
    Arr<T> u[3] = {held(d.f(U1)), held(d.f(U2)), held(d.f(U3))};
    Arr<T> rho = UNI ? nullptr : held(d.rho()), alp = UNI ? nullptr : held(d.alpha());
    T qs[4];   // s11 at planes k-1..k+2
    qs[0] = T(0);
    qs[1] = ldb<T>(s11, o - st[2]);
    qs[2] = ldb<T>(s11, o);
    qs[3] = ldb<T>(s11, o + st[2]);
    T rho_k = UNI ? rho_t : ldb<T>(rho, o), alp_k = UNI ? alp_t : ldb<T>(alp, o);
    T pa[3], pb[3];
    ld_coef(d, i, j, 1, 1, pa, pb);   // half points
    Arr<T> zc = held(d.zab(1));
    Arr<T> mo[3], mn[3];   // own-point variables (forward phi^{aa}, adjoint a phi~^{aa}), taps (adjoint a psi~^{aa})
    hold_mem<T, ADJ>([&](int a) { return d.mem(a, a); }, [&](int a) { return d.mem(a, 3 + a); }, mo, mn);
    T own[3] = {}, near[3][4] = {};
    for (int k = z0; k < z1; ++k, o += st[2], sl.next(k)) {
        T tap[2][4], uold[3], rho_n[3], alp_n[3];
        const T qn = ldb<T>(s11, o + 2 * st[2]);
        taps<T, 0>(s11, o, -1, st[0], tap[0]);
        taps<T, 1>(s11, o, -1, st[1], tap[1]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            uold[c] = ldb<T>(u[c], o);
            rho_n[c] = UNI ? rho_t : (c == 0 ? ldi<T>(rho, o, 1) : ldb<T>(rho, o + st[c]));
            alp_n[c] = UNI ? alp_t : (c == 0 ? ldi<T>(alp, o, 1) : ldb<T>(alp, o + st[c]));
        }
        axes([&](auto A) {
            constexpr int a = decltype(A)::value;
            sl.template ld<a>(mo[a], true, own[a]);
            if (ADJ) sl.template ld4<a>(mn[a], true, -1, near[a]);
        });
        if (sl.own[2]) {
            pa[2] = zc[2 * k];
            pb[2] = zc[2 * k + 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 3; ++n) qs[n] = qs[n + 1];
        qs[3] = qn;
        T acc[3] = {diff4(tap[0]) * h, diff4(tap[1]) * h, diff4(qs) * h};
        axes([&](auto A) {
            constexpr int a = decltype(A)::value;
            if (ADJ) {
                acc[a] = add_near(sl.near[a], acc[a] * dt, near[a], h);
            } else if (sl.own[a]) {
                const T phi = fma(pb[a], own[a], pa[a] * acc[a]);
                sl.template put<a>(mo[a], phi);
                acc[a] += phi;
            }
        });
        T out[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const T rho_c = UNI ? rho_t : T(0.5) * (rho_k + rho_n[c]);
            const T alp_c = UNI ? alp_t : T(0.5) * (alp_k + alp_n[c]);
            const T irho = rcp(rho_c);
            out[c] = fma(uold[c], fma(-dt, alp_c, T(1)), ADJ ? -(acc[c] * irho) : dt * irho * acc[c]);
            stb<T>(u[c], o, out[c]);
            if (EN) kin = fma((double)rho_c * (double)uold[c], (double)out[c], kin);
        }
        rho_k = rho_n[2];
        alp_k = alp_n[2];
        if (ADJ) {
            // g' = a phi~^{aa} <- b g' + a dt r^a
            axes([&](auto A) {
                constexpr int a = decltype(A)::value;
                if (sl.own[a]) sl.template put<a>(mo[a], fma(pb[a], own[a], pa[a] * dt * out[a]));
            });
        }
    }
}

// General columns: component C of the velocity, one wavefront per component.  sh: this lane
// reads the shear stresses (a fluid lane of a mixed sub-tile does not: they are zero there, and
// so are the off-diagonal memory variables that act on it); mp: it reads rho and alpha from the
// maps.  s22 and s33 hold s11's value on a fluid lane's taps (fluid columns store all three,
// fluid tiles the bands next to general tiles).
template <typename T, bool ADJ, bool EN, bool ONCE, int C>
__device__ __forceinline__ void gen_vel(const Dev<T> &d, int i, int j, int z0, int z1, unsigned o, bool sh, bool mp,
                                        T rho_t, T alp_t, double &kin) {
    const T h = d.inv_dx, dt = d.dt;
    const unsigned st[3] = {(unsigned)sizeof(T), d.sy, d.sz};
    Slab<T, ADJ> sl(d, i, j, z0, C == 0 || sh, C == 1 || sh);
    Arr<T> fx = held(d.f(sig(C, 0))), fy = held(d.f(sig(C, 1))), fz = held(d.f(sig(C, 2)));
    Arr<T> u = held(d.f(U1 + C));
    Arr<T> rho = held(d.rho()), alp = held(d.alpha());
    constexpr int t0[3] = {C == 0 ? -1 : -2, C == 1 ? -1 : -2, C == 2 ? -1 : -2};   // first tap: Dp -1, Dm -2
    T qz[4] = {T(0), T(0), T(0), T(0)};
    if (C == 2 || sh) {
#pragma unroll
        for (int n = 0; n < 3; ++n) qz[n + 1] = ldb<T>(fz, o + (unsigned)(t0[2] + n) * st[2]);
    }
    T rho_k = rho_t, alp_k = alp_t;
    if (C == 2 && mp) {
        rho_k = ldb<T>(rho, o);
        alp_k = ldb<T>(alp, o);
    }
    T pa[3], pb[3];
    ld_coef(d, i, j, C == 0, C == 1, pa, pb);   // phi^{Ca}: half points along a == C, integer points otherwise
    Arr<T> zc = held(d.zab(C == 2));
    Arr<T> mo[3], mn[3];
    hold_mem<T, ADJ>([&](int a) { return d.mem(a, C); }, [&](int a) { return d.mem(a, 3 + C); }, mo, mn);
    // values a lane does not load stay as they are: zero
    T tap[2][4] = {}, qn = T(0), own[3] = {}, near[3][4] = {};
    T rho_n = rho_t, alp_n = alp_t;
    for (int k = z0; k < z1; ++k, o += st[2], sl.next(k)) {
        if (C == 0) taps<T, 0>(fx, o, t0[0], st[0], tap[0]);
        if (C == 1) taps<T, 1>(fy, o, t0[1], st[1], tap[1]);
        if (C == 2) qn = ldb<T>(fz, o + (unsigned)(t0[2] + 3) * st[2]);
        if (sh) {
            if (C != 0) taps<T, 0>(fx, o, t0[0], st[0], tap[0]);
            if (C != 1) taps<T, 1>(fy, o, t0[1], st[1], tap[1]);
            if (C != 2) qn = ldb<T>(fz, o + (unsigned)(t0[2] + 3) * st[2]);
        }
        const T uold = ld_own<T, ONCE>(u, o);
        if (mp) {
            if (C < 2) {
                rho_k = ldb<T>(rho, o);
                alp_k = ldb<T>(alp, o);
            }
            rho_n = C == 0 ? ldi<T>(rho, o, 1) : ldb<T>(rho, o + st[C]);
            alp_n = C == 0 ? ldi<T>(alp, o, 1) : ldb<T>(alp, o + st[C]);
        }
        axes([&](auto A) {
            constexpr int a = decltype(A)::value;
            sl.template ld<a>(mo[a], a == C || sh, own[a]);
            if (ADJ) sl.template ld4<a>(mn[a], a == C || sh, t0[a], near[a]);
        });
        if (sl.own[2]) {
            pa[2] = zc[2 * k];
            pb[2] = zc[2 * k + 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 3; ++n) qz[n] = qz[n + 1];
        qz[3] = qn;
        const T df[3] = {diff4(tap[0]), diff4(tap[1]), diff4(qz)};
        T dd[3] = {df[0] * h, df[1] * h, df[2] * h};
        if (ADJ)
            axes([&](auto A) {
                constexpr int a = decltype(A)::value;
                dd[a] = add_near(sl.near[a], dd[a] * dt, near[a], h);
            });
        T acc = ADJ ? dd[0] + dd[1] + dd[2] : fma(h, df[2], fma(h, df[0], dd[1]));
        if (!ADJ) {
            // phi^{Ca} <- b phi^{Ca} + a D_a sigma^{Ca}
            axes([&](auto A) {
                constexpr int a = decltype(A)::value;
                if (!sl.own[a] || !(a != 2 || C == 2 || sh)) return;
                const T phi = fma(pb[a], own[a], pa[a] * dd[a]);
                sl.template put<a>(mo[a], phi);
                acc += phi;
            });
        }
        const T rho_c = T(0.5) * (rho_k + rho_n);
        const T alp_c = T(0.5) * (alp_k + alp_n);
        const T irho = rcp(rho_c);
        const T J = fma(-dt, alp_c, T(1));
        const T out = ADJ ? fma(uold, J, -(acc * irho)) : fma(acc, dt * irho, uold * J);
        st_own<T, ONCE>(u, o, out);
        if (EN) kin = fma((double)rho_c * (double)uold, (double)out, kin);
        if (C == 2) {
            rho_k = rho_n;
            alp_k = alp_n;
        }
        if (ADJ) {
            // g' = a phi~ <- b g' + a dt r   (Gamma^T q with the indicator folded into a)
            axes([&](auto A) {
                constexpr int a = decltype(A)::value;
                if (sl.own[a] && (a != 2 || C == 2 || sh)) sl.template put<a>(mo[a], fma(pb[a], own[a], pa[a] * dt * out));
            });
        }
    }
}

// Sum of v over the block's 256 threads in a fixed order (wavefront butterflies, then the four
// wavefronts in turn): the same double for the same inputs.  Every thread of the block calls it.
__device__ __forceinline__ double block_sum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    __shared__ double part[NT / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += part[w];
    return s;
}

// A block of a fluid entry updates up to four sub-tiles, one per wavefront; a block of a general
// entry updates one sub-tile, its velocity components on wavefronts 0, 1 and 2.
//
// EN (forward only): each wavefront also writes its part of the kinetic energy sum to
// epart[4 blockIdx.x + wavefront], padding blocks included.
//
// Extra blocks after the list's: the forward pass gathers a trace row of the stresses it reads
// (gather_block), the adjoint pass forms the increments of one (scatter_block).
//
// ctr (captured step graphs, el_exec): a device step counter.  The gather blocks write trace row
// *ctr of the traces at row, the scatter blocks read row *ctr - 1 (the stress pass that follows
// advances the counter, or steps it back).
//
// ONCE: see ld_own.
//
// G > 1 (grouped launch): the blocks of member q of the group are first[q] .. first[q+1]-1.
template <typename T, bool ADJ, bool EN, bool ONCE, int G>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 6 : 1))) void k_vel(Grp<T, G> g,
                                                                                              double *epart, int *ctr) {
    static_assert(NT == 256, "gather_block works on blocks of 256 threads");
    static_assert(!(ADJ && EN), "the energy belongs to the forward recursion");
    static_assert(G == 1 || !EN, "the energy is a single plan's");
    const int q = member_of(g);
    const int bid = G > 1 ? (int)blockIdx.x - g.first[q] : (int)blockIdx.x;
    const Dev<T> &d = g.d[q];
    const Tiles &tl = g.tl[q];
    if (bid >= 8 * tl.per) {
        double *row = g.row[q];
        if (!row) return;
        const Rec &r = g.r[q];
        if (ADJ) scatter_block(d, r, ctr ? row + (size_t)(*ctr - 1) * r.nrec : row, bid - 8 * tl.per);
        else gather_block(d, r, ctr ? row + (size_t)(*ctr) * r.nrec : row, bid - 8 * tl.per);
        return;
    }
    double kin = 0.0;
    Block<T> b;
    if (block_of(tl, b, bid)) {
        const int w = wave_id();
        const bool gen = (b.fl & kBlkGen) != 0;
        const int sub = gen ? (int)(b.fl >> kBlkSubShift) & 3 : w;
        const int i = b.x0 + sub_col(sub), j = b.y0 + sub_row(sub);
        const bool active = gen ? w < 3 : ((b.fl >> (kBlkMaskShift + w)) & 1u) != 0;
        if (active && i < d.nx && j < d.ny) {
            const unsigned o = (unsigned)(b.z0 + 2) * d.sz + (unsigned)j * d.sy + (unsigned)i * (unsigned)sizeof(T);
            if (!gen) {
                if ((b.fl >> (kBlkUniShift + w)) & 1u) fluid_vel<T, ADJ, true, EN>(d, i, j, b.z0, b.z1, o, b.rho, b.alpha, kin);
                else fluid_vel<T, ADJ, false, EN>(d, i, j, b.z0, b.z1, o, b.rho, b.alpha, kin);
            } else {
                bool fl, ul;
                fluid_lanes(b, fl, ul);
                if (w == 0) gen_vel<T, ADJ, EN, ONCE, 0>(d, i, j, b.z0, b.z1, o, !fl, !ul, b.rho, b.alpha, kin);
                else if (w == 1) gen_vel<T, ADJ, EN, ONCE, 1>(d, i, j, b.z0, b.z1, o, !fl, !ul, b.rho, b.alpha, kin);
                else gen_vel<T, ADJ, EN, ONCE, 2>(d, i, j, b.z0, b.z1, o, !fl, !ul, b.rho, b.alpha, kin);
            }
        }
    }
    if (EN) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) kin += __shfl_xor(kin, m);
        if ((threadIdx.x & 63) == 0) epart[(size_t)blockIdx.x * (NT / 64) + (threadIdx.x >> 6)] = kin;
    }
}

// ------------------------------------------------------------------------
// stress-shaped pass.  In_ca lives in field u^c (forward) or r^c (adjoint); Dm where a == c,
// Dp elsewhere.
// ------------------------------------------------------------------------
// Normal stresses of a column.  FLUID: fluid columns, whose three normal stresses take the same
// increment lambda tr (mu = 0) and whose s22 and s33 are stored only on the bands that general
// tiles read across a face (put22 and planes outside [zlo, zhi)).  Otherwise the normal stresses
// of a general sub-tile: on its fluid lanes (sh false) mu is zero and s22 = s33 = s11, neither of
// them read.  UNI: lambda comes from the per-tile table instead of the map on every lane, ul: on
// this lane (the same value, so the same results).  Only the diagonal C-PML memory variables
// (psi^{cc}; in the adjoint a phi~^{cc} and a psi~^{cc}) belong to the normal stresses.  inc
// (adjoint, null without scatter points): the sub-tile's increments of Theta^T y (scatter_value),
// which times 3 lambda + 2 mu are added to all three.
template <typename T, bool ADJ, bool FLUID, bool UNI, bool ONCE>
__device__ __forceinline__ void normal_str(const Dev<T> &d, int i, int j, int z0, int z1, unsigned o, T lam_t, bool sh,
                                           bool ul, bool put22, int zlo, int zhi, const T *inc) {
    const T h = d.inv_dx, dt = d.dt;
    const unsigned st[3] = {(unsigned)sizeof(T), d.sy, d.sz};
    Slab<T, ADJ> sl(d, i, j, z0, true, true);
    Arr<T> u1 = held(d.f(U1)), u2 = held(d.f(U2)), u3 = held(d.f(U3));
    Arr<T> s[3] = {held(d.f(S11)), held(d.f(S22)), held(d.f(S33))};
    Arr<T> lamp = UNI ? nullptr : held(d.lam()), mup = FLUID ? nullptr : held(d.mu());
    T qc[4];   // u3 at planes k-2..k+1
    qc[0] = T(0);
    qc[1] = ldb<T>(u3, o - 2 * st[2]);
    qc[2] = ldb<T>(u3, o - st[2]);
    qc[3] = ldb<T>(u3, o);
    T pa[3], pb[3];
    ld_coef(d, i, j, 0, 0, pa, pb);   // integer points
    Arr<T> zc = held(d.zab(0));
    Arr<T> mo[3], mn[3];   // own-point variables (forward psi^{aa}, adjoint a psi~^{aa}), taps (adjoint a phi~^{aa})
    hold_mem<T, ADJ>([&](int a) { return d.mem(a, 3 + a); }, [&](int a) { return d.mem(a, a); }, mo, mn);
    // values a lane does not load stay as they are
    T own[3] = {}, near[3][4] = {}, sold[3] = {}, lam = lam_t, mu = T(0), add = T(0);
    for (int k = z0; k < z1; ++k, o += st[2], sl.next(k)) {
        T tap[2][4];
        const T qn = ldb<T>(u3, o + st[2]);
        taps<T, 0>(u1, o, -2, st[0], tap[0]);
        taps<T, 1>(u2, o, -2, st[1], tap[1]);
        sold[0] = ld_own<T, ONCE>(s[0], o);
        if (!FLUID && sh) {
            sold[1] = ld_own<T, ONCE>(s[1], o);
            sold[2] = ld_own<T, ONCE>(s[2], o);
            mu = ldb<T>(mup, o);
        }
        if (!UNI && !ul) lam = ldb<T>(lamp, o);
        if (ADJ && inc) add = inc[64 * (k - z0) + (int)(threadIdx.x & 63u)];
        axes([&](auto A) {
            constexpr int a = decltype(A)::value;
            sl.template ld<a>(mo[a], true, own[a]);
            if (ADJ) sl.template ld4<a>(mn[a], true, -2, near[a]);
        });
        if (sl.own[2]) {
            pa[2] = zc[2 * k];
            pb[2] = zc[2 * k + 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < 3; ++n) qc[n] = qc[n + 1];
        qc[3] = qn;
        T e[3] = {diff4(tap[0]) * h, diff4(tap[1]) * h, diff4(qc) * h};
        axes([&](auto A) {
            constexpr int a = decltype(A)::value;
            if (ADJ) {
                e[a] = add_near(sl.near[a], e[a] * dt, near[a], h);
            } else if (sl.own[a]) {
                const T psi = fma(pb[a], own[a], pa[a] * e[a]);
                sl.template put<a>(mo[a], psi);
                e[a] += psi;
            }
        });
        const T tr = e[0] + e[1] + e[2];
        const T kf = fma(T(3), lam, mu + mu);   // 3 lambda + 2 mu: what a unit of Theta^T y adds
        T w[3];
        if (FLUID) {
            w[0] = w[1] = w[2] = ADJ ? fma(-lam, tr, sold[0]) : fma(dt, lam * tr, sold[0]);
            const T v = ADJ ? fma(kf, add, w[0]) : w[0];
            stb<T>(s[0], o, v);
            if (put22) stb<T>(s[1], o, v);
            if (k < zlo || k >= zhi) stb<T>(s[2], o, v);
        } else {
            const T lt = lam * tr;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T so = c == 0 || sh ? sold[c] : sold[0], de = fma(mu + mu, e[c], lt);
                w[c] = ADJ ? so - de : fma(dt, de, so);
                st_own<T, ONCE>(s[c], o, ADJ ? fma(kf, add, w[c]) : w[c]);
            }
        }
        if (ADJ) {
            // g = a psi~^{aa} <- b g + a dt w_aa   (Delta^T s; the indicator is folded into a), and
            // a dt times the increment
            axes([&](auto A) {
                constexpr int a = decltype(A)::value;
                if (!sl.own[a]) return;
                const T g = fma(pb[a], own[a], pa[a] * dt * w[a]);
                sl.template put<a>(mo[a], fma(add * kf, pa[a] * dt, g));
            });
        }
    }
}

// Shear stress sigma^{AB} (A < B) of a general column, one wavefront per shear stress.  Lanes of
// fluid columns do not come here: their shear stresses stay zero.
template <typename T, bool ADJ, bool ONCE, int A, int B>
__device__ __forceinline__ void shear_str(const Dev<T> &d, int i, int j, int z0, int z1, unsigned o) {
    static_assert(A < B, "axes in order");
    const T h = d.inv_dx, dt = d.dt;
    const unsigned st[3] = {(unsigned)sizeof(T), d.sy, d.sz};
    Slab<T, ADJ> sl(d, i, j, z0, true, true);
    Arr<T> s = held(d.f(sig(A, B)));
    Arr<T> ua = held(d.f(U1 + A)), ub = held(d.f(U1 + B)), mu = held(d.mu());
    T qz[4];   // u^A at planes k-1..k+2 (B = z)
    T mu0 = T(0), muA = T(0);   // mu at the cell and its +A neighbour of the current plane
    if (B == 2) {
        qz[0] = T(0);
        qz[1] = ldb<T>(ua, o - st[2]);
        qz[2] = ldb<T>(ua, o);
        qz[3] = ldb<T>(ua, o + st[2]);
        mu0 = ldb<T>(mu, o);
        muA = ldb<T>(mu, o + st[A]);
    }
    T pa[3], pb[3];
    ld_coef(d, i, j, 1, 1, pa, pb);   // both memory variables lie at half points of their axis
    Arr<T> zc = B == 2 ? held(d.zab(1)) : nullptr;
    Arr<T> moA = held(d.mem(A, 3 + B)), moB = held(d.mem(B, 3 + A));
    Arr<T> mnA = ADJ ? held(d.mem(A, B)) : nullptr, mnB = ADJ ? held(d.mem(B, A)) : nullptr;
    T ownA = T(0), ownB = T(0), nearA[4] = {}, nearB[4] = {};
    for (int k = z0; k < z1; ++k, o += st[2], sl.next(k)) {
        T ta[4], tb[4];   // D_B u^A and D_A u^B (Dp: -1 .. +2)
        T qn = T(0);
        if (B == 2) {
            qn = ldb<T>(ua, o + 2 * st[2]);
        } else {
            taps<T, B>(ua, o, -1, st[B], ta);
            mu0 = ldb<T>(mu, o);
            muA = ldb<T>(mu, o + st[A]);
        }
        taps<T, A>(ub, o, -1, st[A], tb);
        const T sold = ld_own<T, ONCE>(s, o);
        const T muB = ldb<T>(mu, o + st[B]), muAB = ldb<T>(mu, o + st[A] + st[B]);
        sl.template ld<A>(moA, true, ownA);
        sl.template ld<B>(moB, true, ownB);
        if (ADJ) {
            sl.template ld4<A>(mnA, true, -1, nearA);
            sl.template ld4<B>(mnB, true, -1, nearB);
        }
        if (B == 2 && sl.own[2]) {
            pa[2] = zc[2 * k];
            pb[2] = zc[2 * k + 1];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (B == 2) {
#pragma unroll
            for (int n = 0; n < 3; ++n) qz[n] = qz[n + 1];
            qz[3] = qn;
        }
        T eB = B == 2 ? diff4(qz) * h : diff4(ta) * h, eA = diff4(tb) * h;
        if (ADJ) {
            eB = add_near(sl.near[B], eB * dt, nearB, h);
            eA = add_near(sl.near[A], eA * dt, nearA, h);
        } else {
            // psi^{ca} <- b psi^{ca} + a D_a u^c
            if (sl.own[A]) {
                const T psi = fma(pb[A], ownA, pa[A] * eA);
                sl.template put<A>(moA, psi);
                eA += psi;
            }
            if (sl.own[B]) {
                const T psi = fma(pb[B], ownB, pa[B] * eB);
                sl.template put<B>(moB, psi);
                eB += psi;
            }
        }
        const T m = harmonic4r(rcp(mu0), rcp(muA), rcp(muB), rcp(muAB));
        if (B == 2) {
            mu0 = muB;
            muA = muAB;
        }
        const T w = fma(ADJ ? -m : dt * m, eB + eA, sold);
        st_own<T, ONCE>(s, o, w);
        if (ADJ) {
            if (sl.own[A]) sl.template put<A>(moA, fma(pb[A], ownA, pa[A] * dt * w));
            if (sl.own[B]) sl.template put<B>(moB, fma(pb[B], ownB, pa[B] * dt * w));
        }
    }
}

// A block of a fluid entry updates up to four sub-tiles, one per wavefront; a block of a general
// entry updates one sub-tile, its normal stresses on wavefront 0 and its shear stresses on
// wavefronts 1 to 3.
//
// The adjoint adds the increments Theta^T y that its velocity pass formed (Dev::inc).
//
// ctr (captured step graphs): the pass advances (the adjoint steps back) the device step counter
// that its velocity pass's extra blocks read (all of that launch has completed).  G > 1: grouped
// launch, as k_vel.  ONCE: see ld_own.
template <typename T, bool ADJ, bool ONCE, int G>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 6 : 1))) void k_str(Grp<T, G> g, int *ctr) {
    const int q = member_of(g);
    const int bid = G > 1 ? (int)blockIdx.x - g.first[q] : (int)blockIdx.x;
    const Dev<T> &d = g.d[q];
    const Tiles &tl = g.tl[q];
    if (ctr && bid == 0 && threadIdx.x == 0) *ctr += ADJ ? -1 : 1;
    Block<T> b;
    if (!block_of(tl, b, bid)) return;
    const int w = wave_id();
    const bool gen = (b.fl & kBlkGen) != 0;
    if (!gen && !((b.fl >> (kBlkMaskShift + w)) & 1u)) return;
    const int sub = gen ? (int)(b.fl >> kBlkSubShift) & 3 : w;
    const int i = b.x0 + sub_col(sub), j = b.y0 + sub_row(sub);
    if (i >= d.nx || j >= d.ny) return;
    const unsigned o = (unsigned)(b.z0 + 2) * d.sz + (unsigned)j * d.sy + (unsigned)i * (unsigned)sizeof(T);
    // this sub-tile's increments
    const T *inc = nullptr;
    if (ADJ && (b.fl >> (kBlkIncShift + sub) & 1u)) {
        const int before = __builtin_popcount(b.fl >> kBlkIncShift & ((1u << sub) - 1u));
        inc = d.inc() + (size_t)(b.slot + before * (b.z1 - b.z0)) * 64u;
    }
    if (!gen) {
        // s22 is stored on the rows, s33 on the planes, that general tiles read across a face
        // (everywhere in a general tile's fluid sub-tile)
        const unsigned ed = b.fl >> kBlkEdgeShift;
        const bool keep = (b.fl & kBlkKeep) != 0;
        const bool put22 = keep || ((ed & 1) && j < b.y0 + 2) || ((ed & 2) && j >= b.y0 + TY - 2);
        const int zlo = keep ? b.z1 : ((ed & 4) ? b.z0 + 2 : b.z0), zhi = keep ? b.z0 : ((ed & 8) ? b.z1 - 2 : b.z1);
        const bool uni = ((b.fl >> (kBlkUniShift + w)) & 1u) != 0;
        if (uni) normal_str<T, ADJ, true, true, false>(d, i, j, b.z0, b.z1, o, b.lam, false, true, put22, zlo, zhi, inc);
        else normal_str<T, ADJ, true, false, false>(d, i, j, b.z0, b.z1, o, b.lam, false, false, put22, zlo, zhi, inc);
    } else {
        bool fl, ul;
        fluid_lanes(b, fl, ul);
        if (w == 0) {
            normal_str<T, ADJ, false, false, ONCE>(d, i, j, b.z0, b.z1, o, b.lam, !fl, ul, true, 0, 0, inc);
        } else {
            if (fl) return;
            if (w == 1) shear_str<T, ADJ, ONCE, 1, 2>(d, i, j, b.z0, b.z1, o);
            else if (w == 2) shear_str<T, ADJ, ONCE, 0, 2>(d, i, j, b.z0, b.z1, o);
            else shear_str<T, ADJ, ONCE, 0, 1>(d, i, j, b.z0, b.z1, o);
        }
    }
}

// A plan's own pass as a launch of one member.
template <int G, typename T>
Grp<T, G> one(const Dev<T> &d, const Tiles &tl, const Rec *r = nullptr, double *row = nullptr) {
    Grp<T, G> g{};
    g.d[0] = d;
    g.tl[0] = tl;
    g.r[0] = r ? *r : Rec{};
    g.row[0] = row;
    g.first[0] = 0;
    for (int k = 1; k <= G; ++k) g.first[k] = 1 << 30;
    g.n = 1;
    return g;
}

template <typename T>
hipError_t launch_velocity(const Dev<T> &d, const Tiles &tl, hipStream_t s, const Rec *r, double *grow,
                           double *epart, int *ctr) {
    const bool gat = r && grow && r->nrec > 0;
    const int blocks = 8 * tl.per + (gat ? gather_blocks(r->nrec) : 0);
    const Grp<T, 1> g = one<1>(d, tl, gat ? r : nullptr, gat ? grow : nullptr);
    const auto plain = tl.once ? k_vel<T, false, false, true, 1> : k_vel<T, false, false, false, 1>;
    hipLaunchKernelGGL((epart ? k_vel<T, false, true, false, 1> : plain), dim3(blocks), dim3(NT), 0, s, g, epart, ctr);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_stress(const Dev<T> &d, const Tiles &tl, hipStream_t s, int *ctr) {
    hipLaunchKernelGGL((tl.once ? k_str<T, false, true, 1> : k_str<T, false, false, 1>), dim3(8 * tl.per), dim3(NT), 0, s,
                       one<1>(d, tl), ctr);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_adj_velocity(const Dev<T> &d, const Tiles &tl, hipStream_t s, const Rec *r, const double *y,
                               int *ctr) {
    const bool sc = r && y && r->npts > 0;
    const int blocks = 8 * tl.per + (sc ? scatter_blocks(r->npts) : 0);
    hipLaunchKernelGGL((tl.once ? k_vel<T, true, false, true, 1> : k_vel<T, true, false, false, 1>), dim3(blocks), dim3(NT), 0, s,
                       one<1>(d, tl, sc ? r : nullptr, sc ? const_cast<double *>(y) : nullptr), (double *)nullptr, ctr);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_adj_stress(const Dev<T> &d, const Tiles &tl, hipStream_t s, int *ctr) {
    hipLaunchKernelGGL((tl.once ? k_str<T, true, true, 1> : k_str<T, true, false, 1>), dim3(8 * tl.per), dim3(NT), 0, s,
                       one<1>(d, tl), ctr);
    return hipGetLastError();
}

// Grouped passes: members q < g.n with first[] set by group_blocks.
template <typename T, bool ONCE>
void group_pass(const Grp<T, kGroupMax> &g, int pass, hipStream_t s) {
    const dim3 grid(g.first[g.n]);
    if (pass == 1 || pass == 3)
        hipLaunchKernelGGL((pass == 1 ? k_str<T, false, ONCE, kGroupMax> : k_str<T, true, ONCE, kGroupMax>), grid, dim3(NT), 0, s,
                           g, (int *)nullptr);
    else
        hipLaunchKernelGGL((pass == 0 ? k_vel<T, false, false, ONCE, kGroupMax> : k_vel<T, true, false, ONCE, kGroupMax>), grid,
                           dim3(NT), 0, s, g, (double *)nullptr, (int *)nullptr);
}
template <typename T>
hipError_t launch_group_pass(const Grp<T, kGroupMax> &g, int pass, hipStream_t s) {
    bool once = true;   // of every member's state
    for (int q = 0; q < g.n; ++q) once = once && g.tl[q].once;
    if (once) group_pass<T, true>(g, pass, s);
    else group_pass<T, false>(g, pass, s);
    return hipGetLastError();
}

#pragma clang fp contract(fast)

// Potential part of the modified energy (Sec. 2.2): sigma^T C^+ sigma over the stresses of one
// time level, in double.  At a normal-stress point with moduli lambda, mu
//   (tr s)^2 / (9 K) + |dev s|^2 / (2 mu),   9 K = 3 (3 lambda + 2 mu),
// the second term only where mu > 0 (a fluid cell's deviatoric stress stays zero, Sec. 2.1);
// at a shear point s_ij^2 / mu_ij with the harmonic-mean edge modulus of the stencils, only
// where it is nonzero.  A fluid tile stores s11 alone (s22 = s33 = s11, shear zero), so its
// trace is 3 s11 and it has neither deviatoric nor shear part.  Each tile block writes its
// sum to epart[blockIdx.x].
template <typename T>
__device__ __forceinline__ void pot_tile(const Dev<T> &d, const Tiles &tl, double &pot) {
    Block<T> b;
    if (!block_of(tl, b, (int)blockIdx.x) || !(b.fl & kBlkFirst)) return;
    const bool fast = (b.fl & kBlkFast) != 0;
    const int w = wave_id(), i = b.x0 + sub_col(w), j = b.y0 + sub_row(w);
    if (i >= d.nx || j >= d.ny) return;
    const unsigned sx = sizeof(T), sy = d.sy, sz = d.sz;
    unsigned o = 2 * d.sz + (unsigned)b.z0 * sz + (unsigned)j * sy + (unsigned)i * sx;
    for (int k = b.z0; k < b.z1; ++k, o += sz) {
        const double lam = (double)ldb(d.lam(), o), mu = (double)ldb(d.mu(), o);
        const double s11 = (double)ldb(d.f(S11), o);
        if (fast) {
            const double tr = 3.0 * s11;
            pot += tr * tr / (3.0 * (3.0 * lam + 2.0 * mu));
            continue;
        }
        const double s22 = (double)ldb(d.f(S22), o), s33 = (double)ldb(d.f(S33), o);
        const double tr = s11 + s22 + s33;
        pot += tr * tr / (3.0 * (3.0 * lam + 2.0 * mu));
        if (mu > 0.0) {
            const double m = tr / 3.0, a = s11 - m, b = s22 - m, c = s33 - m;
            pot += (a * a + b * b + c * c) / (2.0 * mu);
        }
        // edge moduli: harmonic means of the four cells around each shear point, as the
        // stencils form them (reciprocals of T, so a zero modulus gives a zero mean)
        const T r0 = rcp(ldb(d.mu(), o)), rx = rcp(ldb(d.mu(), o + sx)), ry = rcp(ldb(d.mu(), o + sy));
        const T rz = rcp(ldb(d.mu(), o + sz)), rxy = rcp(ldb(d.mu(), o + sx + sy));
        const T rxz = rcp(ldb(d.mu(), o + sx + sz)), ryz = rcp(ldb(d.mu(), o + sy + sz));
        const double me[3] = {(double)harmonic4r(r0, ry, rz, ryz), (double)harmonic4r(r0, rx, rz, rxz),
                              (double)harmonic4r(r0, rx, ry, rxy)};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (!(me[q] > 0.0)) continue;
            const double sv = (double)ldb(d.f(S23 + q), o);
            pot += sv * sv / me[q];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(NT) void k_energy_pot(Dev<T> d, Tiles tl, double *epart) {
    double pot = 0.0;
    pot_tile<T>(d, tl, pot);
    const double s = block_sum(pot);
    if (threadIdx.x == 0) epart[blockIdx.x] = s;
}

template <typename T>
hipError_t launch_energy_pot(const Dev<T> &d, const Tiles &tl, double *epart, hipStream_t s) {
    hipLaunchKernelGGL(k_energy_pot<T>, dim3(8 * tl.per), dim3(NT), 0, s, d, tl, epart);
    return hipGetLastError();
}

// Sums of NT consecutive kinetic parts (one per wavefront of the velocity launch), in a fixed
// order.
__global__ __launch_bounds__(NT) void k_energy_blocks(const double *kin, int n, double *kin_block) {
    const int e = (int)blockIdx.x * NT + (int)threadIdx.x;
    const double s = block_sum(e < n ? kin[e] : 0.0);
    if (threadIdx.x == 0) kin_block[blockIdx.x] = s;
}

// out = (sum of kin[0..nk) + sum of pot[0..np)) / 2, in a fixed order.
__global__ __launch_bounds__(NT) void k_energy_final(const double *kin, int nk, const double *pot, int np, double *out) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nk; b += NT) v += kin[b];
    for (int b = threadIdx.x; b < np; b += NT) v += pot[b];
    const double s = block_sum(v);
    if (threadIdx.x == 0) *out = 0.5 * s;
}

hipError_t launch_energy_final(const double *kin, double *kin_block, const double *pot, int nb, double *out,
                               hipStream_t s) {
    const int n = nb * (NT / 64), nk = (n + NT - 1) / NT;
    hipLaunchKernelGGL(k_energy_blocks, dim3(nk), dim3(NT), 0, s, kin, n, kin_block);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(NT), 0, s, kin_block, nk, pot, nb, out);
    return hipGetLastError();
}

// s22 = s33 = s11 on every fluid tile (the state the lean stress loop leaves implicit).
template <typename T>
__global__ __launch_bounds__(NT) void k_fluid_fill(Dev<T> d, Tiles tl) {
    Block<T> b;
    if (!block_of(tl, b, (int)blockIdx.x) || !(b.fl & kBlkFast)) return;
    const int w = wave_id(), i = b.x0 + sub_col(w), j = b.y0 + sub_row(w);
    if (i >= d.nx || j >= d.ny) return;
    unsigned o = 2 * d.sz + (unsigned)b.z0 * d.sz + (unsigned)j * d.sy + (unsigned)i * (unsigned)sizeof(T);
    for (int k = b.z0; k < b.z1; ++k, o += d.sz) {
        const T v = ldb(d.f(S11), o);
        stb(d.f(S22), o, v);
        stb(d.f(S33), o, v);
    }
}

template <typename T>
hipError_t launch_fluid_fill(const Dev<T> &d, const Tiles &tl, hipStream_t s) {
    hipLaunchKernelGGL(k_fluid_fill<T>, dim3(8 * tl.per), dim3(NT), 0, s, d, tl);
    return hipGetLastError();
}

#define EL_STENCIL_INST(T)                                                                  \
    template hipError_t launch_fluid_fill<T>(const Dev<T> &, const Tiles &, hipStream_t);   \
    template hipError_t launch_velocity<T>(const Dev<T> &, const Tiles &, hipStream_t, const Rec *, double *,  \
                                           double *, int *);                                                   \
    template hipError_t launch_energy_pot<T>(const Dev<T> &, const Tiles &, double *, hipStream_t);            \
    template hipError_t launch_stress<T>(const Dev<T> &, const Tiles &, hipStream_t, int *);       \
    template hipError_t launch_adj_velocity<T>(const Dev<T> &, const Tiles &, hipStream_t, const Rec *,            \
                                               const double *, int *);                                             \
    template hipError_t launch_adj_stress<T>(const Dev<T> &, const Tiles &, hipStream_t, int *);                   \
    template hipError_t launch_group_pass<T>(const Grp<T, kGroupMax> &, int, hipStream_t);

EL_STENCIL_INST(float)
EL_STENCIL_INST(double)

}  // namespace el
