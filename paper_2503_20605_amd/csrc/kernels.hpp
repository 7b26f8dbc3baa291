// gfx950 kernels of the IB-LB wetting solver.
//
// Every kernel works on a batch of independent droplets described by a
// device table of DropDev records; a single droplet is a batch of one.
//
//   k_lb              fused pull-stream + BGK collide + Guo source for every
//                     fluid cell (eq. LBE, equilibrium, S_i, moments of eqs.
//                     hydro_var1/hydro_var2); HBM bound, one cell per lane
//   k_force_spread    nodal surface-tension + wetting forces, spread to the
//                     lattice with the Peskin 4-point kernel (eq. force_spread)
//   k_interp_advect   lattice velocity interpolated at the nodes (eq.
//                     vel_interpolation) and forward-Euler advection
//   k_ib_fused2,
//   k_ring2           2D: interpolation and advection of one step fused with
//                     the forces and spreading of the next (few nodes; many)
//   k_force3,
//   k_spread3         3D: forces one lane per vertex (surface tension, an
//                     elastic interface's shear part, wetting), then
//                     spreading summed per chunk of nearby vertices in LDS
//   k_cross2,
//   k_cross3          crossings of the interface with the lattice rows, for
//                     the inside/outside classification of two viscosities
//   k_inside_mask     that classification as a per-cell mask
//   k_tri_ref         reference triangles of an elastic interface
//   k_cell_sums, k_diag_*, k_contact_*, k_cross_dist
//                     FP64 reductions for the diagnostics and the contact
//                     radius
//
// Populations are stored as deviations f_i - w_i (see lattice.hpp), in two
// ping-pong buffers laid out [i][z][y][x] per droplet, x fastest.
//
// The force density F and the velocity U are dense per-cell arrays, but the
// lattice kernel touches them only inside the interface band: the spreading
// kernel raises a one-byte flag for every x strip (8 or 16 cells, see
// Strip) that receives a tap, and only the cells of flagged strips read F, write U for the
// interpolation and clear F (where it is not zero already).  The spread F is accumulated in fixed point (64-bit integers of
// 2^-40 force units, see fq_of), so its value does not depend on the order
// in which the nodes' contributions arrive; a prescribed force field is kept
// in fp32 in an array of its own.  The flags come in two sets, one per step parity: a lattice
// update reads its own parity's set and clears the other one for the
// spreading of the next step.
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include <type_traits>

#include "lattice.hpp"

namespace iblb {

constexpr int kBlock = 256;   // threads per block of every kernel
// Cells per band flag: 8 (an eighth of a wavefront) for 2D lattices in
// 16-bit storage, 16 (a quarter) otherwise.  With 8-cell strips the fp16
// 256-droplet 2D batch's lattice kernel took 121.8 against 128.2 us per
// launch, while the fp32 1024x512 D2Q9 step took 13.68 against 13.48 us and
// the 3D benchmark step 255.9 against 255.0 us.  A row's flags are padded to
// a multiple of the strips of 64 cells, so that a tiled wavefront (64 cells
// of one row, starting at a multiple of 64) finds its strips' flags in one
// aligned word (64 bits for 8-cell strips, 32 for 16-cell ones).  The node
// kernels take the width from the droplet record (DropDev::sshift).
template <int DIM, int S>
struct Strip {
    static constexpr int shift = (DIM == 2 && S != ST_F32) ? 3 : 4;
    static constexpr int n = 1 << shift;
    static constexpr int per64 = 64 >> shift;  // strips of 64 cells (bytes of a word)
    using Word = typename std::conditional<per64 == 8, uint64_t, uint32_t>::type;
};

struct DropDev {
    int nx, ny, nz, nstrip;
    int sshift;           // log2 of the cells per band flag (see Strip)
    int bcx, bcy, bcz, ncell;
    long long f_off;      // element offset of the populations (Q arrays, fst apart)
    long long c_off;      // cell offset; vector arrays start at dim * c_off
    long long flag_off;   // byte offset of the band flags
    float omega, guo;     // 1/tau and 1 - 1/(2 tau)
    int force_mode;       // 0: immersed boundary, 1: prescribed field
    int active;
    int node_off, n_nodes;
    int tri_off, n_tris;
    int grp_off, n_grps;  // this droplet's run in the list of tile groups (cell sums)
    int blk_off, n_blks;  // and in the list of its interface's chunks (diagnostics)
    int wetting, n_exp, m_exp;
    int fst;              // element stride between population arrays (>= ppl nz)
    int ppl;              // elements per z-plane of a population array (>= nx ny):
                          // cell (x, y, z) sits at z ppl + y nx + x
    double sigma, A, xi, zcut;
    // two viscosities (viscosity ratio != 1): cells enclosed by the
    // interface relax with omega_in / guo_in
    int visc;
    int row_off;          // first lattice row (z * ny + y) of this droplet in the crossing tables
    float omega_in, guo_in;
    double win[3];        // classification window [win, win + n) of each axis
    double img_base, img_r;  // x image of cell centre c: c + img_base (+ nx if c < img_r)
    double shear;         // surface shear modulus of an elastic interface (0: liquid)
    double respace;       // rate beta of the tangential re-spacing of a 2D outline (0: off)
};

struct DiagDev {
    double mass_dev;            // sum over cells of rho - 1
    double mom[3];
    double sum_F[3];
    double sum_phi[3];
    double dropped[3];
    double volume, area;
    double min_h, max_h;
    double max_un, max_u;
    double edge_min, edge_max;
    double cross_lo, cross_hi;  // 2D: outermost crossings of y = zcut
    double cross_r;             // 3D: mean distance of crossings to their centre
    double cross_n;
};

// Fixed-point accumulation of the spread force density (eq. force_spread):
// every contribution phi_j Delta is rounded to an integer number of 2^-40
// force units and added with a 64-bit integer atomic.  Integer addition is
// associative, so the sum, and the fp32 value the lattice kernel forms from
// it (one rounding of the exact sum), are the same whatever order the
// contributions arrive in.  A contribution must stay below 2^10 in
// magnitude (then up to 2^12 of them cannot overflow a cell); a larger or
// non-finite one means the run has blown up: it is dropped and the
// droplet flagged unstable (status bit 2).
constexpr double kFqScale = 1099511627776.0;  // 2^40
constexpr float kFqMax = 1024.f;
__device__ __forceinline__ bool fq_ok(float v) { return fabsf(v) < kFqMax; }  // NaN: false
// rint(v 2^40) as a 64-bit integer: adding 1.5 2^52 rounds to a whole number
// (nearest even) and leaves it in the low bits of the sum; |v 2^40| < 2^50.
__device__ __forceinline__ unsigned long long fq_of(float v) {
    const double m = __builtin_fma((double)v, kFqScale, 6755399441055744.0);
    return __builtin_bit_cast(unsigned long long, m) - 0x4338000000000000ull;
}
__device__ __forceinline__ float fq_value(unsigned long long v) {
    return (float)((double)(long long)v * (1.0 / kFqScale));
}

// Has the compiler load these (uniform) values where it stands, in one batch
// of scalar loads, instead of each beside its first use.
__device__ __forceinline__ void wanted() {}
template <typename T, typename... U>
__device__ __forceinline__ void wanted(T v, U... u) {
#ifdef __AMDGCN__
    __asm__ volatile("" ::"s"(v));
#else
    (void)v;
#endif
    wanted(u...);
}

// v (a lane's own), as a value that the compiler cannot form ahead of the
// place of the call; opaque_uniform: v the same for all lanes.
__device__ __forceinline__ int opaque(int v) {
#ifdef __AMDGCN__
    __asm__ volatile("" : "+v"(v));
#endif
    return v;
}
__device__ __forceinline__ int opaque_uniform(int v) {
#ifdef __AMDGCN__
    __asm__ volatile("" : "+s"(v));
#endif
    return v;
}

// Keeps the narrowing of v to fp16 a rounding of its own (the compiler would
// merge it into the fma before it).
__device__ __forceinline__ float unfused(float v) {
#ifdef __AMDGCN__
    __asm__("" : "+v"(v));
#endif
    return v;
}

// One cell's collision in deviation form (eqs. LBE, f^eq, S_i,
// hydro_var1/2), in two parts so that callers can store each population as
// soon as it is relaxed: the constructor takes the streamed deviations
// f_i - w_i and the force (half-force velocity); relax() hands every
// post-collision population to out(i, value): BGK towards the second-order
// equilibrium plus, with FORCED, the Guo source.
//
// A wavefront issues about 250 vector instructions per D2Q9 cell update (330
// before) and its chain from the last load to the first store is as long as
// they are: a lattice that fits the caches (1024x512) waits for that chain,
// the 256-droplet fp16 batch for issue slots.  So no term of a zero velocity
// component is formed (0 u + v is v, but the compiler has to keep it: u may
// be infinite) and the two populations of an opposite pair share c.U and
// (c.U)^2.  Every operation and its rounding is written out (contraction is
// off), so that the result does not depend on the kernel that the code is
// inlined into: the products of the sums below are rounded once, inside the
// fma that takes them.  With the record of the droplet read in one batch
// (k_lb), kernel trace of 1024x512 fp32: 7.3-7.6 -> 6.5-6.9 us per launch with
// plain stores, 10.3 -> 8.7 with non-temporal ones and the late band flag (a
// coupled step of it 14.0 -> 13.8 and 16.6 -> 15.4); the batch's step 245 -> 236
// us.
template <int DIM, int S>
struct Moments {
    float drho, rho, inv, jx, jy, jz, ux, uy, uz, usq, Fx, Fy, Fz;
    __device__ __forceinline__ Moments(const float* f, float fx, float fy, float fz) : Fx(fx), Fy(fy), Fz(fz) {
#pragma clang fp contract(off)
        using L = Lattice<DIM>;
        jx = jy = jz = uz = 0.f;
        drho = f[0];
#pragma unroll
        for (int i = 1; i < L::Q; ++i) {
            drho += f[i];
            if (L::c[i][0] > 0) jx += f[i]; else if (L::c[i][0] < 0) jx -= f[i];
            if (L::c[i][1] > 0) jy += f[i]; else if (L::c[i][1] < 0) jy -= f[i];
            if (DIM == 3) { if (L::c[i][2] > 0) jz += f[i]; else if (L::c[i][2] < 0) jz -= f[i]; }
        }
        rho = 1.f + drho;
        inv = 1.f / rho;
        jx = __builtin_fmaf(0.5f, Fx, jx);
        jy = __builtin_fmaf(0.5f, Fy, jy);
        ux = jx * inv;
        uy = jy * inv;
        usq = DIM == 3 ? __builtin_fmaf(ux, ux, uy * uy) : __builtin_fmaf(uy, uy, ux * ux);
        if (DIM == 3) {
            jz = __builtin_fmaf(0.5f, Fz, jz);
            uz = jz * inv;
            usq = __builtin_fmaf(uz, uz, usq);
        }
    }
    // c_i . U.  With fp32 and fp16 storage the last component of a diagonal
    // enters as the unrounded product j / rho; with bf16 as the rounded u.
    static constexpr bool kFused = S != ST_BF16;
    __device__ __forceinline__ float dot_u(int i) const {
#pragma clang fp contract(off)
        using L = Lattice<DIM>;
        const int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
        const float sx = cx < 0 ? -ux : ux, sy = cy < 0 ? -uy : uy, sz = cz < 0 ? -uz : uz;
        if (DIM == 3 && cz != 0) {
            if (cx == 0 && cy == 0) return sz;
            const float o = cx != 0 ? sx : sy;
            return kFused ? __builtin_fmaf(cz < 0 ? -inv : inv, jz, o) : o + sz;
        }
        if (cy == 0) return sx;
        if (cx == 0) return sy;
        if (!kFused) return sx + sy;
        // 3D: (-1, -1) carries x unrounded, the others y; 2D: (-1, 1) y, the others x
        if (DIM == 3 ? cx < 0 && cy < 0 : !(cx < 0 && cy > 0))
            return __builtin_fmaf(cx < 0 ? -inv : inv, jx, sy);
        return __builtin_fmaf(cy < 0 ? -inv : inv, jy, sx);
    }
    __device__ __forceinline__ float dot_f(int i) const {
        using L = Lattice<DIM>;
        const int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
        const float sx = cx < 0 ? -Fx : Fx, sy = cy < 0 ? -Fy : Fy, sz = cz < 0 ? -Fz : Fz;
        if (DIM == 3 && cz != 0) return cx != 0 ? sx + sz : (cy != 0 ? sy + sz : sz);
        return cx != 0 ? (cy != 0 ? sx + sy : sx) : sy;
    }
    // whether c . U of i + 1 is exactly the negative of that of i (odd i)
    static constexpr bool mirrored(int i) {
        return !kFused || !((DIM == 3 && i == 7) || (DIM == 2 && i == 7));
    }
    template <bool FORCED, typename Out>
    __device__ __forceinline__ void relax(const float* f, float om, float g, Out&& out) const {
#pragma clang fp contract(off)
        using L = Lattice<DIM>;
        // bf16 storage takes the rounded 1.5 u^2 (see kFused)
        const float usq15 = 1.5f * usq;
        float uF = 0.f;
        if (FORCED) {
            uF = DIM == 3 ? __builtin_fmaf(ux, Fx, uy * Fy) : __builtin_fmaf(uy, Fy, ux * Fx);
            if (DIM == 3) uF = __builtin_fmaf(uz, Fz, uF);
        }
        auto one = [&](int i, float cu, float q, float cF) {
            // f_eq - w = w (rho - 1) + w rho (3 cu + 4.5 cu^2 - 1.5 u^2); q = 4.5 cu^2
            const float m = __builtin_fmaf(3.f, cu, q);
            const float e = __builtin_fmaf(rho, kFused ? __builtin_fmaf(-1.5f, usq, m) : m - usq15, drho);
            float v = __builtin_fmaf(-om, __builtin_fmaf(-L::w[i], e, f[i]), f[i]);
            if (FORCED)
                // S_i = (1 - 1/2tau) w_i [3 (c - U).F + 9 (c.U)(c.F)]
                v = __builtin_fmaf(g * L::w[i], __builtin_fmaf(cF, 9.f * cu, 3.f * (cF - uF)), v);
            out(i, S == ST_F16 ? unfused(v) : v);
        };
        one(0, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 1; i < L::Q; i += 2) {
            const float cu = dot_u(i), q = cu * (4.5f * cu), cF = FORCED ? dot_f(i) : 0.f;
            one(i, cu, q, cF);
            if (mirrored(i)) {
                one(i + 1, -cu, q, -cF);
            } else {
                const float cv = dot_u(i + 1);
                one(i + 1, cv, cv * (4.5f * cv), -cF);
            }
        }
    }
};

// ---------------------------------------------------------------------------
// Cells enclosed by the interface (viscosity ratio != 1)
// ---------------------------------------------------------------------------
// The cells inside the closed interface relax with their own tau (Sec.
// IB-LB, last paragraph).  They are found by casting a ray along +x through
// every lattice row (the cell centres of one y, z): the node kernels record,
// per row, the x at which the interface crosses the row's line, and a cell
// is inside when an odd number of crossings lies beyond its centre.  The
// interface is not wrapped across periodic boundaries: rows and cell
// centres are taken at their periodic image inside the droplet's window
// [win, win + n) of each axis, centred on the mean of the node positions.
// Crossing tables: a count per row and kCrossCap x values per row, one pair
// of tables per step parity.
constexpr int kCrossCap = 16;

__device__ __forceinline__ bool cell_inside(const DropDev& D, const int* __restrict__ cnt,
                                            const double* __restrict__ xs, int x, int row) {
    const long long r = (long long)D.row_off + row;
    int n = cnt[r];
    n = n < kCrossCap ? n : kCrossCap;
    const double c = (double)x + 0.5;
    const double xi = c + D.img_base + (c < D.img_r ? (double)D.nx : 0.0);
    bool in = false;
    for (int k = 0; k < n; ++k) in ^= xs[r * kCrossCap + k] > xi;
    return in;
}

// ---------------------------------------------------------------------------
// Lattice kernel
// ---------------------------------------------------------------------------
// NT = 1 writes the new populations with non-temporal stores (fp32 ones
// with sc1 as well, see nt_store_policy): they are not read again before
// the next launch, so they need not displace cached lines.
// NTL = 1 reads the populations with non-temporal loads: each is read once
// per launch (neighbouring wavefronts share only the edges of the lines
// that x-streamed populations straddle).
// VIS = 1 (instantiated only while some droplet of the handle has two
// viscosities) takes each cell's relaxation time from the classification.
// BX = 0 is the flat form: a block takes 256 consecutive cells of the
// droplet in storage order, whatever nx is, so rows that are not a multiple
// of 64 cells long leave no lanes idle (a wavefront may then span two rows,
// and the band flag and the row of the classification are read per lane).
// ONE = 1 (a handle holding a single droplet) reads that droplet's
// parameters without waiting for the block's tile entry, so the two loads
// that open every wavefront are in flight together.
template <int DIM, int S, int BX, int NT, int NTL, int VIS, int ONE>
__global__ __launch_bounds__(kBlock) void k_lb(const DropDev* __restrict__ drops,
                                               const int4* __restrict__ tiles,
                                               const typename Codec<S>::T* __restrict__ fsrc_all,
                                               typename Codec<S>::T* __restrict__ fdst_all,
                                               const float* __restrict__ F_all,
                                               unsigned long long* __restrict__ Fq_all,
                                               float* __restrict__ U_all,
                                               float* __restrict__ rho_all,
                                               float* __restrict__ Fout_all,
                                               const uint8_t* __restrict__ flags_all,
                                               uint8_t* __restrict__ flags_clr, int full,
                                               const int* __restrict__ xcnt,
                                               const double* __restrict__ xpos,
                                               int* __restrict__ xclr) {
    using L = Lattice<DIM>;
    using C = Codec<S>;
    constexpr int Q = L::Q;
    constexpr bool FLAT = BX == 0;
    constexpr int BY = FLAT ? 1 : kBlock / (FLAT ? 1 : BX);
    const int4 tile = tiles[blockIdx.x];  // the host lays the list out in block order
    // The droplet's record is read as a whole at the start: read where they
    // are used, its fields were eight scalar loads in a row, each waited for
    // (see Moments for what it gave).
    const DropDev D = drops[ONE ? 0 : tile.x];
    const int nx = D.nx, ny = D.ny, nz = D.nz;
    wanted(tile.y, tile.z, tile.w, D.nx, D.ny, D.nz, D.nstrip, D.bcx, D.bcy, D.bcz, D.ncell, D.f_off, D.c_off,
           D.flag_off, D.omega, D.guo, D.force_mode, D.fst, D.ppl, fsrc_all, fdst_all, Fq_all, U_all, flags_all,
           flags_clr);
    int x, y, z;
    if constexpr (FLAT) {
        const int c = tile.y * kBlock + (int)threadIdx.x;
        if (c >= D.ncell) return;
        const int r = c / nx;
        x = c - r * nx;
        z = r / ny;
        y = r - z * ny;
    } else {
        x = tile.y * BX + (int)(threadIdx.x % (FLAT ? 1 : BX));
        y = tile.z * BY + (int)(threadIdx.x / (FLAT ? 1 : BX));
        z = tile.w;
        if (x >= nx || y >= ny) return;
    }
    const int ncell = D.ncell, fst = D.fst, ppl = D.ppl;
    const int cell = (z * ny + y) * nx + x;  // field arrays
    const int pc = z * ppl + y * nx + x;      // population arrays
    const typename C::T* __restrict__ fsrc = fsrc_all + D.f_off;
    typename C::T* __restrict__ fdst = fdst_all + D.f_off;

    // Source coordinates for c = +1 (xm) and c = -1 (xp), and whether the
    // source lies beyond a wall: the population was reflected there, and the
    // opposite population of this cell is taken (half-way bounce-back).
    // 2D: wrapped coordinates and selects.  3D: -1 marks a wall; the
    // branches that the compiler makes of it space the nineteen loads out,
    // and 256x256x128 fp32 is 1.4 % faster with them (254.5 against 258.2 us
    // per coupled step).
    int xm = x - 1, xp = x + 1, ym = y - 1, yp = y + 1, zm = z - 1, zp = z + 1;
    bool wxm = false, wxp = false, wym = false, wyp = false;
    if constexpr (DIM == 2) {
        const bool wx = D.bcx != 0, wy = D.bcy != 0;
        wxm = wx & (x == 0);
        wxp = wx & (x == nx - 1);
        wym = wy & (y == 0);
        wyp = wy & (y == ny - 1);
        xm = x == 0 ? nx - 1 : xm;
        xp = x == nx - 1 ? 0 : xp;
        ym = y == 0 ? ny - 1 : ym;
        yp = y == ny - 1 ? 0 : yp;
    } else {
        if (xm < 0) xm = D.bcx ? -1 : nx - 1;
        if (xp >= nx) xp = D.bcx ? -1 : 0;
        if (ym < 0) ym = D.bcy ? -1 : ny - 1;
        if (yp >= ny) yp = D.bcy ? -1 : 0;
        if (zm < 0) zm = D.bcz ? -1 : nz - 1;
        if (zp >= nz) zp = D.bcz ? -1 : 0;
    }

    // The band flag of this cell's strip is requested before the
    // populations: loads return in order, so waiting for the flag then does
    // not wait for the populations, and a band wavefront's F loads overlap
    // them instead of following them.  A lone 2D droplet's kernel in fp32 with
    // non-temporal stores requests it after them: its populations come from
    // beyond L2, and the wavefronts outside the band then do not start on a
    // line that the node kernel wrote just before (us per coupled step, early /
    // late: 512x512 10.9 / 10.5, 1024x512 16.8 / 15.4, 1280x640 19.4 / 18.8, but
    // 2048x1024 36.3 / 37.4).  With plain stores late is slower everywhere
    // (1024x512 13.9 / 14.1, 1024x768 15.8 / 16.6, 2048x1024 30.7 / 31.5), as in
    // the 256-droplet fp16 batch (236 / 246).
    // A tiled wavefront reads its strips' flags as one aligned word.
    using SW = typename Strip<DIM, S>::Word;
    constexpr int SPW = Strip<DIM, S>::per64;
    constexpr bool LATE = DIM == 2 && ONE && S == ST_F32 && NT;
    const long long fi = D.flag_off + (long long)(z * ny + y) * D.nstrip + (x >> Strip<DIM, S>::shift);
    int flag;
    auto get_flag = [&](bool given) {
        if constexpr (FLAT) {
            flag = given ? 1 : (int)flags_all[fi];
        } else {
            const SW word = given ? ~SW(0) : *reinterpret_cast<const SW*>(flags_all + (fi & ~(long long)(SPW - 1)));
            flag = (int)((word >> (8 * (int)(fi & (SPW - 1)))) & 0xffu);
        }
    };
    if (!LATE) get_flag(D.force_mode == 1);
    // Populations move through buffer instructions (32-bit lane offsets,
    // base in scalar registers): one descriptor per opposite pair (i,
    // opp(i)), based at the lower index, so that a lane offset never
    // exceeds 2 fst elements and a bounce-back read of opp(i) stays inside
    // the same descriptor.  Q fst < 2^31 elements keeps every offset and
    // size below 2^31 bytes.
    constexpr int SB = storage_bytes<S>();
    float f[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int cx = L::c[i][0], cy = L::c[i][1], cz = L::c[i][2];
        const int sx = cx > 0 ? xm : (cx < 0 ? xp : x);
        const int sy = cy > 0 ? ym : (cy < 0 ? yp : y);
        const int sz = DIM == 3 ? (cz > 0 ? zm : (cz < 0 ? zp : z)) : 0;
        const int lo = i == 0 ? 0 : ((i & 1) ? i : i - 1);
        const auto rs = buffer_of(fsrc + (long long)lo * fst, (i == 0 ? 1 : 2) * fst * SB);
        int rel;
        if constexpr (DIM == 2) {
            bool wall = false;
            if (cx) wall = wall | (cx > 0 ? wxm : wxp);
            if (cy) wall = wall | (cy > 0 ? wym : wyp);
            const int own = (opp(i) - lo) * fst + pc, from = (i - lo) * fst + sy * nx + sx;
            rel = wall ? own : from;
        } else {
            const bool wall = (sx | sy | sz) < 0;
            rel = wall ? (opp(i) - lo) * fst + pc : (i - lo) * fst + sz * ppl + sy * nx + sx;
        }
        f[i] = C::template load_buf<NTL ? kBufNT : 0>(rs, (unsigned)rel * SB);
    }
    if (LATE) get_flag(false);

    const float* __restrict__ F = F_all + (long long)DIM * D.c_off;
    unsigned long long* __restrict__ Fq = Fq_all + (long long)DIM * D.c_off;
    float* __restrict__ U = U_all + (long long)DIM * D.c_off;
    // band: this lane's strip is flagged (band); a wavefront holding any
    // band lane adds the Guo source on every lane (exactly zero where F is)
    bool band, forced;
    float Fx = 0.f, Fy = 0.f, Fz = 0.f;
    unsigned long long q0 = 0, q1 = 0, q2 = 0;
    if (D.force_mode == 1) {
        band = forced = true;
    } else {
        // band flags of this step (set by the spreading); those of the
        // other parity, read by the step before, are cleared for the
        // spreading of the next step by the first lane of each strip
        band = flag != 0;
        forced = __builtin_amdgcn_ballot_w64(band) != 0;
        if constexpr (FLAT) {
            if (flags_clr && (x & (Strip<DIM, S>::n - 1)) == 0) flags_clr[fi] = 0;
        } else {
            if (flags_clr && (x & 63) == 0) *reinterpret_cast<SW*>(flags_clr + fi) = SW(0);
        }
    }
    if (band) {
        if (D.force_mode == 1) {
            Fx = F[cell];
            Fy = F[ncell + cell];
            if (DIM == 3) Fz = F[2 * ncell + cell];
        } else {
            q0 = Fq[cell];
            q1 = Fq[ncell + cell];
            if (DIM == 3) q2 = Fq[2 * ncell + cell];
            Fx = fq_value(q0);
            Fy = fq_value(q1);
            Fz = fq_value(q2);
        }
    }
    const Moments<DIM, S> M(f, Fx, Fy, Fz);
    const float rho = M.rho, ux = M.ux, uy = M.uy, uz = M.uz;
    float om = D.omega, g = D.guo;
    if (VIS && D.visc) {
        // every lane of a wavefront lies in the same row when BX >= 64
        const int row = FLAT ? z * ny + y : __builtin_amdgcn_readfirstlane(z * ny + y);
        if (cell_inside(D, xcnt, xpos, x, row)) {
            om = D.omega_in;
            g = D.guo_in;
        }
        // the other parity's table was read by the previous step: clear it
        // for the crossings of the next step
        if (x == 0 && xclr) xclr[D.row_off + row] = 0;
    }
    auto put = [&](int i, float fn) {
        const int lo = i == 0 ? 0 : ((i & 1) ? i : i - 1);
        const auto rd = buffer_of(fdst + (long long)lo * fst, (i == 0 ? 1 : 2) * fst * SB);
        C::template store_buf<NT ? nt_store_policy<S>() : 0>(rd, (unsigned)pc * SB, (unsigned)((i - lo) * fst) * SB, fn);
    };
    // 3D and 16-bit storage: the source is a branch of the whole wavefront.
    // 2D in fp32 takes one straight path: there the branch costs a small box
    // 1 us a step in instruction fetches and gives nothing to a large one (4
    // droplets 14.1 against 14.0 us per step, 32: 47.6 both).  fp16: 256
    // droplets 151.7 against 157.0 us per launch; with the flag requested
    // early a lone 128x64 box 8.5 against 8.9 us per step, 8192x4096 without
    // an interface 214 against 229 us.
    constexpr bool SPLIT = DIM == 3 || S != ST_F32;
    if (!SPLIT || forced)
        M.template relax<true>(f, om, g, put);
    else
        M.template relax<false>(f, om, g, put);

    if (band && D.force_mode == 0) {
        // interface band: keep U for the interpolation, hand back a clean F
        U[cell] = ux;
        U[ncell + cell] = uy;
        if (DIM == 3) U[2 * ncell + cell] = uz;
        if (q0) Fq[cell] = 0;
        if (q1) Fq[ncell + cell] = 0;
        if (DIM == 3 && q2) Fq[2 * ncell + cell] = 0;
    }
    if (full) {
        float* __restrict__ Fo = Fout_all + (long long)DIM * D.c_off;
        rho_all[D.c_off + cell] = rho;
        U[cell] = ux;
        U[ncell + cell] = uy;
        Fo[cell] = Fx;
        Fo[ncell + cell] = Fy;
        if (DIM == 3) {
            U[2 * ncell + cell] = uz;
            Fo[2 * ncell + cell] = Fz;
        }
    }
}

// Nodes whose coordinates are not finite or lie absurdly far from any box
// (|q| > 2^24) are never turned into tap indices: converting such a value to
// int is undefined and could yield an index far outside the lattice.  The
// kernels skip the node and flag its droplet unstable instead.
constexpr double kFarCoord = 16777216.0;
__device__ __forceinline__ bool coord_ok(double v) { return fabs(v) <= kFarCoord; }  // NaN: false

// Cell index of tap base + k along an axis of n cells: wrapped on a periodic
// axis, -1 beyond a wall.  base comes from a coordinate that passed coord_ok,
// so base + k cannot overflow.  Almost every tap lies in the box: they leave
// first, the wavefront's others take the branches (selects in their place
// made the node kernels slower: 128x64 7.5 against 7.4, 1024x512 14.1 against
// 13.9 us per coupled step).
__device__ __forceinline__ int tap_index(int base, int k, int n, int wall) {
    int i = base + k;
    if (i >= 0 && i < n) return i;
    if (wall) return -1;
    i %= n;
    return i < 0 ? i + n : i;
}

struct NodeArrays {
    const double* pos;   // [3][stride]
    double* pos_w;       // positions of the next step, written by the advection
    float* phi;          // [3][stride]
    float* qdot;         // [3][stride]
    float* dropped;      // [3][stride]
    const int* node_drop;
    const int* tri;      // [3][tstride] global node ids
    const int* inc;      // incidence entries (triangle << 2 | slot)
    const int* inc_beg;
    const int* inc_end;
    const int* perm;     // node ids in spatial (Morton) order, per droplet
    const double* tref;  // [5][tstride] reference triangles of elastic interfaces
    int stride, tstride, ntot;
};

__device__ __forceinline__ double ipow(double s, int n) {
    double p = 1.0;
    for (int k = 0; k < n; ++k) p *= s;
    return p;
}

// Pi(h) of eq. (disjoin-p)
__device__ __forceinline__ double wetting_pi(const DropDev& D, double h) {
    const double s = D.xi / h;
    return D.A * (ipow(s, D.n_exp) - ipow(s, D.m_exp));
}

// Geometry of a node of a 2D closed CCW polygon from its own position q
// and those of its ring neighbours qm (previous) and qp (next):
// surface-tension force sigma (t_j - t_{j-1}), node normal (mean of the
// adjacent outward edge normals), node length chi = l_{j-1} + l_j.
__device__ __forceinline__ void geom_2d(double sigma, const double qm[2], const double q[2],
                                        const double qp[2], double fs[2], double n[2],
                                        double& chi) {
    const double ex = qp[0] - q[0], ey = qp[1] - q[1];
    const double fx = q[0] - qm[0], fy = q[1] - qm[1];
    const double le = sqrt(ex * ex + ey * ey);
    const double lf = sqrt(fx * fx + fy * fy);
    fs[0] = sigma * (ex / le - fx / lf);
    fs[1] = sigma * (ey / le - fy / lf);
    double nx = ey / le + fy / lf, ny = -ex / le - fx / lf;
    const double nn = sqrt(nx * nx + ny * ny);
    n[0] = nx / nn;
    n[1] = ny / nn;
    chi = le + lf;
}

__device__ __forceinline__ void ring_2d(const DropDev& D, int j, int& jm, int& jp) {
    const int N = D.n_nodes, loc = j - D.node_off;
    jm = D.node_off + (loc == 0 ? N - 1 : loc - 1);
    jp = D.node_off + (loc == N - 1 ? 0 : loc + 1);
}

// Tangential re-spacing of a 2D outline, an addition to the method for long
// runs (a line tension has no tangential stiffness, so nodes carried by the
// fluid drift along the outline and open gaps): node m with ring neighbours
// a and b moves by beta/2 (|q_b - q_m| - |q_m - q_a|) along the unit chord
// q_b - q_a, computed from the positions before the advection and added to
// the advected position.  Uniform spacing is left alone.
__device__ __forceinline__ void respace_move(double beta, const double qa[3], const double qm[3],
                                             const double qb[3], double dq[2]) {
    const double lm = sqrt((qm[0] - qa[0]) * (qm[0] - qa[0]) + (qm[1] - qa[1]) * (qm[1] - qa[1]));
    const double lp = sqrt((qb[0] - qm[0]) * (qb[0] - qm[0]) + (qb[1] - qm[1]) * (qb[1] - qm[1]));
    const double cx = qb[0] - qa[0], cy = qb[1] - qa[1];
    const double c = sqrt(cx * cx + cy * cy);
    const double sc = c > 0.0 ? 0.5 * beta * (lp - lm) / c : 0.0;
    dq[0] = sc * cx;
    dq[1] = sc * cy;
}

__device__ __forceinline__ void node_geom_2d(const DropDev& D, const NodeArrays& A, int j,
                                             double q[2], double fs[2], double n[2],
                                             double& chi) {
    int jm, jp;
    ring_2d(D, j, jm, jp);
    const int st = A.stride;
    const double qm[2] = {A.pos[jm], A.pos[st + jm]}, qp[2] = {A.pos[jp], A.pos[st + jp]};
    q[0] = A.pos[j];
    q[1] = A.pos[st + j];
    geom_2d(D.sigma, qm, q, qp, fs, n, chi);
}

// Elastic interface: the shear part w_s = mu_s (b + 1 - e^a) of the strain
// energy, with the invariants a = (1/2) log det G, b = (1/2) tr G - 1 of
// eq. strain_inv (G = F^T F shares the nonzero eigenvalues of D D^T).  The
// in-plane deformation gradient of triangle t is F = [e1 e2] Ei, Ei the
// inverse of its reference edges in a frame of the reference plane (stored
// with the reference area A0 by k_tri_ref).  With d(a)/dF = F G^-1 and
// d(b)/dF = F the energy gradient is dW/dF = A0 mu_s (F - e^a F G^-1);
// dW/dF Ei^T holds dW/dq1 and dW/dq2 in its columns and
// dW/dq0 = -(dW/dq1 + dW/dq2).  Adds -dW/dq of the triangle's slot s to fs.
__device__ __forceinline__ void shear_force(double mu, const NodeArrays& A, int t, int s,
                                            const double e1[3], const double e2[3], double fs[3]) {
    const int ts = A.tstride;
    const double Ei[2][2] = {{A.tref[t], A.tref[ts + t]}, {A.tref[2 * ts + t], A.tref[3 * ts + t]}};
    const double A0 = A.tref[4 * ts + t];
    double F[3][2];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        F[k][0] = e1[k] * Ei[0][0] + e2[k] * Ei[1][0];
        F[k][1] = e1[k] * Ei[0][1] + e2[k] * Ei[1][1];
    }
    const double g00 = F[0][0] * F[0][0] + F[1][0] * F[1][0] + F[2][0] * F[2][0];
    const double g01 = F[0][0] * F[0][1] + F[1][0] * F[1][1] + F[2][0] * F[2][1];
    const double g11 = F[0][1] * F[0][1] + F[1][1] * F[1][1] + F[2][1] * F[2][1];
    const double det = g00 * g11 - g01 * g01;
    const double ea = sqrt(det);
    const double i00 = g11 / det, i01 = -g01 / det, i11 = g00 / det;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double d0 = A0 * mu * (F[k][0] - ea * (F[k][0] * i00 + F[k][1] * i01));
        const double d1 = A0 * mu * (F[k][1] - ea * (F[k][0] * i01 + F[k][1] * i11));
        const double g1 = d0 * Ei[0][0] + d1 * Ei[0][1];
        const double g2 = d0 * Ei[1][0] + d1 * Ei[1][1];
        fs[k] += s == 0 ? g1 + g2 : (s == 1 ? -g1 : -g2);
    }
}

// Contribution of triangle t (vertices P, node j in slot s) to node j: the
// surface-tension force -sigma/2 n_t x (q_c - q_b) (the gradient of sigma
// times the triangle's area), its unit normal and its area; plus the shear
// part of an elastic interface.
__device__ __forceinline__ void tri_contrib(const DropDev& D, const NodeArrays& A, int t, int s,
                                            const double P[3][3], double fs[3], double ns[3],
                                            double& chi) {
    const double e1[3] = {P[1][0] - P[0][0], P[1][1] - P[0][1], P[1][2] - P[0][2]};
    const double e2[3] = {P[2][0] - P[0][0], P[2][1] - P[0][1], P[2][2] - P[0][2]};
    double nt[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                    e1[0] * e2[1] - e1[1] * e2[0]};
    const double len = sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
    nt[0] /= len;
    nt[1] /= len;
    nt[2] /= len;
    const int sb = s == 2 ? 0 : s + 1, sc = s == 0 ? 2 : s - 1;
    const double d[3] = {P[sc][0] - P[sb][0], P[sc][1] - P[sb][1], P[sc][2] - P[sb][2]};
    fs[0] -= 0.5 * D.sigma * (nt[1] * d[2] - nt[2] * d[1]);
    fs[1] -= 0.5 * D.sigma * (nt[2] * d[0] - nt[0] * d[2]);
    fs[2] -= 0.5 * D.sigma * (nt[0] * d[1] - nt[1] * d[0]);
    ns[0] += nt[0];
    ns[1] += nt[1];
    ns[2] += nt[2];
    chi += 0.5 * len;
    if (D.shear != 0.0) shear_force(D.shear, A, t, s, e1, e2, fs);
}

// Incident triangles of a vertex fetched in one batch (icosphere and cap
// meshes have 5-6 per vertex; a vertex with more takes the plain loop).
constexpr int kIncBatch = 8;

// Geometry of vertex j of a closed 3D triangle mesh (CCW seen from
// outside): surface-tension force -sigma d(area)/dq_j summed over the
// incident triangles, vertex normal (mean of the incident unit normals),
// chi = sum of the incident areas.
__device__ __forceinline__ void node_geom_3d(const DropDev& D, const NodeArrays& A, int j,
                                             double q[3], double fs[3], double n[3],
                                             double& chi) {
    const int st = A.stride, ts = A.tstride;
    q[0] = A.pos[j];
    q[1] = A.pos[st + j];
    q[2] = A.pos[2 * st + j];
    fs[0] = fs[1] = fs[2] = 0.0;
    double ns[3] = {0.0, 0.0, 0.0};
    chi = 0.0;
    const int beg = A.inc_beg[j], end = A.inc_end[j];
    if (end > beg && end - beg <= kIncBatch) {
        // the usual vertex (at most kIncBatch triangles): the incidence
        // entries, then the triangles' vertex ids, then the positions of the
        // two other vertices of each are each fetched in one batch, three
        // round trips in all instead of three per triangle; out-of-range
        // slots repeat the last entry and are not summed
        const int cnt = end - beg;
        int e[kIncBatch];
#pragma unroll
        for (int i = 0; i < kIncBatch; ++i) e[i] = A.inc[beg + (i < cnt ? i : cnt - 1)];
        int vb[kIncBatch], vc[kIncBatch];
#pragma unroll
        for (int i = 0; i < kIncBatch; ++i) {
            const int t = e[i] >> 2, s = e[i] & 3;
            const int sb = s == 2 ? 0 : s + 1, sc = s == 0 ? 2 : s - 1;
            vb[i] = A.tri[sb * ts + t];
            vc[i] = A.tri[sc * ts + t];
        }
        double Pb[kIncBatch][3], Pc[kIncBatch][3];
#pragma unroll
        for (int i = 0; i < kIncBatch; ++i)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                Pb[i][a] = A.pos[a * st + vb[i]];
                Pc[i][a] = A.pos[a * st + vc[i]];
            }
#pragma unroll
        for (int i = 0; i < kIncBatch; ++i) {
            if (i >= cnt) break;
            const int t = e[i] >> 2, s = e[i] & 3;
            const int sb = s == 2 ? 0 : s + 1;
            // vertex slot s of triangle t is node j itself
            double P[3][3];
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int a = 0; a < 3; ++a) P[m][a] = m == s ? q[a] : (m == sb ? Pb[i][a] : Pc[i][a]);
            tri_contrib(D, A, t, s, P, fs, ns, chi);
        }
        const double nn = sqrt(ns[0] * ns[0] + ns[1] * ns[1] + ns[2] * ns[2]);
        n[0] = ns[0] / nn;
        n[1] = ns[1] / nn;
        n[2] = ns[2] / nn;
        return;
    }
    for (int k = beg; k < end; ++k) {
        const int e = A.inc[k];
        const int t = e >> 2, s = e & 3;
        const int v0 = A.tri[t], v1 = A.tri[ts + t], v2 = A.tri[2 * ts + t];
        double P[3][3];
        const int vv[3] = {v0, v1, v2};
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            P[m][0] = A.pos[vv[m]];
            P[m][1] = A.pos[st + vv[m]];
            P[m][2] = A.pos[2 * st + vv[m]];
        }
        tri_contrib(D, A, t, s, P, fs, ns, chi);
    }
    const double nn = sqrt(ns[0] * ns[0] + ns[1] * ns[1] + ns[2] * ns[2]);
    n[0] = ns[0] / nn;
    n[1] = ns[1] / nn;
    n[2] = ns[2] / nn;
}

// ---------------------------------------------------------------------------
// Node kernels: one lane per (node, tap)
// ---------------------------------------------------------------------------
// A node owns a group of TAPS consecutive lanes (16 in 2D: 4 nodes per
// wavefront; 64 in 3D: one wavefront per node).  Every lane of the group
// evaluates the node's geometry (same instructions, broadcast loads), then
// handles one tap of the delta kernel; sums over the taps are shuffles
// inside the group.  This turns a serial chain of 16 or 64 scattered
// memory operations per thread into one per lane.
// Droplet of node j.  ONE: the handle holds a single droplet, so the index
// is a compile-time 0 and its record is read through the scalar cache
// instead of per lane after a lookup.
template <bool ONE>
__device__ __forceinline__ int node_droplet(const NodeArrays& A, int j) {
    return ONE ? 0 : A.node_drop[j];
}

// Workgroup size of the node kernels that give each node a group of tap
// lanes (the groups never straddle a wavefront).  One wavefront per
// workgroup spreads the few thousand lanes of a droplet's nodes over four
// times as many compute units as 256-lane workgroups; measured 1.4% faster
// per coupled 1024x512 step, the same in 3D.
#ifndef IBLB_NODE_BLOCK
#define IBLB_NODE_BLOCK 64
#endif
constexpr int kNodeBlock = IBLB_NODE_BLOCK;


template <int DIM>
struct Taps {
    static constexpr int n = DIM == 2 ? 16 : 64;
};

// Lanes per node of the interpolation kernel: one per tap in 2D; in 3D four
// taps per lane (those of a column of the stencil), 16 lanes per vertex, so
// that a lane forms its x and y weights once for four gathers.  80x80x60 /
// 256x256x128 / 240x240x130 (40 962 vertices): 6.9 / 8.5 / 16.1 us per launch
// against 8.5 / 9.5 / 19.1 us with two taps per lane.
template <int DIM>
struct InterpLanes {
    static constexpr int n = 16;
};
// lanes per workgroup of it (3D: 256 lanes 7.7 / 8.9 / 17.1 us against 8.5 /
// 9.5 / 19.1 us with 64, at two taps per lane)
template <int DIM>
constexpr int interp_block() { return DIM == 3 ? kBlock : kNodeBlock; }

// ---------------------------------------------------------------------------
// Peskin 4-point kernel
// ---------------------------------------------------------------------------
// For a node at coordinate q the four taps are the cells base..base+3 with
// base = floor(q - 1/2) - 1, at distances 1 + r, r, 1 - r, 2 - r from the
// node (r = q - 1/2 - floor(q - 1/2) in [0, 1)).  With s = sqrt(1 + 4r - 4r^2)
// both branches of Psi reduce to
//   Psi(1+r) = (3 - 2r - s)/8, Psi(r) = (3 - 2r + s)/8,
//   Psi(1-r) = (1 + 2r + s)/8, Psi(2-r) = (1 + 2r - s)/8,
// so one square root serves all four taps.
//
// peskin_tap: weight of tap k (0..3) of a node at coordinate q, and the
// index of tap 0.
struct PeskinAxis {
    int base;    // index of tap 0
    float r, s;
    __device__ __forceinline__ explicit PeskinAxis(double q) {
        const double u = q - 0.5;
        const double fl = floor(u);
        r = (float)(u - fl);
        base = (int)fl - 1;
        s = sqrtf(1.f + 4.f * r * (1.f - r));
    }
    __device__ __forceinline__ float weight(int k) const {
        const float a = k < 2 ? 3.f - 2.f * r : 1.f + 2.f * r;
        return (a + ((k == 1 || k == 2) ? s : -s)) * 0.125f;
    }
};
__device__ __forceinline__ float peskin_tap(double q, int k, int& base) {
    const PeskinAxis p(q);
    base = p.base;
    return p.weight(k);
}

template <int G>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Lattice cell of this lane's tap, or -1 when it falls beyond a wall; also
// the tap's row (z * ny + y) and x for the band flag.
template <int DIM>
__device__ __forceinline__ int lane_tap(const DropDev& D, const double q[3], int k, float& w,
                                        int& row, int& ix) {
    int bx, by, bz = 0;
    w = peskin_tap(q[0], k & 3, bx) * peskin_tap(q[1], (k >> 2) & 3, by);
    if (DIM == 3) w *= peskin_tap(q[2], k >> 4, bz);
    ix = tap_index(bx, k & 3, D.nx, D.bcx);
    const int iy = tap_index(by, (k >> 2) & 3, D.ny, D.bcy);
    const int iz = DIM == 3 ? tap_index(bz, k >> 4, D.nz, D.bcz) : 0;
    if ((ix | iy | iz) < 0) return -1;
    row = iz * D.ny + iy;
    return row * D.nx + ix;
}

// This lane's tap of the spreading of nodal force ph at q (eq.
// force_spread); with want_dropped the group's wall losses are summed and
// stored by lane 0.
template <int DIM>
__device__ __forceinline__ void spread_lane(const DropDev& D, const NodeArrays& A, int j, int k,
                                            const double q[3], const float ph[3],
                                            unsigned long long* __restrict__ Fq_all,
                                            uint8_t* __restrict__ flags_all, int want_dropped,
                                            int* __restrict__ status_d) {
    constexpr int T = Taps<DIM>::n;
    float w;
    int row, ix;
    const int cell = lane_tap<DIM>(D, q, k, w, row, ix);
    float lost[3] = {0.f, 0.f, 0.f};
    if (cell < 0) {
#pragma unroll
        for (int a = 0; a < DIM; ++a) lost[a] = ph[a] * w;
    } else {
        unsigned long long* __restrict__ Fq = Fq_all + (long long)DIM * D.c_off;
        bool fine = true;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const float v = ph[a] * w;
            if (fq_ok(v))
                atomicAdd(Fq + a * D.ncell + cell, fq_of(v));
            else
                fine = false;
        }
        if (!fine) atomicOr(status_d, 2);
        flags_all[D.flag_off + row * D.nstrip + (ix >> D.sshift)] = 1;
    }
    if (want_dropped) {
#pragma unroll
        for (int a = 0; a < DIM; ++a) lost[a] = group_sum<T>(lost[a]);
        if (k == 0)
#pragma unroll
            for (int a = 0; a < DIM; ++a) A.dropped[a * A.stride + j] = lost[a];
    }
}

// ---------------------------------------------------------------------------
// Nodal forces + spreading (eq. force_spread)
// ---------------------------------------------------------------------------
template <int DIM, bool ONE>
__global__ __launch_bounds__(kNodeBlock) void k_force_spread(const DropDev* __restrict__ drops,
                                                         NodeArrays A,
                                                         unsigned long long* __restrict__ Fq_all,
                                                         uint8_t* __restrict__ flags_all,
                                                         int* __restrict__ status,
                                                         int want_dropped) {
    constexpr int T = Taps<DIM>::n;
    const int gid = blockIdx.x * kNodeBlock + threadIdx.x;
    const int j = gid / T, k = gid % T;
    if (j >= A.ntot) return;
    const int d = node_droplet<ONE>(A, j);
    const DropDev& D = drops[d];
    if (!D.active || D.force_mode != 0) return;
    double q[3] = {0, 0, 0}, fs[3] = {0, 0, 0}, n[3] = {0, 0, 0}, chi;
    double share;
    if (DIM == 2) {
        node_geom_2d(D, A, j, q, fs, n, chi);
        share = 0.5 * chi;
    } else {
        node_geom_3d(D, A, j, q, fs, n, chi);
        share = chi / 3.0;
    }
    if (D.wetting) {
        const double P = wetting_pi(D, q[DIM - 1]);
#pragma unroll
        for (int a = 0; a < DIM; ++a) fs[a] -= share * P * n[a];
    }
    float ph[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int a = 0; a < DIM; ++a) ph[a] = (float)fs[a];
    if (k == 0)
#pragma unroll
        for (int a = 0; a < DIM; ++a) A.phi[a * A.stride + j] = ph[a];
    bool ok = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) ok &= coord_ok(q[a]);
    if (!ok) {  // the whole group leaves together
        if (k == 0) atomicOr(status + d, 4);
        return;
    }
    spread_lane<DIM>(D, A, j, k, q, ph, Fq_all, flags_all, want_dropped, status + d);
}

// Nodes that do not move this step (droplet inactive, prescribed force
// field, or non-finite input) still carry their positions into the buffer
// of the next step.
template <int DIM>
__device__ __forceinline__ void hold_position(const NodeArrays& A, int j, int k) {
    if (k < DIM) A.pos_w[k * A.stride + j] = A.pos[k * A.stride + j];
}

// ---------------------------------------------------------------------------
// Crossings of the interface with the lattice rows (see cell_inside)
// ---------------------------------------------------------------------------
// Record a crossing of droplet row r (z * ny + y) at x.  More than
// kCrossCap crossings on one row set status bit 8.
__device__ __forceinline__ void add_crossing(const DropDev& D, int* __restrict__ cnt,
                                             double* __restrict__ xs, int r, double x,
                                             int* __restrict__ status, int d) {
    const long long rr = (long long)D.row_off + r;
    const int slot = atomicAdd(cnt + rr, 1);
    if (slot < kCrossCap)
        xs[rr * kCrossCap + slot] = x;
    else
        atomicOr(status + d, 8);
}

// Whether a node lies inside the droplet's classification window along its
// periodic axes (along a wall axis the box itself bounds it).  A node
// outside would make the rows' crossings miss or double the interface: the
// crossing kernels then set status bit 16.
template <int DIM>
__device__ __forceinline__ bool in_window(const DropDev& D, const double* q) {
    bool ok = true;
    if (!D.bcx) ok = ok && q[0] >= D.win[0] && q[0] < D.win[0] + D.nx;
    if (!D.bcy) ok = ok && q[1] >= D.win[1] && q[1] < D.win[1] + D.ny;
    if (DIM == 3 && !D.bcz) ok = ok && q[2] >= D.win[2] && q[2] < D.win[2] + D.nz;
    return ok;
}

// Row index of the image j of a row coordinate along an axis of n rows.
__device__ __forceinline__ int wrap_row(int j, int n) {
    j %= n;
    return j < 0 ? j + n : j;
}

// Edge a -> b of a 2D polygon: crossings with the row lines y = j + 1/2
// inside the window, each edge taken half-open in y so that a line through
// a vertex is crossed once by the two edges that share it.  Coordinates
// have passed coord_ok.
__device__ __forceinline__ void cross_edge_2d(const DropDev& D, int* __restrict__ cnt,
                                              double* __restrict__ xs, const double a[2],
                                              const double b[2], int* __restrict__ status, int d) {
    if (!in_window<2>(D, a)) atomicOr(status + d, 16);  // node a of this edge
    const double wlo = D.win[1], whi = D.win[1] + D.ny;
    const double lo = fmax(fmin(a[1], b[1]), wlo), hi = fmin(fmax(a[1], b[1]), whi);
    if (!(lo <= hi)) return;
    const int j0 = (int)ceil(lo - 0.5), j1 = (int)floor(hi - 0.5);
    for (int j = j0; j <= j1; ++j) {
        const double Y = j + 0.5;
        if ((a[1] <= Y) == (b[1] <= Y) || Y < wlo || Y >= whi) continue;
        const double x = a[0] + (Y - a[1]) * (b[0] - a[0]) / (b[1] - a[1]);
        add_crossing(D, cnt, xs, wrap_row(j, D.ny), x, status, d);
    }
}

// Side of the point (y, z) relative to the directed edge P -> Q of a
// triangle projected onto the y-z plane: the sign of the orientation,
// computed from the edge's endpoints in the order of their node ids so that
// the two triangles sharing an edge evaluate the same number; a zero is
// resolved as for the point moved by (eps, eps^2).  val receives the
// orientation itself (for barycentric weights).
__device__ __forceinline__ int edge_side(const double P[3], int ip, const double Q[3], int iq,
                                         double y, double z, double& val) {
    const bool flip = ip > iq;
    const double* A = flip ? Q : P;
    const double* B = flip ? P : Q;
    const double dy = B[1] - A[1], dz = B[2] - A[2];
    const double o = dy * (z - A[2]) - dz * (y - A[1]);
    int sg = o > 0.0 ? 1 : (o < 0.0 ? -1 : 0);
    if (sg == 0) sg = dz != 0.0 ? (dz > 0.0 ? -1 : 1) : (dy > 0.0 ? 1 : (dy < 0.0 ? -1 : 0));
    val = flip ? -o : o;
    return flip ? -sg : sg;
}

// Triangle (node ids i[3], positions P[3][3]): crossings with the row lines
// (y, z) = (j + 1/2, k + 1/2) inside the window whose projection the
// triangle covers; x by barycentric interpolation.
__device__ __forceinline__ void cross_tri_3d(const DropDev& D, int* __restrict__ cnt,
                                             double* __restrict__ xs, const double P[3][3],
                                             const int id[3], int* __restrict__ status, int d) {
    if (!(in_window<3>(D, P[0]) && in_window<3>(D, P[1]) && in_window<3>(D, P[2])))
        atomicOr(status + d, 16);
    const double ylo = D.win[1], yhi = D.win[1] + D.ny, zlo = D.win[2], zhi = D.win[2] + D.nz;
    const double y0 = fmax(fmin(fmin(P[0][1], P[1][1]), P[2][1]), ylo);
    const double y1 = fmin(fmax(fmax(P[0][1], P[1][1]), P[2][1]), yhi);
    const double z0 = fmax(fmin(fmin(P[0][2], P[1][2]), P[2][2]), zlo);
    const double z1 = fmin(fmax(fmax(P[0][2], P[1][2]), P[2][2]), zhi);
    if (!(y0 <= y1 && z0 <= z1)) return;
    const int j0 = (int)ceil(y0 - 0.5), j1 = (int)floor(y1 - 0.5);
    const int k0 = (int)ceil(z0 - 0.5), k1 = (int)floor(z1 - 0.5);
    for (int k = k0; k <= k1; ++k) {
        const double Z = k + 0.5;
        if (Z < zlo || Z >= zhi) continue;
        for (int j = j0; j <= j1; ++j) {
            const double Y = j + 0.5;
            if (Y < ylo || Y >= yhi) continue;
            double e0, e1, e2;
            const int s0 = edge_side(P[1], id[1], P[2], id[2], Y, Z, e0);
            const int s1 = edge_side(P[2], id[2], P[0], id[0], Y, Z, e1);
            const int s2 = edge_side(P[0], id[0], P[1], id[1], Y, Z, e2);
            if (s0 == 0 || s0 != s1 || s1 != s2) continue;
            const double x = (e0 * P[0][0] + e1 * P[1][0] + e2 * P[2][0]) / (e0 + e1 + e2);
            add_crossing(D, cnt, xs, wrap_row(k, D.nz) * D.ny + wrap_row(j, D.ny), x, status, d);
        }
    }
}

// Crossings of the interfaces at the positions A.pos: of the active
// droplets with two viscosities, or of every droplet with an interface when
// all != 0.  2D: one lane per polygon edge (node j to its ring successor).
template <bool ONE>
__global__ __launch_bounds__(kBlock) void k_cross2(const DropDev* __restrict__ drops, NodeArrays A,
                                                   int* __restrict__ cnt, double* __restrict__ xs,
                                                   int* __restrict__ status, int all) {
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= A.ntot) return;
    const int d = node_droplet<ONE>(A, j);
    const DropDev& D = drops[d];
    if (D.force_mode != 0 || !(all || (D.active && D.visc))) return;
    int jm, jp;
    ring_2d(D, j, jm, jp);
    const int st = A.stride;
    const double a[2] = {A.pos[j], A.pos[st + j]}, b[2] = {A.pos[jp], A.pos[st + jp]};
    if (!(coord_ok(a[0]) && coord_ok(a[1]) && coord_ok(b[0]) && coord_ok(b[1]))) {
        atomicOr(status + d, 4);
        return;
    }
    cross_edge_2d(D, cnt, xs, a, b, status, d);
}

// 3D: one lane per triangle.
template <bool ONE>
__global__ __launch_bounds__(kBlock) void k_cross3(const DropDev* __restrict__ drops, NodeArrays A,
                                                   int ttot, int* __restrict__ cnt,
                                                   double* __restrict__ xs, int* __restrict__ status,
                                                   int all) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= ttot) return;
    const int ts = A.tstride, st = A.stride;
    const int id[3] = {A.tri[t], A.tri[ts + t], A.tri[2 * ts + t]};
    const int d = node_droplet<ONE>(A, id[0]);
    const DropDev& D = drops[d];
    if (D.force_mode != 0 || !(all || (D.active && D.visc))) return;
    double P[3][3];
    bool ok = true;
#pragma unroll
    for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P[m][a] = A.pos[a * st + id[m]];
            ok = ok && coord_ok(P[m][a]);
        }
    if (!ok) {
        atomicOr(status + d, 4);
        return;
    }
    cross_tri_3d(D, cnt, xs, P, id, status, d);
}

// Stress-free reference of droplet d's triangles for the elastic interface
// (see shear_force), from the positions A.pos, one lane per triangle:
// frame t1 along the first edge, t2 in the triangle's plane; the inverse of
// the reference edge matrix and the reference area.
__global__ __launch_bounds__(kBlock) void k_tri_ref(const DropDev* __restrict__ drops, int d, NodeArrays A,
                                                    double* __restrict__ tref) {
    const DropDev& D = drops[d];
    const int l = blockIdx.x * kBlock + threadIdx.x;
    if (l >= D.n_tris) return;
    const int t = D.tri_off + l, ts = A.tstride, st = A.stride;
    const int v[3] = {A.tri[t], A.tri[ts + t], A.tri[2 * ts + t]};
    double r1[3], r2[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r1[k] = A.pos[k * st + v[1]] - A.pos[k * st + v[0]];
        r2[k] = A.pos[k * st + v[2]] - A.pos[k * st + v[0]];
    }
    const double l1 = sqrt(r1[0] * r1[0] + r1[1] * r1[1] + r1[2] * r1[2]);
    const double t1[3] = {r1[0] / l1, r1[1] / l1, r1[2] / l1};
    const double n[3] = {r1[1] * r2[2] - r1[2] * r2[1], r1[2] * r2[0] - r1[0] * r2[2],
                         r1[0] * r2[1] - r1[1] * r2[0]};
    double t2[3] = {n[1] * t1[2] - n[2] * t1[1], n[2] * t1[0] - n[0] * t1[2], n[0] * t1[1] - n[1] * t1[0]};
    const double l2 = sqrt(t2[0] * t2[0] + t2[1] * t2[1] + t2[2] * t2[2]);
    t2[0] /= l2;
    t2[1] /= l2;
    t2[2] /= l2;
    const double a = r1[0] * t1[0] + r1[1] * t1[1] + r1[2] * t1[2];
    const double b = r2[0] * t1[0] + r2[1] * t1[1] + r2[2] * t1[2];
    const double c = r1[0] * t2[0] + r1[1] * t2[1] + r1[2] * t2[2];
    const double e = r2[0] * t2[0] + r2[1] * t2[1] + r2[2] * t2[2];
    const double det = a * e - b * c;
    tref[t] = e / det;
    tref[ts + t] = -b / det;
    tref[2 * ts + t] = -c / det;
    tref[3 * ts + t] = a / det;
    tref[4 * ts + t] = 0.5 * sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
}

// Inside (1) / outside (0) of every cell of droplet d from the crossing
// tables, one lane per cell.
__global__ __launch_bounds__(kBlock) void k_inside_mask(const DropDev* __restrict__ drops, int d,
                                                        const int* __restrict__ cnt,
                                                        const double* __restrict__ xs,
                                                        uint8_t* __restrict__ mask) {
    const DropDev& D = drops[d];
    const int cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= D.ncell) return;
    const int x = cell % D.nx, row = cell / D.nx;
    mask[cell] = cell_inside(D, cnt, xs, x, row) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// Interpolation (eq. vel_interpolation) + forward-Euler advection
// ---------------------------------------------------------------------------
template <int DIM, bool ONE>
__global__ __launch_bounds__(interp_block<DIM>()) void k_interp_advect(const DropDev* __restrict__ drops,
                                                          NodeArrays A,
                                                          const float* __restrict__ U_all,
                                                          int* __restrict__ status) {
    // G lanes per node, each taking T / G taps (k, k + G, ...)
    constexpr int T = Taps<DIM>::n, G = InterpLanes<DIM>::n, R = T / G;
    const int gid = blockIdx.x * interp_block<DIM>() + threadIdx.x;
    const int j = gid / G, k = gid % G;
    if (j >= A.ntot) return;
    const int d = node_droplet<ONE>(A, j);
    const DropDev& D = drops[d];
    if constexpr (ONE)
        wanted(D.nx, D.ny, D.nz, D.bcx, D.bcy, D.bcz, D.ncell, D.c_off, D.active, D.force_mode, D.wetting, A.pos,
               A.pos_w, A.qdot, U_all, status);
    const int st = A.stride;
    if (!D.active || D.force_mode != 0) {
        hold_position<DIM>(A, j, k);
        return;
    }
    double q[3] = {0, 0, 0};
    bool ok = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        q[a] = A.pos[a * st + j];
        ok = ok && coord_ok(q[a]);
    }
    if (!ok) {
        hold_position<DIM>(A, j, k);
        if (k == 0) atomicOr(status + d, 4);
        return;
    }
    const float* __restrict__ U = U_all + (long long)DIM * D.c_off;
    float w[R];
    int cell[R];
    if constexpr (DIM == 3) {
        // the taps of a lane share their column: x and y weights once
        static_assert(G % 16 == 0, "taps of a lane differ in z only");
        const PeskinAxis px(q[0]), py(q[1]), pz(q[2]);
        const float wxy = px.weight(k & 3) * py.weight((k >> 2) & 3);
        const int ix = tap_index(px.base, k & 3, D.nx, D.bcx), iy = tap_index(py.base, (k >> 2) & 3, D.ny, D.bcy);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int kz = (k >> 4) + r * (G / 16), iz = tap_index(pz.base, kz, D.nz, D.bcz);
            w[r] = wxy * pz.weight(kz);
            cell[r] = (ix | iy | iz) < 0 ? -1 : (iz * D.ny + iy) * D.nx + ix;
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int row, ix;
            cell[r] = lane_tap<DIM>(D, q, k + r * G, w[r], row, ix);
        }
    }
    // every gather is issued before any is used: a tap beyond a wall, where
    // the fluid is at rest, reads cell 0 with weight zero
    float u[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int c = cell[r] >= 0 ? cell[r] : 0;
#pragma unroll
        for (int a = 0; a < DIM; ++a) u[r][a] = U[a * D.ncell + c];
    }
    // in 3D taps r and r + 2 first, then the two sums: the order of the tree
    // over 32 lanes of two taps each
    float acc[3];
    float wr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wr[r] = cell[r] >= 0 ? w[r] : 0.f;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        if constexpr (DIM == 3)
            acc[a] = __builtin_fmaf(u[2][a], wr[2], u[0][a] * wr[0]) + __builtin_fmaf(u[3][a], wr[3], u[1][a] * wr[1]);
        else
            acc[a] = __builtin_fmaf(u[0][a], wr[0], 0.f);  // (a bare product would be merged into the sum over lanes)
    }
#pragma unroll
    for (int a = 0; a < DIM; ++a) acc[a] = group_sum<G>(acc[a]);
    if (k != 0) return;
    double dq[2] = {0.0, 0.0};
    if (DIM == 2 && D.respace != 0.0) {
        int jm, jp;
        ring_2d(D, j, jm, jp);
        const double qm[3] = {A.pos[jm], A.pos[st + jm], 0.0}, qp[3] = {A.pos[jp], A.pos[st + jp], 0.0};
        if (!(coord_ok(qm[0]) && coord_ok(qm[1]) && coord_ok(qp[0]) && coord_ok(qp[1]))) {
#pragma unroll
            for (int a = 0; a < DIM; ++a) hold_position<DIM>(A, j, a);
            atomicOr(status + d, 4);
            return;
        }
        respace_move(D.respace, qm, q, qp, dq);
    }
    float sp = 0.f;
    double qn[DIM];
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        qn[a] = (q[a] + (double)acc[a]) + (a < 2 ? dq[a] : 0.0);
        A.qdot[a * st + j] = acc[a];
        A.pos_w[a * st + j] = qn[a];
        sp += acc[a] * acc[a];
    }
    int bad = 0;
    if (!(sp <= 0.09f)) bad |= 2;  // |qdot| > 0.3 or not finite
    if (D.wetting && !(qn[DIM - 1] > 0.0)) bad |= 1;
    if (bad) atomicOr(status + d, bad);
}

// ---------------------------------------------------------------------------
// 3D: nodal forces, then spreading aggregated in LDS (eq. force_spread)
// ---------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ double group_sum_d(double v) {
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Forces of every vertex (membrane + wetting): a group of kForceLanes lanes
// per vertex, each lane taking its own incident triangles (one for the
// usual vertex), their contributions summed across the group; the group's
// first lane adds the wetting term and writes the force.  Against one lane
// per vertex that walks its triangles in turn (three batched rounds of
// loads, then 5-6 FP64 triangle evaluations in sequence) the chain per lane
// is one triangle long and the launch has eight times the wavefronts.
constexpr int kForceLanes = 8;
template <bool ONE>
__global__ __launch_bounds__(kBlock) void k_force3(const DropDev* __restrict__ drops, NodeArrays A) {
    const int gid = blockIdx.x * kBlock + threadIdx.x;
    const int j = gid / kForceLanes, k = gid % kForceLanes;
    if (j >= A.ntot) return;  // the whole group leaves together
    const DropDev& D = drops[node_droplet<ONE>(A, j)];
    if (!D.active || D.force_mode != 0) return;
    const int st = A.stride, ts = A.tstride;
    const double q[3] = {A.pos[j], A.pos[st + j], A.pos[2 * st + j]};
    const int beg = A.inc_beg[j], cnt = A.inc_end[j] - beg;
    double fs[3] = {0.0, 0.0, 0.0}, ns[3] = {0.0, 0.0, 0.0}, chi = 0.0;
    for (int i = k; i < cnt; i += kForceLanes) {
        const int e = A.inc[beg + i];
        const int t = e >> 2, s = e & 3;
        const int sb = s == 2 ? 0 : s + 1, sc = s == 0 ? 2 : s - 1;
        const int vb = A.tri[sb * ts + t], vc = A.tri[sc * ts + t];
        // vertex slot s of triangle t is node j itself
        double P[3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P[s][a] = q[a];
            P[sb][a] = A.pos[a * st + vb];
            P[sc][a] = A.pos[a * st + vc];
        }
        tri_contrib(D, A, t, s, P, fs, ns, chi);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        fs[a] = group_sum_d<kForceLanes>(fs[a]);
        ns[a] = group_sum_d<kForceLanes>(ns[a]);
    }
    chi = group_sum_d<kForceLanes>(chi);
    if (k != 0) return;
    if (D.wetting) {
        const double nn = sqrt(ns[0] * ns[0] + ns[1] * ns[1] + ns[2] * ns[2]);
        const double P = wetting_pi(D, q[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) fs[a] -= (chi / 3.0) * P * (ns[a] / nn);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) A.phi[a * A.stride + j] = (float)fs[a];
}

// A workgroup spreads one chunk of up to kChunk vertices that are close in
// space (consecutive in Morton order, cut by the host where the taps' box
// would grow beyond a budget).  Their 64 taps each overlap heavily,
// so the contributions are first summed in an LDS box that covers the
// chunk's taps, and each touched cell then takes one global atomic add per
// component instead of one per contribution.  The chunks are cut when an
// interface is set; where it has been stretched since, and a chunk's box
// exceeds kBoxCells, the chunk is taken in runs of kRun vertices with a box
// each, one after the other, and only a run whose own box is too large adds
// straight to global memory.  336x336x112, 64 002 vertices, a drop spreading
// from a hemisphere, us per coupled step at the start / after 5 000 / after
// 20 000 steps: 570 / 586 / 597 with chunks that added straight to memory,
// 571 / 575 / 576 with runs of 16, 571 / 582 / 583 with 8, 571 / 577 / 582 with
// 32.  The loop over the runs takes registers: without the bound on them a
// compute unit holds one workgroup (80x80x60: 37.9 against 34.3 us per step).
// What bounds it: the adds to global memory (more than half of the time with
// chunks of 16 vertices on 256 lanes), so chunks are as large as one
// workgroup of 16 wavefronts takes in four rounds.  Kernel time on 80x80x60
// (20 252 vertices, four per cell face), 256x256x128 (20 252) and 240x240x130
// (40 962): 17.2 / 19.8 / 33.3 us with 16 vertices, 256 lanes and a 1024-cell
// box; 12.7 / 14.2 / 26.8 with 32 vertices; 9.9 / 12.0 / 21.8 with 64
// vertices, 1024 lanes and 1536 cells; 10.8 / 12.0 / 24.2 with 128 vertices
// and 2048 cells.
#ifndef IBLB_SPREAD_CHUNK
#define IBLB_SPREAD_CHUNK 64
#endif
#ifndef IBLB_SPREAD_BOX
#define IBLB_SPREAD_BOX 1536
#endif
#ifndef IBLB_SPREAD_BLOCK
#define IBLB_SPREAD_BLOCK 1024
#endif
constexpr int kChunk = IBLB_SPREAD_CHUNK;
constexpr int kBoxCells = IBLB_SPREAD_BOX;
constexpr int kRun = 16;         // vertices of a run of a chunk that has outgrown the box
constexpr int kSpreadWaves = 8;  // wavefronts per SIMD: two workgroups on a compute unit
constexpr int kSpreadBlock = IBLB_SPREAD_BLOCK;  // wavefronts each taking every (block / 64)-th vertex
static_assert(3 * kChunk <= kSpreadBlock, "a lane per vertex and axis");

__global__ __launch_bounds__(kSpreadBlock, kSpreadWaves) void k_spread3(const DropDev* __restrict__ drops, NodeArrays A,
                                                    const int4* __restrict__ chunks,
                                                    unsigned long long* __restrict__ Fq_all,
                                                    uint8_t* __restrict__ flags_all,
                                                    int* __restrict__ status, int want_dropped) {
    __shared__ unsigned long long box[3 * kBoxCells];
    __shared__ uint8_t touched[kBoxCells];
    __shared__ float swt[kChunk][3][4];   // weights of the four taps along each axis
    __shared__ int scell[kChunk][3][4];   // their global index, -1 beyond a wall
    __shared__ int sbase[kChunk][3];      // index of tap 0, not wrapped
    __shared__ float sph[kChunk][3];
    __shared__ int sok[kChunk];
    __shared__ int lo[3], hi[3];
    const int4 ch = chunks[blockIdx.x];  // (droplet, first index into perm, count, -)
    const DropDev& D = drops[ch.x];
    const int t = threadIdx.x, st = A.stride, count = ch.z;
    // the chunk's vertices (positions and forces together) are fetched
    // before the droplet's parameters are checked, not after them; lane
    // 3 v + a takes axis a of vertex v
    const int v0 = t / 3, a0 = t - 3 * v0;
    const bool mine = t < 3 * count;
    double q = 0.0;
    float ph = 0.f;
    if (mine) {
        const int j = A.perm[ch.y + v0];
        q = A.pos[a0 * st + j];
        ph = A.phi[a0 * st + j];
    }
    wanted(D.nx, D.ny, D.nz, D.nstrip, D.sshift, D.bcx, D.bcy, D.bcz, D.ncell, D.c_off, D.flag_off, D.force_mode,
           D.active);
    if (!D.active || D.force_mode != 0) return;
    if (t < kChunk) sok[t] = 1;
    if (t < 3) {
        lo[t] = INT_MAX;
        hi[t] = INT_MIN;
    }
    __syncthreads();
    if (mine && !coord_ok(q)) sok[v0] = 0;
    __syncthreads();
    if (mine) {
        if (sok[v0]) {
            // every tap's weight and index is formed once per vertex and axis
            // (formed by each of the 64 tap lanes, they made the kernel wait
            // for its own arithmetic)
            const PeskinAxis p(q);
            const int n = a0 == 0 ? D.nx : (a0 == 1 ? D.ny : D.nz), wall = a0 == 0 ? D.bcx : (a0 == 1 ? D.bcy : D.bcz);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                swt[v0][a0][k] = p.weight(k);
                scell[v0][a0][k] = tap_index(p.base, k, n, wall);
            }
            sbase[v0][a0] = p.base;
            sph[v0][a0] = ph;
            atomicMin(&lo[a0], p.base);
            atomicMax(&hi[a0], p.base);
        } else if (a0 == 0) {
            atomicOr(status + ch.x, 4);
        }
    }
    __syncthreads();
    // without a finite vertex there is no box; each extent (up to 2^25 + 4) is
    // checked by itself, for their product need not fit 64 bits
    int ex, ey, ez;
    bool fits;
    auto measure = [&]() {
        const bool any = lo[0] <= hi[0];
        ex = any ? hi[0] - lo[0] + 4 : 0;
        ey = any ? hi[1] - lo[1] + 4 : 0;
        ez = any ? hi[2] - lo[2] + 4 : 0;
        fits = any && ex <= kBoxCells && ey <= kBoxCells && ez <= kBoxCells && (long long)ex * ey * ez <= kBoxCells;
        return fits || !any;
    };
    const int run = measure() ? kChunk : kRun;
    unsigned long long* __restrict__ Fq = Fq_all + 3LL * D.c_off;
    bool fine = true;
    for (int first = 0; first < count; first += run) {
        const int last = first + run < count ? first + run : count;
        // (what the compiler would form ahead of the loop, reciprocals and
        // addresses of its later parts, delays the chunks of one round: 80x80x60
        // 34.0 against 33.9 us per step)
        const int nx = opaque_uniform(D.nx), ny = opaque_uniform(D.ny), nz = opaque_uniform(D.nz);
        const int t = opaque(threadIdx.x), k = t & 63;  // tap of this lane; one vertex per wavefront at a time
        const int kx = k & 3, ky = (k >> 2) & 3, kz = k >> 4;
        if (run < kChunk) {  // the run's own box
            __syncthreads();
            if (t < 3) {
                lo[t] = INT_MAX;
                hi[t] = INT_MIN;
            }
            __syncthreads();
            if (v0 < last - first && sok[first + v0]) {
                atomicMin(&lo[a0], sbase[first + v0][a0]);
                atomicMax(&hi[a0], sbase[first + v0][a0]);
            }
            __syncthreads();
            measure();
        }
        const int ncb = fits ? ex * ey * ez : 0;
        for (int c = t; c < ncb; c += kSpreadBlock) {
            box[c] = 0;
            box[kBoxCells + c] = 0;
            box[2 * kBoxCells + c] = 0;
            touched[c] = 0;
        }
        __syncthreads();
        const int ktap = fits ? (kz * ey + ky) * ex + kx : 0;  // its place in the box
        for (int v = first + (t >> 6); v < last; v += kSpreadBlock / 64) {
            if (!sok[v]) continue;  // the same for the whole wavefront
            const float w = swt[v][0][kx] * swt[v][1][ky] * swt[v][2][kz];
            const int gx = scell[v][0][kx], gy = scell[v][1][ky], gz = scell[v][2][kz];
            float lost[3] = {0.f, 0.f, 0.f};
            if ((gx | gy | gz) < 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) lost[a] = sph[v][a] * w;
            } else if (fits) {
                const int c = ((sbase[v][2] - lo[2]) * ey + (sbase[v][1] - lo[1])) * ex + (sbase[v][0] - lo[0]) + ktap;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float val = sph[v][a] * w;
                    if (fq_ok(val))
                        atomicAdd(&box[a * kBoxCells + c], fq_of(val));
                    else
                        fine = false;
                }
                touched[c] = 1;
            } else {
                const int row = gz * ny + gy, cell = row * nx + gx;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float val = sph[v][a] * w;
                    if (fq_ok(val))
                        atomicAdd(Fq + a * D.ncell + cell, fq_of(val));
                    else
                        fine = false;
                }
                flags_all[D.flag_off + row * D.nstrip + (gx >> D.sshift)] = 1;
            }
            if (want_dropped) {
#pragma unroll
                for (int a = 0; a < 3; ++a) lost[a] = group_sum<64>(lost[a]);
                if (k == 0) {
                    const int j = A.perm[ch.y + v];
#pragma unroll
                    for (int a = 0; a < 3; ++a) A.dropped[a * st + j] = lost[a];
                }
            }
        }
        if (!fits) continue;
        __syncthreads();
        // c / ex and (c / ex) / ey of c < kBoxCells by the reciprocal: exact, the
        // half keeps the product 2^-11 away from a whole number at least
        const float rx = 1.f / (float)ex, ry = 1.f / (float)ey;
        for (int c = t; c < ncb; c += kSpreadBlock) {
            if (!touched[c]) continue;
            const int r = (int)(((float)c + 0.5f) * rx), cz = (int)(((float)r + 0.5f) * ry);
            const int cx = c - r * ex, cy = r - cz * ey;
            // a touched cell received a fluid tap, so none of these is -1
            const int gx = tap_index(lo[0], cx, nx, D.bcx), gy = tap_index(lo[1], cy, ny, D.bcy),
                      gz = tap_index(lo[2], cz, nz, D.bcz);
            const int row = gz * ny + gy, cell = row * nx + gx;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const unsigned long long v = box[a * kBoxCells + c];
                if (v != 0) atomicAdd(Fq + a * D.ncell + cell, v);
            }
            flags_all[D.flag_off + row * D.nstrip + (gx >> D.sshift)] = 1;
        }
    }
    if (!fine) atomicOr(status + ch.x, 2);
}

// ---------------------------------------------------------------------------
// 2D: interpolation + advection of step t fused with the forces and the
// spreading of step t + 1
// ---------------------------------------------------------------------------
// The lanes of node j's group also interpolate at its two ring neighbours,
// so the new positions that the force at j needs are formed in registers
// and no grid-wide wait separates the two halves.  Reads positions A.pos
// (step t), writes A.pos_w (step t + 1).
template <bool ONE>
__global__ __launch_bounds__(kNodeBlock) void k_ib_fused2(const DropDev* __restrict__ drops, NodeArrays A,
                                                      const float* __restrict__ U_all,
                                                      unsigned long long* __restrict__ Fq_all,
                                                      uint8_t* __restrict__ flags_all,
                                                      int* __restrict__ status, int want_dropped,
                                                      int* __restrict__ xcnt,
                                                      double* __restrict__ xpos) {
    constexpr int T = Taps<2>::n;
    const int gid = blockIdx.x * kNodeBlock + threadIdx.x;
    const int j = gid / T, k = gid % T;
    if (j >= A.ntot) return;
    const int d = node_droplet<ONE>(A, j);
    const int st = A.stride;
    // a lone droplet's ring is nodes 0 .. ntot - 1, so its positions are
    // fetched alongside the droplet's parameters instead of after them
    int jm = 0, jp = 0;
    double q[3][3];
    if constexpr (ONE) {
        jm = j == 0 ? A.ntot - 1 : j - 1;
        jp = j == A.ntot - 1 ? 0 : j + 1;
        const int id[3] = {jm, j, jp};
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            q[m][0] = A.pos[id[m]];
            q[m][1] = A.pos[st + id[m]];
        }
    }
    const DropDev& D = drops[d];
    if (!D.active || D.force_mode != 0) {
        hold_position<2>(A, j, k);
        return;
    }
    if constexpr (!ONE) {
        ring_2d(D, j, jm, jp);
        const int id[3] = {jm, j, jp};
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            q[m][0] = A.pos[id[m]];
            q[m][1] = A.pos[st + id[m]];
        }
    }
    // with re-spacing, the ring neighbours' moves need their own outer
    // neighbours: qo[0] before jm, qo[1] after jp
    const bool resp = D.respace != 0.0;
    double qo[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    if (resp) {
        int jmm, jpp, dummy;
        ring_2d(D, jm, jmm, dummy);
        ring_2d(D, jp, dummy, jpp);
        qo[0][0] = A.pos[jmm];
        qo[0][1] = A.pos[st + jmm];
        qo[1][0] = A.pos[jpp];
        qo[1][1] = A.pos[st + jpp];
    }
    bool ok = !resp || (coord_ok(qo[0][0]) && coord_ok(qo[0][1]) && coord_ok(qo[1][0]) && coord_ok(qo[1][1]));
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        q[m][2] = 0.0;
        ok = ok && coord_ok(q[m][0]) && coord_ok(q[m][1]);
    }
    if (!ok) {
        hold_position<2>(A, j, k);
        if (k == 0) atomicOr(status + d, 4);
        return;
    }
    const float* __restrict__ U = U_all + 2LL * D.c_off;
    float w[3];
    int cell[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        int row, ix;
        cell[m] = lane_tap<2>(D, q[m], k, w[m], row, ix);
    }
    // all six gathers are issued before any is used (a conditional load per
    // tap would wait for each in turn): a tap beyond a wall, where the fluid
    // is at rest, reads cell 0 with weight zero
    float u[3][2];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int c = cell[m] >= 0 ? cell[m] : 0;
        u[m][0] = U[c];
        u[m][1] = U[D.ncell + c];
    }
    float acc[3][2];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float wm = cell[m] >= 0 ? w[m] : 0.f;
        acc[m][0] = u[m][0] * wm;
        acc[m][1] = u[m][1] * wm;
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        acc[m][0] = group_sum<T>(acc[m][0]);
        acc[m][1] = group_sum<T>(acc[m][1]);
    }
    double qn[3][3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        qn[m][0] = q[m][0] + (double)acc[m][0];
        qn[m][1] = q[m][1] + (double)acc[m][1];
        qn[m][2] = 0.0;
    }
    if (resp) {
        double dq[2];
        respace_move(D.respace, qo[0], q[0], q[1], dq);
        qn[0][0] += dq[0];
        qn[0][1] += dq[1];
        respace_move(D.respace, q[0], q[1], q[2], dq);
        qn[1][0] += dq[0];
        qn[1][1] += dq[1];
        respace_move(D.respace, q[1], q[2], qo[1], dq);
        qn[2][0] += dq[0];
        qn[2][1] += dq[1];
    }
    if (k == 0) {
        A.qdot[j] = acc[1][0];
        A.qdot[st + j] = acc[1][1];
        A.pos_w[j] = qn[1][0];
        A.pos_w[st + j] = qn[1][1];
        int bad = 0;
        if (!(acc[1][0] * acc[1][0] + acc[1][1] * acc[1][1] <= 0.09f)) bad |= 2;
        if (D.wetting && !(qn[1][1] > 0.0)) bad |= 1;
        if (bad) atomicOr(status + d, bad);
    }
    ok = true;
#pragma unroll
    for (int m = 0; m < 3; ++m) ok = ok && coord_ok(qn[m][0]) && coord_ok(qn[m][1]);
    if (!ok) {
        if (k == 0) atomicOr(status + d, 4);
        return;
    }
    // crossings of edge j -> j+1 at the new positions, for the next step
    if (D.visc && k == 1) cross_edge_2d(D, xcnt, xpos, qn[1], qn[2], status, d);
    double fs[2], n[2], chi;
    geom_2d(D.sigma, qn[0], qn[1], qn[2], fs, n, chi);
    if (D.wetting) {
        const double P = wetting_pi(D, qn[1][1]);
        fs[0] -= 0.5 * chi * P * n[0];
        fs[1] -= 0.5 * chi * P * n[1];
    }
    const float ph[3] = {(float)fs[0], (float)fs[1], 0.f};
    if (k == 0) {
        A.phi[j] = ph[0];
        A.phi[st + j] = ph[1];
    }
    spread_lane<2>(D, A, j, k, qn[1], ph, Fq_all, flags_all, want_dropped, status + d);
}

// A workgroup takes up to kRingOwn consecutive nodes of one outline and the
// two neighbours beyond them, four lanes each; a lane takes the four taps of
// one column of the stencil:
//   1. every group interpolates at its node;
//   2. two lanes per node advance it and form its force from the new
//      positions of its ring neighbours, which the workgroup has at hand (no
//      grid-wide wait between the halves of a step);
//   3. every group adds its node's force at the new position to a box of
//      cells in LDS, which is then added to memory: one add per touched cell
//      and component instead of one per tap.  A box that would be too large
//      (nodes far apart) is passed by.
// For batches of many nodes, where the adds to memory, a third of which meet
// in the same cells, and after them the arithmetic are what bounds the node
// kernel: k_ib_fused2 makes an add per tap, interpolates at three nodes per
// node and forms the geometry in all of its 16 lanes.  256 droplets, 118 645
// nodes: 83 us per launch with k_ib_fused2; 77 us in stages with 16 lanes per
// node, 69 us with four (19 us of it left with stores in place of the adds),
// 31.5 us with the box.  Workgroups of one wavefront need no waits between
// the stages: 40.4 / 40.8 us with 32 / 64 slots, 36.1 / 40.0 us with 12 / 10.
// A few thousand nodes finish sooner in k_ib_fused2 (see kRingNodes).
//
// The sum over a node's taps starts with the unrounded product of a lane and
// the rounded one of its partner two rows on (a fused multiply-add), so the
// sums for the lower and the upper two rows may differ in their last bit, as
// the lanes' of k_ib_fused2 do.  Each half of the stencil is spread with its
// own sums (that is what the two lanes of a node are for); the lower half's
// are the ones that are stored.
// Reads positions A.pos (step t), writes A.pos_w (step t + 1).
constexpr int kRingSlots = 16;             // nodes of a workgroup, neighbours included
constexpr int kRingOwn = kRingSlots - 2;
constexpr int kRingBlock = 4 * kRingSlots;
constexpr int kRingBox = 256;              // cells of the box: 14 nodes up to 1.1 apart

__global__ __launch_bounds__(kRingBlock) void k_ring2(const DropDev* __restrict__ drops, NodeArrays A,
                                                      const int4* __restrict__ rings,
                                                      const float* __restrict__ U_all,
                                                      unsigned long long* __restrict__ Fq_all,
                                                      uint8_t* __restrict__ flags_all,
                                                      int* __restrict__ status, int want_dropped,
                                                      int* __restrict__ xcnt,
                                                      double* __restrict__ xpos) {
    __shared__ double sq[kRingSlots + 2][2];     // old positions of the nodes and one more at each end
    __shared__ double sn[2][kRingSlots][2];      // new positions, per half
    __shared__ float sacc[2][kRingSlots][2];     // interpolated velocities, per half
    __shared__ float sph[2][kRingSlots][2];      // forces, per half
    __shared__ uint8_t sok[kRingSlots + 2], sgo[2][kRingSlots];
    __shared__ unsigned long long box[2][kRingBox];
    __shared__ uint8_t touched[kRingBox];
    __shared__ int lo[2], hi[2];  // range of the nodes' first taps
    const int4 rb = rings[blockIdx.x];  // (droplet, first of its nodes, count, -)
    const int d = rb.x, count = rb.z;
    const DropDev& D = drops[d];
    const int N = D.n_nodes, off = D.node_off, st = A.stride;
    wanted(D.nx, D.ny, D.nstrip, D.sshift, D.bcx, D.bcy, D.ncell, D.c_off, D.flag_off, D.force_mode, D.active,
           D.wetting, D.n_exp, D.m_exp, D.sigma, D.A, D.xi, D.visc, D.respace, A.pos, U_all, Fq_all, flags_all);
    const int t = threadIdx.x, slot = t >> 2, l = t & 3;
    auto node_of = [&](int e) {  // node of slot e (-1 .. count + 2)
        int id = rb.y - 1 + e;
        id = id < 0 ? id + N : id;
        return off + (id >= N ? id - N : id);
    };
    if (!D.active || D.force_mode != 0) {
        if (slot >= 1 && slot <= count) hold_position<2>(A, node_of(slot), l);
        return;
    }
    for (int c = t; c < kRingBox; c += kRingBlock) {
        box[0][c] = box[1][c] = 0;
        touched[c] = 0;
    }
    if (t < 2) {
        lo[t] = INT_MAX;
        hi[t] = INT_MIN;
    }
    // stage 1: a slot beyond the workgroup's nodes, or a node that is not
    // finite or far off, has no taps
    const bool live = slot < count + 2;
    double q[3] = {0.0, 0.0, 0.0};
    if (live) {
        const int j = node_of(slot);
        q[0] = A.pos[j];
        q[1] = A.pos[st + j];
    }
    double qe[2] = {0.0, 0.0};
    if (t < count + 4) {
        const int j = node_of(t - 1);
        qe[0] = A.pos[j];
        qe[1] = A.pos[st + j];
    }
    const bool fine = live && coord_ok(q[0]) && coord_ok(q[1]);
    float u[4][2] = {}, w[4] = {};
    if (fine) {
        const float* __restrict__ U = U_all + 2LL * D.c_off;
        const PeskinAxis px(q[0]), py(q[1]);
        const float wx = px.weight(l);
        const int ix = tap_index(px.base, l, D.nx, D.bcx);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int iy = tap_index(py.base, r, D.ny, D.bcy);
            // a tap beyond a wall, where the fluid is at rest, reads cell 0
            // with weight zero
            const bool in = (ix | iy) >= 0;
            const int c = in ? iy * D.nx + ix : 0;
            u[r][0] = U[c];
            u[r][1] = U[D.ncell + c];
            w[r] = in ? wx * py.weight(r) : 0.f;
        }
    }
    if (t < count + 4) {
        sq[t][0] = qe[0];
        sq[t][1] = qe[1];
        sok[t] = coord_ok(qe[0]) && coord_ok(qe[1]);
    }
    float sum[2][2];  // [half][component]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma clang fp contract(off)
            const int r = 2 * h, o = 2 - r;
            sum[h][a] = __builtin_fmaf(u[r][a], w[r], u[o][a] * w[o]) +
                        __builtin_fmaf(u[r + 1][a], w[r + 1], u[o + 1][a] * w[o + 1]);
            sum[h][a] += __shfl_xor(sum[h][a], 2, 64);
            sum[h][a] += __shfl_xor(sum[h][a], 1, 64);
        }
    if (l < 2) {
        sacc[l][slot][0] = l == 0 ? sum[0][0] : sum[1][0];
        sacc[l][slot][1] = l == 0 ? sum[0][1] : sum[1][1];
    }
    __syncthreads();
    // stage 2: a lane per half and slot
    const int h = t / kRingSlots, n = t % kRingSlots;
    const bool resp = D.respace != 0.0, moves = h < 2 && n < count + 2;
    float a0 = 0.f, a1 = 0.f;
    if (moves) {
        a0 = sacc[h][n][0];
        a1 = sacc[h][n][1];
        double x = sq[n + 1][0] + (double)a0, y = sq[n + 1][1] + (double)a1;
        if (resp) {
            double dq[2];
            const double qa[3] = {sq[n][0], sq[n][1], 0.0}, qm[3] = {sq[n + 1][0], sq[n + 1][1], 0.0},
                         qb[3] = {sq[n + 2][0], sq[n + 2][1], 0.0};
            respace_move(D.respace, qa, qm, qb, dq);
            x += dq[0];
            y += dq[1];
        }
        sn[h][n][0] = x;
        sn[h][n][1] = y;
    }
    __syncthreads();
    bool go = false;
    if (moves && n >= 1 && n <= count) {
        const int j = node_of(n);
        // the old positions of the node, its neighbours and, with
        // re-spacing, theirs
        bool ok = sok[n] && sok[n + 1] && sok[n + 2];
        if (resp) ok = ok && sok[n - 1] && sok[n + 3];
        if (!ok) {
            if (h == 0) {
                hold_position<2>(A, j, 0);
                hold_position<2>(A, j, 1);
                atomicOr(status + d, 4);
            }
        } else {
            const double qn[3][3] = {{sn[h][n - 1][0], sn[h][n - 1][1], 0.0},
                                     {sn[h][n][0], sn[h][n][1], 0.0},
                                     {sn[h][n + 1][0], sn[h][n + 1][1], 0.0}};
            if (h == 0) {
                A.qdot[j] = a0;
                A.qdot[st + j] = a1;
                A.pos_w[j] = qn[1][0];
                A.pos_w[st + j] = qn[1][1];
                int bad = 0;
                if (!(a0 * a0 + a1 * a1 <= 0.09f)) bad |= 2;
                if (D.wetting && !(qn[1][1] > 0.0)) bad |= 1;
                if (bad) atomicOr(status + d, bad);
            }
            go = true;
#pragma unroll
            for (int m = 0; m < 3; ++m) go = go && coord_ok(qn[m][0]) && coord_ok(qn[m][1]);
            if (!go) {
                if (h == 0) atomicOr(status + d, 4);
            } else {
                // crossings of edge j -> j + 1 at the new positions, for
                // the next step
                if (D.visc && h == 0) cross_edge_2d(D, xcnt, xpos, qn[1], qn[2], status, d);
                double fs[2], nrm[2], chi;
                geom_2d(D.sigma, qn[0], qn[1], qn[2], fs, nrm, chi);
                if (D.wetting) {
                    const double P = wetting_pi(D, qn[1][1]);
                    fs[0] -= 0.5 * chi * P * nrm[0];
                    fs[1] -= 0.5 * chi * P * nrm[1];
                }
                const float f0 = (float)fs[0], f1 = (float)fs[1];
                sph[h][n][0] = f0;
                sph[h][n][1] = f1;
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    const int b = (int)floor(qn[1][a] - 0.5) - 1;
                    atomicMin(&lo[a], b);
                    atomicMax(&hi[a], b);
                }
                if (h == 0) {
                    A.phi[j] = f0;
                    A.phi[st + j] = f1;
                }
            }
        }
    }
    if (h < 2) sgo[h][n] = go;
    __syncthreads();
    // stage 3
    const bool any = lo[0] <= hi[0];
    const int ex = any ? hi[0] - lo[0] + 4 : 0, ey = any ? hi[1] - lo[1] + 4 : 0;
    const bool boxed = any && (long long)ex * ey <= kRingBox;
    unsigned long long* __restrict__ Fq = Fq_all + 2LL * D.c_off;
    float lost[4][2] = {};
    bool sound = true;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (sgo[h][slot]) {
            const PeskinAxis px(sn[h][slot][0]), py(sn[h][slot][1]);
            const float wx = px.weight(l), ph[2] = {sph[h][slot][0], sph[h][slot][1]};
            const int ix = tap_index(px.base, l, D.nx, D.bcx);
#pragma unroll
            for (int r = 2 * h; r < 2 * h + 2; ++r) {
                const int iy = tap_index(py.base, r, D.ny, D.bcy);
                const float ws = wx * py.weight(r), v[2] = {ph[0] * ws, ph[1] * ws};
                if ((ix | iy) < 0) {
                    lost[r][0] = v[0];
                    lost[r][1] = v[1];
                    continue;
                }
                const int c = boxed ? (py.base + r - lo[1]) * ex + (px.base + l - lo[0]) : 0;
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    if (!fq_ok(v[a]))
                        sound = false;
                    else if (boxed)
                        atomicAdd(&box[a][c], fq_of(v[a]));
                    else
                        atomicAdd(Fq + a * D.ncell + iy * D.nx + ix, fq_of(v[a]));
                }
                if (boxed)
                    touched[c] = 1;
                else
                    flags_all[D.flag_off + iy * D.nstrip + (ix >> D.sshift)] = 1;
            }
        }
    }
    if (!sound) atomicOr(status + d, 2);
    if (want_dropped) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma clang fp contract(off)
            float v = (lost[0][a] + lost[2][a]) + (lost[1][a] + lost[3][a]);
            v += __shfl_xor(v, 2, 64);
            v += __shfl_xor(v, 1, 64);
            if (l == 0 && sgo[0][slot]) A.dropped[a * st + node_of(slot)] = v;
        }
    }
    if (!boxed) return;
    __syncthreads();
    const float rx = 1.f / (float)ex;  // (see k_spread3)
    for (int c = t; c < ex * ey; c += kRingBlock) {
        if (!touched[c]) continue;
        const int cy = (int)(((float)c + 0.5f) * rx), cx = c - cy * ex;
        // a touched cell received a fluid tap, so neither is -1
        const int gx = tap_index(lo[0], cx, D.nx, D.bcx), gy = tap_index(lo[1], cy, D.ny, D.bcy);
#pragma unroll
        for (int a = 0; a < 2; ++a)
            if (box[a][c] != 0) atomicAdd(Fq + a * D.ncell + gy * D.nx + gx, box[a][c]);
        flags_all[D.flag_off + gy * D.nstrip + (gx >> D.sshift)] = 1;
    }
}

// ---------------------------------------------------------------------------
// Population I/O and initialisation
// ---------------------------------------------------------------------------
// Equilibrium populations (eq. f^eq, deviation form f_eq - w =
// w (rho - 1) + w rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2)) from a density field
// (null: 1) and a velocity field [dim][ncell] (null: 0), one lane per cell.
// nxy cells per plane of the fields, ppl elements per plane of the
// population arrays.
__device__ __forceinline__ int pop_cell(int cell, int nxy, int ppl) { return cell + cell / nxy * (ppl - nxy); }

template <int DIM, int S>
__global__ void k_init_eq(typename Codec<S>::T* __restrict__ f, int ncell, int fst, int nxy, int ppl,
                          const float* __restrict__ rho_in, const float* __restrict__ u_in) {
    using L = Lattice<DIM>;
    const int cell = blockIdx.x * kBlock + threadIdx.x;
    if (cell >= ncell) return;
    const int pc = pop_cell(cell, nxy, ppl);
    const float rho = rho_in ? rho_in[cell] : 1.f;
    float u[3] = {0.f, 0.f, 0.f};
    if (u_in)
#pragma unroll
        for (int a = 0; a < DIM; ++a) u[a] = u_in[a * ncell + cell];
    const float usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        const float cu = L::c[i][0] * u[0] + L::c[i][1] * u[1] + (DIM == 3 ? L::c[i][2] * u[2] : 0.f);
        const float v = L::w[i] * ((rho - 1.f) + rho * (3.f * cu + 4.5f * cu * cu - 1.5f * usq));
        Codec<S>::store(f, i * fst + pc, v);
    }
}

// Dense [Q][ncell] doubles on the caller's side, population arrays fst
// elements apart in the workspace, their planes ppl elements apart: one
// workgroup per kPopCells cells of population blockIdx.z, four elements per
// lane in flight.  HBM bound; with one lane per element and its index divided
// by the cell count in 64 bits it was not.  The cells are those of plane
// blockIdx.y (then every gridDim.y-th plane), or, where a plane has fewer than
// kPopCells and most lanes would be idle, of the box (FLAT).  us per call to
// write / read (64-bit divisions; by planes; by the box): 240x240x130 fp16 413
// / 487; 302 / 248; 310 / 311, 32x32x4096 fp16 240 / 281; 175 / 126; 183 / 126,
// 16x16x10000 146 / 182; 139 / 106; 113 / 98, 4x4x100000 106 / 119; 587 / 562;
// 89 / 97.
constexpr int kPopCells = 4 * kBlock;
// Cell c of a box: plane c / nxy = c mul >> shift, exact for c < 2^28 (boxes stay
// below: Q cells < 2^31) as mul = ceil(2^shift / nxy), shift = 28 + ceil(log2 nxy).
struct PopPlanes {
    int nxy, ppl, dz, dr;  // kBlock cells on: dz planes and dr cells
    unsigned mul;
    int shift;
    PopPlanes(int cells, int pitch) : nxy(cells), ppl(pitch), dz(kBlock / cells), dr(kBlock % cells), shift(28) {
        while ((1LL << (shift - 28)) < nxy) ++shift;
        mul = (unsigned)(((1ULL << shift) + nxy - 1) / nxy);
    }
    // the places of cells c0, c0 + kBlock, ... in a population array
    __device__ __forceinline__ void places(int c0, int (&at)[4]) const {
        int z = (int)((unsigned long long)c0 * mul >> shift), r = c0 - z * nxy;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            at[u] = z * ppl + r;
            z += dz;
            r += dr;
            if (r >= nxy) {
                r -= nxy;
                ++z;
            }
        }
    }
};
template <int S, bool FLAT>
__global__ __launch_bounds__(kBlock) void k_pop_write(typename Codec<S>::T* __restrict__ f, int ncell, int fst,
                                                      int nz, PopPlanes P, const double* __restrict__ src) {
    const int i = blockIdx.z, c0 = blockIdx.x * kPopCells + threadIdx.x, n = FLAT ? ncell : P.nxy;
    for (int z = blockIdx.y; z < nz; z += gridDim.y) {
        const double* __restrict__ s = src + (long long)i * ncell + (long long)z * P.nxy;
        typename Codec<S>::T* __restrict__ d = f + (long long)i * fst + (long long)z * P.ppl;
        int at[4];
        if (FLAT) P.places(c0, at);
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = c0 + u * kBlock < n ? __builtin_nontemporal_load(s + c0 + u * kBlock) : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + u * kBlock < n) d[FLAT ? at[u] : c0 + u * kBlock] = Codec<S>::from_double(v[u]);
    }
}

template <int S, bool FLAT>
__global__ __launch_bounds__(kBlock) void k_pop_read(const typename Codec<S>::T* __restrict__ f, int ncell, int fst,
                                                     int nz, PopPlanes P, double* __restrict__ dst) {
    const int i = blockIdx.z, c0 = blockIdx.x * kPopCells + threadIdx.x, n = FLAT ? ncell : P.nxy;
    for (int z = blockIdx.y; z < nz; z += gridDim.y) {
        const typename Codec<S>::T* __restrict__ s = f + (long long)i * fst + (long long)z * P.ppl;
        double* __restrict__ d = dst + (long long)i * ncell + (long long)z * P.nxy;
        int at[4];
        if (FLAT) P.places(c0, at);
        typename Codec<S>::T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = s[c0 + u * kBlock < n ? (FLAT ? at[u] : c0 + u * kBlock) : 0];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (c0 + u * kBlock < n) __builtin_nontemporal_store(Codec<S>::to_double(v[u]), d + c0 + u * kBlock);
    }
}

// Streaming copy used to measure the attainable HBM bandwidth of the device:
// each lane moves four 16-byte vectors, all loads issued before the stores.
typedef float v4f __attribute__((ext_vector_type(4)));

template <int NT>
__global__ __launch_bounds__(kBlock) void k_copy_probe(const v4f* __restrict__ src,
                                                       v4f* __restrict__ dst, long long n) {
    const long long base = (long long)blockIdx.x * (4 * kBlock) + threadIdx.x;
    v4f v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const long long i = base + (long long)u * kBlock;
        if (i < n) v[u] = NT ? __builtin_nontemporal_load(src + i) : src[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const long long i = base + (long long)u * kBlock;
        if (i < n) {
            if (NT)
                __builtin_nontemporal_store(v[u], dst + i);
            else
                dst[i] = v[u];
        }
    }
}

__global__ void k_fill_f32(float* __restrict__ p, long long n, float v) {
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------
// Diagnostics
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Partial sums over the cells of a group of consecutive tiles of one droplet
// (groups: droplet, first tile, tiles): [0] sum of f - w, [1..3] rho U,
// [4..6] F of the last step.  HBM bound: the populations and fields are read
// once.  The host makes the groups so large that a big box leaves a few
// thousand partial sums, not one for every tile: k_diag_final reads them
// with one workgroup per droplet (256x256x128: 32 768 tiles took most of a
// millisecond there).
template <int DIM, int S, int BX>
__global__ __launch_bounds__(kBlock) void k_cell_sums(const DropDev* __restrict__ drops,
                                                      const int4* __restrict__ tiles,
                                                      const int4* __restrict__ groups,
                                                      const typename Codec<S>::T* __restrict__ f_all,
                                                      const float* __restrict__ U_all,
                                                      const float* __restrict__ rho_all,
                                                      const float* __restrict__ Fout_all,
                                                      double* __restrict__ partials) {
    __shared__ double sh[kBlock / 64][7];
    using L = Lattice<DIM>;
    constexpr int BY = kBlock / BX;
    const int4 group = groups[blockIdx.x];
    const DropDev& D = drops[group.x];
    const int ncell = D.ncell;
    const typename Codec<S>::T* __restrict__ f = f_all + D.f_off;
    const float* __restrict__ U = U_all + (long long)DIM * D.c_off;
    const float* __restrict__ Fo = Fout_all + (long long)DIM * D.c_off;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int t = group.y; t < group.y + group.z; ++t) {
        const int4 tile = tiles[t];
        const int x = tile.y * BX + (int)(threadIdx.x % BX);
        const int y = tile.z * BY + (int)(threadIdx.x / BX);
        const int z = tile.w;
        if (x < D.nx && y < D.ny) {
            const int cell = (z * D.ny + y) * D.nx + x;
            const int pc = z * D.ppl + y * D.nx + x;
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < L::Q; ++i) s += (double)Codec<S>::load(f, i * D.fst + pc);
            v[0] += s;
            const float rho = rho_all[D.c_off + cell];
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                v[1 + a] += rho * (double)U[a * ncell + cell];
                v[4 + a] += (double)Fo[a * ncell + cell];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const double w = wave_sum(v[k]);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = w;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        const int k = threadIdx.x;
        double r = sh[0][k];
        for (int w = 1; w < kBlock / 64; ++w) r += sh[w][k];
        partials[(long long)blockIdx.x * 8 + k] = r;
    }
}

// Interface reductions in two launches (three in 3D): each workgroup of
// k_diag_part takes one chunk (droplet, chunk) of kBlock nodes and 2 kBlock
// triangles and leaves its partial results in part; one workgroup per droplet
// joins them, in the order of the chunks, in k_diag_final.  Bound by latency
// (scattered reads of a few MB): one workgroup for a whole 20 252-vertex mesh
// took 1020 us, its chunks on 80 take 20 and 16 to join them.
struct Chunk {
    int c, n;      // this workgroup's chunk of n
    double* part;  // partial results of the droplet's chunks
};
enum PartSlot {
    P_PHI = 0, P_DROP = 3, P_VOL = 6, P_AREA, P_HMIN, P_HMAX, P_UN, P_US, P_EMIN, P_EMAX, P_LO, P_HI,
    P_CX, P_CY, P_CN, P_DIST, P_FLAT, P_SLOTS
};
// how the partial results of a slot are joined: 0 sum, 1 min, 2 max
__device__ __forceinline__ int part_kind(int s) {
    return s == P_HMIN || s == P_EMIN || s == P_LO ? 1 : (s == P_HMAX || s == P_UN || s == P_US || s == P_EMAX || s == P_HI ? 2 : 0);
}
__device__ __forceinline__ double part_none(int s) {
    // of an empty interface: nothing below or above
    return s == P_HMIN || s == P_EMIN || s == P_LO ? 1e300 : (s == P_HMAX || s == P_HI ? -1e300 : 0.0);
}
__device__ __forceinline__ double part_two(int kind, double a, double b) {
    return kind == 0 ? a + b : (kind == 1 ? fmin(a, b) : fmax(a, b));
}
__device__ __forceinline__ double wave_join(int kind, double v) {
    return kind == 0 ? wave_sum(v) : (kind == 1 ? wave_min(v) : wave_max(v));
}
// Partial results of slot s of the chunks, joined by this wavefront; every
// lane gets the result.
__device__ __forceinline__ double part_join(const Chunk& ch, int s) {
    if (ch.n == 1) return ch.part[s];
    const int kind = part_kind(s);
    double v = part_none(s);
    for (int b = (int)(threadIdx.x & 63); b < ch.n; b += 64) v = part_two(kind, v, ch.part[(long long)b * P_SLOTS + s]);
    return wave_join(kind, v);
}
// This workgroup's values of the slots first .. first + n - 1 joined over its
// threads and left in part (chunk: the workgroup's (droplet, chunk) entry);
// one barrier for all of them.
template <int n>
__device__ __forceinline__ void part_put(const Chunk& ch, int first, const double (&v)[n]) {
    __shared__ double sh[kBlock / 64][n];
#pragma unroll
    for (int k = 0; k < n; ++k) {
        const double w = wave_join(part_kind(first + k), v[k]);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = w;
    }
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const int k = threadIdx.x;
        double r = sh[0][k];
        for (int w = 1; w < kBlock / 64; ++w) r = part_two(part_kind(first + k), r, sh[w][k]);
        ch.part[(long long)ch.c * P_SLOTS + first + k] = r;
    }
}

// Calls fn(P, v) for this thread's triangles (vertex positions, node ids).
template <typename Fn>
__device__ __forceinline__ void chunk_tris(const DropDev& D, const NodeArrays& A, const Chunk& ch, Fn&& fn) {
    const int st = A.stride, ts = A.tstride;
    for (int l = ch.c * kBlock + (int)threadIdx.x; l < D.n_tris; l += ch.n * kBlock) {
        const int t = D.tri_off + l;
        const int v[3] = {A.tri[t], A.tri[ts + t], A.tri[2 * ts + t]};
        double P[3][3];
#pragma unroll
        for (int m = 0; m < 3; ++m)
#pragma unroll
            for (int a = 0; a < 3; ++a) P[m][a] = A.pos[a * st + v[m]];
        fn(P, v);
    }
}

// Calls fn(x, y) for the points where a triangle's edges, each taken by the
// one of its two triangles that lists it in ascending order, cross the plane
// at height zc.
template <typename Fn>
__device__ __forceinline__ void edge_crossings(const double P[3][3], const int v[3], double zc, Fn&& fn) {
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int m1 = m == 2 ? 0 : m + 1;
        if (v[m] >= v[m1]) continue;
        const double a0 = P[m][2] - zc, a1 = P[m1][2] - zc;
        if (a0 * a1 < 0.0) {
            const double s = a0 / (a0 - a1);
            fn(P[m][0] + s * (P[m1][0] - P[m][0]), P[m][1] + s * (P[m1][1] - P[m][1]));
        }
    }
}

__device__ __forceinline__ double tri_area(const double P[3][3]) {
    const double e1[3] = {P[1][0] - P[0][0], P[1][1] - P[0][1], P[1][2] - P[0][2]};
    const double e2[3] = {P[2][0] - P[0][0], P[2][1] - P[0][1], P[2][2] - P[0][2]};
    const double nt[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2],
                          e1[0] * e2[1] - e1[1] * e2[0]};
    return 0.5 * sqrt(nt[0] * nt[0] + nt[1] * nt[1] + nt[2] * nt[2]);
}

template <int DIM>
__device__ __forceinline__ void diag_part(const DropDev& D, const NodeArrays& A, const Chunk& ch) {
    const int st = A.stride, N = D.n_nodes, j0 = D.node_off;
    double sphi[3] = {0, 0, 0}, sdrop[3] = {0, 0, 0};
    double vol = 0, area = 0, hmin = 1e300, hmax = -1e300, un = 0, us = 0;
    double emin = 1e300, emax = 0, lo = 1e300, hi = -1e300, cx = 0, cy = 0, cn = 0;
    const double zc = D.zcut;
    for (int l = ch.c * kBlock + (int)threadIdx.x; l < N; l += ch.n * kBlock) {
        const int j = j0 + l;
        double q[3], fs[3], n[3], chi;
        if (DIM == 2) {
            node_geom_2d(D, A, j, q, fs, n, chi);
        } else {
            node_geom_3d(D, A, j, q, fs, n, chi);
        }
        double u2 = 0, udn = 0;
        for (int a = 0; a < DIM; ++a) {
            sphi[a] += A.phi[a * st + j];
            sdrop[a] += A.dropped[a * st + j];
            const double v = A.qdot[a * st + j];
            u2 += v * v;
            udn += v * n[a];
        }
        un = fmax(un, fabs(udn));
        us = fmax(us, sqrt(u2));
        hmin = fmin(hmin, q[DIM - 1]);
        hmax = fmax(hmax, q[DIM - 1]);
        if (DIM == 2) {
            const int jp = j0 + (l == N - 1 ? 0 : l + 1);
            const double x0 = q[0], y0 = q[1], x1 = A.pos[jp], y1 = A.pos[st + jp];
            vol += 0.5 * (x0 * y1 - x1 * y0);
            const double e = sqrt((x1 - x0) * (x1 - x0) + (y1 - y0) * (y1 - y0));
            area += e;
            emin = fmin(emin, e);
            emax = fmax(emax, e);
            const double a0 = y0 - zc, a1 = y1 - zc;
            if (a0 * a1 < 0.0 || (a0 == 0.0 && a1 != 0.0)) {
                const double xs = x0 + a0 / (a0 - a1) * (x1 - x0);
                lo = fmin(lo, xs);
                hi = fmax(hi, xs);
            }
        }
    }
    if (DIM == 3)
        chunk_tris(D, A, ch, [&](const double P[3][3], const int v[3]) {
            const double cr[3] = {P[1][1] * P[2][2] - P[1][2] * P[2][1],
                                  P[1][2] * P[2][0] - P[1][0] * P[2][2],
                                  P[1][0] * P[2][1] - P[1][1] * P[2][0]};
            vol += (P[0][0] * cr[0] + P[0][1] * cr[1] + P[0][2] * cr[2]) / 6.0;
            area += tri_area(P);
            for (int m = 0; m < 3; ++m) {
                const int m1 = m == 2 ? 0 : m + 1;
                const double dx = P[m1][0] - P[m][0], dy = P[m1][1] - P[m][1], dz = P[m1][2] - P[m][2];
                const double e = sqrt(dx * dx + dy * dy + dz * dz);
                emin = fmin(emin, e);
                emax = fmax(emax, e);
            }
            edge_crossings(P, v, zc, [&](double x, double y) {
                cx += x;
                cy += y;
                cn += 1.0;
            });
        });
    const double v[P_DIST] = {sphi[0], sphi[1], sphi[2], sdrop[0], sdrop[1], sdrop[2], vol, area, hmin, hmax,
                              un, us, emin, emax, lo, hi, cx, cy, cn};
    part_put(ch, 0, v);
}

// 3D: sum of the crossings' distances from their centre, which every chunk
// forms from all chunks' partial results.  zcut: height of the plane (NaN:
// the droplet's own).
__device__ __forceinline__ void cross_dist(const DropDev& D, const NodeArrays& A, const Chunk& ch, double zcut) {
    const double n = part_join(ch, P_CN);
    const double mx = part_join(ch, P_CX) / n, my = part_join(ch, P_CY) / n;
    double d = 0.0;
    chunk_tris(D, A, ch, [&](const double P[3][3], const int v[3]) {
        edge_crossings(P, v, zcut == zcut ? zcut : D.zcut, [&](double x, double y) {
            d += sqrt((x - mx) * (x - mx) + (y - my) * (y - my));
        });
    });
    const double v[1] = {d};
    part_put(ch, P_DIST, v);
}

// Cell partials + interface partials of droplet D joined by a workgroup of
// BLK lanes.  partials may be null: interface quantities only (cell sums left
// zero).
template <int DIM, int BLK>
__device__ __forceinline__ void diag_final(const DropDev& D, const double* __restrict__ partials, const Chunk& ch,
                                           DiagDev* __restrict__ out) {
    constexpr int W = BLK / 64;
    __shared__ double cells[W][7];
    __shared__ double joined[P_SLOTS];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    if (partials)
        for (int t = D.grp_off + threadIdx.x; t < D.grp_off + D.n_grps; t += BLK)
#pragma unroll
            for (int k = 0; k < 7; ++k) acc[k] += partials[(long long)t * 8 + k];
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        acc[k] = wave_sum(acc[k]);
        if (lane == 0) cells[w][k] = acc[k];
    }
    for (int s = w; s < P_FLAT; s += W) {
        // the crossings' slots are written in 3D only
        const double v = DIM == 3 || s < P_CX ? part_join(ch, s) : 0.0;
        if (lane == 0) joined[s] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    DiagDev r;
    for (int k = 0; k < 7; ++k) {
        acc[k] = cells[0][k];
        for (int u = 1; u < W; ++u) acc[k] += cells[u][k];
    }
    r.mass_dev = acc[0];
    for (int a = 0; a < 3; ++a) {
        r.mom[a] = acc[1 + a];
        r.sum_F[a] = acc[4 + a];
        r.sum_phi[a] = joined[P_PHI + a];
        r.dropped[a] = joined[P_DROP + a];
    }
    r.volume = joined[P_VOL];
    r.area = joined[P_AREA];
    r.min_h = joined[P_HMIN];
    r.max_h = joined[P_HMAX];
    r.max_un = joined[P_UN];
    r.max_u = joined[P_US];
    r.edge_min = joined[P_EMIN];
    r.edge_max = joined[P_EMAX];
    r.cross_lo = joined[P_LO];
    r.cross_hi = joined[P_HI];
    r.cross_n = joined[P_CN];
    r.cross_r = DIM == 3 ? joined[P_DIST] / joined[P_CN] : 0.0;
    *out = r;
}

// The chunk of this workgroup from the list of all droplets' chunks, and all
// chunks of a droplet for the workgroup that joins them.
__device__ __forceinline__ Chunk chunk_of(const DropDev& D, const int4& blk, double* part) {
    return Chunk{blk.y, D.n_blks, part + (long long)D.blk_off * P_SLOTS};
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_diag_part(const DropDev* __restrict__ drops, NodeArrays A,
                                                      const int4* __restrict__ blocks, double* __restrict__ part) {
    const int4 blk = blocks[blockIdx.x];
    const DropDev& D = drops[blk.x];
    diag_part<DIM>(D, A, chunk_of(D, blk, part));
}
__global__ __launch_bounds__(kBlock) void k_cross_dist(const DropDev* __restrict__ drops, NodeArrays A,
                                                       const int4* __restrict__ blocks, double zcut,
                                                       double* __restrict__ part) {
    const int4 blk = blocks[blockIdx.x];
    const DropDev& D = drops[blk.x];
    cross_dist(D, A, chunk_of(D, blk, part), zcut);
}
constexpr int kFinalBlock = 1024;
template <int DIM>
__global__ __launch_bounds__(kFinalBlock) void k_diag_final(const DropDev* __restrict__ drops,
                                                            const double* __restrict__ partials, double* part,
                                                            DiagDev* __restrict__ out) {
    const DropDev& D = drops[blockIdx.x];
    diag_final<DIM, kFinalBlock>(D, partials, chunk_of(D, make_int4(0, 0, 0, 0), part), out + blockIdx.x);
}
// All of it by one workgroup per droplet that strides over the whole
// interface: for small ones, where the launches would take longer than the
// work.  Up to how many chunks, per dimension (us per call, one workgroup /
// launches): diagnostics 2D 1200 nodes (5 chunks) 61.1 / 61.5, 1700 (7) 62.4 /
// 61.8, 8000 79.8 / 61.4; 3D 362 vertices (2) 76.9 / 78.0, 642 (3) 84.6 / 78.3,
// 4002 177 / 81; contact radius 2D 4000 (16) 34.0 / 36.2, 5000 (20) 35.6 / 36.4,
// 6000 (24) 36.9 / 36.3; 3D 1212 (5) 41.0 / 41.3, 1442 (6) 42.7 / 41.6.
template <int DIM>
constexpr int few_blocks_diag() { return DIM == 2 ? 5 : 2; }
template <int DIM>
constexpr int few_blocks_contact() { return DIM == 2 ? 20 : 5; }
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_diag_one(const DropDev* __restrict__ drops, NodeArrays A,
                                                     const double* __restrict__ partials,
                                                     DiagDev* __restrict__ out) {
    __shared__ double part[P_SLOTS];
    const DropDev& D = drops[blockIdx.x];
    const Chunk ch{0, 1, part};
    diag_part<DIM>(D, A, ch);
    __syncthreads();
    if (DIM == 3) {
        cross_dist(D, A, ch, __builtin_nan(""));
        __syncthreads();
    }
    diag_final<DIM, kBlock>(D, partials, ch, out + blockIdx.x);
}

// Contact radius of one droplet at the positions A.pos by the two protocols
// of Sec. Dynamics.  (i) the interface cut by the plane (2D: line) at height
// zcut: 2D half the distance between the outermost crossings, 3D the mean
// distance of the edge crossings to their centre.  (ii) the flat lower
// region: the elements (2D edges, 3D triangles) whose nodes all lie below
// the mid-height between the lowest and the highest node and differ in
// height by less than tol; 2D half its length, 3D the radius of the disc of
// its area.  Chunks of the droplet (see k_diag_part) on one workgroup each:
// k_contact_height, k_contact_part, in 3D k_cross_dist, then
// k_contact_final, which writes r_i (NaN without crossings), r_ii and the
// number of crossings to out (20 252 vertices: 219 us on one workgroup, about 25
// so).
template <int DIM>
__device__ __forceinline__ void contact_height(const DropDev& D, const NodeArrays& A, const Chunk& ch) {
    double hmin = 1e300, hmax = -1e300;
    for (int l = ch.c * kBlock + (int)threadIdx.x; l < D.n_nodes; l += ch.n * kBlock) {
        const double h = A.pos[(DIM - 1) * A.stride + D.node_off + l];
        hmin = fmin(hmin, h);
        hmax = fmax(hmax, h);
    }
    const double v[2] = {hmin, hmax};
    part_put(ch, P_HMIN, v);
}

template <int DIM>
__device__ __forceinline__ void contact_part(const DropDev& D, const NodeArrays& A, const Chunk& ch, double zcut,
                                             double tol) {
    const int st = A.stride, N = D.n_nodes, j0 = D.node_off;
    const double hmin = part_join(ch, P_HMIN), hmax = part_join(ch, P_HMAX);
    const double mid = 0.5 * (hmin + hmax);
    double lo = 1e300, hi = -1e300, cx = 0.0, cy = 0.0, cn = 0.0, flat = 0.0;
    if (DIM == 2) {
        for (int l = ch.c * kBlock + (int)threadIdx.x; l < N; l += ch.n * kBlock) {
            const int j = j0 + l, jp = j0 + (l == N - 1 ? 0 : l + 1);
            const double x0 = A.pos[j], y0 = A.pos[st + j], x1 = A.pos[jp], y1 = A.pos[st + jp];
            const double a0 = y0 - zcut, a1 = y1 - zcut;
            if (a0 * a1 < 0.0 || (a0 == 0.0 && a1 != 0.0)) {
                const double xs = x0 + a0 / (a0 - a1) * (x1 - x0);
                lo = fmin(lo, xs);
                hi = fmax(hi, xs);
                cn += 1.0;
            }
            if (y0 < mid && y1 < mid && fabs(y1 - y0) < tol)
                flat += sqrt((x1 - x0) * (x1 - x0) + (y1 - y0) * (y1 - y0));
        }
    } else {
        chunk_tris(D, A, ch, [&](const double P[3][3], const int v[3]) {
            edge_crossings(P, v, zcut, [&](double x, double y) {
                cx += x;
                cy += y;
                cn += 1.0;
            });
            const double zlo = fmin(fmin(P[0][2], P[1][2]), P[2][2]);
            const double zhi = fmax(fmax(P[0][2], P[1][2]), P[2][2]);
            if (zhi < mid && zhi - zlo < tol) flat += tri_area(P);
        });
    }
    const double c[5] = {lo, hi, cx, cy, cn}, g[1] = {flat};
    part_put(ch, P_LO, c);
    part_put(ch, P_FLAT, g);
}

// By one wavefront.
template <int DIM>
__device__ __forceinline__ void contact_final(const Chunk& ch, double* __restrict__ out) {
    const double cn = part_join(ch, P_CN), flat = part_join(ch, P_FLAT);
    double ri = __builtin_nan("");
    if (DIM == 2) {
        const double lo = part_join(ch, P_LO), hi = part_join(ch, P_HI);
        if (cn >= 2.0) ri = 0.5 * (hi - lo);
    } else {
        const double dist = part_join(ch, P_DIST);
        if (cn > 0.0) ri = dist / cn;
    }
    if (threadIdx.x == 0) {
        out[0] = ri;
        out[1] = DIM == 2 ? 0.5 * flat : sqrt(flat / 3.14159265358979323846);
        out[2] = cn;
    }
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_contact_height(const DropDev* __restrict__ drops, NodeArrays A,
                                                           const int4* __restrict__ blocks,
                                                           double* __restrict__ part) {
    const int4 blk = blocks[blockIdx.x];
    const DropDev& D = drops[blk.x];
    contact_height<DIM>(D, A, chunk_of(D, blk, part));
}
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_contact_part(const DropDev* __restrict__ drops, NodeArrays A,
                                                         const int4* __restrict__ blocks, double zcut, double tol,
                                                         double* __restrict__ part) {
    const int4 blk = blocks[blockIdx.x];
    const DropDev& D = drops[blk.x];
    contact_part<DIM>(D, A, chunk_of(D, blk, part), zcut, tol);
}
template <int DIM>
__global__ __launch_bounds__(64) void k_contact_final(const DropDev* __restrict__ drops, int d, double* part,
                                                      double* __restrict__ out) {
    contact_final<DIM>(chunk_of(drops[d], make_int4(0, 0, 0, 0), part), out);
}
// One workgroup for a small interface (see k_diag_one).
template <int DIM>
__global__ __launch_bounds__(kBlock) void k_contact_one(const DropDev* __restrict__ drops, int d, NodeArrays A,
                                                        double zcut, double tol, double* __restrict__ out) {
    __shared__ double part[P_SLOTS];
    const DropDev& D = drops[d];
    const Chunk ch{0, 1, part};
    contact_height<DIM>(D, A, ch);
    __syncthreads();
    contact_part<DIM>(D, A, ch, zcut, tol);
    __syncthreads();
    if (DIM == 3) {
        cross_dist(D, A, ch, zcut);
        __syncthreads();
    }
    if (threadIdx.x < 64) contact_final<DIM>(ch, out);
}

}  // namespace iblb
