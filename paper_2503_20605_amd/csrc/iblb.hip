// Host runtime and C ABI of the gfx950 IB-LB wetting solver (see iblb.h).
//
// One handle owns a batch of droplets.  All device arrays are carved from
// the caller's workspace.  A time step in 2D is two launches on the
// caller's stream: k_lb (cells, over a tile list that concatenates every
// active droplet's tiles) and k_ib_fused2 or k_ring2 (nodes: interpolation and
// advection, then the forces and spreading of the next step); in 3D k_lb,
// k_interp_advect, (k_cross3,) k_force3 and k_spread3.  The first step of a
// call spreads its own forces and the last one only interpolates.  Long
// runs replay a hipGraph that holds a fixed, even number of steps, so the
// ping-pong buffers are back in place after every replay.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <tuple>
#include <vector>

// the ABI entry points are the only exported symbols
#pragma GCC visibility push(default)
#include "iblb.h"
#pragma GCC visibility pop
#include "kernels.hpp"

using namespace iblb;

namespace {

// Lattice-kernel variants (autotuner candidates).  The kernel form k = v %
// 16: tiles of 256x1, 128x2 or 64x4 cells per block (shape k % 3),
// ordinary or non-temporal stores ((k / 3) % 2), ordinary or non-temporal
// loads (k / 6) for k < 12; then the flat form (256 consecutive cells per
// block, shape 3) with the four load/store kinds (k = 12 + stores + 2
// loads).  The block order v / 16: 0 deals each XCD one contiguous run of
// tiles, 1 keeps the tiles in storage order (blocks go round-robin to the
// XCDs, so neighbouring tiles run on different XCDs at the same time).
constexpr int kShapes = 4;
constexpr int kForms = 16;
constexpr int kVariants = 2 * kForms;
constexpr int kShapeBX[kShapes] = {256, 128, 64, 0};
constexpr int kShapeBY[kShapes] = {1, 2, 4, 0};
int form_of(int variant) { return variant % kForms; }
int order_of(int variant) { return variant / kForms; }
int shape_of(int variant) { return form_of(variant) < 12 ? form_of(variant) % 3 : 3; }

// Blocks are dealt round-robin to the eight XCDs (block b to XCD b % 8).
// Position of the tile that block b takes when each XCD is to work through
// one contiguous run of the nb tiles (x-neighbouring strips and
// y-neighbouring rows then meet in the same L2).
int xcd_run_tile(int b, int nb) {
    const int q = nb >> 3, r = nb & 7, x = b & 7, l = b >> 3;
    return x < r ? x * (q + 1) + l : r * (q + 1) + (x - r) * q + l;
}
constexpr size_t kAlign = 256;
constexpr int kMaxGraphSteps = 1024;
constexpr int kTimedChunk = 256;  // timed lattice launches between two reads of their events

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

struct Layout {
    // byte offsets into the workspace
    size_t drops, tiles_lb, tiles_all, groups, blocks, rings, part, f0, f1, F, Fq, U, Fout, rho, flags, pos0, pos1, phi, qdot, dropped,
        node_drop, tri, inc, inc_beg, inc_end, perm, chunks, status, partials, diag,
        xcnt0, xcnt1, xpos0, xpos1, tref, total;
    int nchunks;           // capacity of the 3D spreading chunk table
    long long cells;       // sum of cells
    long long flag_bytes;  // sum of band flags
    int ntot, ttot, max_tiles;
    int nblocks = 0;       // interface chunks of all droplets (see k_diag_part)
    int most_blocks = 0;   // of one droplet
    int nrings = 0;        // workgroups of k_ring2, 0: k_ib_fused2 (see kRingNodes)
    int group_tiles = 1;   // tiles per group of the cell sums
    int ngroups = 0;
    long long pop_elems;   // sum over droplets of Q * fst
    std::vector<long long> c_off, flag_off, f_off;
    std::vector<int> fst;
    std::vector<int> node_off, tri_off;
    std::vector<int> row_off;  // first row of each droplet in the crossing tables
    long long rows = 0;        // lattice rows (z, y) of all droplets
};

// Element stride between the Q population arrays of a droplet: the cell
// count rounded up to 64 elements plus kPopPad.  Boxes of power-of-two size
// would otherwise put the Q streams a power of two bytes apart; a pad of 64
// elements measured best over the sizes and storages tried (2-4% faster
// than none on an 8192x4096 D2Q9 box, neutral in 3D).
#ifndef IBLB_POP_PAD
#define IBLB_POP_PAD 64
#endif
constexpr int kPopPad = IBLB_POP_PAD;
#ifndef IBLB_POP_ROUND
#define IBLB_POP_ROUND 64
#endif
constexpr long long kPopRound = IBLB_POP_ROUND;
// Element stride between the z-planes of a 3D population array: nx ny plus
// kPlanePad.  With power-of-two planes the streams of the populations that
// move along z sit a power of two bytes away from those that do not; a pad
// of 32-64 elements made the D3Q19 update 3.5% faster on a 256x256x128 box
// (1024 elements: no gain, 512: 7% slower).  Field arrays (rho, U, F) keep
// the compact [z][y][x] layout.
#ifndef IBLB_PLANE_PAD
#define IBLB_PLANE_PAD 64
#endif
constexpr int kPlanePad = IBLB_PLANE_PAD;

// Nodes from which on the 2D node kernel is k_ring2 (see there): its three
// stages take longer than k_ib_fused2's one, 17.2 against 16.5 us per step of
// 8 droplets (3 700 nodes), and win from 12 on (5 500 nodes:
// 20.8 against 21.3; 32: 33.9 against 40.5).  A lone droplet's k_ib_fused2
// reads its ring without the droplet's record and is ahead for longer where
// the nodes are not crowded: up to four nodes per cell of half the box's
// perimeter, at most kRingMost (k_ib_fused2 / k_ring2, us per step: 512x256
// 5120 nodes 16.5 / 14.2; 1024x512 5120 17.0 / 17.7, 7168 17.7 / 17.8, 8192
// 20.8 / 18.0; 2048x1024 5120 33.0 / 35.3, 7168 34.7 / 35.2, 8192 35.7 / 35.6,
// 16384 43.3 / 36.3; fp16 7168 23.9 / 24.7, 8192 25.8 / 25.2).
constexpr int kRingNodes = 5120;
constexpr int kRingMost = 8192;
int ring_nodes(int n, const iblb_params& p) {
    return n > 1 ? kRingNodes : std::min(kRingMost, std::max(kRingNodes, 4 * (p.nx + p.ny)));
}

// Cell budget of a 3D spreading chunk's tap box when the host cuts chunks
// (see morton_order); the kernel's own limit is kBoxCells.
#ifndef IBLB_CHUNK_BUDGET
#define IBLB_CHUNK_BUDGET 1200
#endif

// Band flags per lattice row: one byte per strip of Strip<dim, storage>::n
// cells, padded to a multiple of the strips of 64 cells so that a row's
// flags start on a word boundary.
int strip_shift(int dim, int storage) {
    if (dim == 2) return storage == ST_F32 ? Strip<2, ST_F32>::shift : Strip<2, ST_F16>::shift;
    return Strip<3, ST_F32>::shift;
}
int strips_of(int nx, int dim, int storage) {
    const int sh = strip_shift(dim, storage), w = 64 >> sh;
    return (ceil_div(nx, 1 << sh) + w - 1) / w * w;
}

long long pop_stride(long long cells) {
    return (cells + kPopRound - 1) / kPopRound * kPopRound + kPopPad;
}

// Elements per z-plane of a population array (2D: the whole box).
long long plane_pitch(const iblb_params& p, int dim) {
    return (long long)p.nx * p.ny + (dim == 3 ? kPlanePad : 0);
}

int tiles_of(const iblb_params& p, int shape) {
    if (kShapeBX[shape] == 0) return ceil_div(p.nx * p.ny * (p.dim == 3 ? p.nz : 1), kBlock);
    const int bx = kShapeBX[shape], by = kShapeBY[shape];
    return ceil_div(p.nx, bx) * ceil_div(p.ny, by) * (p.dim == 3 ? p.nz : 1);
}

// Chunks of kBlock nodes and 2 kBlock triangles of an interface.
int iface_blocks(int nodes, int tris) { return std::max(ceil_div(nodes, kBlock), ceil_div(tris, 2 * kBlock)); }

bool plan(int n, const iblb_params* P, const int* nn, const int* nt, int storage, Layout& L,
          std::string& err) {
    if (n < 1) { err = "n_droplets must be >= 1"; return false; }
    if (!P || !nn) { err = "params and n_nodes must not be NULL"; return false; }
    if (storage < 0 || storage > 2) { err = "storage must be IBLB_F32, IBLB_F16 or IBLB_BF16"; return false; }
    const int dim = P[0].dim;
    if (dim != 2 && dim != 3) { err = "dim must be 2 or 3"; return false; }
    const int Q = dim == 2 ? 9 : 19;
    const int sb = storage == 0 ? 4 : 2;
    L.cells = 0;
    L.flag_bytes = 0;
    L.ntot = 0;
    L.ttot = 0;
    L.max_tiles = 0;
    L.nblocks = 0;
    L.most_blocks = 0;
    L.nrings = 0;
    L.c_off.assign(n, 0);
    L.f_off.assign(n, 0);
    L.fst.assign(n, 0);
    L.pop_elems = 0;
    L.nchunks = 0;
    L.ngroups = 0;
    L.flag_off.assign(n, 0);
    L.node_off.assign(n, 0);
    L.tri_off.assign(n, 0);
    L.row_off.assign(n, 0);
    L.rows = 0;
    int tiles[kShapes] = {0, 0, 0, 0};
    for (int d = 0; d < n; ++d) {
        const iblb_params& p = P[d];
        char buf[256];
        if (p.dim != dim) { err = "all droplets must share dim"; return false; }
        const int nz = dim == 3 ? p.nz : 1;
        if (p.nx < 1 || p.ny < 1 || nz < 1) {
            snprintf(buf, sizeof buf, "droplet %d: lattice sizes must be >= 1", d);
            err = buf;
            return false;
        }
        const long long cells = (long long)p.nx * p.ny * nz;
        const long long pcells = plane_pitch(p, dim) * nz;
        if ((long long)Q * pop_stride(pcells) >= (1LL << 31)) {
            snprintf(buf, sizeof buf, "droplet %d: Q * cells must stay below 2^31", d);
            err = buf;
            return false;
        }
        if (!(p.tau > 0.5)) {
            snprintf(buf, sizeof buf, "droplet %d: tau must exceed 1/2", d);
            err = buf;
            return false;
        }
        for (int a = 0; a < 3; ++a)
            if (p.bc[a] != IBLB_PERIODIC && p.bc[a] != IBLB_WALL) {
                snprintf(buf, sizeof buf, "droplet %d: bad boundary code", d);
                err = buf;
                return false;
            }
        if (nn[d] < 0 || (nn[d] > 0 && nn[d] < 3)) {
            snprintf(buf, sizeof buf, "droplet %d: an interface needs at least 3 nodes", d);
            err = buf;
            return false;
        }
        if (nn[d] > 0 && p.wetting && !(p.xi > 0.0 && p.n_exp > p.m_exp && p.m_exp >= 1)) {
            snprintf(buf, sizeof buf, "droplet %d: wetting needs xi > 0 and n > m >= 1", d);
            err = buf;
            return false;
        }
        const int T = (dim == 3 && nt) ? nt[d] : 0;
        if (dim == 3 && nn[d] > 0 && T < 4) {
            snprintf(buf, sizeof buf, "droplet %d: a closed 3D mesh needs >= 4 triangles", d);
            err = buf;
            return false;
        }
        L.c_off[d] = L.cells;
        L.cells += cells;
        L.fst[d] = pop_stride(pcells);
        L.f_off[d] = L.pop_elems;
        L.pop_elems += (long long)Q * L.fst[d];
        if (L.pop_elems >= (1LL << 40)) { err = "population arrays too large"; return false; }
        L.flag_off[d] = L.flag_bytes;
        L.flag_bytes += (long long)nz * p.ny * strips_of(p.nx, dim, storage);
        L.node_off[d] = L.ntot;
        L.ntot += nn[d];
        if (dim == 3) L.nchunks += nn[d];  // capacity: at worst one vertex per chunk
        L.tri_off[d] = L.ttot;
        L.ttot += T;
        L.nblocks += iface_blocks(nn[d], T);
        if (dim == 2) L.nrings += ceil_div(nn[d], kRingOwn);
        L.most_blocks = std::max(L.most_blocks, iface_blocks(nn[d], T));
        L.row_off[d] = (int)L.rows;
        L.rows += (long long)p.ny * nz;
        if (L.rows >= (1LL << 31) / kCrossCap) { err = "too many lattice rows"; return false; }
        for (int s = 0; s < kShapes; ++s) tiles[s] += tiles_of(p, s);
    }
    for (int s = 0; s < kShapes; ++s) L.max_tiles = std::max(L.max_tiles, tiles[s]);
    // a few thousand groups for a large box, single tiles for a small one
    L.group_tiles = std::max(1, tiles[0] / 8192);
    for (int d = 0; d < n; ++d) L.ngroups += ceil_div(tiles_of(P[d], 0), L.group_tiles);
    const long long C = L.cells;
    const int N = std::max(L.ntot, 1), T = std::max(L.ttot, 1);
    size_t o = 0;
    if (L.ntot < ring_nodes(n, P[0])) L.nrings = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    L.drops = take(sizeof(DropDev) * n);
    L.tiles_lb = take(sizeof(int4) * L.max_tiles);
    // all tiles, their groups, the interfaces' chunks and the outlines' pieces:
    // one list, uploaded at once
    L.tiles_all = take(sizeof(int4) * ((size_t)tiles[0] + L.ngroups + L.nblocks + L.nrings));
    L.groups = L.tiles_all + sizeof(int4) * tiles[0];
    L.blocks = L.groups + sizeof(int4) * L.ngroups;
    L.rings = L.blocks + sizeof(int4) * L.nblocks;
    L.part = take(sizeof(double) * P_SLOTS * std::max(L.nblocks, 1));
    L.f0 = take((size_t)L.pop_elems * sb);
    L.f1 = take((size_t)L.pop_elems * sb);
    L.F = take(sizeof(float) * dim * C);   // prescribed force fields
    L.Fq = take(sizeof(unsigned long long) * dim * C);  // spread force, fixed point
    L.U = take(sizeof(float) * dim * C);
    L.Fout = take(sizeof(float) * dim * C);
    L.rho = take(sizeof(float) * C);
    L.flags = take(2 * (size_t)L.flag_bytes);  // band flags, one set per step parity
    L.pos0 = take(sizeof(double) * 3 * N);  // positions, one buffer per step parity
    L.pos1 = take(sizeof(double) * 3 * N);
    L.phi = take(sizeof(float) * 3 * N);
    L.qdot = take(sizeof(float) * 3 * N);
    L.dropped = take(sizeof(float) * 3 * N);
    L.node_drop = take(sizeof(int) * N);
    L.tri = take(sizeof(int) * 3 * T);
    L.inc = take(sizeof(int) * 3 * T);
    L.tref = take(sizeof(double) * 5 * T);  // reference triangles of elastic interfaces
    L.inc_beg = take(sizeof(int) * N);
    L.inc_end = take(sizeof(int) * N);
    L.perm = take(sizeof(int) * N);
    L.chunks = take(sizeof(int4) * std::max(L.nchunks, 1));
    L.status = take(sizeof(int) * n);
    L.partials = take(sizeof(double) * 8 * L.max_tiles);
    L.diag = take(sizeof(DiagDev) * n);
    // interface crossings of the lattice rows, one table pair per step parity
    L.xcnt0 = take(sizeof(int) * L.rows);
    L.xcnt1 = take(sizeof(int) * L.rows);
    L.xpos0 = take(sizeof(double) * kCrossCap * L.rows);
    L.xpos1 = take(sizeof(double) * kCrossCap * L.rows);
    L.total = o;
    return true;
}

}  // namespace

struct iblb_ctx {
    int n = 0, dim = 2, Q = 9, storage = 0;
    std::vector<iblb_params> params;
    std::vector<int> n_nodes, n_tris;
    std::vector<DropDev> drops;
    Layout L;
    char* ws = nullptr;
    hipStream_t stream = nullptr, cap_stream = nullptr;
    int cur = 0;  // buffer holding the current post-collision populations
    bool any_visc = false;  // some droplet has two viscosities
    int variant = 0;  // lattice-kernel variant; its tile shape is shape_of(variant)
    int ntiles_lb = 0;
    bool tiles_dirty = true;
    std::vector<int4> tiles_h;
    int graph_steps = 64;
    hipGraphExec_t exec[2] = {nullptr, nullptr};
    hipGraphExec_t lexec = nullptr;                // lattice-only launches (time_lattice)
    int lexec_n = 0, lexec_p = 0;                  // its launch count and start parity
    int timing = 0;  // 0: off; n: every n-th lattice launch of a call carries timing events
    double t_lb = 0.0, t_step = 0.0;
    std::vector<hipEvent_t> events;  // [0, 2): around a whole call; then pairs per timed lattice launch
    long long step = 0;
    std::vector<int> status_h;
    std::vector<std::vector<int4>> chunks_h;  // 3D spreading chunks per droplet
    int nchunks = 0;                          // chunks on the device
    std::vector<char> iface_set;
    std::string err;

    template <typename T>
    T* at(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

namespace {

thread_local std::string g_create_err;

int fail(iblb_ctx* c, int code, const std::string& msg) {
    if (c) c->err = msg; else g_create_err = msg;
    return code;
}

#define HIPCHK(ctx, call)                                                                  \
    do {                                                                                   \
        hipError_t e_ = (call);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(ctx, IBLB_EDEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

double* positions(const iblb_ctx* c, int parity) {
    return c->at<double>(parity ? c->L.pos1 : c->L.pos0);
}

// Node arrays of the step whose populations and positions have parity p:
// positions read from buffer p, advected positions written to buffer p ^ 1.
NodeArrays node_arrays(const iblb_ctx* c, int p) {
    NodeArrays A;
    A.pos = positions(c, p);
    A.pos_w = positions(c, p ^ 1);
    A.phi = c->at<float>(c->L.phi);
    A.qdot = c->at<float>(c->L.qdot);
    A.dropped = c->at<float>(c->L.dropped);
    A.node_drop = c->at<int>(c->L.node_drop);
    A.tri = c->at<int>(c->L.tri);
    A.inc = c->at<int>(c->L.inc);
    A.inc_beg = c->at<int>(c->L.inc_beg);
    A.inc_end = c->at<int>(c->L.inc_end);
    A.perm = c->at<int>(c->L.perm);
    A.tref = c->at<double>(c->L.tref);
    A.stride = std::max(c->L.ntot, 1);
    A.tstride = std::max(c->L.ttot, 1);
    A.ntot = c->L.ntot;
    return A;
}

// Classification window of a droplet centred on ref: [ref - n/2, ref + n/2)
// along a periodic axis, [0, n) along a wall axis; and the x image rule
// of the lattice kernel (cell centre c maps to c + img_base, plus nx when
// c < img_r, which lands in the window).
void set_window(DropDev& D, const int* bc, const double* ref) {
    const int n[3] = {D.nx, D.ny, D.nz};
    for (int a = 0; a < 3; ++a) D.win[a] = bc[a] == IBLB_PERIODIC ? ref[a] - 0.5 * n[a] : 0.0;
    const double k0 = floor(D.win[0] / D.nx);
    D.img_base = k0 * D.nx;
    D.img_r = D.win[0] - D.img_base;
}

// Band flags of step parity p: set by the spreading for a step of that
// parity, read by its lattice update.
uint8_t* band_flags(const iblb_ctx* c, int p) {
    return c->at<uint8_t>(c->L.flags) + (p ? c->L.flag_bytes : 0);
}

// Crossing tables of step parity p (see cell_inside).
int* cross_count(const iblb_ctx* c, int p) { return c->at<int>(p ? c->L.xcnt1 : c->L.xcnt0); }
double* cross_x(const iblb_ctx* c, int p) { return c->at<double>(p ? c->L.xpos1 : c->L.xpos0); }

// Record the interface crossings of the lattice rows at the positions of
// parity p into the tables of parity tp (every droplet with an interface
// when all != 0, else the active ones with two viscosities).  The tables
// must hold no crossings of these droplets yet.
void launch_cross(const iblb_ctx* c, hipStream_t s, int p, int tp, int all) {
    const NodeArrays A = node_arrays(c, p);
    const DropDev* D = c->at<DropDev>(c->L.drops);
    const bool one = c->n == 1;
    int* st = c->at<int>(c->L.status);
    if (c->dim == 2) {
        if (c->L.ntot == 0) return;
        hipLaunchKernelGGL(one ? k_cross2<true> : k_cross2<false>, dim3(ceil_div(c->L.ntot, kBlock)),
                           dim3(kBlock), 0, s, D, A, cross_count(c, tp), cross_x(c, tp), st, all);
    } else {
        if (c->L.ttot == 0) return;
        hipLaunchKernelGGL(one ? k_cross3<true> : k_cross3<false>, dim3(ceil_div(c->L.ttot, kBlock)),
                           dim3(kBlock), 0, s, D, A, c->L.ttot, cross_count(c, tp), cross_x(c, tp),
                           st, all);
    }
}

void drop_graphs(iblb_ctx* c) {
    for (int k = 0; k < 2; ++k) {
        if (c->exec[k]) {
            (void)hipGraphExecDestroy(c->exec[k]);
            c->exec[k] = nullptr;
        }
    }
    if (c->lexec) {
        (void)hipGraphExecDestroy(c->lexec);
        c->lexec = nullptr;
    }
}

void release_streams(iblb_ctx* c) {
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    c->cap_stream = nullptr;
}

int upload_drops(iblb_ctx* c) {
    HIPCHK(c, hipMemcpyAsync(c->at<DropDev>(c->L.drops), c->drops.data(),
                             sizeof(DropDev) * c->n, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return IBLB_OK;
}

// Concatenate the per-droplet spreading chunks into the device table.  The
// chunk count is baked into captured graphs, so they are dropped.
int upload_chunks(iblb_ctx* c) {
    std::vector<int4> all;
    for (const auto& v : c->chunks_h) all.insert(all.end(), v.begin(), v.end());
    if ((long long)all.size() > std::max(c->L.nchunks, 1))
        return fail(c, IBLB_EINVAL, "chunk table overflow");
    if (!all.empty())
        HIPCHK(c, hipMemcpyAsync(c->at<int4>(c->L.chunks), all.data(), sizeof(int4) * all.size(),
                                 hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->nchunks = (int)all.size();
    drop_graphs(c);
    return IBLB_OK;
}

// Tiles of droplet d in the given shape, x fastest, then y, then z.
void push_tiles(const iblb_ctx* c, int d, int shape, std::vector<int4>& v) {
    const iblb_params& p = c->params[d];
    if (kShapeBX[shape] == 0) {  // flat: runs of kBlock cells in storage order
        for (int b = 0; b < tiles_of(p, shape); ++b) v.push_back(make_int4(d, b, 0, 0));
        return;
    }
    const int bx = kShapeBX[shape], by = kShapeBY[shape];
    const int ntx = ceil_div(p.nx, bx), nty = ceil_div(p.ny, by);
    const int nz = c->dim == 3 ? p.nz : 1;
    for (int z = 0; z < nz; ++z)
        for (int ty = 0; ty < nty; ++ty)
            for (int tx = 0; tx < ntx; ++tx) v.push_back(make_int4(d, tx, ty, z));
}

int rebuild_tiles(iblb_ctx* c) {
    std::vector<int4> all, lb, groups, blocks, rings;
    for (int d = 0; d < c->n; ++d) {
        // the list of all tiles (diagnostics) always has shape 0
        DropDev& D = c->drops[d];
        const int first = (int)all.size();
        push_tiles(c, d, 0, all);
        D.grp_off = (int)groups.size();
        for (int t = first; t < (int)all.size(); t += c->L.group_tiles)
            groups.push_back(make_int4(d, t, std::min(c->L.group_tiles, (int)all.size() - t), 0));
        D.n_grps = (int)groups.size() - D.grp_off;
        D.blk_off = (int)blocks.size();
        D.n_blks = iface_blocks(c->n_nodes[d], c->n_tris[d]);
        for (int b = 0; b < D.n_blks; ++b) blocks.push_back(make_int4(d, b, 0, 0));
        if (c->L.nrings > 0) {  // the outline in equal pieces of at most kRingOwn nodes
            const long long N = c->n_nodes[d], np = ceil_div(N, kRingOwn);
            for (long long b = 0; b < np; ++b) {
                const int first = (int)(N * b / np);
                rings.push_back(make_int4(d, first, (int)(N * (b + 1) / np) - first, 0));
            }
        }
        if (c->drops[d].active) push_tiles(c, d, shape_of(c->variant), lb);
    }
    if (order_of(c->variant) == 0) {
        // block b takes tile xcd_run_tile(b): the list is laid out in
        // block order, so the kernel reads entry blockIdx.x
        std::vector<int4> runs(lb.size());
        for (size_t b = 0; b < lb.size(); ++b) runs[b] = lb[xcd_run_tile((int)b, (int)lb.size())];
        lb.swap(runs);
    }
    all.insert(all.end(), groups.begin(), groups.end());
    all.insert(all.end(), blocks.begin(), blocks.end());
    all.insert(all.end(), rings.begin(), rings.end());
    c->ntiles_lb = (int)lb.size();
    HIPCHK(c, hipMemcpyAsync(c->at<int4>(c->L.tiles_all), all.data(), sizeof(int4) * all.size(),
                             hipMemcpyHostToDevice, c->stream));
    if (!lb.empty())
        HIPCHK(c, hipMemcpyAsync(c->at<int4>(c->L.tiles_lb), lb.data(), sizeof(int4) * lb.size(),
                                 hipMemcpyHostToDevice, c->stream));
    int rc = upload_drops(c);  // synchronises: the host vectors may go
    if (rc) return rc;
    drop_graphs(c);
    c->tiles_dirty = false;
    return IBLB_OK;
}

// ---- kernel dispatch -------------------------------------------------------

template <int DIM, int S, int VIS, int ONE>
void launch_lb_v(const iblb_ctx* c, hipStream_t s, int src, int full, const hipEvent_t* ev,
                 bool clear) {
    using T = typename Codec<S>::T;
    T* f[2] = {c->at<T>(c->L.f0), c->at<T>(c->L.f1)};
    const dim3 grid(c->ntiles_lb), block(kBlock);
    // ev (timing only, never under graph capture): a pair of events that
    // the dispatch itself marks at the kernel's start and end
    auto go = [&](auto kern) {
        auto args = std::make_tuple(
            c->at<DropDev>(c->L.drops), c->at<int4>(c->L.tiles_lb), (const T*)f[src], f[src ^ 1],
            (const float*)c->at<float>(c->L.F), c->at<unsigned long long>(c->L.Fq), c->at<float>(c->L.U),
            c->at<float>(c->L.rho), c->at<float>(c->L.Fout),
            (const uint8_t*)band_flags(c, src), clear ? band_flags(c, src ^ 1) : nullptr, full,
            (const int*)cross_count(c, src), (const double*)cross_x(c, src),
            clear ? cross_count(c, src ^ 1) : nullptr);
        std::apply(
            [&](auto... a) {
                if (ev)
                    hipExtLaunchKernelGGL(kern, grid, block, 0, s, ev[0], ev[1], 0, a...);
                else
                    hipLaunchKernelGGL(kern, grid, block, 0, s, a...);
            },
            args);
    };
    switch (form_of(c->variant)) {
        case 0: go(k_lb<DIM, S, 256, 0, 0, VIS, ONE>); break;
        case 1: go(k_lb<DIM, S, 128, 0, 0, VIS, ONE>); break;
        case 2: go(k_lb<DIM, S, 64, 0, 0, VIS, ONE>); break;
        case 3: go(k_lb<DIM, S, 256, 1, 0, VIS, ONE>); break;
        case 4: go(k_lb<DIM, S, 128, 1, 0, VIS, ONE>); break;
        case 5: go(k_lb<DIM, S, 64, 1, 0, VIS, ONE>); break;
        case 6: go(k_lb<DIM, S, 256, 0, 1, VIS, ONE>); break;
        case 7: go(k_lb<DIM, S, 128, 0, 1, VIS, ONE>); break;
        case 8: go(k_lb<DIM, S, 64, 0, 1, VIS, ONE>); break;
        case 9: go(k_lb<DIM, S, 256, 1, 1, VIS, ONE>); break;
        case 10: go(k_lb<DIM, S, 128, 1, 1, VIS, ONE>); break;
        case 11: go(k_lb<DIM, S, 64, 1, 1, VIS, ONE>); break;
        case 12: go(k_lb<DIM, S, 0, 0, 0, VIS, ONE>); break;
        case 13: go(k_lb<DIM, S, 0, 1, 0, VIS, ONE>); break;
        case 14: go(k_lb<DIM, S, 0, 0, 1, VIS, ONE>); break;
        default: go(k_lb<DIM, S, 0, 1, 1, VIS, ONE>); break;
    }
}

// The two-viscosity form of the lattice kernel runs only while some droplet
// needs it (graphs are dropped when that changes); a handle of one droplet
// uses the form whose tiles all belong to droplet 0.
template <int DIM, int S>
void launch_lb_t(const iblb_ctx* c, hipStream_t s, int src, int full, const hipEvent_t* ev,
                 bool clear) {
    if (c->any_visc)
        launch_lb_v<DIM, S, 1, 0>(c, s, src, full, ev, clear);
    else if (c->n == 1)
        launch_lb_v<DIM, S, 0, 1>(c, s, src, full, ev, clear);
    else
        launch_lb_v<DIM, S, 0, 0>(c, s, src, full, ev, clear);
}

template <int DIM>
void launch_lb_d(const iblb_ctx* c, hipStream_t s, int src, int full, const hipEvent_t* ev,
                 bool clear) {
    switch (c->storage) {
        case ST_F32: launch_lb_t<DIM, ST_F32>(c, s, src, full, ev, clear); break;
        case ST_F16: launch_lb_t<DIM, ST_F16>(c, s, src, full, ev, clear); break;
        default: launch_lb_t<DIM, ST_BF16>(c, s, src, full, ev, clear); break;
    }
}

// Lattice update of parity src.  With two viscosities the kernel reads the
// crossing tables of parity src and, with clear, empties those of the other
// parity for the next step's crossings.
void launch_lb(const iblb_ctx* c, hipStream_t s, int src, int full, const hipEvent_t* ev,
               bool clear = true) {
    if (c->ntiles_lb == 0) return;
    if (c->dim == 2) launch_lb_d<2>(c, s, src, full, ev, clear);
    else launch_lb_d<3>(c, s, src, full, ev, clear);
}

// Forces at the positions of parity p, spread for the step of parity p.
void launch_spread(const iblb_ctx* c, hipStream_t s, int p, int want_dropped) {
    if (c->L.ntot == 0) return;
    if (c->any_visc) launch_cross(c, s, p, p, 0);
    const NodeArrays A = node_arrays(c, p);
    const int lanes = c->L.ntot * (c->dim == 2 ? Taps<2>::n : Taps<3>::n);
    const dim3 grid(ceil_div(lanes, kNodeBlock)), block(kNodeBlock);
    const DropDev* D = c->at<DropDev>(c->L.drops);
    const bool one = c->n == 1;
    if (c->dim == 2) {
        hipLaunchKernelGGL((one ? k_force_spread<2, true> : k_force_spread<2, false>), grid, block, 0, s, D,
                           A, c->at<unsigned long long>(c->L.Fq), band_flags(c, p), c->at<int>(c->L.status),
                           want_dropped);
        return;
    }
    hipLaunchKernelGGL(one ? k_force3<true> : k_force3<false>, dim3(ceil_div(c->L.ntot * kForceLanes, kBlock)),
                       dim3(kBlock), 0, s, D, A);
    if (c->nchunks == 0) return;
    hipLaunchKernelGGL(k_spread3, dim3(c->nchunks), dim3(kSpreadBlock), 0, s, D, A,
                       (const int4*)c->at<int4>(c->L.chunks), c->at<unsigned long long>(c->L.Fq),
                       band_flags(c, p), c->at<int>(c->L.status), want_dropped);
}

// Node work after the lattice step of parity p: interpolate and advect
// (positions p -> p ^ 1) and, unless this is the last step of the call,
// compute the forces at the new positions and spread them for the next
// step (one fused launch in 2D).
void launch_after(const iblb_ctx* c, hipStream_t s, int p, bool last, int want_dropped) {
    if (c->L.ntot == 0) return;
    const NodeArrays A = node_arrays(c, p);
    const int lanes = c->L.ntot * (c->dim == 2 ? Taps<2>::n : Taps<3>::n);
    const dim3 grid(ceil_div(lanes, kNodeBlock)), block(kNodeBlock);
    const DropDev* D = c->at<DropDev>(c->L.drops);
    const bool one = c->n == 1;
    const float* U = c->at<float>(c->L.U);
    if (c->dim == 2 && !last) {
        if (c->L.nrings > 0)
            hipLaunchKernelGGL(k_ring2, dim3(c->L.nrings), dim3(kRingBlock), 0, s, D, A,
                               (const int4*)c->at<int4>(c->L.rings), U, c->at<unsigned long long>(c->L.Fq),
                               band_flags(c, p ^ 1), c->at<int>(c->L.status), want_dropped, cross_count(c, p ^ 1),
                               cross_x(c, p ^ 1));
        else
            hipLaunchKernelGGL(one ? k_ib_fused2<true> : k_ib_fused2<false>, grid, block, 0, s, D, A, U,
                               c->at<unsigned long long>(c->L.Fq), band_flags(c, p ^ 1), c->at<int>(c->L.status),
                               want_dropped, cross_count(c, p ^ 1), cross_x(c, p ^ 1));
        return;
    }
    if (c->dim == 2)
        hipLaunchKernelGGL((one ? k_interp_advect<2, true> : k_interp_advect<2, false>), grid, block, 0, s, D, A,
                           U, c->at<int>(c->L.status));
    else
        hipLaunchKernelGGL((one ? k_interp_advect<3, true> : k_interp_advect<3, false>),
                           dim3(ceil_div(c->L.ntot * InterpLanes<3>::n, interp_block<3>())), dim3(interp_block<3>()), 0, s, D, A, U,
                           c->at<int>(c->L.status));
    if (!last) launch_spread(c, s, p ^ 1, want_dropped);
}

// One time step of parity p, its forces already spread: lattice update,
// then the node work (see launch_after).  ev (may be null) is the event
// pair that times the lattice launch.
void launch_step(const iblb_ctx* c, hipStream_t s, int p, bool last, int full, int want_dropped,
                 const hipEvent_t* ev = nullptr) {
    launch_lb(c, s, p, full, ev);
    launch_after(c, s, p, last, want_dropped);
}

int ensure_events(iblb_ctx* c, int need) {
    while ((int)c->events.size() < need) {
        hipEvent_t ev;
        HIPCHK(c, hipEventCreate(&ev));
        c->events.push_back(ev);
    }
    return IBLB_OK;
}

// Graph of graph_steps steps starting from buffer `parity` (none of them
// the last step of a call).
int ensure_graph(iblb_ctx* c, int parity) {
    hipGraphExec_t* slot = &c->exec[parity];
    if (*slot) return IBLB_OK;
    hipGraph_t g = nullptr;
    HIPCHK(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
    int src = parity;
    for (int k = 0; k < c->graph_steps; ++k) {
        launch_step(c, c->cap_stream, src, false, 0, 0);
        src ^= 1;
    }
    hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
    if (e != hipSuccess) return fail(c, IBLB_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e));
    e = hipGraphInstantiate(slot, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        *slot = nullptr;
        return fail(c, IBLB_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(e));
    }
    return IBLB_OK;
}

// Sum of the elapsed times (ms) of the first n event pairs that timed
// lattice launches (events 2 + 2k, 3 + 2k).  Synchronises the stream.
int read_lb_events(iblb_ctx* c, int n, double& ms) {
    HIPCHK(c, hipStreamSynchronize(c->stream));
    ms = 0.0;
    for (int k = 0; k < n; ++k) {
        float t = 0.f;
        HIPCHK(c, hipEventElapsedTime(&t, c->events[2 + 2 * k], c->events[3 + 2 * k]));
        ms += (double)t;
    }
    return IBLB_OK;
}

int check_droplet(const iblb_ctx* c, int d) {
    return c && d >= 0 && d < c->n;
}

template <int S>
void launch_pop_io(iblb_ctx* c, int d, const double* in, double* out) {
    using T = typename Codec<S>::T;
    T* f = c->at<T>(c->cur ? c->L.f1 : c->L.f0) + c->drops[d].f_off;
    const DropDev& D = c->drops[d];
    const PopPlanes P(D.nx * D.ny, D.ppl);
    const bool flat = P.nxy < kPopCells;
    const int nz = flat ? 1 : D.nz;  // rounds over planes
    const dim3 grid(ceil_div(flat ? D.ncell : P.nxy, kPopCells), std::min(nz, 65535), c->Q);
    if (in)
        hipLaunchKernelGGL((flat ? k_pop_write<S, true> : k_pop_write<S, false>), grid, dim3(kBlock), 0, c->stream, f,
                           D.ncell, D.fst, nz, P, in);
    else
        hipLaunchKernelGGL((flat ? k_pop_read<S, true> : k_pop_read<S, false>), grid, dim3(kBlock), 0, c->stream,
                           (const T*)f, D.ncell, D.fst, nz, P, out);
}

int pop_io(iblb_ctx* c, int d, const double* in, double* out) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (!in && !out) return fail(c, IBLB_EINVAL, "NULL population array");
    switch (c->storage) {
        case ST_F32: launch_pop_io<ST_F32>(c, d, in, out); break;
        case ST_F16: launch_pop_io<ST_F16>(c, d, in, out); break;
        default: launch_pop_io<ST_BF16>(c, d, in, out); break;
    }
    HIPCHK(c, hipGetLastError());
    return IBLB_OK;
}

int reset_droplet(iblb_ctx* c, int d) {
    const DropDev& D = c->drops[d];
    const size_t sb = c->storage == ST_F32 ? 4 : 2;
    // zero deviation = rest state, in both buffers
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.f0 + D.f_off * sb, 0, (size_t)c->Q * D.fst * sb, c->stream));
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.f1 + D.f_off * sb, 0, (size_t)c->Q * D.fst * sb, c->stream));
    const size_t vb = sizeof(float) * c->dim * D.ncell, vo = sizeof(float) * c->dim * D.c_off;
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.F + vo, 0, vb, c->stream));
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.Fq + 2 * vo, 0, 2 * vb, c->stream));
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.U + vo, 0, vb, c->stream));
    HIPCHK(c, hipMemsetAsync(c->ws + c->L.Fout + vo, 0, vb, c->stream));
    const iblb_params& p = c->params[d];
    const size_t fb = (size_t)(c->dim == 3 ? p.nz : 1) * p.ny * strips_of(p.nx, c->dim, c->storage);
    HIPCHK(c, hipMemsetAsync(band_flags(c, 0) + D.flag_off, 0, fb, c->stream));
    HIPCHK(c, hipMemsetAsync(band_flags(c, 1) + D.flag_off, 0, fb, c->stream));
    hipLaunchKernelGGL(k_fill_f32, dim3(ceil_div(D.ncell, kBlock)), dim3(kBlock), 0, c->stream,
                       c->at<float>(c->L.rho) + D.c_off, (long long)D.ncell, 1.0f);
    HIPCHK(c, hipGetLastError());
    HIPCHK(c, hipMemsetAsync(c->at<int>(c->L.status) + d, 0, sizeof(int), c->stream));
    return IBLB_OK;
}

double angle_from_height(int dim, double volume, double height) {
    const double ell = 0.5 * height;
    if (!(ell > 0.0) || !(volume > 0.0)) return NAN;
    if (dim == 3) {
        // tan^2(theta/2) = 3 l^3 / (R0^3 - l^3), R0 of the equal-volume sphere
        const double R03 = 3.0 * volume / (4.0 * M_PI);
        const double l3 = ell * ell * ell;
        if (l3 >= R03) return M_PI;
        return 2.0 * atan(sqrt(3.0 * l3 / (R03 - l3)));
    }
    // circular cap of angle theta: area / l^2 = (theta - sin cos) / sin^4(theta/2),
    // decreasing on (0, pi)
    const double target = volume / (ell * ell);
    auto g = [](double th) {
        const double s = sin(0.5 * th);
        return (th - sin(th) * cos(th)) / (s * s * s * s);
    };
    double lo = 1e-6, hi = M_PI;
    if (target <= g(hi)) return M_PI;
    for (int k = 0; k < 200; ++k) {
        const double mid = 0.5 * (lo + hi);
        if (g(mid) > target) lo = mid; else hi = mid;
    }
    return 0.5 * (lo + hi);
}

template <int DIM, int S>
void launch_cell_sums(iblb_ctx* c) {
    using T = typename Codec<S>::T;
    const T* f = c->at<T>(c->cur ? c->L.f1 : c->L.f0);
    const dim3 grid(c->L.ngroups), block(kBlock);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, block, 0, c->stream, c->at<DropDev>(c->L.drops),
                           c->at<int4>(c->L.tiles_all), c->at<int4>(c->L.groups), f, c->at<float>(c->L.U), c->at<float>(c->L.rho),
                           c->at<float>(c->L.Fout), c->at<double>(c->L.partials));
    };
    go(k_cell_sums<DIM, S, 256>);  // tiles of shape 0
}

template <int DIM>
void launch_diag_d(iblb_ctx* c, bool cells = true) {
    if (cells) {
        switch (c->storage) {
            case ST_F32: launch_cell_sums<DIM, ST_F32>(c); break;
            case ST_F16: launch_cell_sums<DIM, ST_F16>(c); break;
            default: launch_cell_sums<DIM, ST_BF16>(c); break;
        }
    }
    const DropDev* D = c->at<DropDev>(c->L.drops);
    const NodeArrays A = node_arrays(c, c->cur);
    const int4* blocks = c->at<int4>(c->L.blocks);
    double* part = c->at<double>(c->L.part);
    const double* sums = cells ? (const double*)c->at<double>(c->L.partials) : nullptr;
    if (c->L.most_blocks <= few_blocks_diag<DIM>()) {
        hipLaunchKernelGGL(k_diag_one<DIM>, dim3(c->n), dim3(kBlock), 0, c->stream, D, A, sums,
                           c->at<DiagDev>(c->L.diag));
        return;
    }
    if (c->L.nblocks > 0) {
        const dim3 grid(c->L.nblocks), block(kBlock);
        hipLaunchKernelGGL(k_diag_part<DIM>, grid, block, 0, c->stream, D, A, blocks, part);
        if (DIM == 3)
            hipLaunchKernelGGL(k_cross_dist, grid, block, 0, c->stream, D, A, blocks, (double)NAN, part);
    }
    hipLaunchKernelGGL(k_diag_final<DIM>, dim3(c->n), dim3(kFinalBlock), 0, c->stream, D,
                       sums, part, c->at<DiagDev>(c->L.diag));
}

template <int DIM>
void launch_contact(iblb_ctx* c, int d, double z_cut, double flat_tol, double* out) {
    const DropDev* D = c->at<DropDev>(c->L.drops);
    const NodeArrays A = node_arrays(c, c->cur);
    // the droplet's own chunks; their partial results lie at its offset
    const int4* blocks = c->at<int4>(c->L.blocks) + c->drops[d].blk_off;
    double* part = c->at<double>(c->L.part);
    const dim3 grid(c->drops[d].n_blks), block(kBlock);
    if (c->drops[d].n_blks <= few_blocks_contact<DIM>()) {
        hipLaunchKernelGGL(k_contact_one<DIM>, dim3(1), block, 0, c->stream, D, d, A, z_cut, flat_tol, out);
        return;
    }
    hipLaunchKernelGGL(k_contact_height<DIM>, grid, block, 0, c->stream, D, A, blocks, part);
    hipLaunchKernelGGL(k_contact_part<DIM>, grid, block, 0, c->stream, D, A, blocks, z_cut, flat_tol, part);
    if (DIM == 3) hipLaunchKernelGGL(k_cross_dist, grid, block, 0, c->stream, D, A, blocks, z_cut, part);
    hipLaunchKernelGGL(k_contact_final<DIM>, dim3(1), dim3(64), 0, c->stream, D, d, part, out);
}

}  // namespace

// ============================================================================
// C ABI
// ============================================================================

extern "C" {

size_t iblb_workspace_bytes(int n_droplets, const iblb_params* params, const int* n_nodes,
                            const int* n_tris, int storage) {
    Layout L;
    std::string err;
    if (!plan(n_droplets, params, n_nodes, n_tris, storage, L, err)) {
        fail(nullptr, IBLB_EINVAL, err);
        return 0;
    }
    return L.total;
}

int iblb_create(int n, const iblb_params* P, const int* nn, const int* nt, int storage,
                void* d_ws, size_t ws_bytes, void* stream, iblb_ctx** out) {
    if (!out) return fail(nullptr, IBLB_EINVAL, "out must not be NULL");
    *out = nullptr;
    Layout L;
    std::string err;
    if (!plan(n, P, nn, nt, storage, L, err)) return fail(nullptr, IBLB_EINVAL, err);
    if (!d_ws) return fail(nullptr, IBLB_EINVAL, "NULL workspace");
    if (ws_bytes < L.total) {
        char buf[160];
        snprintf(buf, sizeof buf, "workspace of %zu bytes is smaller than the %zu needed", ws_bytes,
                 L.total);
        return fail(nullptr, IBLB_ENOMEM, buf);
    }
    if (reinterpret_cast<uintptr_t>(d_ws) % kAlign)
        return fail(nullptr, IBLB_EINVAL, "workspace must be 256-byte aligned");
    iblb_ctx* c = new iblb_ctx();
    c->n = n;
    c->dim = P[0].dim;
    c->Q = c->dim == 2 ? 9 : 19;
    c->storage = storage;
    c->params.assign(P, P + n);
    c->n_nodes.assign(nn, nn + n);
    c->n_tris.assign(n, 0);
    if (c->dim == 3 && nt) c->n_tris.assign(nt, nt + n);
    c->L = L;
    c->ws = static_cast<char*>(d_ws);
    c->stream = static_cast<hipStream_t>(stream);
    c->status_h.assign(n, 0);
    c->iface_set.assign(n, 0);
    c->drops.resize(n);
    for (int d = 0; d < n; ++d) {
        const iblb_params& p = P[d];
        DropDev& D = c->drops[d];
        memset(&D, 0, sizeof D);
        D.nx = p.nx;
        D.ny = p.ny;
        D.nz = c->dim == 3 ? p.nz : 1;
        D.nstrip = strips_of(p.nx, c->dim, c->storage);
        D.sshift = strip_shift(c->dim, c->storage);
        D.bcx = p.bc[0];
        D.bcy = p.bc[1];
        D.bcz = c->dim == 3 ? p.bc[2] : 0;
        D.ncell = p.nx * p.ny * D.nz;
        D.f_off = L.f_off[d];
        D.fst = L.fst[d];
        D.ppl = (int)plane_pitch(p, c->dim);
        D.c_off = L.c_off[d];
        D.flag_off = L.flag_off[d];
        D.omega = (float)(1.0 / p.tau);
        D.guo = (float)(1.0 - 0.5 / p.tau);
        D.visc = 0;
        D.omega_in = D.omega;
        D.guo_in = D.guo;
        D.row_off = L.row_off[d];
        D.force_mode = 0;
        D.active = 1;
        D.node_off = L.node_off[d];
        D.n_nodes = nn[d];
        D.tri_off = L.tri_off[d];
        D.n_tris = c->n_tris[d];
        D.wetting = p.wetting ? 1 : 0;
        D.n_exp = p.n_exp;
        D.m_exp = p.m_exp;
        D.sigma = p.sigma;
        D.xi = p.xi;
        // eq. (A_choice)
        D.A = p.wetting ? p.sigma * (double)((p.m_exp - 1) * (p.n_exp - 1)) /
                              ((double)(p.n_exp - p.m_exp) * p.xi) * (1.0 + cos(p.theta_eq))
                        : 0.0;
        // minimum of Pi(h): h* = xi (n/m)^(1/(n-m))
        D.zcut = p.wetting ? p.xi * pow((double)p.n_exp / p.m_exp, 1.0 / (p.n_exp - p.m_exp))
                           : p.xi;
        const double centre[3] = {0.5 * p.nx, 0.5 * p.ny, 0.5 * D.nz};
        set_window(D, p.bc, centre);
    }
    hipError_t e = hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
        g_create_err = std::string("hipStreamCreate: ") + hipGetErrorString(e);
        release_streams(c);
        delete c;
        return IBLB_EDEVICE;
    }
    // node -> droplet table; positions zero until set
    std::vector<int> nd(std::max(L.ntot, 1), 0);
    for (int d = 0; d < n; ++d)
        for (int k = 0; k < nn[d]; ++k) nd[L.node_off[d] + k] = d;
    int rc = IBLB_OK;
    auto chk = [&](hipError_t ee, const char* what) {
        if (ee != hipSuccess && rc == IBLB_OK) {
            g_create_err = std::string(what) + ": " + hipGetErrorString(ee);
            rc = IBLB_EDEVICE;
        }
    };
    chk(hipMemsetAsync(c->ws, 0, L.total, c->stream), "hipMemsetAsync");
    chk(hipMemcpyAsync(c->at<int>(L.node_drop), nd.data(), sizeof(int) * nd.size(),
                       hipMemcpyHostToDevice, c->stream), "hipMemcpyAsync");
    // spatial order of the vertices: identity until an interface is set
    std::vector<int> perm(std::max(L.ntot, 1), 0);
    for (int k = 0; k < L.ntot; ++k) perm[k] = k;
    chk(hipMemcpyAsync(c->at<int>(L.perm), perm.data(), sizeof(int) * perm.size(),
                       hipMemcpyHostToDevice, c->stream), "hipMemcpyAsync");
    if (c->dim == 3) {
        c->chunks_h.assign(n, {});
        for (int d = 0; d < n; ++d)
            for (int b = 0; b < nn[d]; b += kChunk)
                c->chunks_h[d].push_back(make_int4(d, L.node_off[d] + b, std::min(kChunk, nn[d] - b), 0));
    }
    chk(hipStreamSynchronize(c->stream), "hipStreamSynchronize");
    if (rc == IBLB_OK) {
        for (int d = 0; d < n && rc == IBLB_OK; ++d) {
            int r = reset_droplet(c, d);
            if (r) { g_create_err = c->err; rc = r; }
        }
    }
    if (rc == IBLB_OK) {
        int r = rebuild_tiles(c);
        if (!r) r = upload_chunks(c);
        if (r) { g_create_err = c->err; rc = r; }
    }
    if (rc != IBLB_OK) {
        release_streams(c);
        delete c;
        return rc;
    }
    *out = c;
    return IBLB_OK;
}

int iblb_destroy(iblb_ctx* c) {
    if (!c) return IBLB_OK;
    drop_graphs(c);
    for (auto ev : c->events) (void)hipEventDestroy(ev);
    release_streams(c);
    delete c;
    return IBLB_OK;
}

const char* iblb_last_error(const iblb_ctx* c) { return c ? c->err.c_str() : g_create_err.c_str(); }

}  // extern "C"

namespace {

// Spread the low 10 bits of v to every third bit.
uint32_t spread_bits3(uint32_t v) {
    v &= 0x3ff;
    v = (v | (v << 16)) & 0x030000ff;
    v = (v | (v << 8)) & 0x0300f00f;
    v = (v | (v << 4)) & 0x030c30c3;
    v = (v | (v << 2)) & 0x09249249;
    return v;
}

// Global node ids off + 0..N-1 sorted by the Morton code of their position
// (SoA [3][N]) quantised to 1024 steps per axis over the vertices' bounding
// box, so that consecutive vertices are close in space.
void morton_order(const double* pos, int N, int off, std::vector<int>& perm, int d,
                  std::vector<int4>& chunks) {
    double lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = *std::min_element(pos + (size_t)a * N, pos + (size_t)(a + 1) * N);
        hi[a] = *std::max_element(pos + (size_t)a * N, pos + (size_t)(a + 1) * N);
    }
    const double span = std::max({hi[0] - lo[0], hi[1] - lo[1], hi[2] - lo[2], 1e-300});
    std::vector<std::pair<uint32_t, int>> key(N);
    for (int k = 0; k < N; ++k) {
        uint32_t m = 0;
        for (int a = 0; a < 3; ++a) {
            const double u = (pos[(size_t)a * N + k] - lo[a]) / span * 1023.0;
            m |= spread_bits3((uint32_t)std::min(std::max(u, 0.0), 1023.0)) << a;
        }
        key[k] = {m, k};
    }
    std::sort(key.begin(), key.end());
    perm.resize(N);
    for (int k = 0; k < N; ++k) perm[k] = off + key[k].second;
    // Cut the order into chunks of at most kChunk vertices whose taps fit a
    // box of kChunkBudget cells (below the kernel's kBoxCells, so that the
    // vertices can move a little before a chunk outgrows it and is taken in
    // runs).
    // (in doubles: any finite position is accepted, and the product of far
    // extents has to stay a large number)
    constexpr double kChunkBudget = IBLB_CHUNK_BUDGET;
    chunks.clear();
    double blo[3] = {0, 0, 0}, bhi[3] = {0, 0, 0};
    int first = 0, cnt = 0;
    for (int r = 0; r < N; ++r) {
        const int k = key[r].second;
        double b[3];
        for (int a = 0; a < 3; ++a) b[a] = std::floor(pos[(size_t)a * N + k] - 0.5) - 1;
        if (cnt > 0) {
            double cells = 1;
            for (int a = 0; a < 3; ++a) cells *= std::max(bhi[a], b[a]) - std::min(blo[a], b[a]) + 4;
            if (cnt == kChunk || cells > kChunkBudget) {
                chunks.push_back(make_int4(d, off + first, cnt, 0));
                cnt = 0;
            }
        }
        if (cnt == 0) {
            first = r;
            for (int a = 0; a < 3; ++a) blo[a] = bhi[a] = b[a];
        }
        for (int a = 0; a < 3; ++a) {
            blo[a] = std::min(blo[a], b[a]);
            bhi[a] = std::max(bhi[a], b[a]);
        }
        ++cnt;
    }
    if (cnt > 0) chunks.push_back(make_int4(d, off + first, cnt, 0));
}

}  // namespace

extern "C" {

int iblb_set_interface(iblb_ctx* c, int d, const double* h_pos, const int32_t* h_tris) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    const int N = c->n_nodes[d];
    if (N == 0) return IBLB_OK;
    if (!h_pos) return fail(c, IBLB_EINVAL, "NULL positions");
    const DropDev& D = c->drops[d];
    const int st = std::max(c->L.ntot, 1);
    for (int a = 0; a < c->dim; ++a)
        for (int k = 0; k < N; ++k)
            if (!std::isfinite(h_pos[(size_t)a * N + k]))
                return fail(c, IBLB_EINVAL, "non-finite node position");
    if (c->params[d].wetting)
        for (int k = 0; k < N; ++k)
            if (!(h_pos[(size_t)(c->dim - 1) * N + k] > 0.0))
                return fail(c, IBLB_EINVAL, "a node lies at or below the substrate (h <= 0)");
    std::vector<double> pos(h_pos, h_pos + (size_t)c->dim * N);
    {
        // window of the inside/outside classification: centred on the mean
        // of the nodes
        double ref[3] = {0.5 * D.nx, 0.5 * D.ny, 0.5 * D.nz};
        for (int a = 0; a < c->dim; ++a) {
            double sum = 0.0;
            for (int k = 0; k < N; ++k) sum += pos[(size_t)a * N + k];
            ref[a] = sum / N;
        }
        set_window(c->drops[d], c->params[d].bc, ref);
    }
    for (int a = 0; a < c->dim; ++a)
        HIPCHK(c, hipMemcpyAsync(positions(c, c->cur) + (size_t)a * st + D.node_off,
                                 pos.data() + (size_t)a * N, sizeof(double) * N,
                                 hipMemcpyHostToDevice, c->stream));
    std::vector<int> tri, inc, beg, end, perm;
    if (c->dim == 3) {
        const int T = c->n_tris[d];
        if (!h_tris) return fail(c, IBLB_EINVAL, "NULL triangle list");
        const int ts = std::max(c->L.ttot, 1);
        std::vector<int> cnt(N, 0);
        for (int t = 0; t < T; ++t)
            for (int s = 0; s < 3; ++s) {
                const int v = h_tris[3 * t + s];
                if (v < 0 || v >= N) return fail(c, IBLB_EINVAL, "triangle vertex index out of range");
                cnt[v]++;
            }
        for (int k = 0; k < N; ++k)
            if (cnt[k] == 0) return fail(c, IBLB_EINVAL, "a vertex belongs to no triangle");
        // incidence list (CSR by vertex), global triangle and node ids
        beg.resize(N);
        end.resize(N);
        int acc = 3 * D.tri_off;
        for (int k = 0; k < N; ++k) {
            beg[k] = acc;
            acc += cnt[k];
            end[k] = beg[k];
        }
        inc.assign(3 * T, 0);
        tri.assign(3 * T, 0);
        for (int t = 0; t < T; ++t)
            for (int s = 0; s < 3; ++s) {
                const int v = h_tris[3 * t + s];
                tri[(size_t)s * T + t] = D.node_off + v;
                inc[end[v] - 3 * D.tri_off] = ((D.tri_off + t) << 2) | s;
                end[v]++;
            }
        for (int s = 0; s < 3; ++s)
            HIPCHK(c, hipMemcpyAsync(c->at<int>(c->L.tri) + (size_t)s * ts + D.tri_off,
                                     tri.data() + (size_t)s * T, sizeof(int) * T,
                                     hipMemcpyHostToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(c->at<int>(c->L.inc) + 3 * D.tri_off, inc.data(), sizeof(int) * 3 * T,
                                 hipMemcpyHostToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(c->at<int>(c->L.inc_beg) + D.node_off, beg.data(), sizeof(int) * N,
                                 hipMemcpyHostToDevice, c->stream));
        HIPCHK(c, hipMemcpyAsync(c->at<int>(c->L.inc_end) + D.node_off, end.data(), sizeof(int) * N,
                                 hipMemcpyHostToDevice, c->stream));
        morton_order(pos.data(), N, D.node_off, perm, d, c->chunks_h[d]);
        HIPCHK(c, hipMemcpyAsync(c->at<int>(c->L.perm) + D.node_off, perm.data(), sizeof(int) * N,
                                 hipMemcpyHostToDevice, c->stream));
        int rc = upload_chunks(c);
        if (rc) return rc;
    }
    HIPCHK(c, hipMemsetAsync(c->at<int>(c->L.status) + d, 0, sizeof(int), c->stream));
    c->iface_set[d] = 1;
    return upload_drops(c);  // synchronises: host staging vectors go out of scope
}

int iblb_init_rest(iblb_ctx* c, int d) {
    if (!c) return IBLB_EINVAL;
    if (d == -1) {
        for (int k = 0; k < c->n; ++k) {
            int rc = reset_droplet(c, k);
            if (rc) return rc;
        }
        return IBLB_OK;
    }
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    return reset_droplet(c, d);
}

}  // extern "C"

namespace {

template <int S>
void launch_init_eq(iblb_ctx* c, int d, const float* rho, const float* u) {
    using T = typename Codec<S>::T;
    const DropDev& D = c->drops[d];
    T* f = c->at<T>(c->cur ? c->L.f1 : c->L.f0) + D.f_off;
    const dim3 grid(ceil_div(D.ncell, kBlock)), block(kBlock);
    if (c->dim == 2)
        hipLaunchKernelGGL((k_init_eq<2, S>), grid, block, 0, c->stream, f, D.ncell, D.fst, D.nx * D.ny, D.ppl,
                           rho, u);
    else
        hipLaunchKernelGGL((k_init_eq<3, S>), grid, block, 0, c->stream, f, D.ncell, D.fst, D.nx * D.ny, D.ppl,
                           rho, u);
}

}  // namespace

extern "C" {

int iblb_init_fields(iblb_ctx* c, int d, const float* d_rho, const float* d_u) {
    if (!c) return IBLB_EINVAL;
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    int rc = reset_droplet(c, d);  // clears F, U, the band flags and both population buffers
    if (rc) return rc;
    switch (c->storage) {
        case ST_F32: launch_init_eq<ST_F32>(c, d, d_rho, d_u); break;
        case ST_F16: launch_init_eq<ST_F16>(c, d, d_rho, d_u); break;
        default: launch_init_eq<ST_BF16>(c, d, d_rho, d_u); break;
    }
    HIPCHK(c, hipGetLastError());
    return IBLB_OK;
}

int iblb_write_populations(iblb_ctx* c, int d, const double* d_fdev) {
    return pop_io(c, d, d_fdev, nullptr);
}

int iblb_read_populations(iblb_ctx* c, int d, double* d_fdev) { return pop_io(c, d, nullptr, d_fdev); }

int iblb_set_force_field(iblb_ctx* c, int d, const float* d_F) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    DropDev& D = c->drops[d];
    const size_t vb = sizeof(float) * c->dim * D.ncell, vo = sizeof(float) * c->dim * D.c_off;
    if (d_F) {
        HIPCHK(c, hipMemcpyAsync(c->ws + c->L.F + vo, d_F, vb, hipMemcpyDeviceToDevice, c->stream));
        D.force_mode = 1;
    } else {
        HIPCHK(c, hipMemsetAsync(c->ws + c->L.F + vo, 0, vb, c->stream));
        HIPCHK(c, hipMemsetAsync(c->ws + c->L.Fq + 2 * vo, 0, 2 * vb, c->stream));
        D.force_mode = 0;
    }
    return upload_drops(c);
}

int iblb_step(iblb_ctx* c, int n_steps) {
    if (!c) return IBLB_EINVAL;
    if (n_steps < 0) return fail(c, IBLB_EINVAL, "n_steps must be >= 0");
    if (n_steps == 0) return IBLB_OK;
    for (int d = 0; d < c->n; ++d)
        if (c->n_nodes[d] > 0 && !c->iface_set[d] && c->drops[d].force_mode == 0) {
            char buf[96];
            snprintf(buf, sizeof buf, "droplet %d: interface not set", d);
            return fail(c, IBLB_EINVAL, buf);
        }
    if (c->tiles_dirty) {
        int rc = rebuild_tiles(c);
        if (rc) return rc;
    }
    if (c->any_visc) {
        // the first step's crossings are recorded by launch_spread into the
        // current tables; later steps find theirs cleared by the lattice
        // kernel of the step before
        HIPCHK(c, hipMemsetAsync(cross_count(c, c->cur), 0, sizeof(int) * c->L.rows, c->stream));
    }
    if (c->timing) {
        // Every step launched directly (a dispatch that marks events cannot
        // be captured in a graph), each lattice launch between a pair of
        // events marked by its own dispatch; the events are read every
        // kTimedChunk launches.  The final field-storing step is not part
        // of the kernel average.
        int rc = ensure_events(c, 2 + 2 * kTimedChunk);
        if (rc) return rc;
        hipEvent_t* ev = c->events.data();
        double lb = 0.0, ms = 0.0;
        long long nlb = 0;
        int pending = 0;
        HIPCHK(c, hipEventRecord(ev[0], c->stream));
        launch_spread(c, c->stream, c->cur, n_steps == 1);
        for (int rem = n_steps, k = 0; rem > 1; --rem, ++k) {
            // with a stride above one only every timing-th launch carries
            // the events, so that they perturb the run less
            const bool timed = k % c->timing == 0;
            if (timed && pending == kTimedChunk) {
                if ((rc = read_lb_events(c, pending, ms))) return rc;
                lb += ms;
                nlb += pending;
                pending = 0;
            }
            launch_step(c, c->stream, c->cur, false, 0, rem == 2, timed ? ev + 2 + 2 * pending : nullptr);
            if (timed) ++pending;
            c->cur ^= 1;
            c->step++;
        }
        launch_step(c, c->stream, c->cur, true, 1, 0);
        c->cur ^= 1;
        c->step++;
        HIPCHK(c, hipEventRecord(ev[1], c->stream));
        HIPCHK(c, hipGetLastError());
        if ((rc = read_lb_events(c, pending, ms))) return rc;
        lb += ms;
        nlb += pending;
        float total = 0.f;
        HIPCHK(c, hipEventElapsedTime(&total, ev[0], ev[1]));
        c->t_lb = nlb ? lb / nlb : 0.0;
        c->t_step = total / n_steps;
    } else {
        // forces for the first step; every later spread is launched by the
        // node work of the step before it; the drops lost at walls are
        // recorded by the spread that feeds the last step
        launch_spread(c, c->stream, c->cur, n_steps == 1);
        int rem = n_steps;
        while (rem > 1) {
            if (c->graph_steps > 0 && rem >= c->graph_steps + 2) {
                int rc = ensure_graph(c, c->cur);
                if (rc) return rc;
                HIPCHK(c, hipGraphLaunch(c->exec[c->cur], c->stream));
                rem -= c->graph_steps;
                c->step += c->graph_steps;
            } else {
                launch_step(c, c->stream, c->cur, false, 0, rem == 2);
                c->cur ^= 1;
                rem--;
                c->step++;
            }
        }
        launch_step(c, c->stream, c->cur, true, 1, 0);
        c->cur ^= 1;
        c->step++;
        HIPCHK(c, hipGetLastError());
    }
    if (n_steps & 1) {
        // a frozen droplet's populations stay in the buffer that was current
        // when the call began; after an odd number of steps the other buffer
        // is current, so carry them over
        const size_t sb = c->storage == ST_F32 ? 4 : 2;
        char* now = c->ws + (c->cur ? c->L.f1 : c->L.f0);
        const char* was = c->ws + (c->cur ? c->L.f0 : c->L.f1);
        for (int d = 0; d < c->n; ++d) {
            const DropDev& D = c->drops[d];
            if (D.active) continue;
            const size_t off = (size_t)D.f_off * sb, bytes = (size_t)c->Q * D.fst * sb;
            HIPCHK(c, hipMemcpyAsync(now + off, was + off, bytes, hipMemcpyDeviceToDevice, c->stream));
        }
    }
    HIPCHK(c, hipMemcpyAsync(c->status_h.data(), c->at<int>(c->L.status), sizeof(int) * c->n,
                             hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (int d = 0; d < c->n; ++d)
        if (c->status_h[d] && c->drops[d].active) {
            char buf[256];
            const int code = c->status_h[d];
            snprintf(buf, sizeof buf, "droplet %d %s (code %d:%s%s%s%s%s) by step %lld", d,
                     (code & 7) ? "unstable" : "over a fixed limit", code,
                     (code & 1) ? " node at or below the substrate" : "",
                     (code & 2) ? " node speed above 0.3 or not finite" : "",
                     (code & 4) ? " node position not finite or far outside the box" : "",
                     (code & 8) ? " more than 16 interface crossings on one lattice row" : "",
                     (code & 16) ? " a node left the window of the inside/outside classification" : "",
                     (long long)c->step);
            return fail(c, (code & 7) ? IBLB_EUNSTABLE : IBLB_ELIMIT, buf);
        }
    return IBLB_OK;
}

int iblb_read_fields(iblb_ctx* c, int d, float* d_rho, float* d_u, float* d_F) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    const DropDev& D = c->drops[d];
    const size_t vb = sizeof(float) * c->dim * D.ncell, vo = sizeof(float) * c->dim * D.c_off;
    if (d_rho)
        HIPCHK(c, hipMemcpyAsync(d_rho, c->at<float>(c->L.rho) + D.c_off, sizeof(float) * D.ncell,
                                 hipMemcpyDeviceToDevice, c->stream));
    if (d_u) HIPCHK(c, hipMemcpyAsync(d_u, c->ws + c->L.U + vo, vb, hipMemcpyDeviceToDevice, c->stream));
    if (d_F) HIPCHK(c, hipMemcpyAsync(d_F, c->ws + c->L.Fout + vo, vb, hipMemcpyDeviceToDevice, c->stream));
    return IBLB_OK;
}

int iblb_read_nodes(iblb_ctx* c, int d, double* h_pos, float* h_vel, float* h_force) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    const int N = c->n_nodes[d];
    const int st = std::max(c->L.ntot, 1);
    const int o = c->drops[d].node_off;
    for (int a = 0; a < c->dim && N > 0; ++a) {
        if (h_pos)
            HIPCHK(c, hipMemcpyAsync(h_pos + (size_t)a * N, positions(c, c->cur) + (size_t)a * st + o,
                                     sizeof(double) * N, hipMemcpyDeviceToHost, c->stream));
        if (h_vel)
            HIPCHK(c, hipMemcpyAsync(h_vel + (size_t)a * N, c->at<float>(c->L.qdot) + (size_t)a * st + o,
                                     sizeof(float) * N, hipMemcpyDeviceToHost, c->stream));
        if (h_force)
            HIPCHK(c, hipMemcpyAsync(h_force + (size_t)a * N, c->at<float>(c->L.phi) + (size_t)a * st + o,
                                     sizeof(float) * N, hipMemcpyDeviceToHost, c->stream));
    }
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return IBLB_OK;
}

static void fill_diag(const iblb_ctx* c, int d, const DiagDev& r, int st, iblb_diag* out) {
    memset(out, 0, sizeof *out);
    out->step = c->step;
    out->mass = (double)c->drops[d].ncell + r.mass_dev;
    for (int a = 0; a < 3; ++a) {
        out->momentum[a] = r.mom[a];
        out->sum_phi[a] = r.sum_phi[a];
        out->sum_F[a] = r.sum_F[a];
        out->dropped_F[a] = r.dropped[a];
    }
    const bool has_iface = c->n_nodes[d] > 0;
    out->volume = has_iface ? r.volume : 0.0;
    out->area = has_iface ? r.area : 0.0;
    out->height = has_iface ? r.max_h - r.min_h : 0.0;
    out->min_h = has_iface ? r.min_h : NAN;
    out->max_normal_speed = r.max_un;
    out->max_speed = r.max_u;
    out->edge_min = has_iface ? r.edge_min : NAN;
    out->edge_max = has_iface ? r.edge_max : NAN;
    if (c->dim == 2)
        out->contact_radius = (has_iface && r.cross_hi > r.cross_lo) ? 0.5 * (r.cross_hi - r.cross_lo) : NAN;
    else
        out->contact_radius = (has_iface && r.cross_n > 0) ? r.cross_r : NAN;
    out->theta_meas = has_iface ? angle_from_height(c->dim, r.volume, out->height) : NAN;
    out->status = st ? IBLB_EUNSTABLE : IBLB_OK;
}

int iblb_diagnostics(iblb_ctx* c, int d, iblb_diag* out) {
    if (!c) return IBLB_EINVAL;
    if (d != -1 && !check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (!out) return fail(c, IBLB_EINVAL, "NULL output");
    if (c->tiles_dirty) {
        int rc = rebuild_tiles(c);
        if (rc) return rc;
    }
    if (c->dim == 2) launch_diag_d<2>(c);
    else launch_diag_d<3>(c);
    HIPCHK(c, hipGetLastError());
    std::vector<DiagDev> r(c->n);
    std::vector<int> st(c->n);
    HIPCHK(c, hipMemcpyAsync(r.data(), c->at<DiagDev>(c->L.diag), sizeof(DiagDev) * c->n,
                             hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipMemcpyAsync(st.data(), c->at<int>(c->L.status), sizeof(int) * c->n,
                             hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (d >= 0) {
        fill_diag(c, d, r[d], st[d], out);
    } else {
        for (int k = 0; k < c->n; ++k) fill_diag(c, k, r[k], st[k], out + k);
    }
    return IBLB_OK;
}

int iblb_run_to_rest(iblb_ctx* c, double tol, double angle_tol, int check_every, int hold,
                     long long max_steps, long long* steps_out) {
    if (!c) return IBLB_EINVAL;
    if (!steps_out || !(tol > 0.0) || !(angle_tol >= 0.0) || check_every < 1 || hold < 1 || max_steps < 1)
        return fail(c, IBLB_EINVAL, "run_to_rest: bad arguments");
    if (c->tiles_dirty) {
        int rc = rebuild_tiles(c);
        if (rc) return rc;
    }
    std::vector<int> below(c->n, 0);
    std::vector<DiagDev> r(c->n);
    // measured angles of the last hold + 1 checks of every droplet (ring)
    // and how many of them have been taken
    std::vector<double> angles((size_t)c->n * (hold + 1), 0.0);
    std::vector<int> nang(c->n, 0);
    int live = 0;
    for (int d = 0; d < c->n; ++d) {
        const bool tracked = c->drops[d].active && c->n_nodes[d] > 0;
        steps_out[d] = tracked ? -1 : 0;
        live += tracked;
    }
    const long long start = c->step;
    while (live > 0 && c->step - start < max_steps) {
        const int n = (int)std::min<long long>(check_every, max_steps - (c->step - start));
        int rc = iblb_step(c, n);
        if (rc == IBLB_EUNSTABLE || rc == IBLB_ELIMIT) {
            // freeze the droplets that failed; the others carry on
            for (int d = 0; d < c->n; ++d)
                if (c->status_h[d] && c->drops[d].active) {
                    iblb_set_active(c, d, 0);
                    steps_out[d] = -2;
                    --live;
                }
            if (c->tiles_dirty && (rc = rebuild_tiles(c))) return rc;
            continue;
        }
        if (rc) return rc;
        if (c->dim == 2) launch_diag_d<2>(c, false);
        else launch_diag_d<3>(c, false);
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipMemcpyAsync(r.data(), c->at<DiagDev>(c->L.diag), sizeof(DiagDev) * c->n,
                                 hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        for (int d = 0; d < c->n; ++d) {
            if (steps_out[d] != -1) continue;
            below[d] = r[d].max_un < tol ? below[d] + 1 : 0;
            bool steady = true;
            if (angle_tol > 0.0) {
                // the angle from the half-height must also have stayed within
                // angle_tol over the window: this check and the hold before
                double* a = angles.data() + (size_t)d * (hold + 1);
                for (int k = hold; k > 0; --k) a[k] = a[k - 1];
                a[0] = angle_from_height(c->dim, r[d].volume, r[d].max_h - r[d].min_h);
                nang[d] = std::min(nang[d] + 1, hold + 1);
                if (nang[d] <= hold) {
                    steady = false;
                } else {
                    double lo = a[0], hi = a[0];
                    for (int k = 1; k <= hold; ++k) {
                        lo = std::min(lo, a[k]);
                        hi = std::max(hi, a[k]);
                    }
                    steady = hi - lo < angle_tol;  // false for a NaN angle
                }
            }
            if (below[d] >= hold && steady) {
                steps_out[d] = c->step - start;
                iblb_set_active(c, d, 0);
                --live;
            }
        }
    }
    return IBLB_OK;
}

int iblb_set_lb_variant(iblb_ctx* c, int variant, int* variant_out) {
    if (!c) return IBLB_EINVAL;
    if (variant >= kVariants || variant < -1)
        return fail(c, IBLB_EINVAL, "lattice-kernel variant must be -1 or 0..31");
    if (variant >= 0 && variant != c->variant) {
        c->variant = variant;
        c->tiles_dirty = true;
    }
    if (variant_out) *variant_out = c->variant;
    return IBLB_OK;
}

int iblb_set_graph_steps(iblb_ctx* c, int steps) {
    if (!c) return IBLB_EINVAL;
    if (steps < 0 || steps == 1 || (steps & 1) || steps > kMaxGraphSteps)
        return fail(c, IBLB_EINVAL, "graph steps must be 0 or an even number in 2..1024");
    if (steps != c->graph_steps) {
        drop_graphs(c);
        c->graph_steps = steps;
    }
    return IBLB_OK;
}

int iblb_set_active(iblb_ctx* c, int d, int active) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    const int a = active ? 1 : 0;
    if (c->drops[d].active != a) {
        c->drops[d].active = a;
        c->tiles_dirty = true;
    }
    return IBLB_OK;
}

int iblb_set_viscosity_ratio(iblb_ctx* c, int d, double lambda) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (!(lambda > 0.0) || !std::isfinite(lambda))
        return fail(c, IBLB_EINVAL, "viscosity ratio must be positive and finite");
    if (c->n_nodes[d] == 0) return fail(c, IBLB_EINVAL, "droplet has no interface");
    const double tau = c->params[d].tau;
    if (!std::isfinite(tau)) return fail(c, IBLB_EINVAL, "viscosity ratio needs a finite tau");
    // mu = rho cs^2 (tau - 1/2) on both sides, lambda = mu_in / mu_out
    const double tau_in = 0.5 + lambda * (tau - 0.5);
    DropDev& D = c->drops[d];
    D.visc = lambda != 1.0;
    D.omega_in = (float)(1.0 / tau_in);
    D.guo_in = (float)(1.0 - 0.5 / tau_in);
    bool any = false;
    for (int k = 0; k < c->n; ++k) any = any || c->drops[k].visc;
    if (any != c->any_visc) {
        c->any_visc = any;
        drop_graphs(c);  // whether the crossing launches run is baked into them
    }
    return upload_drops(c);
}

int iblb_set_membrane_shear(iblb_ctx* c, int d, double mu_s) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (c->dim != 3) return fail(c, IBLB_EINVAL, "an elastic interface needs a 3D triangle mesh");
    if (!(mu_s >= 0.0) || !std::isfinite(mu_s))
        return fail(c, IBLB_EINVAL, "shear modulus must be finite and >= 0");
    if (c->n_nodes[d] == 0 || !c->iface_set[d]) return fail(c, IBLB_EINVAL, "droplet has no interface");
    DropDev& D = c->drops[d];
    if (mu_s != 0.0) {
        hipLaunchKernelGGL(k_tri_ref, dim3(ceil_div(D.n_tris, kBlock)), dim3(kBlock), 0, c->stream,
                           c->at<DropDev>(c->L.drops), d, node_arrays(c, c->cur), c->at<double>(c->L.tref));
        HIPCHK(c, hipGetLastError());
    }
    D.shear = mu_s;
    return upload_drops(c);
}

int iblb_set_node_respacing(iblb_ctx* c, int d, double beta) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (c->dim != 2) return fail(c, IBLB_EINVAL, "node re-spacing applies to a 2D outline");
    if (!(beta >= 0.0 && beta < 1.0)) return fail(c, IBLB_EINVAL, "re-spacing rate must lie in [0, 1)");
    if (c->n_nodes[d] == 0 || !c->iface_set[d]) return fail(c, IBLB_EINVAL, "droplet has no interface");
    c->drops[d].respace = beta;
    return upload_drops(c);
}

int iblb_inside_mask(iblb_ctx* c, int d, uint8_t* d_mask) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (!d_mask) return fail(c, IBLB_EINVAL, "NULL mask");
    if (c->n_nodes[d] == 0 || !c->iface_set[d] || c->drops[d].force_mode != 0)
        return fail(c, IBLB_EINVAL, "droplet has no interface");
    int before = 0, code = 0;
    HIPCHK(c, hipMemcpyAsync(&before, c->at<int>(c->L.status) + d, sizeof(int), hipMemcpyDeviceToHost,
                             c->stream));
    // the current tables are rebuilt at the start of the next step call
    HIPCHK(c, hipMemsetAsync(cross_count(c, c->cur), 0, sizeof(int) * c->L.rows, c->stream));
    launch_cross(c, c->stream, c->cur, c->cur, 1);
    hipLaunchKernelGGL(k_inside_mask, dim3(ceil_div(c->drops[d].ncell, kBlock)), dim3(kBlock), 0,
                       c->stream, c->at<DropDev>(c->L.drops), d, (const int*)cross_count(c, c->cur),
                       (const double*)cross_x(c, c->cur), d_mask);
    HIPCHK(c, hipGetLastError());
    HIPCHK(c, hipMemcpyAsync(&code, c->at<int>(c->L.status) + d, sizeof(int), hipMemcpyDeviceToHost,
                             c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    code &= ~before;
    if (code & 4) return fail(c, IBLB_EUNSTABLE, "inside mask: node position not finite");
    if (code & 8) return fail(c, IBLB_ELIMIT, "inside mask: more than 16 crossings on one lattice row");
    if (code & 16)
        return fail(c, IBLB_ELIMIT, "inside mask: a node lies outside the classification window "
                                    "(the droplet spans more than the box along a periodic axis)");
    return IBLB_OK;
}

int iblb_contact_radius(iblb_ctx* c, int d, double z_cut, double flat_tol, double* out) {
    if (!check_droplet(c, d)) return fail(c, IBLB_EINVAL, "bad droplet index");
    if (!out) return fail(c, IBLB_EINVAL, "NULL output");
    if (c->n_nodes[d] == 0 || !c->iface_set[d]) return fail(c, IBLB_EINVAL, "droplet has no interface");
    if (!std::isfinite(z_cut) || !(flat_tol >= 0.0))
        return fail(c, IBLB_EINVAL, "z_cut must be finite and flat_tol >= 0");
    double* dev = c->at<double>(c->L.partials);
    if (c->dim == 2) launch_contact<2>(c, d, z_cut, flat_tol, dev);
    else launch_contact<3>(c, d, z_cut, flat_tol, dev);
    HIPCHK(c, hipGetLastError());
    HIPCHK(c, hipMemcpyAsync(out, dev, 3 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return IBLB_OK;
}

int iblb_set_timing(iblb_ctx* c, int on) {
    if (!c) return IBLB_EINVAL;
    if (on < 0) return fail(c, IBLB_EINVAL, "timing: the stride must be >= 0");
    c->timing = on;
    return IBLB_OK;
}

int iblb_last_timing(const iblb_ctx* c, double* lb_ms, double* step_ms) {
    if (!c) return IBLB_EINVAL;
    if (lb_ms) *lb_ms = c->t_lb;
    if (step_ms) *step_ms = c->t_step;
    return IBLB_OK;
}

int iblb_time_lattice(iblb_ctx* c, int launches, double* ms_per_launch) {
    if (!c || !ms_per_launch) return IBLB_EINVAL;
    if (launches < 2 || launches > 1024 || launches % 2)
        return fail(c, IBLB_EINVAL, "time_lattice: launches must be even, 2..1024");
    if (c->tiles_dirty) {
        int rc = rebuild_tiles(c);
        if (rc) return rc;
    }
    if (c->lexec && (c->lexec_n != launches || c->lexec_p != c->cur)) {
        (void)hipGraphExecDestroy(c->lexec);
        c->lexec = nullptr;
    }
    if (!c->lexec) {
        hipGraph_t g = nullptr;
        HIPCHK(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
        for (int k = 0; k < launches; ++k)
            launch_lb(c, c->cap_stream, c->cur ^ (k & 1), 0, nullptr, false);
        hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
        if (e != hipSuccess) return fail(c, IBLB_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e));
        e = hipGraphInstantiate(&c->lexec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) {
            c->lexec = nullptr;
            return fail(c, IBLB_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(e));
        }
        c->lexec_n = launches;
        c->lexec_p = c->cur;
    }
    if (c->any_visc) {
        // every launch classifies the cells at the current node positions:
        // both parities' tables hold those crossings and are not cleared
        // (the next step call rebuilds its own)
        for (int tp = 0; tp < 2; ++tp) {
            HIPCHK(c, hipMemsetAsync(cross_count(c, tp), 0, sizeof(int) * c->L.rows, c->stream));
            launch_cross(c, c->stream, c->cur, tp, 0);
        }
    }
    int rc = ensure_events(c, 2);
    if (rc) return rc;
    hipEvent_t* ev = c->events.data();
    HIPCHK(c, hipGraphLaunch(c->lexec, c->stream));  // warm-up replay
    HIPCHK(c, hipEventRecord(ev[0], c->stream));
    HIPCHK(c, hipGraphLaunch(c->lexec, c->stream));
    HIPCHK(c, hipEventRecord(ev[1], c->stream));
    HIPCHK(c, hipEventSynchronize(ev[1]));
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, ev[0], ev[1]));
    c->step += 2LL * launches;
    *ms_per_launch = (double)ms / launches;
    return IBLB_OK;
}

int iblb_autotune(iblb_ctx* c, int steps, const char* cache_path, int* chosen, double* ms_out) {
    if (!c) return IBLB_EINVAL;
    if (steps < 2) return fail(c, IBLB_EINVAL, "autotune needs at least 2 steps per variant");
    // cache key: device, lattice, storage, total cells and droplet count (log2 buckets)
    int dev = 0;
    hipDeviceProp_t prop;
    HIPCHK(c, hipGetDevice(&dev));
    HIPCHK(c, hipGetDeviceProperties(&prop, dev));
    int cb = 0, db = 0;
    while ((1LL << cb) < c->L.cells) ++cb;
    while ((1 << db) < c->n) ++db;
    char key[256];
    snprintf(key, sizeof key, "%s/%d D%dQ%d storage=%d cells=2^%d droplets=2^%d", prop.gcnArchName,
             prop.multiProcessorCount, c->dim, c->Q, c->storage, cb, db);
    if (cache_path) {
        FILE* f = fopen(cache_path, "r");
        if (f) {
            char line[512];
            while (fgets(line, sizeof line, f)) {
                char* bar = strrchr(line, '|');
                if (!bar) continue;
                *bar = 0;
                if (strcmp(line, key) == 0) {
                    const int v = atoi(bar + 1);
                    fclose(f);
                    if (v < 0 || v >= kVariants) break;
                    int rc = iblb_set_lb_variant(c, v, chosen);
                    if (ms_out)
                        for (int k = 0; k < kVariants; ++k) ms_out[k] = -1.0;
                    return rc;
                }
            }
            fclose(f);
        }
    }
    // Each variant runs `steps` coupled steps twice: the first call builds
    // its graphs and warms the caches, the second is timed between two
    // events, so the choice is made on what a caller's steps cost (kernel
    // execution, dispatch and drain, and the node work in between), not on
    // the lattice kernel's own execution span alone.
    int rc = ensure_events(c, 2);
    if (rc) return rc;
    hipEvent_t* ev = c->events.data();
    const int was_timing = c->timing;
    c->timing = 0;
    double ms[kVariants];
    double best_ms = 1e300;
    for (int v = 0; v < kVariants; ++v) {
        float t = 0.f;
        rc = iblb_set_lb_variant(c, v, nullptr);
        if (!rc) rc = iblb_step(c, steps);
        if (!rc && hipEventRecord(ev[0], c->stream) != hipSuccess)
            rc = fail(c, IBLB_EDEVICE, "autotune: event record failed");
        if (!rc) rc = iblb_step(c, steps);
        if (!rc && (hipEventRecord(ev[1], c->stream) != hipSuccess ||
                    hipEventSynchronize(ev[1]) != hipSuccess ||
                    hipEventElapsedTime(&t, ev[0], ev[1]) != hipSuccess))
            rc = fail(c, IBLB_EDEVICE, "autotune: event timing failed");
        if (rc) {
            c->timing = was_timing;
            return rc;
        }
        ms[v] = (double)t / steps;
        if (ms_out) ms_out[v] = ms[v];
        best_ms = std::min(best_ms, ms[v]);
    }
    c->timing = was_timing;
    // the lowest-numbered variant within 2% of the fastest: near-ties (run
    // to run noise) then resolve the same way every time
    int best = 0;
    while (ms[best] > 1.02 * best_ms) ++best;
    rc = iblb_set_lb_variant(c, best, chosen);
    if (rc) return rc;
    if (cache_path) {
        FILE* f = fopen(cache_path, "a");
        if (f) {
            fprintf(f, "%s|%d\n", key, best);
            fclose(f);
        }
    }
    return IBLB_OK;
}

int iblb_probe_copy(void* d_dst, const void* d_src, size_t bytes, int reps, void* stream,
                    double* gbs) {
    if (!d_dst || !d_src || !gbs || reps < 1 || bytes < 16 || bytes % 16)
        return fail(nullptr, IBLB_EINVAL, "probe: bad arguments (bytes must be a multiple of 16)");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const long long n = (long long)(bytes / 16);
    const int grid = ceil_div(n, 4LL * kBlock);
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return fail(nullptr, IBLB_EDEVICE, "probe: event");
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(nullptr, IBLB_EDEVICE, "probe: event");
    }
    // best of plain and non-temporal accesses
    double best = 0.0;
    int rc = IBLB_OK;
    for (int nt = 0; nt < 2 && rc == IBLB_OK; ++nt) {
        double total = 0.0;
        for (int r = 0; r <= reps && rc == IBLB_OK; ++r) {
            const v4f* src = static_cast<const v4f*>(d_src);
            v4f* dst = static_cast<v4f*>(d_dst);
            if (nt)
                hipExtLaunchKernelGGL(k_copy_probe<1>, dim3(grid), dim3(kBlock), 0, s, e0, e1, 0,
                                      src, dst, n);
            else
                hipExtLaunchKernelGGL(k_copy_probe<0>, dim3(grid), dim3(kBlock), 0, s, e0, e1, 0,
                                      src, dst, n);
            float ms = 0.f;
            if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
                rc = fail(nullptr, IBLB_EDEVICE, "probe: timing");
            if (r > 0) total += ms;  // the first launch warms up
        }
        if (rc == IBLB_OK) best = std::max(best, 2.0 * (double)bytes * reps / (total * 1e-3) / 1e9);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc == IBLB_OK) *gbs = best;
    return rc;
}

}  // extern "C"
