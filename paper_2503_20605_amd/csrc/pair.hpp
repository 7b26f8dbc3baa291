// Two lattice updates in one pass over the populations.
#pragma once

#include "kernels.hpp"

namespace iblb {

// A barrier of the workgroup that orders LDS accesses only: global loads
// that are in flight stay in flight across it (__syncthreads waits for
// them).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A population as it is stored, loaded without being widened (so that a
// load can stay in flight) through a buffer descriptor: voff per lane, soff
// the same for all lanes.
template <int S>
struct Raw;
template <>
struct Raw<ST_F32> {
    using T = unsigned;
    static __device__ __forceinline__ T load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0);
    }
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, T v) {
        __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)voff, (int)soff, kBufNT);
    }
    static __device__ __forceinline__ float widen(T v) { return __builtin_bit_cast(float, v); }
    static __device__ __forceinline__ T narrow(float v) { return __builtin_bit_cast(unsigned, v); }
};
template <int S>
struct Raw16 {
    using T = unsigned short;
    static __device__ __forceinline__ T load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
        return __builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
    }
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, T v) {
        __builtin_amdgcn_raw_buffer_store_b16(v, r, (int)voff, (int)soff, kBufNT);
    }
};
template <>
struct Raw<ST_F16> : Raw16<ST_F16> {
    static __device__ __forceinline__ float widen(T v) { return (float)__builtin_bit_cast(_Float16, v); }
    static __device__ __forceinline__ T narrow(float v) { return __builtin_bit_cast(unsigned short, (_Float16)v); }
};
template <>
struct Raw<ST_BF16> : Raw16<ST_BF16> {
    static __device__ __forceinline__ float widen(T v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ T narrow(float v) { return to_bf16(v); }
};

// LDS slot of population i: those that move within the plane, in order.
template <int DIM>
constexpr bool in_plane(int i) {
    return Lattice<DIM>::c[i][0] != 0 || (DIM == 3 && Lattice<DIM>::c[i][1] != 0);
}
template <int DIM>
constexpr int lds_slot(int i) {
    int n = 0;
    for (int k = 0; k < i; ++k) n += in_plane<DIM>(k) ? 1 : 0;
    return n;
}
template <int DIM>
struct PairSlots {
    static constexpr int n = lds_slot<DIM>(Lattice<DIM>::Q);
};

template <int DIM, int S, int NT, int VIS>
__global__ __launch_bounds__(NT, 4) void k_lb_pair(const DropDev* __restrict__ drops, const int4* __restrict__ tiles,
                                                const typename Codec<S>::T* __restrict__ fsrc_all,
                                                typename Codec<S>::T* __restrict__ fdst_all,
                                                const float* __restrict__ F_all,
                                                unsigned long long* __restrict__ Fq_all,
                                                float* __restrict__ U_all,
                                                const uint8_t* __restrict__ flags1,
                                                const uint8_t* __restrict__ flags2,
                                                const int* __restrict__ xcnt1, const double* __restrict__ xpos1,
                                                const int* __restrict__ xcnt2, const double* __restrict__ xpos2) {
    using L = Lattice<DIM>;
    using R = Raw<S>;
    using T = typename R::T;
    constexpr int Q = L::Q, A = DIM - 1;  // A: the axis that is marched along
    constexpr unsigned SB = storage_bytes<S>();
    __shared__ T lds[2][PairSlots<DIM>::n][NT];
    const int4 ta = tiles[2 * blockIdx.x], tb = tiles[2 * blockIdx.x + 1];
    const DropDev& D = drops[ta.x];
    const int x0 = ta.y, w = ta.z, y0 = ta.w, h = tb.x, m0 = tb.y, m1 = tb.y + tb.z;
    const int nx = D.nx, ny = D.ny;
    const int M = DIM == 3 ? D.nz : ny, wall = DIM == 3 ? D.bcz : D.bcy;
    const unsigned plB = SB * (unsigned)(DIM == 3 ? D.ppl : nx);  // bytes per plane of a population array
    const unsigned fstB = SB * (unsigned)D.fst;
    const unsigned fpl = (unsigned)(DIM == 3 ? nx * ny : nx);      // cells per plane of the fields
    const int HX = w + 2, t = threadIdx.x;
    const int hy = DIM == 3 ? t / HX : 0, hx = t - hy * HX;
    const bool act = DIM == 3 ? hy < h + 2 : hx < HX;
    const bool inner = act && hx >= 1 && hx <= w && (DIM == 2 || (hy >= 1 && hy <= h));
    int x = 0, y = 0;
    if (act) {
        x = x0 + hx - 1;
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        if (DIM == 3) {
            y = y0 + hy - 1;
            y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
        }
    }
    // byte offsets within a plane: columns x - 1, x, x + 1, rows y - 1, y, y + 1
    const unsigned xs[3] = {SB * (x == 0 ? nx - 1 : x - 1), SB * x, SB * (x == nx - 1 ? 0 : x + 1)};
    const unsigned ys[3] = {SB * nx * (y == 0 ? ny - 1 : y - 1), SB * nx * y, SB * nx * (y == ny - 1 ? 0 : y + 1)};
    const unsigned own = ys[1] + xs[1], own1 = own / SB;
    const unsigned ncell = (unsigned)D.ncell;
    const auto rs = buffer_of(fsrc_all + D.f_off, (int)(Q * fstB));
    const auto rd = buffer_of(fdst_all + D.f_off, (int)(Q * fstB));
    const auto rF = buffer_of(F_all + (long long)DIM * D.c_off, (int)(4 * DIM * ncell));
    const auto rq = buffer_of(Fq_all + (long long)DIM * D.c_off, (int)(8 * DIM * ncell));
    const auto rU = buffer_of(U_all + (long long)DIM * D.c_off, (int)(4 * DIM * ncell));
    const unsigned frow = (unsigned)(DIM == 3 ? D.nstrip * ny : D.nstrip);  // flags per plane
    const auto rg1 = buffer_of(flags1 + D.flag_off, (int)(frow * M));
    const auto rg2 = buffer_of(flags2 + D.flag_off, (int)(frow * M));
    const unsigned fcol = (unsigned)((DIM == 3 ? y * D.nstrip : 0) + (x >> Strip<DIM, S>::shift));
    const bool given = D.force_mode == 1;

    auto wrap = [&](int z) { return z < 0 ? z + M : (z >= M ? z - M : z); };
    auto row_of = [&](int z) { return DIM == 3 ? z * ny + y : z; };
    T pre[Q];
    // populations that arrive in plane z: source planes z - 1, z, z + 1
    auto fetch = [&](int z) {
        const unsigned lo = plB * (unsigned)(z > 0 ? z - 1 : M - 1), mid = plB * (unsigned)z,
                       hi = plB * (unsigned)(z < M - 1 ? z + 1 : 0);
        const bool blo = wall && z == 0, bhi = wall && z == M - 1;
        unsigned so = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i, so += fstB) {
            const int cx = L::c[i][0], cy = DIM == 3 ? L::c[i][1] : 0, ca = L::c[i][A];
            const unsigned off = ys[1 - cy] + xs[1 - cx];
            if (ca == 0) {
                pre[i] = R::load(rs, off, so + mid);
            } else {
                // beyond a wall: the opposite population of this cell (half-way bounce-back)
                const bool b = ca > 0 ? blo : bhi;
                const unsigned sb = opp(i) > i ? so + fstB : so - fstB;
                pre[i] = R::load(rs, b ? own : off, b ? sb + mid : so + (ca > 0 ? lo : hi));
            }
        }
    };
    unsigned f1[3] = {0, 0, 0};
    auto fetch_f1 = [&](int z) {
#pragma unroll
        for (int a = 0; a < DIM; ++a)
            f1[a] = __builtin_amdgcn_raw_buffer_load_b32(rF, (int)(4 * own1), (int)(4 * (a * ncell + z * fpl)), 0);
    };
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 q2[3] = {{0, 0}, {0, 0}, {0, 0}};
    auto fetch_f2 = [&](int z) {
#pragma unroll
        for (int a = 0; a < DIM; ++a)
            q2[a] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rq, (int)(8 * own1), (int)(8 * (a * ncell + z * fpl)), 0));
    };
    auto flag1 = [&](int z) -> int {
        return given ? 1 : (int)__builtin_amdgcn_raw_buffer_load_b8(rg1, (int)fcol, (int)(frow * z), 0);
    };
    auto flag2 = [&](int z) -> int {
        return given ? 1 : (int)__builtin_amdgcn_raw_buffer_load_b8(rg2, (int)fcol, (int)(frow * z), 0);
    };

    float hp1[Q], hp2[Q], h0[Q], sp = 0.f;
#pragma unroll
    for (int i = 0; i < Q; ++i) hp1[i] = hp2[i] = h0[i] = 0.f;
    const int zb = wall && m0 == 0 ? 0 : m0 - 1, ze = m1;
    int fa = 0, fan = 0, fb = 0, fbn = 0;
    if (act) {
        fa = flag1(wrap(zb));
        if (zb + 1 < M || !wall) fan = flag1(wrap(zb + 1));
        if (inner) fbn = flag2(wrap(zb));
        if (fa) fetch_f1(wrap(zb));
        fetch(wrap(zb));
    }
    for (int zp = zb; zp <= ze; ++zp) {
        const bool real = !(wall && zp == M);
        const int par = zp & 1;
        float s[Q];
        if (real && act) {
            const float Fx = fa ? __builtin_bit_cast(float, f1[0]) : 0.f, Fy = fa ? __builtin_bit_cast(float, f1[1]) : 0.f,
                        Fz = DIM == 3 && fa ? __builtin_bit_cast(float, f1[2]) : 0.f;
            const bool forced = __builtin_amdgcn_ballot_w64(fa != 0) != 0;
            float om = D.omega, g = D.guo;
            if (VIS && D.visc && cell_inside(D, xcnt1, xpos1, x, row_of(wrap(zp)))) {
                om = D.omega_in;
                g = D.guo_in;
            }
            float f[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) f[i] = R::widen(pre[i]);
            const Moments<DIM, S> m(f, Fx, Fy, Fz);
            auto put = [&](int i, float fn) {
                const T v = R::narrow(fn);
                s[i] = R::widen(v);
                if (in_plane<DIM>(i)) lds[par][lds_slot<DIM>(i)][t] = v;
            };
            if (forced)
                m.template relax<true>(f, om, g, put);
            else
                m.template relax<false>(f, om, g, put);
        }
        // the next plane's loads
        if (act && zp < ze && !(wall && zp + 1 == M)) {
            fa = fan;
            fan = flag1(wrap(zp + 2 < M || !wall ? zp + 2 : zp + 1));
            if (fa) fetch_f1(wrap(zp + 1));
            fetch(wrap(zp + 1));
        }
        lds_barrier();
        const int zt = zp - 1;
        if (inner) {
            auto arrived = [&](int i) {
                const int cx = L::c[i][0], cy = DIM == 3 ? L::c[i][1] : 0;
                const int tn = cy > 0 ? t - HX : (cy < 0 ? t + HX : t);
                return in_plane<DIM>(i) ? R::widen(lds[par][lds_slot<DIM>(i)][tn - cx]) : s[i];
            };
            if (zt >= m0) {
                float f[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const int ca = L::c[i][A];
                    if (ca > 0)
                        f[i] = hp2[i];
                    else if (ca == 0)
                        f[i] = h0[i];
                    else if (real)
                        f[i] = arrived(i);
                    else  // the wall above: this cell's own populations come back
                        f[i] = in_plane<DIM>(i) ? R::widen(lds[par ^ 1][lds_slot<DIM>(opp(i))][t]) : sp;
                }
                float Fc[3] = {0.f, 0.f, 0.f};
                if (fb) {
#pragma unroll
                    for (int a = 0; a < DIM; ++a)
                        Fc[a] = given ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                                      rF, (int)(4 * own1), (int)(4 * (a * ncell + zt * fpl)), 0))
                                      : fq_value(__builtin_bit_cast(unsigned long long, q2[a]));
                }
                const bool forced = __builtin_amdgcn_ballot_w64(fb != 0) != 0;
                float om = D.omega, g = D.guo;
                if (VIS && D.visc && cell_inside(D, xcnt2, xpos2, x, row_of(zt))) {
                    om = D.omega_in;
                    g = D.guo_in;
                }
                const Moments<DIM, S> m(f, Fc[0], Fc[1], Fc[2]);
                const unsigned so = plB * (unsigned)zt;
                auto put = [&](int i, float fn) { R::store(rd, own, so + (unsigned)i * fstB, R::narrow(fn)); };
                if (forced)
                    m.template relax<true>(f, om, g, put);
                else
                    m.template relax<false>(f, om, g, put);
                if (fb && !given) {
                    const float uu[3] = {m.ux, m.uy, m.uz};
#pragma unroll
                    for (int a = 0; a < DIM; ++a) {
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, uu[a]), rU, (int)(4 * own1),
                                                              (int)(4 * (a * ncell + zt * fpl)), 0);
                        if (q2[a].x | q2[a].y)
                            __builtin_amdgcn_raw_buffer_store_b64(u32x2{0, 0}, rq, (int)(8 * own1),
                                                                  (int)(8 * (a * ncell + zt * fpl)), 0);
                    }
                }
            }
            // the second update of plane zp comes next
            fb = fbn;
            if (zp + 1 < m1) fbn = flag2(wrap(zp + 1));
            if (fb && !given && zp >= m0 && zp < m1) fetch_f2(zp);
            if (real) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const int ca = L::c[i][A];
                    if (ca > 0) {
                        hp2[i] = wall && zp == 0 ? s[opp(i)] : hp1[i];
                        hp1[i] = arrived(i);
                        if (!in_plane<DIM>(i)) sp = s[i];
                    } else if (ca == 0) {
                        h0[i] = arrived(i);
                    }
                }
            }
        }
    }
}

}  // namespace iblb
