// gfx950 kernels of the learned warm start: a small fully connected network
// trained and evaluated with bf16 operands on the matrix cores (fp32
// accumulation), fp32 master weights, Adam.
//
//   k_gemm_bf16     C = A B with A, B bf16 (either operand k-contiguous or
//                   not), fp32 result: a 64x64 tile of C per workgroup, K in
//                   panels staged through LDS with 16-byte loads along the
//                   operand's contiguous index, the next panel fetched while
//                   the current one is multiplied, one 32x32 tile per
//                   wavefront through gfx950's v_mfma_f32_32x32x16_bf16;
//                   optional split of K over workgroups (fp32 atomic
//                   accumulation); epilogue: + bias, optional GELU (keeps
//                   the fp32 pre-activation and writes the bf16
//                   activation), or the GELU backward dZ = C * GELU'(Z)
//   k_mlp_rows      a narrow network's whole forward (or forward and backward)
//                   pass, 32 rows of the batch per workgroup
//   k_wgrad         the weight gradients of all its layers
//   k_pack          its weights in the order of the matrix instruction (when they
//                   are set; k_adam keeps them so)
//   k_mse_colsum    loss, dY = 2 (Y - T) / (B n) and the last layer's bias
//                   gradient (column sums of dY): 64 columns x 256 rows
//                   per workgroup, reduced in LDS, then added atomically
//   k_adam          Adam update of the fp32 master weights + bf16 copy
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lattice.hpp"

namespace iblb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMlpBlock = 256;  // 4 wavefronts, a 64x64 tile of C

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float z) {
    const float cdf = 0.5f * (1.f + erff(z * 0.70710678118654752f));
    const float pdf = 0.39894228040143268f * expf(-0.5f * z * z);
    return cdf + z * pdf;
}

// C(i, j) = sum_k A(i, k) B(k, j) (+ bias[j]) with A, B bf16 and fp32
// accumulation.  Operand layouts (template arguments):
//   AT = 0: A(i, k) = A[i * lda + k]  (k contiguous);  AT = 1: A[k * lda + i]
//   BT = 0: B(k, j) = B[j * ldb + k]  (k contiguous);  BT = 1: B[k * ldb + j]
// A workgroup takes a 64x64 tile of C and walks K in panels of KP: every
// thread fetches its share of the next panel of both operands (KP / 32
// 16-byte pieces of eight elements along the operand's contiguous index)
// while the wavefronts multiply the current one out of LDS, where tiles are
// kept k-contiguous (rows of KP + 8 elements, so every lane's eight MFMA
// operands are one aligned 16-byte read).  avec / bvec = 0 fetches the
// pieces element by element (an operand whose contiguous extent or leading
// dimension is not a multiple of 8, or is not 16-byte aligned).  Elements
// outside M x N x [kbeg, kend) read as zero.
// Epilogue (act): 0: Cf = C + bias; 1: Cf = Z = C + bias, Hb = bf16(GELU(Z));
// 2: Cf = C * GELU'(Zpre), Hb = its bf16 copy (the backward of a GELU layer,
// Zpre its pre-activation, same layout as Hb; Cf may be null), and, when
// colsum is given, colsum[j] += the sum of column j over the rows (added
// atomically).  With gridDim.z = S > 1 the
// workgroups of z take k in [z kc, (z + 1) kc) and add their partial
// products to Cf atomically (Cf zeroed beforehand; no bias, act = 0).
//
// Operand and result layout of one 32x32x16 product (lane l of 64):
//   A: row l % 32, k = 8 (l / 32) + 0..7;  B: column l % 32, same k;
//   result register r: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Piece v (0 .. 64 KP / 8 - 1) of a 64 x KP panel of operand X whose rows r
// (i of A, j of B) start at rb and whose k start at k0.  T = 0: piece v
// holds row v / (KP / 8), k 8 (v % (KP / 8)) + 0..7; T = 1: k v / 8, rows
// 8 (v % 8) + 0..7.
template <int T, int KP>
__device__ __forceinline__ u32x4 panel_fetch(const uint16_t* __restrict__ X, long long ld, int R, int kend,
                                            int rb, int k0, int v, int vec) {
    int r, k;
    if (T == 0) {
        r = rb + v / (KP / 8);
        k = k0 + 8 * (v % (KP / 8));
    } else {
        k = k0 + v / 8;
        r = rb + 8 * (v % 8);
    }
    u32x4 out = {0u, 0u, 0u, 0u};
    if (vec) {
        // the contiguous extent is a multiple of 8: a piece lies wholly
        // inside or wholly outside
        if (r < R && k < kend)
            out = *reinterpret_cast<const u32x4*>(X + (T == 0 ? (long long)r * ld + k : (long long)k * ld + r));
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int ru = T == 0 ? r : r + u, ku = T == 0 ? k + u : k;
            const uint32_t e =
                (ru < R && ku < kend) ? X[T == 0 ? (long long)ru * ld + ku : (long long)ku * ld + ru] : 0u;
            out[u >> 1] |= e << (16 * (u & 1));
        }
    }
    return out;
}

// Piece v into the k-contiguous LDS tile S (rows of KP + 8 elements).
template <int T, int KP>
__device__ __forceinline__ void panel_stash(uint16_t* __restrict__ S, int v, u32x4 x) {
    constexpr int LD = KP + 8;
    if (T == 0) {
        *reinterpret_cast<u32x4*>(S + (v / (KP / 8)) * LD + 8 * (v % (KP / 8))) = x;
    } else {
        const int k = v / 8, r = 8 * (v % 8);
#pragma unroll
        for (int u = 0; u < 8; ++u) S[(r + u) * LD + k] = (uint16_t)(x[u >> 1] >> (16 * (u & 1)));
    }
}

template <int AT, int BT, int KP>
__device__ __forceinline__ void gemm_tile(
    const uint16_t* __restrict__ A, long long lda, const uint16_t* __restrict__ B, long long ldb,
    float* __restrict__ Cf, uint16_t* __restrict__ Hb, long long ldc, const float* __restrict__ bias,
    const float* __restrict__ Zpre, float* __restrict__ colsum, int M, int N, int K, int act, int kc,
    int avec, int bvec, int bx, int by, int bz, bool split) {
    constexpr int LD = KP + 8, NV = KP / 32;
    __shared__ __attribute__((aligned(16))) uint16_t As[64 * LD];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[64 * LD];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int ib = by * 64, jb = bx * 64;
    const int kbeg = bz * kc, kend = K < kbeg + kc ? K : kbeg + kc;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    u32x4 ra[NV], rb[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        ra[u] = panel_fetch<AT, KP>(A, lda, M, kend, ib, kbeg, t + kMlpBlock * u, avec);
        rb[u] = panel_fetch<BT, KP>(B, ldb, N, kend, jb, kbeg, t + kMlpBlock * u, bvec);
    }
    for (int k0 = kbeg; k0 < kend; k0 += KP) {
        if (k0 != kbeg) __syncthreads();  // the previous panel's reads are done
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            panel_stash<AT, KP>(As, t + kMlpBlock * u, ra[u]);
            panel_stash<BT, KP>(Bs, t + kMlpBlock * u, rb[u]);
        }
        __syncthreads();
        if (k0 + KP < kend) {
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                ra[u] = panel_fetch<AT, KP>(A, lda, M, kend, ib, k0 + KP, t + kMlpBlock * u, avec);
                rb[u] = panel_fetch<BT, KP>(B, ldb, N, kend, jb, k0 + KP, t + kMlpBlock * u, bvec);
            }
        }
        // k steps of 16 past kend hold zeros only: skipped
        const int nsteps = (kend - k0 < KP ? kend - k0 + 15 : KP) / 16;
#pragma unroll
        for (int s = 0; s < KP / 16; ++s) {
            if (s < nsteps) {
                const int kq = 16 * s + (lane >> 5) * 8;
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(As + (wi + (lane & 31)) * LD + kq);
                const bf16x8 b = *reinterpret_cast<const bf16x8*>(Bs + (wj + (lane & 31)) * LD + kq);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
            }
        }
    }
    const int j = jb + wj + (lane & 31);
    if (j >= N) return;
    if (split) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = ib + wi + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (i < M) unsafeAtomicAdd(Cf + (long long)i * ldc + j, acc[r]);
        }
        return;
    }
    const float bj = bias ? bias[j] : 0.f;
    float cs = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = ib + wi + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (i >= M) continue;
        const long long o = (long long)i * ldc + j;
        if (act == 2) {
            const float g = acc[r] * gelu_grad(Zpre[o]);
            if (Cf) Cf[o] = g;
            Hb[o] = to_bf16(g);
            cs += g;
        } else {
            const float z = acc[r] + bj;
            Cf[o] = z;
            if (act) Hb[o] = to_bf16(gelu(z));
        }
    }
    if (act == 2 && colsum) {
        // the column sums of dZ (the bias gradient of the layer below):
        // lanes l and l ^ 32 hold the two halves of column j's 32 rows
        cs += __shfl_xor(cs, 32, 64);
        if (lane < 32) unsafeAtomicAdd(colsum + j, cs);
    }
}

template <int AT, int BT, int KP>
__global__ __launch_bounds__(kMlpBlock) void k_gemm_bf16(
    const uint16_t* __restrict__ A, long long lda, const uint16_t* __restrict__ B, long long ldb,
    float* __restrict__ Cf, uint16_t* __restrict__ Hb, long long ldc, const float* __restrict__ bias,
    const float* __restrict__ Zpre, float* __restrict__ colsum, int M, int N, int K, int act, int kc,
    int avec, int bvec) {
    gemm_tile<AT, BT, KP>(A, lda, B, ldb, Cf, Hb, ldc, bias, Zpre, colsum, M, N, K, act, kc, avec, bvec,
                          blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z > 1);
}

// The weight gradients of every layer in one launch: grad W_l = H_l^T dZ_l
// over the batch, both operands as k_mlp_rows left them (batch index
// contiguous, rows beyond the batch zero), added atomically to grad (zeroed
// beforehand) by the workgroups that share a tile's batch range.  tile0[l]
// is layer l's first 64x64 tile among all; blockIdx.y: batch range of kc.
struct MlpWgrad {
    int L, K, kc;
    int w[17], tile0[17];
    long long ld, ht[16], dt[16], woff[16];
};
__global__ __launch_bounds__(kMlpBlock) void k_wgrad(MlpWgrad P, const uint16_t* __restrict__ tbuf,
                                                     float* __restrict__ grad) {
    int l = 0;
    while (l + 1 < P.L && (int)blockIdx.x >= P.tile0[l + 1]) ++l;
    const int t = (int)blockIdx.x - P.tile0[l], in = P.w[l], out = P.w[l + 1], nx = (out + 63) / 64;
    gemm_tile<0, 0, 128>(tbuf + P.ht[l], P.ld, tbuf + P.dt[l], P.ld, grad + P.woff[l], nullptr, out, nullptr, nullptr,
                         nullptr, in, out, P.K, 0, P.kc, 1, 1, t % nx, t / nx, blockIdx.y, true);
}

// The loss gradient of the last layer and its column sums: dY = 2 (Y - T) /
// (M N) for Y, T of M rows and N columns (row-major), written in bf16 for
// the products; colsum[j] += sum_i dY(i, j) (zeroed beforehand; the bias
// gradient); partial[block] = sum of (Y - T)^2 over the block's elements in
// fp64 (the loss, summed on the host in block order).  Workgroup (bx, by)
// takes 64 columns and rows [by kColsumRows, (by + 1) kColsumRows); its 16
// lane groups take every 16th row; the partial sums meet in LDS and each
// column's goes out with one atomic.
constexpr int kColsumBlock = 1024;
constexpr int kColsumRows = 256;
__global__ __launch_bounds__(kColsumBlock) void k_mse_colsum(const float* __restrict__ Y,
                                                              const float* __restrict__ T,
                                                              uint16_t* __restrict__ dYb,
                                                              float* __restrict__ colsum,
                                                              double* __restrict__ partial, int M, int N) {
    __shared__ float part[16][64];
    __shared__ double sq[16][64];
    const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + c;
    const int i0 = blockIdx.y * kColsumRows, i1 = i0 + kColsumRows < M ? i0 + kColsumRows : M;
    const float scale = 2.f / (float)((long long)M * N);
    float s = 0.f;
    double e2 = 0.0;
    if (j < N)
        for (int i = i0 + g; i < i1; i += 16) {
            const long long o = (long long)i * N + j;
            const float e = Y[o] - T[o];
            const float d = scale * e;
            dYb[o] = to_bf16(d);
            s += d;
            e2 += (double)e * e;
        }
    part[g][c] = s;
    sq[g][c] = e2;
    __syncthreads();
    if (g == 0) {
        float t = 0.f;
        double q = 0.0;
        for (int k = 0; k < 16; ++k) {
            t += part[k][c];
            q += sq[k][c];
        }
        if (j < N) unsafeAtomicAdd(colsum + j, t);
        sq[0][c] = q;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double q = 0.0;
        for (int k = 0; k < 64; ++k) q += sq[0][k];
        partial[blockIdx.y * gridDim.x + blockIdx.x] = q;
    }
}

// ---------------------------------------------------------------------------
// Whole passes of a narrow network (every input and hidden width at most
// kRowsWidth) in one launch
// ---------------------------------------------------------------------------
// A workgroup takes 32 rows of the batch through all layers: their
// activations stay in LDS (bf16), a wavefront forms a 32x32 tile of a
// layer's output at a time, and the weights come straight from the caches in
// the order in which the matrix instruction takes them (packed once, when
// the weights change).  One launch per layer spent 11-17 us each on one
// dependent fetch - product - epilogue chain with a workgroup per compute
// unit: 4096 rows of 4-256-256-256-1280 took 59 us forward and 130 us with
// the backward pass through the activations, 29 and 56 so (64 rows: 43 and
// 17 us forward).  What is left is the serial chain through the layers, of
// which the exact GELU of 16 values per lane takes about half.
//
// The products take k in the same order, with the same instruction, as
// k_gemm_bf16: the results are the same bit for bit.
constexpr int kRowsBlock = 512;             // 8 wavefronts
constexpr int kRows = 32;                   // batch rows per workgroup
constexpr int kRowsWidth = 256;             // widest input or hidden layer
constexpr int kRowsLd = kRowsWidth + 8;     // LDS row, elements
constexpr int kMaxLayers = 16;

struct MlpRows {
    int L, batch;
    int w[kMaxLayers + 1];
    long long wp[kMaxLayers];    // packed weights of layer l (elements): B(k, j) = W[k][j]
    long long wt[kMaxLayers];    // packed transposed weights: B(k, j) = W[j][k]
    long long boff[kMaxLayers];  // biases in the parameter vector
    // training
    long long ld;                // row length of the transposed operands below: batch rounded up to 32
    long long z[kMaxLayers];     // pre-activations of layer l (floats), in the lanes' own order: per workgroup
                                 // 1024 for each 32x32 tile
    long long ht[kMaxLayers];    // input of layer l, transposed: [w[l]][ld] bf16
    long long dt[kMaxLayers];    // gradient at the output of layer l, transposed: [w[l + 1]][ld] bf16
};

// 16-byte pieces of a packed K x N operand: piece ((s NT + t) 64 + lane)
// holds B(16 s + 8 (lane / 32) + 0..7, 32 t + lane % 32), zero outside.
__host__ __device__ __forceinline__ long long packed_pieces(int K, int N) {
    return (long long)((K + 15) / 16) * ((N + 31) / 32) * 64;
}

// The pieces of n-tile t of a packed operand (NT n-tiles) for k steps s0 to
// s0 + ks - 1, all requested at once (steps beyond repeat the last), so that
// they can be in flight while the operand before them is still worked on.
struct Pieces {
    u32x4 b[kRowsWidth / 16];
    __device__ __forceinline__ void load(const u32x4* __restrict__ Bp, int ks, int s0, int t, int NT, int lane) {
        const u32x4* __restrict__ p = Bp + ((long long)s0 * NT + t) * 64;
        const int step = NT * 64;
#pragma unroll
        for (int s = 0; s < kRowsWidth / 16; ++s) {
            b[s] = p[lane];
            p += s + 1 < ks ? step : 0;
        }
    }
    // acc += A B for the 32 rows of A in LDS, k steps 0 to ks - 1
    __device__ __forceinline__ f32x16 times(f32x16 acc, const uint16_t* __restrict__ A, int ks, int lane) const {
        const uint16_t* __restrict__ a0 = A + (lane & 31) * kRowsLd + 8 * (lane >> 5);
        if (ks == kRowsWidth / 16) {  // (a branch per step would wait for each LDS read in turn)
#pragma unroll
            for (int s = 0; s < kRowsWidth / 16; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(a0 + 16 * s),
                                                              __builtin_bit_cast(bf16x8, b[s]), acc, 0, 0, 0);
            return acc;
        }
#pragma unroll
        for (int s = 0; s < kRowsWidth / 16; ++s)
            if (s < ks)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(a0 + 16 * s),
                                                              __builtin_bit_cast(bf16x8, b[s]), acc, 0, 0, 0);
        return acc;
    }
};
__device__ __forceinline__ int k_steps(int K) { return (K + 15) / 16; }
__device__ __forceinline__ int n_tiles(int N) { return (N + 31) / 32; }

// Row of result register r of a 32x32 product.
__device__ __forceinline__ int result_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// A tile's column j (this lane's 16 rows, as bf16) into the LDS operand and,
// transposed, into memory: G[j ld + row0 + row] (four consecutive rows are
// one 8-byte store).
__device__ __forceinline__ void rows_put(uint16_t* __restrict__ A, int col, int lane, const uint16_t h[16],
                                         uint16_t* __restrict__ G, bool write) {
#pragma unroll
    for (int r = 0; r < 16; ++r) A[result_row(r, lane) * kRowsLd + col] = h[r];
    if (write) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint64_t v = (uint64_t)h[4 * q] | (uint64_t)h[4 * q + 1] << 16 | (uint64_t)h[4 * q + 2] << 32 |
                               (uint64_t)h[4 * q + 3] << 48;
            *reinterpret_cast<uint64_t*>(G + 8 * q + 4 * (lane >> 5)) = v;
        }
    }
}

// TRAIN = 0: y = the network's output for x; gridDim.y workgroups share the
// last layer's columns of the same rows, and each of them reads the rows of x,
// so y must not overlap x (X = uint16_t: x already rounded to bf16, see
// rows_forward).
// TRAIN = 1: the loss of y against tgt (partial[block], summed on the host in
// block order), the gradients at every layer's output and the inputs of
// every layer (transposed, for k_wgrad), and the bias gradients (column sums,
// added to grad atomically).
__device__ __forceinline__ uint16_t as_bf16(float v) { return to_bf16(v); }
__device__ __forceinline__ uint16_t as_bf16(uint16_t v) { return v; }
template <int TRAIN, typename X>
__global__ __launch_bounds__(kRowsBlock) void k_mlp_rows(MlpRows P, const X* __restrict__ x,
                                                         const uint16_t* __restrict__ packed,
                                                         const float* __restrict__ master, float* __restrict__ y,
                                                         const float* __restrict__ tgt, float* __restrict__ zbuf,
                                                         uint16_t* __restrict__ tbuf, float* __restrict__ grad,
                                                         double* __restrict__ partial) {
    __shared__ __attribute__((aligned(16))) uint16_t buf[2][kRows * kRowsLd];
    __shared__ double sq[kRowsBlock / 64];
    // (the wavefront index is the same for all lanes: keep it scalar)
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63, L = P.L;
    const int row0 = blockIdx.x * kRows, M = P.batch;
    auto fwd = [&](int l) { return reinterpret_cast<const u32x4*>(packed + P.wp[l]); };
    auto bwd = [&](int l) { return reinterpret_cast<const u32x4*>(packed + P.wt[l]); };
    const int K = P.w[L - 1], N = P.w[L], NT = n_tiles(N), KS = k_steps(K);  // of the last layer
    const int t0 = TRAIN ? 0 : (int)((long long)NT * blockIdx.y / gridDim.y);
    const int t1 = TRAIN ? NT : (int)((long long)NT * (blockIdx.y + 1) / gridDim.y);
    Pieces B;
    // request the pieces of layer l's tile of this wavefront (the last layer:
    // its first tile)
    auto request = [&](int l) {
        const int nt = n_tiles(P.w[l + 1]), t = l < L - 1 ? wave : t0 + wave;
        if (t < nt) B.load(fwd(l), k_steps(P.w[l]), 0, t, nt, lane);
    };
    request(0);
    // the input, rounded to bf16; columns up to the next multiple of 16 and
    // rows beyond the batch are zero
    const int K0 = P.w[0], K0p = (K0 + 15) / 16 * 16;
    for (int e = threadIdx.x; e < kRows * K0p; e += kRowsBlock) {
        const int r = e / K0p, k = e - r * K0p;
        const bool in = row0 + r < M && k < K0;
        const uint16_t v = in ? as_bf16(x[(long long)(row0 + r) * K0 + k]) : (uint16_t)0;
        buf[0][r * kRowsLd + k] = v;
        if (TRAIN && k < K0) tbuf[P.ht[0] + k * P.ld + row0 + r] = v;
    }
    __syncthreads();
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.f;
    // this wavefront's tile of a hidden layer's pre-activations
    auto zw = [&](int l) { return zbuf + P.z[l] + ((long long)blockIdx.x * n_tiles(P.w[l + 1]) + wave) * 1024 + lane; };
    int cur = 0;
    for (int l = 0; l < L - 1; ++l) {
        const int Nl = P.w[l + 1];
        const bool mine = wave < n_tiles(Nl);
        f32x16 acc = zero;
        if (mine) acc = B.times(zero, buf[cur], k_steps(P.w[l]), lane);
        request(l + 1);
        if (mine) {
            const int j = 32 * wave + (lane & 31);
            const float bj = j < Nl ? master[P.boff[l] + j] : 0.f;
            uint16_t h[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float z = acc[r] + bj;
                if (TRAIN) zw(l)[r * 64] = z;
                const bool in = j < Nl && (!TRAIN || row0 + result_row(r, lane) < M);
                const uint16_t v = to_bf16(gelu(z));
                h[r] = in ? v : (uint16_t)0;
            }
            rows_put(buf[cur ^ 1], j, lane, h, TRAIN ? tbuf + P.ht[l + 1] + (long long)j * P.ld + row0 : nullptr,
                     TRAIN && j < Nl);
        }
        cur ^= 1;
        __syncthreads();
    }
    const uint16_t* __restrict__ H = buf[cur];
    if (!TRAIN) {
        for (int t = t0 + wave; t < t1; t += kRowsBlock / 64) {
            const f32x16 acc = B.times(zero, H, KS, lane);
            if (t + kRowsBlock / 64 < t1) B.load(fwd(L - 1), KS, 0, t + kRowsBlock / 64, NT, lane);
            const int j = 32 * t + (lane & 31);
            const float bj = j < N ? master[P.boff[L - 1] + j] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = row0 + result_row(r, lane);
                if (i < M && j < N) y[(long long)i * N + j] = acc[r] + bj;
            }
        }
        return;
    }
    // training: the last layer in chunks of kRowsWidth columns; each chunk's
    // loss gradient is at once multiplied into the gradient at the layer below
    const float scale = 2.f / (float)((long long)M * N);
    const int JT = L > 1 ? n_tiles(K) : 0;  // tiles of the layer below
    __shared__ __attribute__((aligned(16))) uint16_t dy[2][kRows * kRowsLd];
    f32x16 down = zero;
    double e2 = 0.0;
    int par = 0;
    for (int c = 0; c < N; c += kRowsWidth, par ^= 1) {
        const int t = c / 32 + wave, j = 32 * t + (lane & 31);
        const int kc = N - c < kRowsWidth ? N - c : kRowsWidth;
        Pieces D;  // of the product with the transposed weights
        if (wave < JT) D.load(bwd(L - 1), k_steps(kc), c / 16, wave, JT, lane);
        if (t < NT) {
            // the targets are requested together (elements outside: a valid
            // one instead, not used)
            float tv[16];
            const int jc = j < N ? j : N - 1;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = row0 + result_row(r, lane);
                tv[r] = tgt[(long long)(i < M ? i : M - 1) * N + jc];
            }
            const float bj = master[P.boff[L - 1] + jc];
            const f32x16 acc = B.times(zero, H, KS, lane);
            if (t + kRowsBlock / 64 < NT) B.load(fwd(L - 1), KS, 0, t + kRowsBlock / 64, NT, lane);
            uint16_t h[16];
            float cs = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = row0 + result_row(r, lane) < M && j < N;
                const float e = in ? (acc[r] + bj) - tv[r] : 0.f;
                const float d = scale * e;
                e2 += (double)e * e;
                cs += d;
                h[r] = to_bf16(d);
            }
            rows_put(dy[par], 32 * wave + (lane & 31), lane, h, tbuf + P.dt[L - 1] + (long long)j * P.ld + row0, j < N);
            cs += __shfl_xor(cs, 32, 64);
            if (lane < 32 && j < N) unsafeAtomicAdd(grad + P.boff[L - 1] + j, cs);
        }
        __syncthreads();
        if (wave < JT) down = D.times(down, dy[par], k_steps(kc), lane);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) e2 += __shfl_xor(e2, o, 64);
    if (lane == 0) sq[wave] = e2;
    // gradients at the hidden layers' outputs, from the last one down
    for (int l = L - 2; l >= 0; --l) {
        const int Nl = P.w[l + 1], Tl = n_tiles(P.w[l]);
        const bool mine = wave < n_tiles(Nl);
        float z[16];
        if (mine)
#pragma unroll
            for (int r = 0; r < 16; ++r) z[r] = zw(l)[r * 64];
        if (l > 0 && wave < Tl) B.load(bwd(l), k_steps(Nl), 0, wave, Tl, lane);
        __syncthreads();  // every wavefront is done with the operand below
        if (mine) {
            const int j = 32 * wave + (lane & 31);
            uint16_t h[16];
            float cs = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = j < Nl && row0 + result_row(r, lane) < M;
                const float gz = down[r] * gelu_grad(z[r]);
                const float g = in ? gz : 0.f;
                cs += g;
                h[r] = to_bf16(g);
            }
            rows_put(dy[0], j, lane, h, tbuf + P.dt[l] + (long long)j * P.ld + row0, j < Nl);
            cs += __shfl_xor(cs, 32, 64);
            if (lane < 32 && j < Nl) unsafeAtomicAdd(grad + P.boff[l] + j, cs);
        }
        if (l == 0) break;
        __syncthreads();
        if (wave < Tl) down = B.times(zero, dy[0], k_steps(Nl), lane);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double q = 0.0;
        for (int k = 0; k < kRowsBlock / 64; ++k) q += sq[k];
        partial[blockIdx.x] = q;
    }
}

// The weights of every layer packed for Pieces, both ways (both; else for
// forward passes only), from the bf16 copy wb (row-major [w[l]][w[l + 1]] at woff): one lane per 16-byte
// piece, layer blockIdx.y.
struct MlpPack {
    int L, both;
    int w[kMaxLayers + 1];
    long long woff[kMaxLayers], wp[kMaxLayers], wt[kMaxLayers];
};
__global__ __launch_bounds__(kMlpBlock) void k_pack(MlpPack P, const uint16_t* __restrict__ wb,
                                                    uint16_t* __restrict__ packed) {
    const int l = blockIdx.y, in = P.w[l], out = P.w[l + 1];
    const uint16_t* __restrict__ W = wb + P.woff[l];
    const long long nf = packed_pieces(in, out), nt = P.both ? packed_pieces(out, in) : 0;
    for (long long v = (long long)blockIdx.x * kMlpBlock + threadIdx.x; v < nf + nt;
         v += (long long)gridDim.x * kMlpBlock) {
        const bool tr = v >= nf;  // transposed: B(k, j) = W[j][k]
        const long long p = tr ? v - nf : v;
        const int K = tr ? out : in, N = tr ? in : out, NT = (N + 31) / 32;
        const int lane = (int)(p & 63), t = (int)((p >> 6) % NT), s = (int)((p >> 6) / NT);
        const int j = 32 * t + (lane & 31), k0 = 16 * s + 8 * (lane >> 5);
        u32x4 o = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + u;
            const uint32_t e = (k < K && j < N) ? W[tr ? (long long)j * out + k : (long long)k * out + j] : 0u;
            o[u >> 1] |= e << (16 * (u & 1));
        }
        reinterpret_cast<u32x4*>(packed + (tr ? P.wt[l] : P.wp[l]))[p] = o;
    }
}

// The packed copies of parameter i, h its bf16 value (biases have none).
__device__ __forceinline__ void put_packed(const MlpPack& P, uint16_t* __restrict__ packed, long long i, uint16_t h) {
    int l = 0;
    while (l + 1 < P.L && i >= P.woff[l + 1]) ++l;
    const unsigned in = P.w[l], out = P.w[l + 1];
    const long long o = i - P.woff[l];
    if (o >= (long long)in * out) return;
    const unsigned k = (unsigned)o / out, j = (unsigned)o - k * out;  // (in <= kRowsWidth: 32 bits)
    auto at = [](unsigned r, unsigned c, unsigned NT) {  // element B(r, c) of a packed operand
        return ((long long)(r / 16 * NT + c / 32) * 64 + (c & 31) + 32 * (r / 8 & 1)) * 8 + (r & 7);
    };
    packed[P.wp[l] + at(k, j, (out + 31) / 32)] = h;
    if (P.both) packed[P.wt[l] + at(j, k, (in + 31) / 32)] = h;
}

// x[i] = 0 for i < n
__global__ void k_zero_f32(float* __restrict__ x, long long n) {
    const long long i = (long long)blockIdx.x * kMlpBlock + threadIdx.x;
    if (i < n) x[i] = 0.f;
}

// Adam (Kingma & Ba) on the fp32 master copy; bc1 = 1 - beta1^t,
// bc2 = 1 - beta2^t.  Writes the bf16 copy used by the products and, with
// PACK, its packed form, element by element (a launch of k_pack after every
// step instead: 16-2048 69 us per training step against 46, 4-256-256-256-1280
// 142 against 140).
template <bool PACK>
__global__ void k_adam(float* __restrict__ w, uint16_t* __restrict__ wb, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, long long n, float lr,
                       float beta1, float beta2, float eps, float bc1, float bc2, MlpPack K,
                       uint16_t* __restrict__ packed) {
    const long long i = (long long)blockIdx.x * kMlpBlock + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    w[i] = wi;
    const uint16_t h = to_bf16(wi);
    wb[i] = h;
    if (PACK) put_packed(K, packed, i, h);
}

// fp32 -> bf16 (nearest even), n elements
__global__ void k_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, long long n) {
    const long long i = (long long)blockIdx.x * kMlpBlock + threadIdx.x;
    if (i < n) y[i] = to_bf16(x[i]);
}

}  // namespace iblb
