// Alternating low-rank initialisation of the adapter (Sec. 4.1, "Using LoftQ as low-rank
// initializer"; App. D): starting from B A = 0, every step quantizes the residual W - B A with the
// layer's widths and tables and then fits B A to what the quantized weights miss, E = W - What.
//
// The paper takes the rank-r fit from an SVD.  Here it is a block power (subspace) iteration, which
// only needs products with E and E^T -- the two tall-skinny kernels this library already has:
//   Y = E A^T   [N, r]   (lora_side.hip, contraction over the input features)
//   Z = Y^T E   [r, K]   (adapter_grads.hip, contraction over the channels)
//   A <- rows of Z made orthonormal (Gram matrix, Cholesky factor, triangular solve: below)
// and, after the last round, B = E A^T, so that B A is the projection of E onto the row space
// found.  The start is a random A the caller passes in; later steps start from the previous
// step's A, whose row space hardly moves between steps.  E, Y, A and B are bf16 (B and A are what
// the linear calls consume), Z and the orthonormalisation are fp32 / fp64.
#include <algorithm>

#include "gemm_common.h"

namespace lowra {

hipError_t launch_skinny(const uint16_t* P, int ldp, int M, const uint16_t* Q, int ldq, int r, int Kc,
                         float s, uint16_t* out, int RP, hipStream_t st);
size_t tn_partial_bytes(int C, int M, int RP);
hipError_t launch_tn_partial(const uint16_t* P, int C, int M, const uint16_t* Q, float* partial, int* chunks, hipStream_t st);

constexpr int LQ_RP = 64;      // rank padded to the side products' row length
constexpr int LQ_GT = 32;      // columns of Z per tile of its Gram matrix
constexpr int LQ_GBLOCKS = 136, LQ_GENTRIES = 16 * LQ_GBLOCKS;       // 4 x 4 blocks on and below the diagonal of a 64 x 64 matrix

// ---- F = W - Y At^T: Y [N][64] bf16 (B, padded with zero columns), At [K][64] bf16 (A^T, padded)
// A wavefront owns 32 channels x 128 input features: its 32 x 64 piece of Y stays in registers,
// each 32 x 32 tile is 4 MFMAs, W is read and F written in 128-byte segments, 4 side by side per row.
__global__ __launch_bounds__(256) void residual_kernel(const float* __restrict__ W, const uint16_t* __restrict__ Y,
                                                       const uint16_t* __restrict__ At, float* __restrict__ F, int N, int K) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 31, h = lane >> 5;
    const int n0 = blockIdx.x * 32;
    const int kbase = blockIdx.y * 512 + wave * 128;
    if (kbase >= K) return;                                        // whole wavefront; the kernel has no barrier
    const int nrow = min(n0 + i, N - 1);                           // rows past N: a valid row, never stored
    bf16x8_t yf[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) yf[kk] = *reinterpret_cast<const bf16x8_t*>(Y + (size_t)nrow * LQ_RP + 16 * kk + 8 * h);
    // K is a multiple of 64: a 32-wide tile is in or out as a whole
    floatx16_t acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
        const int kr = min(kbase + 32 * t + i, K - 1);               // a tile past K: valid rows of At, result unused
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const bf16x8_t af = *reinterpret_cast<const bf16x8_t*>(At + (size_t)kr * LQ_RP + 16 * kk + 8 * h);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(yf[kk], af, acc[t], 0, 0, 0);
        }
    }
    // acc[t][v] = (Y At^T)[n0 + 8 (v/4) + 4 h + v%4][kbase + 32 t + i]: row by row, the wavefront's 4 tiles side by side
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int n = n0 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (n < N) {
            float w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) w[t] = kbase + 32 * t < K ? W[(size_t)n * K + kbase + 32 * t + i] : 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (kbase + 32 * t < K) F[(size_t)n * K + kbase + 32 * t + i] = w[t] - acc[t][v];
        }
    }
}

// ---- E = bf16(W - What), What decoded on the fly (App. A.2: table level times the group's absmax, fp32):
// one workgroup per channel, 8 weights per lane and pass; nothing but E is written.
__global__ __launch_bounds__(256) void residual_of_decode_kernel(const RowInfo* __restrict__ rows, const uint8_t* __restrict__ packed,
                                                                 const float* __restrict__ absmax, const float* __restrict__ mappings,
                                                                 const float* __restrict__ W, uint16_t* __restrict__ E, int K) {
    __shared__ float tab[kTableStride];
    const int n = blockIdx.x, tid = threadIdx.x, units = K >> 3;
    const RowInfo ri = rows[n];
    const int bits = ri.bits();
    if (tid < kTableStride) tab[tid] = mappings[(size_t)ri.cb() * kTableStride + tid];
    __syncthreads();
    const uint8_t* row = packed + ri.offset;
    const float* am = absmax + (size_t)n * (K / kGroup);
    const float4* w4 = reinterpret_cast<const float4*>(W + (size_t)n * K);
    uint4* e4 = reinterpret_cast<uint4*>(E + (size_t)n * K);
    const uint32_t mask = (1u << bits) - 1u;
    for (int base = 0; base < units; base += 512) {
        uint32_t c[2];
        float a[2];
        float4 w[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int u = min(base + tid + q * 256, units - 1);          // past the row's end: in bounds, never stored
            c[q] = load_codes8(row, u, bits);
            a[q] = am[u >> 3];
            w[q][0] = w4[2 * u]; w[q][1] = w4[2 * u + 1];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int u = base + tid + q * 256;
            if (u < units) {
                float d[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) d[i] = tab[(c[q] >> (i * bits)) & mask] * a[q];
                e4[u] = make_uint4(pack_bf16x2(w[q][0].x - d[0], w[q][0].y - d[1]), pack_bf16x2(w[q][0].z - d[2], w[q][0].w - d[3]),
                                   pack_bf16x2(w[q][1].x - d[4], w[q][1].y - d[5]), pack_bf16x2(w[q][1].z - d[6], w[q][1].w - d[7]));
            }
        }
    }
}

// ---- Z = the sum of its chunks' partial sums [nchunks][K][64], in chunk order, left as Zt [K][64]; and partial Gram matrices
// of it (fp64): the sum over a workgroup's columns k of Z[i][k] Z[j][k], block by block, Gp[workgroup][block][4 u + v] being entry
// (4 bi + u, 4 bj + v) of block bi (bi + 1) / 2 + bj, bj <= bi.
// A workgroup takes `per` tiles of 32 columns one after the other.  The contraction is bound by a compute unit's fp64 rate, so
// the tiles are small (128 workgroups at 4096 columns); wavefront w takes the rows [16 w, 16 w + 16) of the result, lane
// (bi, bj) the 4 x 4 block of rows 16 w + 4 bi .., columns 4 bj ..: no sum over wavefronts.  At 64 x 4096 with four chunks
// 6.2 us; a launch for the sum, transposed, and one for the Gram matrices took 3.9 + 7.1.
__global__ __launch_bounds__(256) void zsum_gram_kernel(const float* __restrict__ partial, int nchunks, int K, float* __restrict__ Zt,
                                                        double* __restrict__ Gp, int per) {
    constexpr int ZS = 68;                                           // row stride of zt: 16-byte aligned rows
    __shared__ __align__(16) float zt[LQ_GT * ZS];                   // zt[k][i]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, bi = lane >> 4, bj = lane & 15;
    const int row0 = 16 * wave + 4 * bi, lc = tid >> 3, lr = (tid & 7) * 8;      // I bring ranks lr .. + 7 of column lc
    double g[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) g[u][v] = 0.0;
    const int t_hi = min(((int)blockIdx.x + 1) * per, K / LQ_GT);    // K is a multiple of 64
    for (int t = blockIdx.x * per; t < t_hi; ++t) {
        const size_t at = (size_t)(t * LQ_GT + lc) * 64 + lr;
        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
        for (int k0 = 0; k0 < nchunks; k0 += 4) {                    // four chunks in flight
            float4 p[4], q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float* src = partial + (size_t)min(k0 + k, nchunks - 1) * K * 64 + at;
                p[k] = *reinterpret_cast<const float4*>(src); q[k] = *reinterpret_cast<const float4*>(src + 4);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k0 + k < nchunks) {
                    a.x += p[k].x; a.y += p[k].y; a.z += p[k].z; a.w += p[k].w;
                    b.x += q[k].x; b.y += q[k].y; b.z += q[k].z; b.w += q[k].w;
                }
        }
        *reinterpret_cast<float4*>(Zt + at) = a; *reinterpret_cast<float4*>(Zt + at + 4) = b;
        __syncthreads();                                             // the tile before has been read
        *reinterpret_cast<float4*>(zt + lc * ZS + lr) = a; *reinterpret_cast<float4*>(zt + lc * ZS + lr + 4) = b;
        __syncthreads();
        if (4 * bj <= row0) {                                        // blocks above the diagonal: nothing to do
#pragma unroll 4
            for (int k = 0; k < LQ_GT; ++k) {
                const float4 a4 = *reinterpret_cast<const float4*>(zt + k * ZS + row0);
                const float4 b4 = *reinterpret_cast<const float4*>(zt + k * ZS + 4 * bj);
                const double x[4] = {a4.x, a4.y, a4.z, a4.w}, y[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[u][v] = fma(x[u], y[v], g[u][v]);
            }
        }
    }
    if (4 * bj <= row0) {
        const int r4 = row0 >> 2;
        double* out = Gp + (size_t)blockIdx.x * LQ_GENTRIES + (r4 * (r4 + 1) / 2 + bj) * 16;
#pragma unroll
        for (int u = 0; u < 4; ++u) *reinterpret_cast<double4*>(out + 4 * u) = make_double4(g[u][0], g[u][1], g[u][2], g[u][3]);
    }
}

// ---- G [64][64] (the blocks on and below the diagonal) = the sum of the partial matrices.  A kernel of its own because one
// compute unit fetches about 30 GB/s: the partial matrices took a single workgroup of the factorisation 18 us; spread over
// the chip it takes 4 us, launch included.  Four threads share an entry, a run of partial matrices each, added in their order.
__global__ __launch_bounds__(256) void gram_sum_kernel(const double* __restrict__ Gp, int parts, double* __restrict__ G) {
    __shared__ double run[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;                            // entry 4 u + v of a block
    const int each = (parts + 3) / 4, hi = min((q + 1) * each, parts);
    double sum = 0.0;
    for (int c0 = q * each; c0 < hi; c0 += 16) {
        double part[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) part[i] = Gp[(size_t)min(c0 + i, hi - 1) * LQ_GENTRIES + e];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (c0 + i < hi) sum += part[i];
    }
    run[q][lane] = sum;
    __syncthreads();
    if (q > 0) return;
    int bi = 0;
    while ((bi + 1) * (bi + 2) / 2 <= e >> 4) ++bi;
    const int bj = (e >> 4) - bi * (bi + 1) / 2;
    G[(4 * bi + ((e >> 2) & 3)) * 64 + 4 * bj + (e & 3)] = ((run[0][lane] + run[1][lane]) + run[2][lane]) + run[3][lane];
}
static_assert(LQ_GENTRIES % 64 == 0, "whole workgroups of entries");

// ---- G = L L^T (fp64) and A = L^-1 Z by forward substitution: orthonormal rows, written as bf16 [64][K] (rows >= r zero)
// and transposed, At [K][64].  One workgroup of eight wavefronts per 64 columns of Z; every workgroup factors G for
// itself, since a serial 64 x 64 factorisation takes one compute unit as long as it takes sixty-four, and a launch of
// its own cost its gap and a round trip of the factor through memory.
// A pivot that vanishes (a row of Z inside the span of the earlier ones, a row >= r, or Z = 0) gets a zero column and
// a zero reciprocal: that row of A comes out zero and the rest stays orthonormal.
// The factorisation is a chain of 64 pivots, each waiting for the one before: what bounds it is the latency of one
// pivot.  So wavefront p keeps panel p, columns 8 p .. 8 p + 7, with one row per lane: its eight pivots need no LDS and
// no barrier and solve all rows below the panel on the way; the panel is then published through LDS (double
// buffered) and every wavefront to its right takes the rank-8 product off its own, the next one first: a 16-byte LDS read
// of one address costs as much as one of 64 (eight cycles of the unit's LDS), and with all seven at it each waited for 250
// of them.  The next pivot's value is formed beside the column, from two entries read before the reciprocal root is known,
// so that only arithmetic is on the chain.
// The substitution goes by blocks of 16 rows on the matrix cores (fp32): the blocks on L's diagonal are inverted in fp64
// -- each by a wavefront that has nothing left to factor, while the factorisation goes on -- and
//     a_b = L_bb^-1 s_b,   a_b += L_bb^-1 (s_b - L_bb a_b),   s_c -= L_cb a_b   for the blocks c below.
// (The second product makes it as exact as row-by-row substitution: without it the rounding of the inverse costs up to
// twice that error where the rows are nearly dependent.)
// A wavefront takes 16 columns through all four blocks: with k = 4 (lane / 16) + v as the contraction index of the v-th
// MFMA, a result lies in the registers as the next product reads it, so there is no barrier and no LDS on that chain.
// Measured at 64 x 4096: 15.9 us, of them 1.2 the loads, 9.8 the factorisation (3600 cycles a panel: its eight pivots
// 1500, the product off the next panel 950, the rest LDS and barriers), 1.8 the last block's inverse and 1.9 the
// substitution (in fp64 on the matrix cores this alone took 4 us more).  The two launches before, a panel of four columns
// over sixteen lanes of one workgroup and a substitution on the vector units with L broadcast from LDS, took 16.3 + 8 us.
// 1 / sqrt(d) for d > 0 from the hardware's approximation and one Newton step (about 1e-13; the factor is rounded to fp32
// afterwards): the library's correctly rounded division and square root are some forty instructions each, and one
// reciprocal root sits on the critical path of every pivot.
__device__ __forceinline__ double lq_rsqrt(double d) {
    const double r = __builtin_amdgcn_rsq(d);
    return r * fma(-0.5 * d * r, r, 1.5);
}

// v of lane `lane` (the same for the whole wavefront) as a wavefront-uniform value
__device__ __forceinline__ double lq_readlane(double v, int lane) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// lane `c` of my row of sixteen lanes (c < 16, a constant)
template <int C>
__device__ __forceinline__ double lq_row_bcast(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, 0x150 + C, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), 0x150 + C, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// one step of the inversion below: the rows under row C lose their share of it (l[C] is zero in the others)
template <int C>
__device__ __forceinline__ void lq_invert_from(double (&x)[4], const double (&l)[16], const double* rd) {
    const double rc = rd[C];
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = fma(-l[C], lq_row_bcast<C>(x[v]) * rc, x[v]);
    if constexpr (C < 14) lq_invert_from<C + 1>(x, l, rd);
}

constexpr int LQ_APPLY_THREADS = 512;
constexpr int LQ_LS = 68;                                            // row stride of Ls: 16-byte reads of 16 rows meet all banks
__global__ __launch_bounds__(LQ_APPLY_THREADS) void factor_apply_kernel(const float* __restrict__ Zt, const double* __restrict__ G, int K, int r,
                                                                        uint16_t* __restrict__ A, uint16_t* __restrict__ At) {
    __shared__ double2 pan[2][4][64];                                // [buffer][pair of columns of the panel][row]
    __shared__ double2 diag[4][16][8];                               // the 16 x 16 blocks on L's diagonal (below their diagonals)
    __shared__ __align__(16) float Lb[4][16][20];                    // the same blocks whole, for the substitution
    __shared__ __align__(16) double rdiag[64];                       // 1 / L[i][i]
    __shared__ __align__(16) float Ls[64 * LQ_LS];                   // L below its diagonal blocks, these blocks' inverses
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, h = lane >> 4;
    const int k = blockIdx.x * 64 + 16 * w + i;                      // K is a multiple of 64: wavefronts 0 .. 3 have a column per i
    double g[8], is[8];                                              // row `lane` of my panel (rows above it are never used); 1 / its pivots
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double2 v = lane >= 8 * w ? reinterpret_cast<const double2*>(G + lane * 64 + 8 * w)[q] : make_double2(0.0, 0.0);
        g[2 * q] = v.x; g[2 * q + 1] = v.y;
    }
    double maxdiag = G[lane * 65];
    floatx4_t s[4];                                                  // s[b][v]: row 16 b + 4 h + v of column k
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        s[b] = floatx4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (w < 4) {                                                 // (columns of Zt from r on are zeros: the matching ones of Y are)
            const float4 z = *reinterpret_cast<const float4*>(Zt + (size_t)k * 64 + 16 * b + 4 * h);
            s[b] = floatx4_t{z.x, z.y, z.z, z.w};
        }
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) maxdiag = fmax(maxdiag, __shfl_xor(maxdiag, o, 64));
    const double tiny = 1e-12 * fmax(maxdiag, 0.0);
    auto factor = [&](int p) {                                       // my panel, p == w: factored and published
        double pv = lq_readlane(g[0], 8 * p);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            is[j] = pv > tiny ? lq_rsqrt(pv) : 0.0;
            double l = 0.0;
            if (j < 7) {                                             // the same operations as in the column below
                l = lq_readlane(g[j], 8 * p + j + 1) * is[j];
                pv = fma(-l, l, lq_readlane(g[j + 1], 8 * p + j + 1));
            }
            g[j] *= is[j];
#pragma unroll
            for (int c = j + 1; c < 8; ++c) g[c] = fma(-g[j], c == j + 1 ? l : lq_readlane(g[j], 8 * p + c), g[c]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) pan[p & 1][q][lane] = make_double2(g[2 * q], g[2 * q + 1]);
    };
    auto update = [&](int p) {                                       // my panel less panel p's rank-8 product
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double2 mine = pan[p & 1][q][lane];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const double2 l = pan[p & 1][q][8 * w + c];
                g[c] = fma(-mine.y, l.y, fma(-mine.x, l.x, g[c]));
            }
        }
    };
    if (w == 0) factor(0);
    for (int p = 0; p < 8; ++p) {
        __syncthreads();                                             // panel p is published
        if (w == p + 1) update(p);                                   // the next panel first, with the LDS to itself
        if (w == p) {
            if (h == p >> 1) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    diag[h][i][4 * (p & 1) + q] = make_double2(g[2 * q], g[2 * q + 1]);
                    const int c = 8 * (p & 1) + 2 * q;
                    *reinterpret_cast<float2*>(&Lb[h][i][c]) = make_float2(c <= i ? (float)g[2 * q] : 0.0f, c + 1 <= i ? (float)g[2 * q + 1] : 0.0f);
                }
            }
            if (lane == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) reinterpret_cast<double2*>(rdiag + 8 * p)[q] = make_double2(is[2 * q], is[2 * q + 1]);
            }
            if (h > p >> 1) {
                float4* dst = reinterpret_cast<float4*>(Ls + lane * LQ_LS + 8 * p);
                dst[0] = make_float4((float)g[0], (float)g[1], (float)g[2], (float)g[3]);
                dst[1] = make_float4((float)g[4], (float)g[5], (float)g[6], (float)g[7]);
            }
        }
        __syncthreads();
        if (w == p + 1) factor(p + 1);
        else if (w > p) update(p);
        else if ((p & 1) && w == p - 1) {                            // block p / 2 of the diagonal is complete: its inverse
            const int b = p >> 1;
            double l[16], x[4];                                      // row i of L's block; entries 4 h + v of row i of the inverse
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double2 v = diag[b][i][q];
                l[2 * q] = i > 2 * q ? v.x : 0.0; l[2 * q + 1] = i > 2 * q + 1 ? v.y : 0.0;
            }
            const double mine = rdiag[16 * b + i];
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = i == 4 * h + v ? 1.0 : 0.0;
            lq_invert_from<0>(x, l, rdiag + 16 * b);
            *reinterpret_cast<float4*>(Ls + (16 * b + i) * LQ_LS + 16 * b + 4 * h) =
                make_float4((float)(x[0] * mine), (float)(x[1] * mine), (float)(x[2] * mine), (float)(x[3] * mine));
        }
    }
    __syncthreads();
    if (w >= 4) return;                                              // whole wavefronts; no barrier follows
    auto block = [&](const float* at, float sign, const floatx4_t& x, floatx4_t acc) {   // acc + sign times the block at `at`, x
        const float4 l = *reinterpret_cast<const float4*>(at);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sign * l.x, x[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sign * l.y, x[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sign * l.z, x[2], acc, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(sign * l.w, x[3], acc, 0, 0, 0);
    };
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const float* at = Ls + (16 * b + i) * LQ_LS + 16 * b + 4 * h;
        floatx4_t a = block(at, 1.0f, s[b], floatx4_t{0.0f, 0.0f, 0.0f, 0.0f});
        a = block(at, 1.0f, block(&Lb[b][i][4 * h], -1.0f, a, s[b]), a);
#pragma unroll
        for (int c = b + 1; c < 4; ++c) s[c] = block(at + 16 * (c - b) * LQ_LS, -1.0f, a, s[c]);
        const uint32_t lo = pack_bf16x2(a[0], a[1]), hi = pack_bf16x2(a[2], a[3]);
        uint16_t* dst = A + (size_t)(16 * b + 4 * h) * K + k;
        dst[0] = (uint16_t)lo; dst[K] = (uint16_t)(lo >> 16); dst[2 * (size_t)K] = (uint16_t)hi; dst[3 * (size_t)K] = (uint16_t)(hi >> 16);
        *reinterpret_cast<uint2*>(At + (size_t)k * LQ_RP + 16 * b + 4 * h) = make_uint2(lo, hi);
    }
}

// dst [rows][cols] = src [rows][ld] restricted to its first `cols` columns
__global__ __launch_bounds__(256) void copy_cols_kernel(const uint16_t* __restrict__ src, int ld, size_t rows, int cols, uint16_t* __restrict__ dst) {
    const size_t tot = rows * (size_t)cols;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < tot; e += (size_t)gridDim.x * 256)
        dst[e] = src[(e / cols) * ld + (e % cols)];
}

static inline size_t lq_align(size_t v) { return (v + 255) & ~(size_t)255; }

// Gp: the partial Gram matrices.  They lie in the place of F, which is used up by the time of the first round, or, with so few
// channels that F is smaller than 32 KB per 128 features, in a place of their own.
struct LoftqWs {
    size_t F, E, Y, Z, partial, Gp, Gp_bytes, G, A, At, total;
};
static LoftqWs loftq_ws(int N, int K) {
    LoftqWs w;
    size_t o = 0;
    w.F = o; o += lq_align((size_t)N * K * 4);
    w.E = o; o += lq_align((size_t)N * K * 2);
    w.Y = o; o += lq_align((size_t)N * LQ_RP * 2);
    w.Z = o; o += lq_align((size_t)LQ_RP * K * 4);
    w.partial = o; o += lq_align(tn_partial_bytes(K, N, LQ_RP));
    w.Gp = w.F; w.Gp_bytes = (size_t)N * K * 4;
    const size_t own = (size_t)((K + 127) / 128) * 4096 * sizeof(double);
    if (w.Gp_bytes < own) { w.Gp = o; w.Gp_bytes = own; o += lq_align(own); }
    w.G = o; o += lq_align(4096 * sizeof(double));
    w.A = o; o += lq_align((size_t)LQ_RP * K * 2);
    w.At = o; o += lq_align((size_t)K * LQ_RP * 2);
    w.total = o;
    return w;
}
size_t loftq_workspace_bytes(const lowra_layout& L, int r) { return r > 0 ? loftq_ws(L.N, L.K).total : 0; }

static unsigned lq_grid(size_t items) { return (unsigned)std::min<size_t>((items + 255) / 256, 16384); }

hipError_t launch_loftq(const lowra_layout& L, const float* W, const float* thresholds, const float* mappings, int r, int steps,
                        int iters, const uint16_t* omega, uint8_t* packed, float* absmax, uint16_t* A_out, uint16_t* B_out,
                        void* workspace, hipStream_t st) {
    const int N = L.N, K = L.K;
    hipError_t e;
    if (r == 0) return launch_quantize(L, W, thresholds, packed, absmax, st);      // nothing to fit: plain quantization
    const LoftqWs o = loftq_ws(N, K);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    float* F = reinterpret_cast<float*>(ws + o.F);
    uint16_t* E = reinterpret_cast<uint16_t*>(ws + o.E);
    uint16_t* Y = reinterpret_cast<uint16_t*>(ws + o.Y);
    float* Zt = reinterpret_cast<float*>(ws + o.Z);
    float* partial = reinterpret_cast<float*>(ws + o.partial);
    double* Gp = reinterpret_cast<double*>(ws + o.Gp);
    const int tiles = K / LQ_GT, room = (int)std::min<size_t>(o.Gp_bytes / (LQ_GENTRIES * sizeof(double)), (size_t)tiles);     // a partial matrix per tile, or fewer
    const int per = (tiles + room - 1) / room, parts = (tiles + per - 1) / per;
    double* G = reinterpret_cast<double*>(ws + o.G);
    uint16_t* A = reinterpret_cast<uint16_t*>(ws + o.A);
    uint16_t* At = reinterpret_cast<uint16_t*>(ws + o.At);
    for (int t = 0; t < steps; ++t) {
        const float* src = W;
        if (t > 0) {                                                 // residual of the previous step's factors
            residual_kernel<<<dim3((N + 31) / 32, (K + 511) / 512), dim3(256), 0, st>>>(W, Y, At, F, N, K);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            src = F;
        }
        if ((e = launch_quantize(L, src, thresholds, packed, absmax, st)) != hipSuccess) return e;
        residual_of_decode_kernel<<<dim3(N), dim3(256), 0, st>>>(L.d_rows, packed, absmax, mappings, W, E, K);   // E = W - What
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const uint16_t* Aq = t == 0 ? omega : A;
        for (int it = 0; it < iters; ++it) {
            if ((e = launch_skinny(E, K, N, Aq, K, r, K, 1.0f, Y, LQ_RP, st)) != hipSuccess) return e;              // Y = E A^T
            int chunks;
            if ((e = launch_tn_partial(E, K, N, Y, partial, &chunks, st)) != hipSuccess) return e;                  // Z = Y^T E
            zsum_gram_kernel<<<dim3(parts), dim3(256), 0, st>>>(partial, chunks, K, Zt, Gp, per);
            gram_sum_kernel<<<dim3(LQ_GENTRIES / 64), dim3(256), 0, st>>>(Gp, parts, G);
            factor_apply_kernel<<<dim3((K + 63) / 64), dim3(LQ_APPLY_THREADS), 0, st>>>(Zt, G, K, r, A, At);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            Aq = A;
        }
        if ((e = launch_skinny(E, K, N, A, K, r, K, 1.0f, Y, LQ_RP, st)) != hipSuccess) return e;                  // B = E A^T
    }
    copy_cols_kernel<<<dim3(lq_grid((size_t)r * K)), dim3(256), 0, st>>>(A, K, (size_t)r, K, A_out);
    copy_cols_kernel<<<dim3(lq_grid((size_t)N * r)), dim3(256), 0, st>>>(Y, LQ_RP, (size_t)N, r, B_out);
    return hipGetLastError();
}

}  // namespace lowra
