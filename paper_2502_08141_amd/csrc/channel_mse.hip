// Per-channel error table (paper Sec. 6.1: every channel's MSE under 1-, 2- and 4-bit
// quantization, the input of the precision assignment), and a greedy budgeted assignment that
// stands in for the paper's two-level ILP (Sec. 6).
//
//   mse[n][p] = (1/K) sum_k ( W[n,k] - mappings[p][code_p] * absmax )^2      p = 0, 1, 2: 1, 2, 4 bits
// with absmax, normalisation and binning exactly as in the quantize kernel (App. A.1) and the fp32
// decode of App. A.2: quantize -> decode -> squared error fused in one pass over W, nothing packed.
//
// Mapping: one workgroup per channel or two, a lane owns 8 consecutive weights (a block is 8 adjacent
// lanes), all three widths from the same registers; the narrow widths' levels are selected in
// registers.  What bounds it is plain-ALU work per weight, beside 4 bytes from HBM once.  The 4-bit code
// -- the number of thresholds strictly below u, App. A.1 -- is found by bisection (14 instructions and
// three LDS reads) or, in long rows, by buckets: [-1, 1] is cut into 64; a bucket's entry holds the one threshold
// inside it and the levels on its two sides, so that a scaled conversion, three LDS reads without conflicts, one
// compare and one select give the level.  The bucket of a value is a monotone function of it, the same for
// thresholds and weights, so thresholds of lower buckets are below u and those of higher ones are not: the code is
// the bisection's.  Tables with two thresholds in one bucket, or out of order, keep the bisection.
// The form by sizes, kernel times of calls in a graph (bisection, one channel per workgroup | buckets, one | two):
//   below 4096 features the entries cost more than they save: 11008 x 2048 23.3 | 28.7 | 25.4 us, 2048 x 1024 5.4 |
//   7.2 | 6.4; 4096 x 11008 38.4 | 34.3 | 35.5, 11008 x 4096 37.6 | 39.1 | 36.9 us (4.9 TB/s);
//   two channels share the entries from 2048 channels on: 16384 x 4096 54.0 | 55.7 | 52.1, 2048 x 4096 9.9 | 10.5 |
//   10.1; fewer leave half of the workgroups' places empty: 1536 x 11008 18.8 | 16.8 | 18.2, 128 x 4096 4.0 | 4.6 | 6.1.
#include <algorithm>
#include <queue>
#include <tuple>
#include <type_traits>
#include <vector>

#include "lowra_host.h"

namespace lowra {

constexpr int kMseBuckets = 64;
// (clamped before the conversion: thresholds and the u of a block of subnormal weights may be infinite, or not numbers)
__device__ __forceinline__ int mse_bucket(float u) { return (int)fminf(fmaxf(fmaf(u, 32.0f, 32.0f), 0.0f), kMseBuckets - 1.0f); }

struct MseTabs { float t1, t2a, t2b, t2c, t4_3, t4_7, t4_11, m1a, m1b, m2a, m2b, m2c, m2d; };
// squared errors of one channel at 1, 2 and 4 bits, this thread's share
template <bool BISECT>
__device__ __forceinline__ void mse_row(const float4* __restrict__ w4, int units, int tid, const float (&bucket)[3][kMseBuckets],
                                        const float (&thr4)[16], const float (&lev4)[16], const MseTabs T, float& e1, float& e2, float& e4) {
    for (int base = 0; base < units; base += 2 * 256) {   // two passes requested together: a K = 4096 row is in flight at once
        float4 q0[2], q1[2];
#pragma unroll
        for (int ps = 0; ps < 2; ++ps) {
            const int un = min(base + ps * 256 + tid, units - 1);        // past the row: clamped, unused
            q0[ps] = w4[2 * un]; q1[ps] = w4[2 * un + 1];
        }
#pragma unroll
        for (int ps = 0; ps < 2; ++ps) {
            __builtin_amdgcn_sched_barrier(0);            // one pass after the other: interleaved they need 114 registers
            const int un = base + ps * 256 + tid;
            if (un < units) {                             // units is a multiple of 8: the 8 lanes of a block agree
                const float v[8] = {q0[ps].x, q0[ps].y, q0[ps].z, q0[ps].w, q1[ps].x, q1[ps].y, q1[ps].z, q1[ps].w};
                float a = 0.0f;
#pragma unroll
                for (int i = 0; i < 8; ++i) a = fmaxf(a, fabsf(v[i]));
                a = dpp_max_f32<0xB1>(a);
                a = dpp_max_f32<0x4E>(a);
                a = dpp_max_f32<0x141>(a);                // the block's other four lanes (half-row mirror; quads agree by now)
                const float inv = (a == 0.0f) ? 0.0f : 1.0f / a;  // IEEE division, once per block
                float u[8], l4[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) u[i] = v[i] * inv;
                if (BISECT) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        // thresholds ascending: #{j : T[j] < u} by bisection, the code's bits from the top
                        const int b3 = (T.t4_7 < u[i]) ? 1 : 0;
                        int c4 = 2 * b3 + (((b3 ? T.t4_11 : T.t4_3) < u[i]) ? 1 : 0);
                        c4 = 2 * c4 + ((thr4[4 * c4 + 1] < u[i]) ? 1 : 0);
                        c4 = 2 * c4 + ((thr4[2 * c4] < u[i]) ? 1 : 0);
                        l4[i] = lev4[c4];
                    }
                } else {
                    float t[8], hi[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int q = mse_bucket(u[i]);
                        t[i] = bucket[0][q]; l4[i] = bucket[1][q]; hi[i] = bucket[2][q];
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) l4[i] = (t[i] < u[i]) ? hi[i] : l4[i];
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float l1 = (T.t1 < u[i]) ? T.m1b : T.m1a;
                    float l2 = (T.t2a < u[i]) ? T.m2b : T.m2a;         // the highest threshold below u decides
                    l2 = (T.t2b < u[i]) ? T.m2c : l2;
                    l2 = (T.t2c < u[i]) ? T.m2d : l2;
                    // the decoded weight is the product ROUNDED to fp32: a weight that equals it has no error
                    const float d1 = v[i] - l1 * a, d2 = v[i] - l2 * a, d4 = v[i] - l4[i] * a;
                    e1 = fmaf(d1, d1, e1); e2 = fmaf(d2, d2, e2); e4 = fmaf(d4, d4, e4);   // (the build does not contract on its own)
                }
            }
        }
    }
}

template <bool BUCKETS>
__global__ __launch_bounds__(256) void channel_mse_kernel(const float* __restrict__ W, const float* __restrict__ thr3,
                                                          const float* __restrict__ map3, float* __restrict__ mse, int N, int K, int per) {
    __shared__ float bucket[3][kMseBuckets];                      // threshold; level below it; level above it: bank = bucket, no conflicts
    __shared__ float lev4[16];
    __shared__ float thr4[16];                                    // sorted, entry 15 unused
    __shared__ double part[4][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int units = K >> 3;
    if (tid < 16) { lev4[tid] = map3[2 * kTableStride + tid]; thr4[tid] = thr3[2 * kTableStride + tid]; }
    const MseTabs tab = {thr3[0], thr3[kTableStride], thr3[kTableStride + 1], thr3[kTableStride + 2],
                         thr3[2 * kTableStride + 3], thr3[2 * kTableStride + 7], thr3[2 * kTableStride + 11],
                         map3[0], map3[1], map3[kTableStride], map3[kTableStride + 1], map3[kTableStride + 2], map3[kTableStride + 3]};
    __syncthreads();
    bool crowded = !BUCKETS;
    if (BUCKETS && tid < kMseBuckets) {
        int below = 0, inside = 0;
#pragma unroll
        for (int j = 0; j < 15; ++j) {
            const float t = thr4[j];
            const int q = mse_bucket(t);
            if (!(t >= 1.5f)) { below += q < tid ? 1 : 0; inside += q == tid ? 1 : 0; }   // (larger ones are above every |u| <= 1 + 2^-23)
        }
        crowded = inside > 1;
        bucket[0][tid] = inside ? thr4[below] : __builtin_inff();
        bucket[1][tid] = lev4[below];
        bucket[2][tid] = lev4[min(below + 1, 15)];
    }
    // an infinite u (a block of subnormal weights) may pass any threshold: those tables keep the bisection as well, and so
    // do thresholds that are not ascending (the bucket counts below would name another one than the bucket's own)
    crowded = crowded || (tid < 15 && thr4[tid] >= 1.5f) || (tid < 14 && !(thr4[tid] <= thr4[tid + 1]));
    const bool bisect = !BUCKETS || __syncthreads_or(crowded) != 0;
    for (int n = blockIdx.x * per; n < min((int)blockIdx.x * per + per, N); ++n) {
        const float4* w4 = reinterpret_cast<const float4*>(W + (size_t)n * K);
        float e1 = 0.0f, e2 = 0.0f, e4 = 0.0f;
        if (!BUCKETS || bisect) mse_row<true>(w4, units, tid, bucket, thr4, lev4, tab, e1, e2, e4);
        else mse_row<false>(w4, units, tid, bucket, thr4, lev4, tab, e1, e2, e4);
        const double s1 = wave_sum((double)e1), s2 = wave_sum((double)e2), s4 = wave_sum((double)e4);
        __syncthreads();                                          // the previous channel's sums have been read
        if (lane == 0) { part[wave][0] = s1; part[wave][1] = s2; part[wave][2] = s4; }
        __syncthreads();
        if (tid < 3) mse[(size_t)n * 3 + tid] = (float)((part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid]) / (double)K);
    }
}

hipError_t launch_channel_mse(int N, int K, const float* W, const float* thr3, const float* map3, float* mse, hipStream_t st) {
    if (N == 0) return hipSuccess;
    KernelTimer timer(st);
    const int per = K >= 4096 && N >= 2048 ? 2 : 1;               // channels per workgroup
    if (K >= 4096) channel_mse_kernel<true><<<dim3((N + per - 1) / per), dim3(256), 0, st>>>(W, thr3, map3, mse, N, K, per);
    else channel_mse_kernel<false><<<dim3(N), dim3(256), 0, st>>>(W, thr3, map3, mse, N, K, 1);
    return hipGetLastError();
}

// Greedy assignment on the host.  Every channel starts at 1 bit; an upgrade is 1 -> 2 bits (cost
// params bits) or, once a channel is at 2 bits, 2 -> 4 (cost 2 params); the upgrade with the
// largest error reduction per bit that still fits the budget and reduces the error is applied
// until none is left; ties go to the lower channel.  An upgrade that does not fit never fits
// later (the remaining budget only shrinks), so a heap of the currently available upgrades is
// enough.  fp64 throughout, the same expressions as the reference statement of the rule.
bool assign_greedy_host(int N, const int64_t* params, const float* mse, double budget_bpp, uint8_t* bits) {
    if (N < 0 || !(budget_bpp >= 1.0)) return false;
    double total = 0.0;
    for (int n = 0; n < N; ++n) {
        if (params[n] <= 0) return false;
        total += (double)params[n];
        bits[n] = 1;
    }
    double remaining = budget_bpp * total - total;
    struct Up { double eff; int n; };
    auto worse = [](const Up& x, const Up& y) { return x.eff < y.eff || (x.eff == y.eff && x.n > y.n); };
    std::priority_queue<Up, std::vector<Up>, decltype(worse)> heap(worse);
    auto offer = [&](int n) {
        if (bits[n] == 4) return;
        const double pn = (double)params[n];
        const double cost = bits[n] == 1 ? pn : 2.0 * pn;
        const double gain = bits[n] == 1 ? pn * ((double)mse[n * 3] - (double)mse[n * 3 + 1])
                                         : pn * ((double)mse[n * 3 + 1] - (double)mse[n * 3 + 2]);
        if (!(gain > 0.0)) return;
        heap.push(Up{gain / cost, n});
    };
    for (int n = 0; n < N; ++n) offer(n);
    while (!heap.empty()) {
        const Up u = heap.top();
        heap.pop();
        const double cost = bits[u.n] == 1 ? (double)params[u.n] : 2.0 * (double)params[u.n];
        if (cost > remaining) continue;                      // never fits again
        remaining -= cost;
        bits[u.n] = bits[u.n] == 1 ? 2 : 4;
        offer(u.n);
    }
    return true;
}

}  // namespace lowra
