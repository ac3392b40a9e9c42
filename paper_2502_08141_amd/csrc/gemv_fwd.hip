// Small-token forward (M <= 16):  y = x What^T + (s x A^T) B^T, streaming the packed codes once.
//
// Bandwidth-bound: per weight the method moves bits/8 + 1/16 bytes (codes + fp32 group scale), a
// whole Llama-sized matrix is a few MB, about what the chip must have outstanding to cover one HBM
// round trip.  So every wavefront issues ALL its loads of codes and scales before it touches the
// first result, and every load is as wide as the layout allows.
//
// Workgroup = 16 output channels (one MFMA tile, walked in the width-sorted order of their 256-row
// tile so a wavefront mostly sees one width) x all of K.  Its wavefronts split K in blocks of 256.
// In a block, lane (i, kg) LOADS one whole 64-wide group of channel i -- group 4 blk + kg, a
// contiguous run of the packed row (8/16/32 bytes, one or two 16-byte loads) -- and the four scales
// of the block.  v_mfma_f32_16x16x32_bf16 step (g, h) then contracts k = 64 g + 32 h + 8 kg + e, so
// both steps of a group see ONE group in all four kg lanes: the lanes of a channel trade pieces of
// their groups first (a 4 x 4 dword transpose with v_permlane32_swap / v_permlane16_swap).
//
// Decode: two codes (2, 4 or 8 bits) index the channel's pair table in LDS, whose entry is the two
// UNSCALED levels as bf16 (App. A.2's lookup); the absmax multiplies the fp32 dot product of the
// group instead of every weight -- the same sum in another order, with one bf16 rounding per level
// instead of per product.  One table read per two weights for every width, no per-group set-up.
// Tokens are the MFMA rows and channels its columns, so a lane's results belong to its own channel.
//
// The activations of a block (16 tokens x 256 columns, 8 KB, the same for every workgroup: L2)
// come by global->LDS DMA into buffers private to the wavefront -- all rounds at once when they
// fit, else one round ahead -- so that no operand load of x ever is a per-lane request and no
// round needs a barrier.
//
// The rank-r term needs t = x A^T first: a small kernel writes partial sums of t per 256-column block, the
// main kernel's threads share them out (a few KB from L2), and the wavefront that adds up the results multiplies [B rows] [t]^T
// with one MFMA per 32 ranks.  For short contractions and low ranks the workgroups form t themselves, beside the products with
// the codes (FUSE), and the small kernel falls away.
//
// A call on one matrix is a chain of round trips and of instructions that every wavefront of a workgroup issues (four per
// SIMD: 16 cycles an instruction).  So the chain's head, the row record, is asked for first; the levels come by one
// load of one wavefront; nothing waits for t before the end; and few blocks take fewer wavefronts.  A call in a captured graph,
// before -> after: 256 x 512, rank 8, 16 tokens 9.0 -> 5.0 us; 4096 x 1024, 4 tokens, rank 16 8.7 -> 6.0, rank 64 11.1 -> 9.3;
// 11008 x 4096, rank 16, 1 token 15.9 -> 14.5; three 4096 x 4096 matrices in one launch 17.7 -> 16.1; and level: one 4096 x 4096
// matrix, 1 token, rank 16 8.65, rank 64 10.9 -> 11.0.
#include <algorithm>
#include <cmath>

#include "gemm_common.h"
#include "gemv_t.h"

namespace lowra {

constexpr int GV_XROW = 512;                 // bytes per token row of a staged activation block (256 bf16)
constexpr int GV_MAXR = 8;                   // blocks (rounds) per multiplying wavefront at most
constexpr int GV_TABROW = 1024 + 16;         // bytes per channel of the pair tables: 256 entries, rows skewed by 4 banks

__global__ __launch_bounds__(64) void gemv_t_partial_kernel(const uint16_t* __restrict__ x, int M, int K,
                                                           const uint16_t* __restrict__ A, int r, int RT,
                                                           float* __restrict__ tp) {
    t_partial_body(x, M, K, A, r, RT, tp, blockIdx.x);
}

// the same for every matrix of a batch in one launch: workgroup = one 256-column block of one matrix.
// owner[id] names the matrix of workgroup id and first[m] its first workgroup: two dependent scalar
// loads (a search over the prefix sums would be a chain of eight).
__global__ __launch_bounds__(64) void gemv_t_partial_batch_kernel(const GemvParams* __restrict__ descs, const int* __restrict__ blk0,
                                                                 const int* __restrict__ owner) {
    const int m = owner[blockIdx.x];
    const GemvParams& p = descs[m];
    t_partial_body(p.x, p.M, p.K, p.A, p.r, p.RT, p.tp, (int)blockIdx.x - blk0[m]);
}

// ---------------------------------------------------------------------------------------------
typedef unsigned int uint2v_t __attribute__((ext_vector_type(2)));

// 4 x 4 transpose of dwords over the four lanes (i, kg = 0..3) of a channel: lane kg ends up with
// z[kg] of lanes 0, 1, 2, 3.  v_permlane32_swap trades the upper half of the first register for
// the lower half of the second, v_permlane16_swap the odd 16-lane rows for the even ones.
__device__ __forceinline__ void transpose4(uint32_t (&z)[4]) {
    const uint2v_t p02 = __builtin_amdgcn_permlane32_swap(z[0], z[2], false, false);
    const uint2v_t p13 = __builtin_amdgcn_permlane32_swap(z[1], z[3], false, false);
    const uint2v_t r01 = __builtin_amdgcn_permlane16_swap(p02.x, p13.x, false, false);
    const uint2v_t r23 = __builtin_amdgcn_permlane16_swap(p02.y, p13.y, false, false);
    z[0] = r01.x; z[1] = r01.y; z[2] = r23.x; z[3] = r23.y;
}

constexpr int GV_LEV = 20;                   // floats per channel of the staged levels
constexpr int GV_FIXED = 16 * GV_TABROW + 16 * GV_LEV * 4 + 64;      // LDS in front of t
// Sums that a workgroup keeps per entry of t: one of every wavefront's block (FUSE), with several rounds one of the blocks that
// each of an entry's threads adds up, else the whole sum, scaled and rounded to bf16; and their bytes
constexpr int gemv_t_parts(int W, int PER, int RT, bool fuse) { return RT == 0 ? 0 : fuse ? W : PER > 1 && 16 * RT < W * 64 ? W * 64 / (16 * RT) : 1; }
constexpr int gemv_t_bytes(int W, int PER, int RT, bool fuse) { return gemv_t_parts(W, PER, RT, fuse) * 16 * RT * (PER > 1 || fuse ? 4 : 2); }

// FUSE: t comes from the workgroup itself (one round, r <= 16); else from the partial sums in p.tp
template <int W, int PER, bool FUSE>
__device__ __forceinline__ void gemv_body(const GemvParams& p, const int strip) {
    static_assert(!FUSE || PER == 1, "a wavefront forms t beside the products of its only block");
    extern __shared__ __align__(16) uint8_t gv_smem[];
    // LDS: pair tables [16 channels][GV_TABROW bytes] | levels [16][GV_LEV] | channel numbers [16] | t: sums [tparts][16 tokens][RT] or bf16 [16][RT] |
    //      [xbufs buffers][W pieces][rows2 KB] activations (rows2 = pairs of token rows; xbufs = all
    //      rounds when they fit, else 2).  After its last round a wavefront reuses the head of its
    //      piece of buffer 0 for its partial results [16 channels][16 tokens].
    constexpr int LEV0 = 16 * GV_TABROW, NL0 = LEV0 + 16 * GV_LEV * 4, T0 = GV_FIXED;
    const int nt = 16 * p.RT, X0 = T0 + p.tparts * nt * (PER > 1 || FUSE ? 4 : 2);
    float* t_lds = reinterpret_cast<float*>(gv_smem + T0);
    const int rows2 = (min(p.M, 16) + 1) >> 1;
    const int XPIECE = rows2 * 1024, XBUF = W * XPIECE;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(lptr_t)gv_smem;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = lane & 15, kg = lane >> 4;
    const int nblk = (p.G + 3) >> 2;                               // blocks of 4 groups
    const int per = PER == 1 ? 1 : (nblk + W - 1) / W;             // rounds: blocks per wavefront (<= PER)
    const int blk0 = wave * per;
    const bool live = blk0 < nblk;                                 // (with few blocks some wavefronts have none)
    const bf16x8_t zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

    // What a strip waits for is a chain: row record -> codes, scales and levels -> pair tables -> products.  So the record is
    // asked for first, and A, which takes longest, behind it.  Loads come back in order and the compiler does not count the
    // transfers: what it waits for, it waits for with transfers behind it.  So with one round activations and sums of t are
    // asked for behind the levels, which the pair tables wait for (4096 x 4096, rank 64, 1 to 16 tokens: 1.2 % less than in
    // front of the levels' write); with several rounds they fill the wait for the record (11008 x 4096: 16.4 -> 15.2 us).
    const SortedRow rec = p.sorted_rows[strip * 16 + i];
    bf16x8_t af[8];                                                // FUSE: A[i][32 j + 8 kg ..] of my block
    constexpr int TU = PER == 1 ? 16 : 4 * PER < 16 ? 4 * PER : 16;    // else: sums of the blocks tpart, tpart + tparts, .. of entry `to`
    float tsum[TU];
    int tpart = 0, to = threadIdx.x;
    if (FUSE) {
        if (live) {
            const uint16_t* ar = p.A + (size_t)min(i, p.r - 1) * p.K + blk0 * 256 + 8 * kg;
#pragma unroll
            for (int j = 0; j < 8; ++j) af[j] = blk0 * 256 + 32 * j < p.K ? *reinterpret_cast<const bf16x8_t*>(ar + 32 * j) : zero8;
        }
    }

    // One DMA instruction moves 2 token rows x 512 B of my block of round q into that round's
    // buffer; chunk c of token row m lands at chunk c ^ (m & 15).
    const int tok = lane >> 5;
    const bool x_all = PER == 1 || p.xbufs >= per;                 // every round has a buffer of its own: all asked for at once
    auto xbuf_of = [&](int q) { return x_all ? q : (q & 1); };
    auto issue_x = [&](int q) {
        const int blk = min(blk0 + q, nblk - 1);
        const uint32_t left = (uint32_t)p.K - (uint32_t)blk * 256u, dst = smem_lds + X0 + xbuf_of(q) * XBUF + wave * XPIECE;
        if (left >= 256u) {                                        // uniform
            for (int pr = 0; pr < rows2; ++pr) {                    // uniform
                const int m = 2 * pr + tok;
                const uint32_t col = (uint32_t)blk * 256u + (uint32_t)(((lane & 31) ^ (m & 15)) * 8);
                dma16_s(p.x, ((uint32_t)min(m, p.M - 1) * (uint32_t)p.K + col) * 2u, dst + pr * 1024);
            }
        } else {
            // Features past K are zeros, by a buffer descriptor: another value times a zero scale or a zero of A would be none if
            // it is infinite.  (A path of its own: through the descriptor the other blocks take up to 7 % of a call longer.)
            const bufdesc_t xd = buffer_desc(p.x);
            for (int pr = 0; pr < rows2; ++pr) {
                const int m = 2 * pr + tok;
                const uint32_t c = (uint32_t)(((lane & 31) ^ (m & 15)) * 8);
                const uint32_t off = ((uint32_t)min(m, p.M - 1) * (uint32_t)p.K + (uint32_t)blk * 256u + c) * 2u;
                dma16_b(xd, c < left ? off : 0x80000000u, 0u, dst + pr * 1024);
            }
        }
    };
    auto ask_inputs = [&]() __attribute__((always_inline)) {       // activations, sums of t
        if (live) {
            if (x_all) {
                for (int q = 0; q < per; ++q) issue_x(q);            // uniform
            } else {
                issue_x(0);
            }
        }
        if (!FUSE && p.RT > 0) {
            for (int w = wave * 64; w >= nt; w -= nt) ++tpart;     // uniform: nt is a multiple of 256
            to -= tpart * nt;
#pragma unroll
            for (int u = 0; u < TU; ++u) {
                const int b = tpart + u * p.tparts;
                tsum[u] = tpart < p.tparts && b < nblk ? p.tp[(size_t)b * nt + to] : 0.0f;     // uniform condition
            }
        }
    };
    if (PER > 1) ask_inputs();
    const int bits = (int)(rec.bits_cb & 0xffu);
    const bool row_ok = rec.n >= 0;                                // padding rows are recorded as 1-bit rows
    const int nc = row_ok ? rec.n : 0;
    const bool two = bits == 2, four = bits == 4;
    // The levels of the strip's channels, 64 bytes each, by one wavefront's single load (gathered entry by entry for the pair
    // tables they were 128 wavefront instructions of the unit's one address pipe).
    const float* mrow = p.mappings + (size_t)(rec.bits_cb >> 8) * kTableStride;
    float4 lv = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (wave == 0) lv = *reinterpret_cast<const float4*>(mrow + 4 * kg);

    // every load of codes and scales of all my rounds, back to back
    const bool wave_has4 = __builtin_amdgcn_ballot_w64(four) != 0;
    const bool vec_sc = (p.G & 3) == 0;                            // a block's four scales are one aligned 16-byte load
    uint4 ca[PER], cb[PER];
    float4 sc[PER];
    bool hi8[PER];
    const uint8_t* rowp = p.packed + rec.offset;
    const uint8_t* pend16 = p.packed + p.packed_bytes - 16;
    const float* ar = p.absmax + (size_t)nc * p.G;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int blk = blk0 + q;
        ca[q] = cb[q] = zero4(); sc[q] = make_float4(0.0f, 0.0f, 0.0f, 0.0f); hi8[q] = false;
        if (q < per && blk < nblk) {                                // uniform
            const int g = min(4 * blk + kg, p.G - 1);              // clamped: groups past the row get a zero scale below
            const uint8_t* a0 = rowp + (size_t)(g * 8 * bits);
            const uint8_t* a0c = a0 < pend16 ? a0 : pend16;         // a 1-bit group is 8 B: its 16-byte load may be pulled back
            hi8[q] = a0 != a0c && bits == 1;                        // ... then the group sits in the upper 8 bytes
            ca[q] = *reinterpret_cast<const uint4*>(a0c);
            if (wave_has4) cb[q] = *reinterpret_cast<const uint4*>(four ? a0 + 16 : a0c);
            if (vec_sc) {
                sc[q] = *reinterpret_cast<const float4*>(ar + 4 * blk);
            } else {
                sc[q].x = ar[4 * blk]; sc[q].y = ar[min(4 * blk + 1, p.G - 1)];
                sc[q].z = ar[min(4 * blk + 2, p.G - 1)]; sc[q].w = ar[min(4 * blk + 3, p.G - 1)];
            }
        }
    }
    // my fragments of B for the first 64 ranks, asked for with everything else
    bf16x8_t bfr0 = zero8, bfr1 = zero8;
    if (wave == 0 && p.RT > 0 && (p.r & 7) == 0) {
        if (row_ok && kg * 8 < p.r) bfr0 = *reinterpret_cast<const bf16x8_t*>(p.B + (size_t)nc * p.r + kg * 8);
        if (!FUSE && row_ok && 32 + kg * 8 < p.r) bfr1 = *reinterpret_cast<const bf16x8_t*>(p.B + (size_t)nc * p.r + 32 + kg * 8);
    }

    float* lev = reinterpret_cast<float*>(gv_smem + LEV0) + i * GV_LEV;
    if (wave == 0) {
        *reinterpret_cast<float4*>(lev + 4 * kg) = lv;
        if (kg == 0) reinterpret_cast<int*>(gv_smem + NL0)[i] = rec.n;
    }
    if (PER == 1) ask_inputs();
    __syncthreads();                                               // the levels
    // my channel's pair table, entry e = two codes (low, high) -> two bf16 (unscaled levels; the group scale multiplies the
    // group's dot product)
    uint8_t* tabp = gv_smem + i * GV_TABROW;
    const int nent = 1 << (2 * bits);
    for (int e = (int)(threadIdx.x >> 4); e < nent; e += 4 * W)
        *reinterpret_cast<uint32_t*>(tabp + 4 * e) = pack_bf16x2(lev[e & ((1 << bits) - 1)], lev[e >> bits]);
    if (!FUSE && p.RT > 0 && tpart < p.tparts) {
        for (int o = to; o < nt; o += W * 64) {                    // (more entries than threads: one part, the later entries from memory)
            float v = 0.0f;
            if (o == to) {
#pragma unroll
                for (int u = 0; u < TU; ++u) v += tsum[u];
            }
            int b = o == to ? tpart + TU * p.tparts : tpart;
            if (W == 8 && PER >= 6 && p.tparts == 1) {             // long contractions of higher ranks: more of them in flight (4096 x 11008,
                for (; b < nblk; b += 16) {                        // 16 tokens, rank 64: 24.4 -> 23.0 us; shorter ones have no registers to spare)
                    float w[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) w[u] = p.tp[(size_t)min(b + u, nblk - 1) * nt + o];
#pragma unroll
                    for (int u = 0; u < 16; ++u) v += b + u < nblk ? w[u] : 0.0f;
                }
            }
            for (; b < nblk; b += 4 * p.tparts) {         // four loads in flight
                float w[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = p.tp[(size_t)min(b + u * p.tparts, nblk - 1) * nt + o];
#pragma unroll
                for (int u = 0; u < 4; ++u) v += b + u * p.tparts < nblk ? w[u] : 0.0f;
            }
            if (PER == 1) reinterpret_cast<uint16_t*>(t_lds)[o] = (uint16_t)(pack_bf16x2(v * p.s, 0.0f) & 0xffffu);
            else t_lds[tpart * nt + o] = v;
        }
    }
    __syncthreads();                                               // pair tables

    // + [s t as bf16] x [B rows], t the sum of `parts` of them
    auto fragment_b = [&](int j0) __attribute__((always_inline)) -> bf16x8_t {
        bf16x8_t f = zero8;
        if (row_ok && j0 < p.r) {
            const uint16_t* br = p.B + (size_t)nc * p.r + j0;
            if ((p.r & 7) == 0) {
                f = *reinterpret_cast<const bf16x8_t*>(br);
            } else {
                uint32_t tmp[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) tmp[e] = j0 + e < p.r ? (uint32_t)br[e] : 0u;
                f = __builtin_bit_cast(bf16x8_t, make_uint4(tmp[0] | (tmp[1] << 16), tmp[2] | (tmp[3] << 16), tmp[4] | (tmp[5] << 16), tmp[6] | (tmp[7] << 16)));
            }
        }
        return f;
    };
    auto fragment_t = [&](int j0, int parts) __attribute__((always_inline)) -> bf16x8_t {
        if (PER == 1 && !FUSE) return j0 < p.RT ? *reinterpret_cast<const bf16x8_t*>(reinterpret_cast<const uint16_t*>(t_lds) + i * p.RT + j0) : zero8;
        float t[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (j0 < p.RT) {
            for (int q = 0; q < parts; ++q) {
                const float* src = t_lds + q * nt + i * p.RT + j0;
                const float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + 4);
                t[0] += a.x; t[1] += a.y; t[2] += a.z; t[3] += a.w; t[4] += b.x; t[5] += b.y; t[6] += b.z; t[7] += b.w;
            }
            if (FUSE) {                                            // (a rank past r is the last one again)
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = j0 + e < p.r ? t[e] : 0.0f;
            }
        }
        return __builtin_bit_cast(bf16x8_t, make_uint4(pack_bf16x2(t[0] * p.s, t[1] * p.s), pack_bf16x2(t[2] * p.s, t[3] * p.s),
                                                       pack_bf16x2(t[4] * p.s, t[5] * p.s), pack_bf16x2(t[6] * p.s, t[7] * p.s)));
    };
    auto rank_r = [&](floatx4_t acc, int parts) __attribute__((always_inline)) -> floatx4_t {
        if (p.RT == 0) return acc;                                 // uniform, as the rest
        const bool at_hand = (p.r & 7) == 0;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fragment_t(kg * 8, parts), at_hand ? bfr0 : fragment_b(kg * 8), acc, 0, 0, 0);
        if (FUSE || p.RT <= 32) return acc;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fragment_t(32 + kg * 8, parts), at_hand ? bfr1 : fragment_b(32 + kg * 8), acc, 0, 0, 0);
        for (int e0 = 64; e0 < p.RT; e0 += 32) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fragment_t(e0 + kg * 8, parts), fragment_b(e0 + kg * 8), acc, 0, 0, 0);
        return acc;
    };
    if (live) {
        const uint32_t fw2 = 2u * (uint32_t)bits;                  // bits of one table index (two codes)
        floatx4_t tot = {0.0f, 0.0f, 0.0f, 0.0f}, tf = tot;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int blk = blk0 + q;
            if (q < per && blk < nblk) {                            // uniform
                // my block of this round has landed (so has everything else I asked for); ask for the next
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (!x_all && q + 1 < per) issue_x(q + 1);
                const float a4[4] = {row_ok ? sc[q].x : 0.0f, row_ok && 4 * blk + 1 < p.G ? sc[q].y : 0.0f,
                                     row_ok && 4 * blk + 2 < p.G ? sc[q].z : 0.0f, row_ok && 4 * blk + 3 < p.G ? sc[q].w : 0.0f};
                // I loaded group kg of my channel; MFMA step (g, h) wants from me the 8 codes
                // k = 64 g + 32 h + 8 kg .. + 8 of group g: piece kg of each half of the group goes
                // to lane kg of the lane that loaded it
                const uint32_t c0 = hi8[q] ? ca[q].z : ca[q].x, c1 = hi8[q] ? ca[q].w : ca[q].y;     // a 1-bit row uses 8 of its 16 bytes
                const uint32_t D[8] = {ca[q].x, ca[q].y, ca[q].z, ca[q].w, cb[q].x, cb[q].y, cb[q].z, cb[q].w};
                uint32_t za[4], zb[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t a2 = D[k >> 1] >> (16 * (k & 1)), b2 = D[2 + (k >> 1)] >> (16 * (k & 1));
                    const uint32_t a1 = c0 >> (8 * k), b1 = c1 >> (8 * k);
                    za[k] = four ? D[k] : (two ? a2 : a1);
                    zb[k] = four ? D[4 + k] : (two ? b2 : b1);
                }
                transpose4(za);
                transpose4(zb);
                const uint8_t* xp = gv_smem + X0 + xbuf_of(q) * XBUF + wave * XPIECE + min(i, p.M - 1) * GV_XROW;
                // tokens are the rows, channels the columns: lane (i, kg) gets y[token 4 kg + v][channel i].
                // Token rows past M repeat row M - 1 and are never stored.
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    floatx4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t cs = h ? zb[g] : za[g];
                        uint32_t d[4];
#pragma unroll
                        for (int pp = 0; pp < 4; ++pp)
                            d[pp] = *reinterpret_cast<const uint32_t*>(tabp + 4u * __builtin_amdgcn_ubfe(cs, pp * fw2, fw2));
                        const bf16x8_t xf = *reinterpret_cast<const bf16x8_t*>(xp + (((8 * g + 4 * h + kg) ^ i) << 4));
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, __builtin_bit_cast(bf16x8_t, make_uint4(d[0], d[1], d[2], d[3])), acc, 0, 0, 0);
                        if (FUSE) tf = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2 * g + h], xf, tf, 0, 0, 0);      // rank 4 kg + v of token i
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) tot[v] += a4[g] * acc[v];
                }
            }
        }
        if (!FUSE && wave == 0) tot = rank_r(tot, p.tparts);
        // my piece of buffer 0 is dead (all my rounds are done, all transfers have landed)
        float* part = reinterpret_cast<float*>(gv_smem + X0 + wave * XPIECE);
        *reinterpret_cast<float4*>(part + i * 16 + 4 * kg) = make_float4(tot[0], tot[1], tot[2], tot[3]);   // [channel][token]
        if (FUSE) *reinterpret_cast<float4*>(t_lds + wave * 256 + i * 16 + 4 * kg) = make_float4(tf[0], tf[1], tf[2], tf[3]);     // [token][rank]
    }
    __syncthreads();

    // the sum over the wavefronts, in their order, stored as bf16
    const int waves = PER == 1 ? min(W, nblk) : (nblk + per - 1) / per;
    if (FUSE) {                                                    // by one wavefront, which has the rank-r term to add
        if (wave != 0) return;
        floatx4_t tot = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int w = 0; w < waves; ++w) {
            const float4 v = *reinterpret_cast<const float4*>(gv_smem + X0 + w * XPIECE + (i * 16 + 4 * kg) * 4);
            tot[0] += v.x; tot[1] += v.y; tot[2] += v.z; tot[3] += v.w;
        }
        tot = rank_r(tot, waves);
        if (row_ok) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * kg + v < p.M) p.y[(size_t)(4 * kg + v) * p.N + nc] = (uint16_t)(pack_bf16x2(tot[v], 0.0f) & 0xffffu);
        }
        return;
    }
    for (int o = threadIdx.x; o < 256; o += W * 64) {
        const int m = o & 15, n = reinterpret_cast<const int*>(gv_smem + NL0)[o >> 4];
        if (m < p.M && n >= 0) {
            float v = 0.0f;
            for (int w = 0; w < waves; ++w) v += reinterpret_cast<const float*>(gv_smem + X0 + w * XPIECE)[o];
            p.y[(size_t)m * p.N + n] = (uint16_t)(pack_bf16x2(v, 0.0f) & 0xffffu);
        }
    }
}

template <int W, int PER, bool FUSE>
__global__ __launch_bounds__(W * 64) void gemv_fwd_kernel(GemvParams p) {
    gemv_body<W, PER, FUSE>(p, blockIdx.x);
}
// every matrix of a batch that takes this instantiation, in one launch: workgroup = one 16-channel strip of one matrix
template <int W, int PER, bool FUSE>
__global__ __launch_bounds__(W * 64) void gemv_fwd_batch_kernel(const GemvParams* __restrict__ descs, const int* __restrict__ strip0,
                                                                const int* __restrict__ owner) {
    const int m = owner[blockIdx.x];
    const GemvParams p = descs[m];
    gemv_body<W, PER, FUSE>(p, (int)blockIdx.x - strip0[m]);
}

struct GemvChoice { int W, PER, fuse; };
// LDS bytes of an instantiation for this matrix (0: does not fit), and its number of activation buffers
static size_t gemv_lds(const GemvParams& p, const GemvChoice& c, int* xbufs) {
    constexpr int kMaxLds = 160 * 1024;
    const int rows2 = (std::min(p.M, 16) + 1) / 2;
    const int nblk = (p.G + 3) / 4, per = (nblk + c.W - 1) / c.W;
    const size_t base = (size_t)GV_FIXED + gemv_t_bytes(c.W, c.PER, p.RT, c.fuse), xbuf = (size_t)c.W * rows2 * 1024;
    int bufs = base + per * xbuf <= (size_t)kMaxLds ? per : 2;     // a buffer per round when they fit
    // ... but not at the price of the second workgroup on a compute unit (5120 features, 6 tokens, three matrices of 5120
    // channels: 34 -> 25 us)
    if (c.W == 8 && per > 2 && 2 * (base + per * xbuf) > (size_t)kMaxLds && 2 * (base + 2 * xbuf) <= (size_t)kMaxLds) bufs = 2;
    *xbufs = bufs;
    const size_t sh = base + (size_t)bufs * xbuf;
    return sh > (size_t)kMaxLds ? 0 : sh;
}
template <int W, int PER, bool FUSE>
static size_t gemv_lds(GemvParams& p) {
    p.tparts = gemv_t_parts(W, PER, p.RT, FUSE);
    return gemv_lds(p, GemvChoice{W, PER, FUSE}, &p.xbufs);
}
template <int W, int PER, bool FUSE>
static hipError_t gemv_attr() {
    static hipError_t a0 = hipFuncSetAttribute(reinterpret_cast<const void*>(gemv_fwd_kernel<W, PER, FUSE>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    static hipError_t a1 = hipFuncSetAttribute(reinterpret_cast<const void*>(gemv_fwd_batch_kernel<W, PER, FUSE>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return a0 != hipSuccess ? a0 : a1;
}
template <int W, int PER, bool FUSE>
static hipError_t launch_one(GemvParams p, hipStream_t st) {
    const hipError_t attr = gemv_attr<W, PER, FUSE>();
    if (attr != hipSuccess) return attr;
    const size_t sh = gemv_lds<W, PER, FUSE>(p);
    if (sh == 0) return hipErrorInvalidValue;
    const dim3 grid((p.N + 15) / 16);
    gemv_fwd_kernel<W, PER, FUSE><<<grid, dim3(W * 64), sh, st>>>(p);
    return hipGetLastError();
}

static int compute_units_cached() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
        cus = v;
    }
    return cus;
}

// 8 wavefronts x GV_MAXR rounds x 256 columns
bool gemv_fwd_fits(int K) { return (K + 255) / 256 <= 8 * GV_MAXR; }

// The instantiation a matrix takes.  Rounds per wavefront fix the register footprint, so the kernel is
// compiled for a few depths; the smallest of 4, 8 and 16 wavefronts that covers the blocks (16 beyond: 4 per SIMD hide the
// LDS and decode latencies better), some of them idle, whenever its activation buffers fit; with more strips than compute
// units two 8-wavefront workgroups per unit (when their buffers fit twice) overlap one strip's loads with the other's
// arithmetic.
// Whether the workgroups form t = x A^T themselves.  It saves the partial sums' launch (2.7 us on the GPU, 2.6 us on the host) and
// costs every workgroup A: a compute unit gathers about 30 GB/s, 64 KB in 2 us, and pays that for each round of strips.
// `strips`: of the launch.  (GPU time, formed here against the launch: 2048 features, rank 16 0.95; 4096, rank 8 1.01, rank 16 1.12.)
static bool gemv_fuses(const GemvParams& p, int strips) {
    const long long rounds = (strips + compute_units_cached() - 1) / compute_units_cached();
    return p.r > 0 && p.r <= 16 && rounds * p.r * p.K <= 32768;
}
// LDS of an instantiation with two activation buffers per wavefront, or one where it has one round
static size_t gemv_lds_least(const GemvParams& p, const GemvChoice& c) {
    const int nblk = (p.G + 3) / 4, rows2 = (std::min(p.M, 16) + 1) / 2;
    return (size_t)GV_FIXED + gemv_t_bytes(c.W, c.PER, p.RT, c.fuse) + (size_t)std::min((nblk + c.W - 1) / c.W, 2) * c.W * rows2 * 1024;
}
// strips: of the launch
static GemvChoice gemv_choose(const GemvParams& p, int strips) {
    constexpr size_t kMaxLds = 160 * 1024;
    const int nblk = (p.G + 3) / 4;
    const bool fuses = gemv_fuses(p, strips);
    // (up to 24 blocks: 5120 features, three rounds; one token, three matrices of 5120 channels 34 -> 24 us, two of 13824
    // 59 -> 38 us against one 16-wavefront workgroup per unit; a batch whose strips have a unit each takes the 16, as a call does:
    // one 2048 x 2048 matrix, 4 tokens, rank 16 9.2 -> 7.2 us, one of 4096 9.95 -> 9.3)
    const size_t lds8 = gemv_lds_least(p, {8, 2, 0});
    const bool pair8 = strips > compute_units_cached() && 2 * lds8 <= (size_t)150 * 1024 && nblk <= 24;
    if (!pair8) {
        // What counts is the LDS of the form that the call will have: with 15 and 16 tokens the sums of 16 wavefronts that form t
        // are 1.5 KB too many, and then t comes from its own launch rather than through half as many wavefronts (4096 x 4096,
        // 16 tokens, rank 8: 10.4 -> 10.15 us; 2048 x 2048, rank 16, where 8 wavefronts fit either way, 9.75 -> 7.6).
        GemvChoice c = nblk <= 4 ? GemvChoice{4, 1, 0} : nblk <= 8 ? GemvChoice{8, 1, 0} : nblk <= 16 ? GemvChoice{16, 1, 0}      // K <= 4096
                     : nblk <= 32 ? GemvChoice{16, 2, 0} : nblk <= 48 ? GemvChoice{16, 3, 0} : GemvChoice{16, 4, 0};               // K <= 12288: three
        c.fuse = c.PER == 1 && fuses;
        if (c.fuse && gemv_lds_least(p, c) > kMaxLds) c.fuse = 0;
        // nor is it formed in the workgroup where several rounds of strips would then have a unit each to themselves (three
        // 2048 x 2048 matrices in a launch, 13 tokens, rank 8: 12.6 -> 10.7 us)
        if (c.fuse && strips > compute_units_cached() && 2 * gemv_lds_least(p, c) > kMaxLds && 2 * gemv_lds_least(p, {c.W, c.PER, 0}) <= kMaxLds) c.fuse = 0;
        if (gemv_lds_least(p, c) <= kMaxLds) return c;
    }
    if (nblk <= 4) return {4, 1, fuses};
    if (nblk <= 8) return {4, 2, 0};
    if (nblk <= 16) return {8, 2, 0};       // K <= 4096
    if (nblk <= 32) return {8, 4, 0};
    if (nblk <= 48) return {8, 6, 0};       // K = 11008
    return {8, 8, 0};
}
// The instantiations of a batch's matrices.  Those of one round whose strips together fill the chip once at most take the widest
// of theirs: every further instantiation is a launch of its own, 4 us and more behind the one before, and idle wavefronts cost
// less (1024 x 1024 and 1024 x 2816, 16 tokens, rank 16: 14.9 -> 8.8 us, 16 tokens without a rank-r term 10.5 -> 5.7).
static std::vector<GemvChoice> gemv_choose_batch(const std::vector<GemvParams>& items) {
    int strips = 0, strips1 = 0, W = 0;
    for (const GemvParams& p : items) strips += (p.N + 15) / 16;
    std::vector<GemvChoice> out;
    for (const GemvParams& p : items) {
        out.push_back(gemv_choose(p, strips));
        if (out.back().PER == 1) { strips1 += (p.N + 15) / 16; W = std::max(W, out.back().W); }
    }
    if (strips1 > compute_units_cached()) return out;
    bool fuse = true;                                              // all of them or none: one launch
    for (size_t i = 0; i < items.size(); ++i)
        if (out[i].PER == 1 && out[i].W < W) {
            out[i].W = W;
            if (gemv_lds_least(items[i], out[i]) > (size_t)160 * 1024) out[i].fuse = 0;
        }
    for (const GemvChoice& c : out) fuse = fuse && (c.PER != 1 || c.fuse);
    for (GemvChoice& c : out)
        if (c.PER == 1) c.fuse = fuse;
    return out;
}
void gemv_plan(int N, int K, int M, int r, int batch_strips, int* wavefronts, int* rounds, int* fused) {
    GemvParams p{};
    p.N = N; p.K = K; p.G = K / kGroup; p.M = M; p.r = r; p.RT = r > 0 ? (r + 15) / 16 * 16 : 0;
    const GemvChoice c = gemv_choose(p, batch_strips > 0 ? batch_strips : (N + 15) / 16);
    *wavefronts = c.W; *rounds = ((p.G + 3) / 4 + c.W - 1) / c.W; *fused = c.fuse;
}
// calls f.template operator()<W, PER, FUSE>() for the chosen instantiation
template <typename F>
static hipError_t gemv_dispatch(GemvChoice c, F&& f) {
    if (c.W == 4 && c.PER == 1) return c.fuse ? f.template operator()<4, 1, true>() : f.template operator()<4, 1, false>();
    if (c.W == 8 && c.PER == 1) return c.fuse ? f.template operator()<8, 1, true>() : f.template operator()<8, 1, false>();
    if (c.W == 16 && c.PER == 1) return c.fuse ? f.template operator()<16, 1, true>() : f.template operator()<16, 1, false>();
    if (c.fuse) return hipErrorInvalidValue;
    if (c.W == 16 && c.PER == 2) return f.template operator()<16, 2, false>();
    if (c.W == 16 && c.PER == 3) return f.template operator()<16, 3, false>();
    if (c.W == 16 && c.PER == 4) return f.template operator()<16, 4, false>();
    if (c.W == 4 && c.PER == 2) return f.template operator()<4, 2, false>();
    if (c.W == 8 && c.PER == 2) return f.template operator()<8, 2, false>();
    if (c.W == 8 && c.PER == 4) return f.template operator()<8, 4, false>();
    if (c.W == 8 && c.PER == 6) return f.template operator()<8, 6, false>();
    if (c.W == 8 && c.PER == 8) return f.template operator()<8, 8, false>();
    return hipErrorInvalidValue;
}
struct LaunchSingle {
    const GemvParams& p; hipStream_t st;
    template <int W, int PER, bool FUSE> hipError_t operator()() const { return launch_one<W, PER, FUSE>(p, st); }
};

hipError_t launch_gemv_fwd(const GemvParams& p, hipStream_t st) {
    const GemvChoice c = gemv_choose(p, (p.N + 15) / 16);
    if (p.RT > 0 && !c.fuse) {
        gemv_t_partial_kernel<<<dim3((p.G + 3) / 4), dim3(64), 0, st>>>(p.x, p.M, p.K, p.A, p.r, p.RT, p.tp);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return gemv_dispatch(c, LaunchSingle{p, st});
}

// Which kernel a batch takes: estimated times, fits to 13824 batches (the projections of layers of nine sizes, 1024 x 2816 to
// 6144 x 16384, one to seven matrices, every token count from 1 to 16, ranks 0, 8, 16 and 32, 1.15 to 2.5 bits with and without
// 4-bit rows; least squares of the relative error, batches that both kernels run in about the same time counted up to eleven times:
// 8 % here, 6 % for the streaming kernel).
// This kernel takes its instantiations' launches one after the other; each takes as many rounds as its strips fill the compute
// units with as many workgroups as they hold.  A round costs a fixed part, a part per block of 256 features that a wavefront walks
// and a part by the wavefronts that have a block (12 of 16 at 3072 features: without it q,k,v,o there were put at 21.0 us for 18.5,
// and at 26.5 for 27.1 at 4096).  The streaming kernel pays 11 us before and behind its stream, and with a rank-r term its t
// kernel, which is a chain over the features.  A decoder layer of 4096 x 11008 taken apart by data dependence, 4 tokens, rank 16:
// q,k,v 17.7 us here against 26.8, o 10.3 / 20.3, gate,up 27.6 / 30.4, down 17.4 / 39.1; all seven matrices in one batch 53.8 /
// 55.5, and without a rank-r term 48.3 / 38.6.
double gemv_batch_us(const std::vector<GemvParams>& items, const std::vector<int>& n4) {
    if (items.empty()) return 0.0;
    const std::vector<GemvChoice> choices = gemv_choose_batch(items);
    struct Launch { GemvChoice c; size_t lds; double strips, blocks, busy, wide; };
    std::vector<Launch> launches;
    double kmax = 0.0;
    bool t_launch = false;
    for (size_t i = 0; i < items.size(); ++i) {
        const GemvParams& p = items[i];
        const GemvChoice c = choices[i];
        int xbufs;
        const size_t lds = gemv_lds(p, c, &xbufs);
        size_t l = 0;
        while (l < launches.size() && !(launches[l].c.W == c.W && launches[l].c.PER == c.PER && launches[l].c.fuse == c.fuse && launches[l].lds == lds)) ++l;
        if (l == launches.size()) launches.push_back(Launch{c, lds, 0.0, 0.0, 0.0, 0.0});
        const int strips = (p.N + 15) / 16, nblk = (p.G + 3) / 4;
        const double busy = (double)strips * nblk / c.W;
        launches[l].strips += strips; launches[l].blocks += (double)strips * ((nblk + c.W - 1) / c.W);
        launches[l].busy += busy; launches[l].wide += busy * n4[i] / p.N;
        kmax = std::max(kmax, (double)p.K);
        t_launch = t_launch || (p.RT > 0 && !c.fuse);
    }
    const double M = items[0].M, ranks = items[0].RT / 16;
    double t = 1.42 + (t_launch ? 2.47 + 0.56 * (1.0 + ranks) * kmax / 4096.0 : 0.0);
    for (const Launch& l : launches) {
        // workgroups of a unit by LDS and by registers
        const int most = l.c.W == 16 ? (l.c.PER == 1 ? 2 : 1) : l.c.W == 8 ? (l.c.PER <= 2 ? 3 : l.c.PER <= 4 ? 2 : 1) : (l.c.PER == 1 ? 7 : 6);
        const int n = std::max(1, std::min(most, (int)((size_t)160 * 1024 / std::max<size_t>(l.lds, 1))));
        double rounds = l.strips / (double)(compute_units_cached() * n);
        rounds = n == 1 ? std::ceil(rounds - 1e-9) : rounds < 1.0 ? 0.5 + 0.5 * rounds : rounds;
        const double fixed = l.c.W == 16 ? (n == 1 ? 1.69 : 4.1) : l.c.W == 4 ? 5.02 : n == 1 ? 2.62 : n == 2 ? 3.91 : 3.66;
        const double busy = l.c.W == 16 ? (n == 1 ? 2.08 : 2.16) : l.c.W == 4 ? 0.17 : n == 1 ? 0.44 : n == 2 ? 0.89 : 2.34;
        t += rounds * (fixed + (l.busy * (busy + 0.035 * M) + l.wide * 2.36 + l.blocks * 0.68) / l.strips + 0.45 * ranks + (l.c.fuse ? 1.9 : 0.0));
    }
    return t;
}
double gemv_stream_batch_us(const std::vector<GemvParams>& items, const std::vector<int>& n4) {
    if (items.empty()) return 0.0;
    double units = 0.0, kmax = 0.0;                                // strips x chunks of 4096 features, 4-bit ones twice, per compute unit
    for (size_t i = 0; i < items.size(); ++i) {
        const GemvParams& p = items[i];
        units += (double)((p.N + 15) / 16) * ((p.K + 4095) / 4096) * (1.0 + (double)n4[i] / p.N) / compute_units_cached();
        kmax = std::max(kmax, (double)p.K);
    }
    const double M = items[0].M, r = items[0].r;
    return 11.48 + 0.049 * M + units * (1.191 + 0.053 * M) + (kmax > 4096.0 ? 4.77 : 0.0) +
           (r > 0 ? 1.62 + kmax / 4096.0 * (2.9 + 0.165 * r + 0.118 * M) : 0.0);
}

// ---- several matrices in one launch per instantiation.  The descriptors (every pointer of every matrix)
// are fixed when the batch is built and live in device memory; a run is one launch of the partial-sum
// kernel over all matrices that have a LoRA term and one launch of the main kernel per group of
// matrices that take the same instantiation with the same LDS size.
struct PrepareDesc {
    GemvParams& p; size_t& sh;
    template <int W, int PER, bool FUSE> hipError_t operator()() const {
        const hipError_t attr = gemv_attr<W, PER, FUSE>();
        if (attr != hipSuccess) return attr;
        sh = gemv_lds<W, PER, FUSE>(p);
        return sh ? hipSuccess : hipErrorInvalidValue;
    }
};
struct LaunchGroup {
    const GemvBatchGroup& g; hipStream_t st;
    template <int W, int PER, bool FUSE> hipError_t operator()() const {
        gemv_fwd_batch_kernel<W, PER, FUSE><<<dim3(g.nstrips), dim3(W * 64), g.sh, st>>>(g.d_descs, g.d_strip0, g.d_owner);
        return hipGetLastError();
    }
};

void gemv_batch_free(lowra_fwd_batch& b) {
    for (auto& g : b.groups) { (void)hipFree(g.d_descs); (void)hipFree(g.d_strip0); (void)hipFree(g.d_owner); }
    b.groups.clear();
    (void)hipFree(b.d_tdescs); (void)hipFree(b.d_blk0); (void)hipFree(b.d_towner);
    b.d_tdescs = nullptr; b.d_blk0 = nullptr; b.d_towner = nullptr;
}

template <typename T>
static hipError_t to_device(const std::vector<T>& v, T** out) {
    hipError_t e = hipMalloc(reinterpret_cast<void**>(out), v.size() * sizeof(T));
    if (e != hipSuccess) return e;
    return hipMemcpy(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
}

hipError_t gemv_batch_build(std::vector<GemvParams>& items, lowra_fwd_batch& b) {
    hipError_t e;
    struct Key { int W, PER, fuse; size_t sh; };
    std::vector<Key> keys;
    std::vector<std::vector<GemvParams>> members;
    const std::vector<GemvChoice> choices = gemv_choose_batch(items);
    std::vector<GemvParams> tdescs;
    std::vector<int> blk0(1, 0);
    for (size_t i = 0; i < items.size(); ++i) {
        GemvParams& p = items[i];
        const GemvChoice c = choices[i];
        if (p.RT > 0 && !c.fuse) { tdescs.push_back(p); blk0.push_back(blk0.back() + (p.G + 3) / 4); }
        size_t sh = 0;
        if ((e = gemv_dispatch(c, PrepareDesc{p, sh})) != hipSuccess) return e;
        size_t k = 0;
        while (k < keys.size() && !(keys[k].W == c.W && keys[k].PER == c.PER && keys[k].fuse == c.fuse && keys[k].sh == sh)) ++k;
        if (k == keys.size()) { keys.push_back(Key{c.W, c.PER, c.fuse, sh}); members.emplace_back(); }
        members[k].push_back(p);
    }
    for (size_t k = 0; k < keys.size(); ++k) {
        GemvBatchGroup g{};
        g.W = keys[k].W; g.PER = keys[k].PER; g.fuse = keys[k].fuse; g.sh = keys[k].sh; g.nmat = (int)members[k].size();
        std::vector<int> strip0(members[k].size() + 1, 0);
        for (size_t m = 0; m < members[k].size(); ++m) strip0[m + 1] = strip0[m] + (members[k][m].N + 15) / 16;
        g.nstrips = strip0.back();
        std::vector<int> owner((size_t)g.nstrips);
        for (size_t m = 0; m < members[k].size(); ++m)
            for (int w = strip0[m]; w < strip0[m + 1]; ++w) owner[(size_t)w] = (int)m;
        b.groups.push_back(g);                                       // pushed first so that a failure below is freed with the rest
        if ((e = to_device(members[k], &b.groups.back().d_descs)) != hipSuccess) return e;
        if ((e = to_device(strip0, &b.groups.back().d_strip0)) != hipSuccess) return e;
        if ((e = to_device(owner, &b.groups.back().d_owner)) != hipSuccess) return e;
    }
    b.nt = (int)tdescs.size(); b.nblk_total = blk0.back();
    if (b.nt > 0) {
        std::vector<int> owner((size_t)b.nblk_total);
        for (int m = 0; m < b.nt; ++m)
            for (int w = blk0[(size_t)m]; w < blk0[(size_t)m + 1]; ++w) owner[(size_t)w] = m;
        if ((e = to_device(tdescs, &b.d_tdescs)) != hipSuccess) return e;
        if ((e = to_device(blk0, &b.d_blk0)) != hipSuccess) return e;
        if ((e = to_device(owner, &b.d_towner)) != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t gemv_batch_run(const lowra_fwd_batch& b, hipStream_t st) {
    if (b.nt > 0) {
        gemv_t_partial_batch_kernel<<<dim3(b.nblk_total), dim3(64), 0, st>>>(b.d_tdescs, b.d_blk0, b.d_towner);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (b.groups.empty()) return hipSuccess;
    KernelTimer timer(st);
    for (const auto& g : b.groups) {
        const hipError_t e = gemv_dispatch(GemvChoice{g.W, g.PER, g.fuse}, LaunchGroup{g, st});
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lowra
