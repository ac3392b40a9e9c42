// Fused dequant-GEMMs for the token counts between the small-token kernels and the large output grids: the forward
// y = [x | s x A^T] [What | B]^T and the input gradient dX = [dY | s dY B] [What ; A] (Sec. 2.1 LoRA form; App. A.2
// decode).
//
// The 256-column kernels of gemm_fwd.hip and gemm_bwd.hip hold a compute unit with one workgroup of 256 x (128..256)
// outputs that walks the whole contraction.  With few output tiles that leaves most of the chip idle: 128 tokens of a
// 4096 x 4096 matrix are 16 workgroups and 64 steps in a row.  Here a workgroup owns 128 output columns x 32 TM tokens
// (TM = 1..4 or 6), up to five of them share a compute unit and cover each other's latencies, and the contraction is split
// between workgroups until they fill the chip; the splits leave fp32 partial tiles in accumulator order that
// mid_sum_kernel adds in split order (deterministic, no atomics).  Any K from 128 on (an odd number of groups
// included), any mix of widths, any number of codebooks.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "gemm_mid.h"

namespace lowra {

namespace {

constexpr int MID_COLS = kMidCols;       // output columns per workgroup: 32 per wavefront
constexpr int MID_THREADS = 256;

typedef unsigned int u32x2a4_t __attribute__((ext_vector_type(2), aligned(4)));
typedef unsigned int u32x4a4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4v_t __attribute__((ext_vector_type(4)));
typedef short mid_v4i16_t __attribute__((ext_vector_type(4)));
typedef short mid_v8i16_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) mid_v4i16_t* mid_lds_v4i16_ptr;

// packed rows start at multiples of 8 bytes only (K = 64 x an odd number): no 16-byte alignment to rely on
__device__ __forceinline__ uint4 load16_u(const uint8_t* q) {
    const u32x4a4_t v = *reinterpret_cast<const u32x4a4_t*>(q);
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 load8_u(const uint8_t* q) {
    const u32x2a4_t v = *reinterpret_cast<const u32x2a4_t*>(q);
    return make_uint2(v.x, v.y);
}
// A group's scale as it is stored, fp32 or bf16 bits; scale_of() widens it.  Apart, because a conversion beside the load
// would wait for it there, and for every transfer under way with it.
__device__ __forceinline__ uint32_t load_scale(const MidParams& p, size_t i) {
    return p.scale_bf16 ? static_cast<const uint16_t*>(p.absmax)[i] : static_cast<const uint32_t*>(p.absmax)[i];
}
__device__ __forceinline__ uint32_t scale_of(const MidParams& p, uint32_t bits) { return bits << (p.scale_bf16 ? 16 : 0); }
__device__ __forceinline__ bf16x8_t frag_of(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const u32x4v_t v = {a, b, c, d};
    return __builtin_bit_cast(bf16x8_t, v);
}

// The unified decode of a 1- or 2-bit row (gemm_fwd.hip): byte tables of the row's levels times the group's absmax,
// rounded to bf16, and per-lane constants that make both widths one instruction stream.
struct NarrowConsts { uint32_t mul, mask, orc, sell, selh, width; };
__device__ __forceinline__ NarrowConsts narrow_consts(bool two) {
    NarrowConsts c;
    c.mul = two ? 0x404101u : 0x808101u;
    c.mask = two ? 0x03030303u : 0x01010101u;
    c.orc = two ? 0x04000400u : 0x02000200u;
    c.sell = two ? 0x06040200u : 0x03010200u;
    c.selh = two ? 0x07050301u : 0x03010200u;
    c.width = two ? 4u : 2u;                    // bits per pair of codes
    return c;
}
// 8 codes (low bits of cw) -> 8 bf16
__device__ __forceinline__ bf16x8_t narrow8(uint32_t cw, uint32_t SL, uint32_t SH, const NarrowConsts& c) {
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t q = __builtin_amdgcn_ubfe(cw, j * c.width, c.width);
        d[j] = __builtin_amdgcn_perm(SH, SL, (__umul24(q, c.mul) & c.mask) | c.orc);
    }
    return frag_of(d[0], d[1], d[2], d[3]);
}

// What both kernels do at the end.  Accumulator register v of token tile t: column 32 wave + 8 (v/4) + 4 (lane/32) + v%4,
// token 32 t + lane%32.
template <int TM>
__device__ __forceinline__ void mid_epilogue(const MidParams& p, const floatx16_t (&acc)[TM], uint8_t* smem, int wave, int lane,
                                             int split, int tile, int c0, int m0, int cols) {
    const int fi = lane & 31, h = lane >> 5;
    if (p.splits > 1) {
        const int ntiles = p.ntiles;
        float4* dst = reinterpret_cast<float4*>(p.part) + (((size_t)split * ntiles + tile) * 4 + wave) * (TM * 256) + lane;
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                dst[(t * 4 + vq) * 64] = make_float4(acc[t][4 * vq], acc[t][4 * vq + 1], acc[t][4 * vq + 2], acc[t][4 * vq + 3]);
        return;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            const uint2 v = make_uint2(pack_bf16x2(acc[t][4 * vq], acc[t][4 * vq + 1]), pack_bf16x2(acc[t][4 * vq + 2], acc[t][4 * vq + 3]));
            *reinterpret_cast<uint2*>(smem + (32 * t + fi) * 256 + (((wave * 4 + vq) ^ (fi & 15)) << 4) + 8 * h) = v;
        }
    __syncthreads();
    const int c = threadIdx.x & 15;
    if (c0 + 8 * c < cols) {                                          // cols is a multiple of 8
#pragma unroll
        for (int it = 0; it < 2 * TM; ++it) {
            const int r = it * 16 + (threadIdx.x >> 4);
            if (m0 + r < p.M)
                *reinterpret_cast<uint4*>(p.out + (size_t)(m0 + r) * cols + c0 + 8 * c) =
                    *reinterpret_cast<const uint4*>(smem + r * 256 + ((c ^ (r & 15)) << 4));
        }
    }
}

// ---- forward.  Wavefront w owns channels c0 + 32 w .. + 31 (weights as the A operand, decoded straight into operand
// registers) x all tokens of the tile; the activations come through a ring of three LDS stages by global -> LDS
// transfers two steps ahead.  A superstep is 256 input features: lane (row, h) decodes the 128 features from 128 h on,
// which are 16, 32 or 64 contiguous bytes of its row, so that its codes are asked for once per superstep, one
// superstep ahead.  Step j (0..3) contracts features 32 j .. + 31 of both halves; LDS chunk c (16 bytes) of a token
// row holds half c / 4, features 8 (c % 4) .. + 7 of the step, at physical chunk c ^ ((row >> 1) & 7).
// WIDE: the matrix has 4-bit rows.  Every wavefront then keeps the levels of its 32 rows in LDS, level q of row i at
// 128 q + 4 i (a lookup's bank follows from the row alone: no conflicts), and a looked-up level times the group's absmax is
// rounded to bf16 (App. A.2 as written).
//
// What bounds it: plain-ALU issue.  The decode is 1.3 (WIDE 2) instructions per weight, that is 20 to 34 beside the TM MFMAs
// of a slice, whatever TM is: two workgroups on a unit are busy for the sum of the decode's and the MFMAs' issue times.
// Hence (a) a superstep of 16 slices without a branch: transfers past an end are zeroed by a buffer descriptor, codes and
// scales are staged in LDS by counted transfers, an odd number of groups is its own instantiation; with a branch at every
// transfer the compiler emptied the matrix pipe at each.  4096 x 4096, 512 tokens, 50/50 % of 1-/2-bit rows 39 -> 30 us;
// 4096 x 1024, 777 tokens with 4-bit rows 19.8 -> 17.1.  (b) Tiles of 192 tokens, which halve the decode of tiles of 96:
// 11008 x 4096, 333 tokens, 50/25/25 %: 77 us -> 70 (a) -> 55 in calls that follow each other (waited for, or in a kernel
// trace, a launch takes 58 to 62).  They leave LDS for one workgroup per unit.
template <int TM, bool WIDE, bool ODD>
struct FwdLds {
    static constexpr int STAGE = TM * 4096;                           // 32 TM token rows x 128 bytes
    static constexpr int NP = WIDE ? 4 : 2;                           // 16-byte pieces of a lane's codes per superstep
    static constexpr int TAB0 = 3 * STAGE;                            // WIDE: 2 KB of levels per wavefront
    static constexpr int CODE0 = TAB0 + (WIDE ? 4 * 2048 : 0);        // per wavefront: two scales (256 bytes each), then the pieces, 1 KB each
    static constexpr int CODE = 512 + (NP + (ODD ? 1 : 0)) * 1024;    // (an odd number of groups: rows may start at 8 mod 16, one piece more)
    static constexpr int BYTES = CODE0 + 4 * CODE;
};

template <int TM, bool WIDE, bool ODD>
__global__ __launch_bounds__(MID_THREADS, 2) void mid_fwd_kernel(MidParams p) {
    extern __shared__ __align__(16) uint8_t smem[];
    using L = FwdLds<TM, WIDE, ODD>;
    constexpr int STAGE = L::STAGE, NP = L::NP;
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(lptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = lane & 31, h = lane >> 5;
    const int ntiles = p.ntiles;
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    const int split = __builtin_amdgcn_readfirstlane(w / ntiles);
    const int tile = p.tile0 + w - split * ntiles;
    const int mt = __builtin_amdgcn_readfirstlane(tile / p.tiles_c);
    const int n0 = (tile - mt * p.tiles_c) * MID_COLS, m0 = mt * (32 * TM);
    const int G = p.G, K = p.K;
    const int nsuper = (G + 3) >> 2;
    const int s_lo = split * p.per_split, s_hi = min(s_lo + p.per_split, nsuper);
    const int k_hi = min(K, s_hi * 256);

    // my row (past N: the last one again, into output columns that are never stored)
    const int nc = min(n0 + wave * 32 + fi, p.N - 1);
    const RowInfo rec = p.rows[nc];

    // Activation transfers: wavefront w moves rows 8 (w TM + i) .. + 7, i < TM.  They go through a buffer descriptor: a lane
    // whose features lie past k_hi gets an offset past its end, and zeros land in LDS without a branch around the transfer
    // (an infinity times a stand-in weight would not be none; and a branch per transfer cuts the slices' schedule to pieces).
    const int m_last = p.M - 1 - m0;
    const bufdesc_t act = buffer_desc(p.act + (size_t)m0 * K);
    uint32_t voff[TM];
    const int half0 = (((lane & 7) ^ ((wave * TM * 4 + (lane >> 4)) & 7)) >> 2) * 128;    // even i; odd i: the other half
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = (wave * TM + i) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        voff[i] = (uint32_t)min(r, m_last) * (uint32_t)K * 2u + (uint32_t)((c >> 2) * 128 + (c & 3) * 8) * 2u;     // rows past M are clamped (never stored)
    }
    auto issue1 = [&](int ss, int j, int stage, int i) __attribute__((always_inline)) {   // of step j of superstep ss
        const int left = k_hi - ss * 256 - j * 32;                    // uniform
        const uint32_t v = ((i & 1) ? 128 - half0 : half0) < left ? voff[i] : 0x80000000u;
        dma16_b(act, v, (uint32_t)(ss * 512 + j * 64), smem_lds + stage * STAGE + wave * (TM * 1024) + i * 1024);
    };
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < (j < 2 ? TM : TM / 4); ++i) issue1(s_lo, j, j, i);

    const int bits = rec.bits();
    const float* tab = p.mappings + (size_t)rec.cb() * kTableStride;
    const bool one = bits == 1, four = bits == 4;
    const NarrowConsts nk = narrow_consts(bits == 2);

    // My codes and scales of one superstep travel as the activations do, counted with them: a register load among
    // transfers that the compiler does not know would be waited for with all of them.  Pieces past the row's are its last
    // one again.  The last superstep of an odd number of groups, inside which the row ends at 8 mod 16, is not staged.
    const int s_staged = ODD ? max(min(s_hi, nsuper - 1), 1) - 1 : s_hi - 1;
    uint8_t* const my_code = smem + L::CODE0 + wave * L::CODE;
    const uint32_t code_lds = smem_lds + L::CODE0 + wave * L::CODE;
    const uint32_t mis = ODD ? rec.offset & 8u : 0u;                  // the 16-byte pieces start this much before my codes
    const uint32_t srow = (uint32_t)nc * (uint32_t)G;
    const int scale_sh = p.scale_bf16 ? 1 : 0;                        // bf16: the dword that holds the scale
    constexpr int NCODE = NP + 2 + (ODD ? 1 : 0);
    auto issue_codes = [&](int ss_) __attribute__((always_inline)) {
        const int ss = min(ss_, s_staged);
        int gh = ss * 4 + 2 * h;                                      // my two groups
        if (gh + 1 >= G) gh = ss * 4;                                 // past the row's end: any of the row's, its scale becomes zero
        const uint32_t c0 = rec.offset - mis + (uint32_t)(gh * 8 * bits);
        const int last = bits - 1 + (int)(mis >> 3);
        dma4_s(p.absmax, ((srow + (uint32_t)gh) >> scale_sh) * 4u, code_lds);
        dma4_s(p.absmax, ((srow + (uint32_t)gh + 1u) >> scale_sh) * 4u, code_lds + 256);
#pragma unroll
        for (int q = 0; q < NP + (ODD ? 1 : 0); ++q) dma16_s(p.packed, c0 + 16u * (uint32_t)min(q, last), code_lds + 512 + q * 1024);
    };
    issue_codes(s_lo);

    floatx16_t acc[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
    int kof[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kof[kk] = fi * 128 + (((4 * h + kk) ^ ((fi >> 1) & 7)) << 4);
    uint8_t* mytab = smem + L::TAB0 + wave * 2048 + fi * 4;
    float lev[4];
#pragma unroll
    for (int q = 0; q < (WIDE ? 16 : 4); q += 4) {
        const float4 v = *reinterpret_cast<const float4*>(tab + q);
        if (WIDE) {
            float* d = reinterpret_cast<float*>(mytab + 128 * q);
            d[0] = v.x; d[32] = v.y; d[64] = v.z; d[96] = v.w;        // (both halves write the same values)
        } else {
            lev[0] = v.x; lev[1] = v.y; lev[2] = v.z; lev[3] = v.w;
        }
    }

    struct Codes { uint32_t c[4 * NP]; float a0, a1; };               // of one superstep: 128 codes and two scales
    auto fetch = [&](int ss, Codes& o) __attribute__((always_inline)) {
        const int gh = ss * 4 + 2 * h;
        uint32_t b0, b1;
        if (!ODD || ss + 1 < nsuper) {                                // uniform
            uint32_t d[4 * NP + 4];
#pragma unroll
            for (int q = 0; q < NP + (ODD ? 1 : 0); ++q) {
                const uint4 v = *reinterpret_cast<const uint4*>(my_code + 512 + q * 1024 + lane * 16);
                d[4 * q] = v.x; d[4 * q + 1] = v.y; d[4 * q + 2] = v.z; d[4 * q + 3] = v.w;
            }
            b0 = *reinterpret_cast<const uint32_t*>(my_code + lane * 4);
            b1 = *reinterpret_cast<const uint32_t*>(my_code + 256 + lane * 4);
            const uint32_t e = srow + (uint32_t)gh;                   // (a zeroed scale's parity does not matter)
            b0 >>= (e & scale_sh) * 16; b1 >>= (~e & scale_sh) * 16;
#pragma unroll
            for (int i = 0; i < 4 * NP; ++i) o.c[i] = ODD && mis ? d[ODD ? i + 2 : i] : d[i];
        } else {
            b0 = load_scale(p, srow + min(gh, G - 1));
            b1 = load_scale(p, srow + min(gh + 1, G - 1));
            const uint8_t* q0 = p.packed + rec.offset + (size_t)gh * 8 * bits;
            const int have = min(max(G - gh, 0), 2) * 8 * bits;
#pragma unroll
            for (int q = 0; q < 2 * NP; ++q) {
                const uint2 v = 8 * q + 8 <= have ? load8_u(q0 + 8 * q) : make_uint2(0u, 0u);
                o.c[2 * q] = v.x; o.c[2 * q + 1] = v.y;
            }
        }
        o.a0 = gh < G ? __builtin_bit_cast(float, scale_of(p, b0)) : 0.0f;
        o.a1 = gh + 1 < G ? __builtin_bit_cast(float, scale_of(p, b1)) : 0.0f;
    };
    Codes cur, nxt;
    uint32_t SL = 0, SH = 0;
    // Slice q (0..15) of a superstep: 16 of a step's 64 features, step q / 4.  q = 16, 17: the next superstep's first.
    auto word = [&](int q, bool want4) __attribute__((always_inline)) -> uint32_t {
        const Codes& o = q < 16 ? cur : nxt;
        const int j = (q >> 2) & 3, kk = q & 3;
        const uint32_t c2 = o.c[2 * j + (kk >> 1)] >> (16 * (kk & 1)), c1 = o.c[j] >> (8 * kk);
        const uint32_t c21 = one ? c1 : c2;
        return want4 && four ? o.c[(q & 15) % (4 * NP)] : c21;
    };
    auto new_group = [&](float a) __attribute__((always_inline)) {    // narrow rows: the byte tables of the next group
        const uint32_t P01 = pack_bf16x2(lev[0] * a, lev[1] * a), P23 = pack_bf16x2(lev[2] * a, lev[3] * a);
        SL = __builtin_amdgcn_perm(P23, P01, nk.sell);
        SH = __builtin_amdgcn_perm(P23, P01, nk.selh);
    };
    auto look = [&](int q, float (&e)[8]) __attribute__((always_inline)) {
        const uint32_t cw = word(q, true);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            e[i] = *reinterpret_cast<const float*>(mytab + (__builtin_amdgcn_ubfe(cw, (uint32_t)(i * bits), (uint32_t)bits) << 7));
    };
    auto pack = [&](int q, const float (&e)[8]) __attribute__((always_inline)) -> bf16x8_t {
        const float a = q < 8 ? cur.a0 : q < 16 ? cur.a1 : nxt.a0;
        return frag_of(pack_bf16x2(e[0] * a, e[1] * a), pack_bf16x2(e[2] * a, e[3] * a), pack_bf16x2(e[4] * a, e[5] * a), pack_bf16x2(e[6] * a, e[7] * a));
    };
    struct Acts { bf16x8_t f[TM]; };
    auto read_act = [&](int stage, int kk, Acts& o) __attribute__((always_inline)) {
        const uint8_t* sb = smem + stage * STAGE + kof[kk];
#pragma unroll
        for (int tt = 0; tt < TM; ++tt) o.f[tt] = *reinterpret_cast<const bf16x8_t*>(sb + tt * 4096);
    };
    // The instruction order of a slice: after each MFMA a share of the work that prepares the next ones (MFMAs issued back
    // to back hold the wavefront at its next one for 32 cycles each).
    auto spread = [&]() __attribute__((always_inline)) {
        constexpr int NV = WIDE ? 34 : 22, ND = WIDE ? TM + 8 : TM;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, (NV + TM - 1) / TM, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, (ND + TM - 1) / TM, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                  // all three activation tiles, the first codes
    __syncthreads();
    fetch(s_lo, cur);
    Acts ac[2];
    bf16x8_t wf[2];
    float e[2][8];
    if (WIDE) {
        look(0, e[0]);
        look(1, e[1]);
        wf[0] = pack(0, e[0]);
    } else {
        new_group(cur.a0);
        wf[0] = narrow8(word(0, false), SL, SH, nk);
    }
    read_act(0, 0, ac[0]);

    // Step t.  Its barrier sits before the last slice, when every wavefront holds that slice's operands: stage t % 3 is
    // then free for tile t + 3, whose transfers go out one per slice from there on (several at once hold up the
    // wavefront), and the operands of (step t + 1, slice 0) are read under the last slice's MFMAs.  The codes of superstep
    // ss + 1 are sent for in its predecessor's first step, into a place that has been read, and read in the last.
    int st = 0;                                                       // stage of step t
    for (int ss = s_lo; ss < s_hi; ++ss) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int j = q >> 2, kk = q & 3;
            const int stn = st == 2 ? 0 : st + 1, stp = st == 0 ? 2 : st - 1;
            if (kk == 3) {
                // tile t + 1 has landed when no more is outstanding than was issued for tile t + 2 and, in a superstep's
                // second step, for the codes before it
                if (j == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(TM + NCODE) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(TM) : "memory");
                __syncthreads();
                if (j == 0) issue_codes(ss + 1);
#pragma unroll
                for (int i = 0; i < TM / 4; ++i) issue1(j == 0 ? ss : ss + 1, (j + 3) & 3, st, i);
                read_act(stn, 0, ac[(q + 1) & 1]);
            } else {
#pragma unroll
                for (int i = (kk + 1) * TM / 4; i < (kk + 2) * TM / 4; ++i) {
                    if (j < 2) issue1(ss, j + 2, stp, i);
                    else issue1(ss + 1, j - 2, stp, i);
                }
                if (q == 12) fetch(ss + 1, nxt);
                read_act(st, kk + 1, ac[(q + 1) & 1]);
            }
            if (WIDE) {
                look(q + 2, e[q & 1]);
                wf[(q + 1) & 1] = pack(q + 1, e[(q + 1) & 1]);
            } else {
                if (q == 7) new_group(cur.a1);
                if (q == 15) new_group(nxt.a0);
                wf[(q + 1) & 1] = narrow8(word(q + 1, false), SL, SH, nk);
            }
#pragma unroll
            for (int tt = 0; tt < TM; ++tt) acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q & 1], ac[q & 1].f[tt], acc[tt], 0, 0, 0);
            spread();
            if (kk == 3) st = stn;
        }
        cur = nxt;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                  // transfers past the end: none may land in what comes next

    // the rank-r term: the last split contracts over t = s x A^T, 64 ranks at a time; rank 64 e + 16 kk + 8 h + i
    if (p.r > 0 && s_hi == nsuper) {
        for (int e = 0; e * 64 < p.r; ++e) {
            __syncthreads();                                          // the stage's last reader is done
            const uint32_t dst = smem_lds + wave * (TM * 1024);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = (wave * TM + i) * 8 + (lane >> 3);
                dma16_s(p.ext_act + (size_t)m0 * p.RP + e * 64,
                        (uint32_t)min(r, m_last) * (uint32_t)p.RP * 2u + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) << 4), dst + i * 1024);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int r0 = e * 64 + 16 * kk;
                if (r0 >= p.r) break;                                 // uniform
                const uint16_t* src = p.lora + (size_t)nc * p.r + r0 + 8 * h;
                bf16x8_t wf;
                if ((p.r & 7) == 0) {                                 // uniform: 16-byte pieces, in or out as a whole
                    const uint4 v = r0 + 8 * h < p.r ? *reinterpret_cast<const uint4*>(src) : make_uint4(0u, 0u, 0u, 0u);
                    wf = frag_of(v.x, v.y, v.z, v.w);
                } else {
                    uint32_t v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = r0 + 8 * h + i < p.r ? src[i] : 0u;
                    wf = frag_of(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
                }
#pragma unroll
                for (int tt = 0; tt < TM; ++tt) {
                    const bf16x8_t f = *reinterpret_cast<const bf16x8_t*>(smem + (32 * tt + fi) * 128 + (((2 * kk + h) ^ ((fi >> 1) & 7)) << 4));
                    acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, f, acc[tt], 0, 0, 0);
                }
            }
        }
    }
    mid_epilogue<TM>(p, acc, smem, wave, lane, split, tile - p.tile0, n0, m0, p.N);
}

// ---- input gradient.  The contraction runs over channels while codes are packed along k (gemm_bwd.hip): a step's
// 64 channels x 128 input features are decoded into an LDS tile [channel][k] and read back transposed.  Two roles per
// thread: as mover (row 16 w + lane / 4, piece lane % 4) it brings 16 bytes of a row's codes, four of its levels and
// its scales into registers two steps ahead and into LDS one step ahead, so that a row's 16, 32 or 64 code bytes are
// one run of neighbouring lanes; as decoder (row lane, features 32 w .. + 31) it decodes 32 weights of ONE row and ONE
// group.  Wavefront w multiplies output columns c0 + 32 w .. + 31 (weights as the A operand) with all tokens.
constexpr int BM_WROW = 256;                                          // bytes per row of the weight tile: 128 k x bf16
__device__ __forceinline__ int bmid_swz(int r, int c) { return r * BM_WROW + ((c ^ (((r & 3) << 2) | ((r >> 2) & 3))) << 4); }

template <int TM, bool WIDE>
struct BwdLds {
    static constexpr int A = TM * 4096, W = 64 * BM_WROW;
    static constexpr int C = WIDE ? 4096 : 2048;                      // staged codes: 64 rows x 64 (32) bytes
    static constexpr int W0 = 2 * A, C0 = W0 + 2 * W, META0 = C0 + 2 * C, TAB0 = META0 + 2 * 1024;
    // TAB0: WIDE with shared tables: all of them, once; else two buffers of a step's 64 rows (64 or 16 bytes each)
};

// SHARED (with WIDE): at most kMidLutBooks codebooks, kept in LDS as a whole.
// What bounds it: plain-ALU and LDS issue of the decode, 160 and 50 instructions per step beside 4 TM MFMAs (11008 x 4096, 333
// tokens: VALU 30 % of a wavefront's life, LDS busy 40 % of the unit's, a quarter of that in conflicts).  So a step is one run
// of instructions without branches (68.0 -> 64.2 us; 4096 x 1024, 777 tokens 30.3 -> 28.6), and tiles of 192 tokens halve the
// decode of those of 96 (68.7 -> 63.2).
template <int TM, bool WIDE, bool SHARED>
__global__ __launch_bounds__(MID_THREADS, 2) void mid_bwd_kernel(MidParams p) {
    extern __shared__ __align__(16) uint8_t smem[];
    using L = BwdLds<TM, WIDE>;
    constexpr int ROWTAB = WIDE ? 64 : 16;                            // bytes of a row's staged levels
    const uint32_t smem_lds = (uint32_t)(uintptr_t)(lptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = lane & 31, h = lane >> 5;
    const int ntiles = p.ntiles;
    const int wg = xcd_tile(blockIdx.x, gridDim.x);
    const int split = __builtin_amdgcn_readfirstlane(wg / ntiles);
    const int tile = p.tile0 + wg - split * ntiles;
    const int mt = __builtin_amdgcn_readfirstlane(tile / p.tiles_c);
    const int k0 = (tile - mt * p.tiles_c) * MID_COLS, m0 = mt * (32 * TM);
    const int G = p.G, K = p.K, N = p.N;
    const int nsteps = (N + 63) >> 6;
    const int s_lo = split * p.per_split, s_hi = min(s_lo + p.per_split, nsteps);
    if (SHARED)
        for (int e = tid; e < p.C * kTableStride; e += MID_THREADS) reinterpret_cast<float*>(smem + L::TAB0)[e] = p.mappings[e];

    // ---- activations: dY[m0.., 64 s ..], 128 bytes per token row, chunk c at c ^ ((row >> 1) & 7)
    const int m_last = p.M - 1 - m0;
    const bufdesc_t act = buffer_desc(p.act + (size_t)m0 * N);
    uint32_t voff[TM];
    int coff[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = (wave * TM + i) * 8 + (lane >> 3);
        coff[i] = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
        voff[i] = (uint32_t)min(r, m_last) * (uint32_t)N * 2u + (uint32_t)coff[i] * 2u;
    }
    auto issue = [&](int s, int buf) __attribute__((always_inline)) {
        const uint32_t dst = smem_lds + buf * L::A + wave * (TM * 1024);
        const int left = N - s * 64;                                  // channels past N are zeros, against the last row's weights again
#pragma unroll
        for (int i = 0; i < TM; ++i) dma16_b(act, coff[i] < left ? voff[i] : 0x80000000u, (uint32_t)s * 128u, dst + i * 1024);
    };

    // ---- mover role
    const int mrow = 16 * wave + (lane >> 2), piece = lane & 3;
    const int g0 = k0 >> 6;
    const bool two_groups = g0 + 1 < G;
    // the scale I bring: piece 1 the tile's second group's (in the last column tile, where there is none, the first again, for
    // columns that are never stored), the others the first's
    const int my_group = g0 + (piece == 1 && two_groups ? 1 : 0);
    struct Raw { uint4 codes; float4 lev; uint32_t a, e; RowInfo rec; };
    const int sh = p.scale_bf16 ? 1 : 0;                              // bf16: the dword that holds the scale, no branch
    const uint32_t* const scales = static_cast<const uint32_t*>(p.absmax);
    auto load_rec = [&](int s) -> RowInfo { return p.rows[min(s * 64 + mrow, N - 1)]; };
    auto load_raw = [&](int s, const RowInfo& rec, Raw& d) __attribute__((always_inline)) {
        const int ncl = min(s * 64 + mrow, N - 1), bits = rec.bits();
        const int row_bytes = K / 8 * bits;
        // a piece past the row's codes of this tile fetches the last one again; 16 bytes before the row's end at the latest
        const int off = min(k0 / 8 * bits + 16 * min(piece, bits - 1), row_bytes - 16);
        d.codes = load16_u(p.packed + (uint32_t)(rec.offset + (uint32_t)off));
        if (!SHARED) d.lev = *reinterpret_cast<const float4*>(p.mappings + (size_t)rec.cb() * kTableStride + (WIDE ? 4 * piece : 0));
        d.e = (uint32_t)ncl * (uint32_t)G + (uint32_t)my_group;
        d.a = scales[d.e >> sh];
        d.rec = rec;
    };
    // (without branches: the four movers of a row write its record's four words, and what pieces past a narrow row's second
    // repeat goes to the same place)
    const int slot = WIDE ? piece : min(piece, 1);
    auto stage_in = [&](int buf, const Raw& d) __attribute__((always_inline)) {
        *reinterpret_cast<uint4*>(smem + L::C0 + buf * L::C + mrow * (WIDE ? 64 : 32) + ((slot ^ (WIDE ? (mrow >> 2) & 3 : (mrow >> 3) & 1)) << 4)) = d.codes;
        const uint32_t scale = (d.a >> ((d.e & sh) * 16)) << (sh * 16);
        *reinterpret_cast<uint32_t*>(smem + L::META0 + buf * 1024 + mrow * 16 + piece * 4) = piece == 2 ? d.rec.bits_cb : scale;
        if (WIDE && !SHARED) {                                        // level q of row r at 256 q + 4 r: a lookup touches bank r whatever the code
            float* tab = reinterpret_cast<float*>(smem + L::TAB0 + buf * (64 * ROWTAB) + piece * 1024 + mrow * 4);
            tab[0] = d.lev.x; tab[64] = d.lev.y; tab[128] = d.lev.z; tab[192] = d.lev.w;
        } else if (!WIDE) {
            *reinterpret_cast<float4*>(smem + L::TAB0 + buf * (64 * ROWTAB) + mrow * ROWTAB) = d.lev;
        }
    };

    // ---- decoder role: 32 weights of row `lane`, features 32 wave .. + 31 of the tile (group wave / 2)
    const bool tail_shift = !two_groups && K >= 128;                  // a 1-bit row's 16 bytes then start one group early
    constexpr int tab_shift = SHARED ? 2 : 8;
    struct Dec { uint32_t lo, hi, c4[4]; float a, v[2][8]; int bits; const uint8_t* tb; uint32_t SL, SH; };
    Dec d;
    auto decode_begin = [&](int buf) __attribute__((always_inline)) {
        const uint4 meta = *reinterpret_cast<const uint4*>(smem + L::META0 + buf * 1024 + lane * 16);
        d.a = __builtin_bit_cast(float, (wave >> 1) ? meta.y : meta.x);
        d.bits = (int)(meta.z & 0xffu);
        const bool one = d.bits == 1;
        // my 32 codes: 4 bits: piece `wave`; 2 bits: half (wave & 1) of piece wave / 2; 1 bit: dword `wave` of piece 0
        const int pc = d.bits == 4 ? wave : one ? 0 : wave >> 1;
        const uint4 q = *reinterpret_cast<const uint4*>(smem + L::C0 + buf * L::C + lane * (WIDE ? 64 : 32) +
                                                        ((pc ^ (WIDE ? (lane >> 2) & 3 : (lane >> 3) & 1)) << 4));
        const int d1 = (wave + (tail_shift ? 2 : 0)) & 3;             // uniform
        const uint32_t q1 = d1 == 0 ? q.x : d1 == 1 ? q.y : d1 == 2 ? q.z : q.w;
        d.lo = one ? q1 : (wave & 1) ? q.z : q.x;
        d.hi = (wave & 1) ? q.w : q.y;
        if (WIDE) {
            d.c4[0] = q.x; d.c4[1] = q.y; d.c4[2] = q.z; d.c4[3] = q.w;
            d.tb = smem + L::TAB0 + (SHARED ? (int)(meta.z >> 8) * (kTableStride * 4) : buf * (64 * ROWTAB) + lane * 4);
        } else {
            const NarrowConsts nk = narrow_consts(!one);
            const float4 lv = *reinterpret_cast<const float4*>(smem + L::TAB0 + buf * (64 * ROWTAB) + lane * ROWTAB);
            const uint32_t P01 = pack_bf16x2(lv.x * d.a, lv.y * d.a), P23 = pack_bf16x2(lv.z * d.a, lv.w * d.a);
            d.SL = __builtin_amdgcn_perm(P23, P01, nk.sell); d.SH = __builtin_amdgcn_perm(P23, P01, nk.selh);
        }
    };
    auto decode_look = [&](int kk) __attribute__((always_inline)) {   // WIDE: the lookups of chunk kk
        if (!WIDE) return;
        const uint32_t c2 = ((kk >> 1) ? d.hi : d.lo) >> (16 * (kk & 1)), c1 = d.lo >> (8 * kk);
        const uint32_t c21 = d.bits == 1 ? c1 : c2;
        const uint32_t cw = d.bits == 4 ? d.c4[kk] : c21;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            d.v[kk & 1][i] = *reinterpret_cast<const float*>(d.tb + (__builtin_amdgcn_ubfe(cw, (uint32_t)(i * d.bits), (uint32_t)d.bits) << tab_shift));
    };
    auto decode_put = [&](int kk, uint8_t* wt) __attribute__((always_inline)) {
        if (WIDE) {
            const float (&v)[8] = d.v[kk & 1];
            *reinterpret_cast<uint4*>(wt + bmid_swz(lane, wave * 4 + kk)) =
                make_uint4(pack_bf16x2(v[0] * d.a, v[1] * d.a), pack_bf16x2(v[2] * d.a, v[3] * d.a), pack_bf16x2(v[4] * d.a, v[5] * d.a),
                           pack_bf16x2(v[6] * d.a, v[7] * d.a));
        } else {
            const uint32_t c2 = ((kk >> 1) ? d.hi : d.lo) >> (16 * (kk & 1)), c1 = d.lo >> (8 * kk);
            *reinterpret_cast<bf16x8_t*>(wt + bmid_swz(lane, wave * 4 + kk)) =
                narrow8(d.bits == 1 ? c1 : c2, d.SL, d.SH, narrow_consts(d.bits != 1));
        }
    };

    // ---- multiplier role
    floatx16_t acc[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
    int aoff[4], troff[2];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) aoff[kk] = fi * 128 + (((2 * kk + h) ^ ((fi >> 1) & 7)) << 4);
    {   // transposing reads: lane L of a 16-lane group points at channel L / 4 of its four, 8 bytes at k 4 (L % 4)
        const int L16 = lane & 15, grp = (lane >> 4) & 1;
#pragma unroll
        for (int eb = 0; eb < 2; ++eb)
            troff[eb] = bmid_swz(h * 8 + eb * 4 + (L16 >> 2), wave * 4 + grp * 2 + ((L16 & 3) >> 1)) + (L16 & 1) * 8;
    }
    struct Slice { bf16x8_t f[TM], wf; };
    auto read_slice = [&](const uint8_t* at, uint32_t wt_lds, int kk, Slice& o) __attribute__((always_inline)) {
        const mid_v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mid_lds_v4i16_ptr)(uintptr_t)(wt_lds + troff[0] + kk * 16 * BM_WROW));
        const mid_v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((mid_lds_v4i16_ptr)(uintptr_t)(wt_lds + troff[1] + kk * 16 * BM_WROW));
        const mid_v8i16_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        o.wf = __builtin_bit_cast(bf16x8_t, v);
#pragma unroll
        for (int t = 0; t < TM; ++t) o.f[t] = *reinterpret_cast<const bf16x8_t*>(at + aoff[kk] + t * 4096);
    };
    auto multiply = [&](const Slice& o) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TM; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.wf, o.f[t], acc[t], 0, 0, 0);
    };

    // Pipeline.  Step s, buffers s & 1: slices 0..2 multiply while the weight tile of step s + 1 is decoded from the staged
    // codes; then the step's barrier (tile s + 1 is complete, the buffers of step s are free); under slice 3 the first
    // operands of step s + 1 are read, the activations of step s + 2 are sent for, the raw data of step s + 3 goes from
    // registers to LDS and that of step s + 4 is asked for.  Steps past the end fetch the last one again: what is decoded
    // of them is never multiplied.
    const int s_end = s_hi - 1;
    Raw raw;
    RowInfo rec = load_rec(s_lo);
    issue(s_lo, s_lo & 1);
    issue(min(s_lo + 1, s_end), (s_lo + 1) & 1);
    load_raw(s_lo, rec, raw);
    rec = load_rec(min(s_lo + 1, s_end));
    stage_in(s_lo & 1, raw);
    load_raw(min(s_lo + 1, s_end), rec, raw);
    rec = load_rec(min(s_lo + 2, s_end));
    stage_in((s_lo + 1) & 1, raw);
    load_raw(min(s_lo + 2, s_end), rec, raw);
    rec = load_rec(min(s_lo + 3, s_end));
    __syncthreads();
    decode_begin(s_lo & 1);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) { decode_look(kk); decode_put(kk, smem + L::W0 + (s_lo & 1) * L::W); }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    stage_in(s_lo & 1, raw);                                          // step s_lo + 2
    load_raw(min(s_lo + 3, s_end), rec, raw);
    rec = load_rec(min(s_lo + 4, s_end));
    Slice sl[2];
    read_slice(smem + (s_lo & 1) * L::A, smem_lds + L::W0 + (s_lo & 1) * L::W, 0, sl[0]);

    auto step = [&](int s, auto B_) __attribute__((always_inline)) {
        constexpr int b = decltype(B_)::value;
        const uint8_t* at = smem + b * L::A;
        const uint32_t wt_lds = smem_lds + L::W0 + b * L::W;
        uint8_t* wn = smem + L::W0 + (b ^ 1) * L::W;
        decode_begin(b ^ 1);
        read_slice(at, wt_lds, 1, sl[1]);
        decode_look(0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(sl[0]);
        decode_look(1);
        read_slice(at, wt_lds, 2, sl[0]);
        decode_put(0, wn);
        __builtin_amdgcn_sched_barrier(0);
        multiply(sl[1]);
        decode_look(2);
        read_slice(at, wt_lds, 3, sl[1]);
        decode_put(1, wn);
        __builtin_amdgcn_sched_barrier(0);
        multiply(sl[0]);
        decode_look(3);
        decode_put(2, wn);
        decode_put(3, wn);
        // the activation transfers of step s + 1 are older than the loads for the steps ahead: at least three of those
        // (codes, scale, record) may stay in flight
        asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
        __syncthreads();
        stage_in(b ^ 1, raw);                                         // step s + 3
        asm volatile("" : "+v"(rec.offset), "+v"(rec.bits_cb));       // wait for the record here, not behind the transfers below
        read_slice(smem + (b ^ 1) * L::A, smem_lds + L::W0 + (b ^ 1) * L::W, 0, sl[0]);
        __builtin_amdgcn_sched_barrier(0);
        multiply(sl[1]);
        issue(min(s + 2, s_end), b);
        __builtin_amdgcn_sched_barrier(0);
        load_raw(min(s + 4, s_end), rec, raw);
        rec = load_rec(min(s + 5, s_end));
    };
    int s = s_lo;
    if (s & 1) step(s++, std::integral_constant<int, 1>{});
    for (; s + 2 <= s_hi; s += 2) {
        step(s, std::integral_constant<int, 0>{});
        step(s + 1, std::integral_constant<int, 1>{});
    }
    if (s < s_hi) step(s, std::integral_constant<int, 0>{});

    // the rank-r term: the last split contracts over u = s dY B against the rows of A, 64 ranks at a time
    if (p.r > 0 && s_hi == nsteps) {
        for (int e = 0; e * 64 < p.r; ++e) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // no transfer of the steps above lands here any more
            __syncthreads();                                          // ... and the buffers' last readers are done
            const uint32_t dst = smem_lds + wave * (TM * 1024);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                dma16_s(p.ext_act + (size_t)m0 * p.RP + e * 64,
                        (uint32_t)min((wave * TM + i) * 8 + (lane >> 3), m_last) * (uint32_t)p.RP * 2u + (uint32_t)coff[i] * 2u, dst + i * 1024);
            const int j = e * 64 + lane;
            const bool ok = j < p.r && k0 + 32 * wave < K;
            const uint4* src = reinterpret_cast<const uint4*>(p.lora + (size_t)(ok ? j : 0) * K + (ok ? k0 + 32 * wave : 0));
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                *reinterpret_cast<uint4*>(smem + L::W0 + bmid_swz(lane, wave * 4 + kk)) = ok ? src[kk] : make_uint4(0u, 0u, 0u, 0u);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) { read_slice(smem, smem_lds + L::W0, kk, sl[0]); multiply(sl[0]); }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                  // transfers past the end: none may land in the output stage
    mid_epilogue<TM>(p, acc, smem, wave, lane, split, tile - p.tile0, k0, m0, K);
}

// out = bf16(sum of the splits' partial tiles, in split order).  A thread owns four columns of one token.
__global__ __launch_bounds__(256) void mid_sum_kernel(const float4* __restrict__ part, int splits, int ntiles, int tile0, int tiles_c, int TM,
                                                      int M, int cols, uint16_t* __restrict__ out) {
    const size_t per = (size_t)ntiles * TM * 1024;                    // float4 per split
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= per) return;
    float4 a = part[e];
    int s = 1;
    for (; s + 3 < splits; s += 4) {
        const float4 b0 = part[s * per + e], b1 = part[(s + 1) * per + e], b2 = part[(s + 2) * per + e], b3 = part[(s + 3) * per + e];
        a.x = (((a.x + b0.x) + b1.x) + b2.x) + b3.x; a.y = (((a.y + b0.y) + b1.y) + b2.y) + b3.y;
        a.z = (((a.z + b0.z) + b1.z) + b2.z) + b3.z; a.w = (((a.w + b0.w) + b1.w) + b2.w) + b3.w;
    }
    for (; s < splits; ++s) {
        const float4 b = part[s * per + e];
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    const int lane = (int)(e & 63), vq = (int)(e >> 6) & 3;
    const int q = (int)(e >> 8), t = q % TM, wt = q / TM, wave = wt & 3, tile = tile0 + (wt >> 2);
    const int col = (tile % tiles_c) * MID_COLS + 32 * wave + 8 * vq + 4 * (lane >> 5);
    const int m = (tile / tiles_c) * (32 * TM) + 32 * t + (lane & 31);
    if (m < M && col < cols) *reinterpret_cast<uint2*>(out + (size_t)m * cols + col) = make_uint2(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w));
}

template <int TM, bool WIDE, bool ODD>
hipError_t launch_mid_fwd(const MidParams& p, unsigned grid, hipStream_t st) {
    constexpr int sh = FwdLds<TM, WIDE, ODD>::BYTES;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mid_fwd_kernel<TM, WIDE, ODD>), hipFuncAttributeMaxDynamicSharedMemorySize, sh);
    if (attr != hipSuccess) return attr;
    mid_fwd_kernel<TM, WIDE, ODD><<<dim3(grid), dim3(MID_THREADS), sh, st>>>(p);
    return hipGetLastError();
}

template <int TM, bool WIDE>
hipError_t launch_mid_fwd_any(const MidParams& p, hipStream_t st) {
    const unsigned grid = (unsigned)(p.ntiles * p.splits);
    return (p.G & 1) ? launch_mid_fwd<TM, WIDE, true>(p, grid, st) : launch_mid_fwd<TM, WIDE, false>(p, grid, st);
}

template <int TM, bool WIDE, bool SHARED>
hipError_t launch_mid_bwd(const MidParams& p, unsigned grid, hipStream_t st) {
    using L = BwdLds<TM, WIDE>;
    constexpr int most = L::TAB0 + 2 * 64 * (WIDE ? 64 : 16);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mid_bwd_kernel<TM, WIDE, SHARED>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (attr != hipSuccess) return attr;
    const int sh = SHARED ? L::TAB0 + p.C * kTableStride * 4 : most;
    static_assert(kMidLutBooks * kTableStride * 4 <= 2 * 64 * 64, "either table scheme fits the region");
    mid_bwd_kernel<TM, WIDE, SHARED><<<dim3(grid), dim3(MID_THREADS), sh, st>>>(p);
    return hipGetLastError();
}

template <int TM, bool WIDE>
hipError_t launch_mid_variant(const MidParams& p, int op, hipStream_t st) {
    const unsigned grid = (unsigned)(p.ntiles * p.splits);
    if (op == 0) {
        return launch_mid_fwd_any<TM, WIDE>(p, st);
    } else {
        const bool shared = WIDE && p.C <= kMidLutBooks;
        const hipError_t e = shared ? launch_mid_bwd<TM, WIDE, WIDE>(p, grid, st) : launch_mid_bwd<TM, WIDE, false>(p, grid, st);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace

// ---- which calls take these kernels, with which tile height and how many splits: the shortest estimated time.  The
// estimate of a plan is a launch cost, the steps of a workgroup times the time of a step, a cost per round of workgroups,
// and with splits the partial tiles' way out and back.  A step takes `solo` us while its compute unit has few workgroups
// and `share` us per resident workgroup once their instructions fill it.  The figures are fits to timings of every height
// with 1 to 24 splits (8 shapes from 1024 x 1024 to 5120 x 13824, an odd group count among them, 24 to 2048 tokens; calls
// repeated on two sets of buffers, without a rank-r term).  Forward: 5040 timings, rms error 8 %, the plan picked within
// 0.4 to 0.9 % of the best one measured on average.  Input gradient: 5721, 7 - 8 %, 0.4 to 0.7 %.  The 256-column kernels'
// time is compared with it: they win once their tiles fill the chip.  Forward, 4096 x 4096, 2048
// tokens: 50/50 % of 1-/2-bit rows 72 us against 73 here, 50/25/25 % of 1-/2-/4-bit rows 96 against 88; input gradient 80
// against 94, and with 4-bit rows level (98.6), from about 1000 tokens on.
// The 256-column input gradient is taken as rounds of workgroups, each with a fixed part (prologue, pipeline fill, output), its
// steps, those outside the pipeline 2.4 times as long, and the partial tiles: 896 timings of PATH_GEMM at each mix (72 to 5120
// channels, 256 to 13824 features, 257 to 4096 tokens), rms error 6 % and 5 %.  As a launch and steps of one length (rms error 45 %)
// it was put at less than half its time for few channels and for K % 256 != 0: 264 x 5504, 3072 tokens took 62 us where 128-column
// tiles take 30, 4096 x 4160, 2048 tokens 228 for 117.
constexpr int kHeights = 5;
static const int kMidHeight[kHeights] = {1, 2, 3, 4, 6};              // TM: 32 tokens each
struct MidCost {
    double solo[kHeights], share[kHeights];  // us per step (64 of the contraction)
    double launch, round, split, per_byte;   // us per call; per round of workgroups; more when split; per byte of partial tiles
};
static const MidCost kMidCost[2][3] = {
    // forward: 1- and 2-bit rows only; with 4-bit rows, up to kMidLutBooks codebooks; with 4-bit rows, more codebooks
    {{{0.35, 0.34, 0.43, 0.52, 0.70}, {0.23, 0.29, 0.36, 0.43, 0.57}, 3.6, 0.3, 3.2, 3.5e-7},
     {{0.46, 0.51, 0.61, 0.69, 0.81}, {0.35, 0.41, 0.47, 0.54, 0.74}, 5.6, 0.1, 2.9, 3.1e-7},
     {{0.46, 0.53, 0.61, 0.68, 0.80}, {0.33, 0.42, 0.47, 0.57, 0.81}, 5.4, 0.3, 3.2, 2.9e-7}},
    // input gradient
    {{{0.56, 0.61, 0.71, 0.89, 0.98}, {0.38, 0.46, 0.51, 0.63, 0.87}, 4.5, 0.1, 2.9, 4.2e-7},
     {{0.56, 0.73, 0.82, 0.90, 1.13}, {0.46, 0.56, 0.62, 0.71, 1.13}, 5.4, 1.0, 2.9, 3.3e-7},
     {{0.69, 0.69, 0.80, 0.92, 1.37}, {0.53, 0.54, 0.66, 0.50, 1.29}, 5.5, 1.0, 2.2, 3.9e-7}}};
// The 256-column kernels, by class as above.  Forward: us per call, us per step of a 256 x 256 tile.  Input gradient: us per call,
// per round of workgroups, per step in the pipeline and in general form, more when split, per byte of partial tiles (with more
// codebooks: the earlier fit, a launch and steps).
static const double kBigFwd[3][2] = {{5.0, 1.29}, {10.7, 1.70}, {11.6, 1.73}};
struct BigBwdCost { double launch, round, pipelined, general, split, per_byte; };
static const BigBwdCost kBigBwd[3] = {{0.0, 14.2, 1.41, 3.33, 3.3, 1.8e-7}, {0.0, 13.1, 2.07, 2.07, 2.3, 2.1e-7}, {6.9, 0.0, 2.72, 2.72, 5.0, 3.9e-7}};
// Workgroups per compute unit that the fits were made with: what the kernels hold by registers and LDS, by class as above.
static const int kMidResident[2][3][kHeights] = {{{5, 4, 3, 2, 1}, {4, 3, 2, 2, 1}, {4, 3, 2, 2, 1}}, {{3, 2, 2, 2, 1}, {3, 2, 2, 2, 1}, {2, 2, 2, 1, 1}}};

static std::atomic<int> g_mid_forced{0};                              // rows << 8 | splits
void force_mid_plan(int rows, int splits) { g_mid_forced.store(rows << 8 | splits); }

MidPlan plan_mid(int op, int N, int K, int M, bool wide, int C, size_t part_bytes) {
    MidPlan best{0, 0, 0, 0, 0};
    const int cols = op == 0 ? N : K, unit = op == 0 ? 4 : 1;         // steps that a split takes as a whole
    const int units = op == 0 ? (K / 64 + 3) / 4 : (N + 63) / 64;
    const int tiles_c = (cols + kMidCols - 1) / kMidCols, cus = device_compute_units();
    const size_t cap = std::min(part_bytes, kMidPartMax);
    if (const int forced = g_mid_forced.load()) {
        const int TM = (forced >> 8) / 32, per = (units + (forced & 255) - 1) / (forced & 255);
        best = MidPlan{TM, tiles_c, (M + 32 * TM - 1) / (32 * TM), (units + per - 1) / per, per};
        if (best.splits > 1 && mid_part_bytes(best) > cap) { best.splits = 1; best.per_split = units; }
        return best;
    }
    if ((long long)tiles_c * ((M + 127) / 128) > 16LL * cus) return best;   // far beyond what is compared below
    const int cls = !wide ? 0 : C <= kMidLutBooks ? 1 : 2;
    const MidCost& mc = kMidCost[op][cls];
    double best_t = 1e300;
    for (int i = 0; i < kHeights && (i == 0 || 32 * kMidHeight[i - 1] < M); ++i) {
        const int TM = kMidHeight[i];
        MidPlan pl{TM, tiles_c, (M + 32 * TM - 1) / (32 * TM), 0, 0};
        const int res = kMidResident[op][cls][i];
        for (int S = 1; S <= kMidMaxSplits && S <= units; S += S < 6 ? 1 : S < 12 ? 2 : 4) {
            pl.per_split = (units + S - 1) / S;
            pl.splits = (units + pl.per_split - 1) / pl.per_split;
            if (pl.splits > 1 && mid_part_bytes(pl) > cap) break;
            const long long wgs = (long long)pl.tiles_c * pl.tiles_m * pl.splits, n = (wgs + cus - 1) / cus;
            auto step = [&](long long k) { return k ? std::max(mc.solo[i], (double)k * mc.share[i]) : 0.0; };
            double t = mc.launch + (double)pl.per_split * unit * ((double)(n / res) * step(res) + step(n % res)) + (double)((n + res - 1) / res) * mc.round;
            if (pl.splits > 1) t += mc.split + (double)mid_part_bytes(pl) * mc.per_byte;
            if (t < best_t * (1.0 - 1e-9)) { best_t = t; best = pl; }
        }
    }
    // About level: the 256-column kernels need no partial tiles.  Input gradient: of 13464 calls 1063 change kernel by the costs above,
    // 989 away from 256 columns at 0.75 times the time on average, 74 to them level; 35 take over 3 % longer, 40 with 1.02 here.
    const double kLevel = op == 0 || cls == 2 ? 1.02 : 1.04;
    double big_t;
    if (op == 0) {
        const double launch = kBigFwd[cls][0], step = kBigFwd[cls][1];
        big_t = launch + step * gemm_fwd_steps(N, K, M, (kLevel * best_t - launch) / step);
    } else {
        const BigBwdCost& bc = kBigBwd[cls];
        const BwdWork w = gemm_bwd_work(N, K, M, wide);
        big_t = bc.launch + w.rounds * bc.round + w.pipelined * bc.pipelined + w.general * bc.general;
        if (w.part_bytes > 0.0) big_t += bc.split + w.part_bytes * bc.per_byte;
    }
    if (big_t <= kLevel * best_t) best = MidPlan{0, 0, 0, 0, 0};
    return best;
}

hipError_t launch_gemm_mid(const MidParams& p_in, int op, int TM, bool wide, hipStream_t st) {
    MidParams p = p_in;
    const int tiles = p.tiles_c * p.tiles_m, cols = op == 0 ? p.N : p.K;
    const int fit = p.splits > 1 ? (int)std::min<size_t>(p.part_bytes / mid_tile_bytes(p.splits, TM), (size_t)tiles) : tiles;
    if (fit < 1) return hipErrorInvalidValue;
    const int pieces = (tiles + fit - 1) / fit, per = (tiles + pieces - 1) / pieces;     // equal ones: a short last one costs as much
    for (p.tile0 = 0; p.tile0 < tiles; p.tile0 += per) {
        p.ntiles = std::min(per, tiles - p.tile0);
        hipError_t e = hipErrorInvalidValue;
        if (TM == 1) e = wide ? launch_mid_variant<1, true>(p, op, st) : launch_mid_variant<1, false>(p, op, st);
        if (TM == 2) e = wide ? launch_mid_variant<2, true>(p, op, st) : launch_mid_variant<2, false>(p, op, st);
        if (TM == 3) e = wide ? launch_mid_variant<3, true>(p, op, st) : launch_mid_variant<3, false>(p, op, st);
        if (TM == 4) e = wide ? launch_mid_variant<4, true>(p, op, st) : launch_mid_variant<4, false>(p, op, st);
        if (TM == 6) e = wide ? launch_mid_variant<6, true>(p, op, st) : launch_mid_variant<6, false>(p, op, st);
        if (e != hipSuccess) return e;
        if (p.splits <= 1) continue;
        mid_sum_kernel<<<dim3((unsigned)((size_t)p.ntiles * TM * 4)), dim3(256), 0, st>>>(reinterpret_cast<const float4*>(p.part), p.splits, p.ntiles, p.tile0,
                                                                                         p.tiles_c, TM, p.M, cols, p.out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lowra
