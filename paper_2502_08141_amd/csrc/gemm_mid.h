// The mid-token fused GEMMs (gemm_mid.hip): parameters and plan.
#pragma once
#include "gemm_common.h"

namespace lowra {

constexpr int kMidCols = 128;            // output columns per workgroup
constexpr int kMidMaxSplits = 32;
static_assert(kMidMaxSplits * 192 * kMidCols * sizeof(float) <= kMidTileMax, "32 TM = 192 rows at most");
constexpr int kMidLutBooks = 64;         // codebooks the input gradient keeps in LDS as a whole (more: a step's 64 rows are staged)

struct MidParams {
    const RowInfo* rows;
    const uint8_t* packed;
    const void* absmax;          // fp32, or bf16 with scale_bf16
    const float* mappings;
    const uint16_t* act;         // x [M,K] or dY [M,N]
    const uint16_t* ext_act;     // s x A^T or s dY B, bf16 [M,RP]
    const uint16_t* lora;        // B [N,r] (forward) or A [r,K] (input gradient)
    uint16_t* out;               // y [M,N] or dX [M,K]
    float* part;                 // splits > 1: fp32 partial tiles of the launch's tiles
    size_t part_bytes;           // room there
    int M, N, K, G, C, r, RP, scale_bf16;
    int tiles_c, tiles_m;        // output tiles: 128 columns x 32 TM tokens
    int tile0, ntiles;           // this launch: tiles [tile0, tile0 + ntiles) of them
    int splits, per_split;       // workgroups per output tile; contraction steps of each (forward: 256 features; input gradient: 64 channels)
};

struct MidPlan { int TM, tiles_c, tiles_m, splits, per_split; };         // TM == 0: the call belongs to another kernel
// contraction steps of a whole 256 x 256 tile that the 256-column forward's plan comes to (any value above `enough` may stand
// for a larger one)
double gemm_fwd_steps(int N, int K, int M, double enough);
BwdWork gemm_bwd_work(int N, int K, int M, bool any4);
BwdSplitPlan gemm_bwd_split_plan(int N, int K, int M);
MidPlan plan_mid(int op, int N, int K, int M, bool wide, int C, size_t part_bytes);
void force_mid_plan(int rows, int splits);         // lowra_set_mid_tiling; 0, 0: the planner
inline size_t mid_tile_bytes(int splits, int TM) { return (size_t)splits * TM * (32 * kMidCols * sizeof(float)); }
inline size_t mid_part_bytes(const MidPlan& pl) { return mid_tile_bytes(pl.splits, pl.TM) * pl.tiles_c * pl.tiles_m; }
// With room for some of a plan's partial tiles only, as many output tiles as fit can be computed and summed at a time: the
// same sums in the same order.  At most kMidPieces such pieces (0: more would be needed).  Only for calls that promise the
// bits of the whole plan: a piece fills a part of the chip only, and fewer splits are the better plan for the time (half the
// room: 1.2x, a third 1.5x, an eighth up to 4x).
constexpr int kMidPieces = 3;
inline int mid_pieces(const MidPlan& pl, size_t room) {
    const size_t fit = room / mid_tile_bytes(pl.splits, pl.TM), tiles = (size_t)pl.tiles_c * pl.tiles_m;
    return fit == 0 || (tiles + fit - 1) / fit > (size_t)kMidPieces ? 0 : (int)((tiles + fit - 1) / fit);
}

hipError_t launch_gemm_mid(const MidParams& p, int op, int TM, bool wide, hipStream_t st);

}  // namespace lowra
