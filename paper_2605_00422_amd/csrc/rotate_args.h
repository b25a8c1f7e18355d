// Arguments of the rotation launches, and the roles of the workgroups behind the rotation's own.
#pragma once
#include "rotate_common.h"
#include "psp_block_device.h"

struct RqArgs {
    const void* X; int64_t M, K; int n1, n2, r;
    const float* R1; const float* R2; const __half* U;
    int8_t* q; float* scale; int32_t* qsum; float* T;
    int* counters; float* partials; int S;
    float* xs; float* pmax;  // split rotation: rotated values (M x K) and per-workgroup extremes (M x G x 2)
    float qmax;              // largest code: 2^(bits-1) - 1
    int tp;                  // row pitch of T (= r, or r + 1 for a layer with row shifts)
    float* tmode;            // T + (PSP rank): first of the entries the layer's mode adds to a row, or NULL
    int asym, shift;         // the layer's mode: asymmetric activation codes, row shift
    int64_t rot_blocks;      // workgroups below this index rotate token blockIdx.x, the rest project
    int JG;                  // projection workgroups per (token tile, slice): groups of rank tiles
    const uint16_t* R1p; const uint16_t* R2p;          // bf16 term planes of the factors
};

namespace {

// workgroup pb behind the rotation's own in a launch that adds up the partial tiles of the launch in front (a.S < 0)
__device__ __forceinline__ void psp_sum_at(const RqArgs& a, int pb) {
    const int W = a.r <= 16 ? 16 : a.r <= 32 ? 32 : 64;                // bwla_psp_prefill_tile_cols
    bwla_psp_sum_tiles(bwla_psp_tiles{a.partials, a.T, a.M, a.r, a.tp, -a.S, a.JG, W, (int)(gridDim.x - a.rot_blocks)}, pb);
}
// projection workgroup pb of a launch: slice fastest, then the group of rank tiles, then the token tile.  EITHER: or the role
// above, in one kernel, told apart by a word that both load anyway (56 bytes more of arguments cost small launches 0.1 us).
template <bool BF16, bool EITHER = false>
__device__ __forceinline__ void psp_block_at(char* lds, const RqArgs& a, int pb, bool finish = true) {
    if (EITHER && a.S < 0) {
        psp_sum_at(a, pb);
        return;
    }
    const int s = pb % a.S, rest = pb / a.S;
    psp_block<BF16>(lds, a.X, a.M, a.K, a.r, a.U, a.T, a.counters, a.partials, a.S, rest / a.JG, s, a.tp, finish,
                    rest % a.JG, a.JG);
}

}  // namespace
