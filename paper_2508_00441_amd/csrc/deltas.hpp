// Operand::deltas from Operand::exps: by a launch of its own (launch_deltas), or by the one pass where it finds vectors off the ladder.
#pragma once
#include <string.h>

#include "layout.hpp"

namespace ozaki {

struct DeltaOperand {
    const int32_t* exps;
    int32_t* deltas;
    const int32_t* l1;
    int32_t* bounds;
    const uint8_t* off_ladder;
    int64_t rows, rows_pad;
};
// The first tiles_first workgroups of a block's belong to the first operand, the rest to the second.
struct DeltaArgs {
    DeltaOperand o[2];
    unsigned tiles_first, tiles;
    int s, b;
};

inline DeltaArgs delta_args(const Plan& pl, const Operand* op0, const Operand* op1) {
    DeltaArgs a;
    memset(&a, 0, sizeof(a));
    const Operand* ops[2] = {op0, op1};
    for (int i = 0; i < 2; ++i)
        if (ops[i] != nullptr && ops[i]->rows > 0)
            a.o[i] = DeltaOperand{ops[i]->exps, ops[i]->deltas, ops[i]->l1, ops[i]->bounds, ops[i]->off_ladder, ops[i]->rows, ops[i]->rows_pad};
    a.tiles_first = (unsigned)(a.o[0].rows_pad / TILE);
    a.tiles = a.tiles_first + (unsigned)(a.o[1].rows_pad / TILE);
    a.s = pl.s; a.b = pl.b;
    return a;
}

#if defined(__HIPCC__)
// 256 threads, 256 vectors of block t, one half-wave per group of 32 vectors: is c_p - c_(p+1) the same for all real vectors of the group?
__device__ __forceinline__ void fill_delta(const DeltaArgs& a, unsigned tile_index, int64_t t, int p) {
    const bool second = tile_index >= a.tiles_first;
    const DeltaOperand& o = a.o[second ? 1 : 0];
    const int64_t row = (int64_t)(tile_index - (second ? a.tiles_first : 0u)) * TILE + threadIdx.x;
    const int lane = threadIdx.x & 63, half = lane & 32;
    const int32_t* const e = o.exps + ((size_t)t * a.s + p) * o.rows_pad + row;
    const bool last = p + 1 == a.s;
    const int d = last ? 0 : e[0] - e[o.rows_pad];
    // the first vector of a group is a real one, or the whole group is padding (then every d is 0)
    const int ref = __shfl(d, half, 64);
    const unsigned long long ok = __ballot(row >= o.rows || d == ref);
    const bool same = !last && (uint32_t)(ok >> half) == 0xFFFFFFFFu;
    if ((lane & 31) == 0) o.deltas[((size_t)t * a.s + p) * (o.rows_pad / LINK_ROWS) + row / LINK_ROWS] = same ? ref : DELTA_IRREGULAR;
}
#endif

}  // namespace ozaki
