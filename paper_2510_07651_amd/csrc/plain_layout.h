// Where the general path's kernels find the logits of a piece (host and device: a test walks every address that is asked for).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace obc {

// What one launch works on: KV heads bg0 .. bg0 + gridDim.z - 1, their window rows r0 .. r0 + nr - 1 (of the G*W rows
// that share the KV head), tokens s0 .. s1 - 1.  Buffers of the group are indexed from (bg0, r0, s0).
struct Piece {
    int bg0, r0, nr, s0, s1;
    int z_stride;                // floats between the logits of consecutive rows
};

// Floats ahead of the 16 x 16 logits of a row block and of the 16 tokens from `token` on (score_fixed.h):
//   z       [head][row / 16][token / 16][token % 16 / 4][row % 16][token % 4]
__host__ __device__ inline size_t z_block(const Piece &w, int hl, int row_block, int token) {
    return (((size_t)hl * ((w.nr + 15) / 16) + row_block) * (w.z_stride / 16) + (token - w.s0) / 16) * 256;
}

// The 16 tokens whose logits a wave of fixed_score fetches while it works on those from t0 + p0 on, one of `part_tokens` of its own in each
// tile: those it scores next, and behind its last ones, where nothing is scored any more, the same again.
__host__ __device__ inline int next_scored(int t0, int p0, int part, int part_tokens, int tile, int t_end) {
    if (p0 + 16 < (part + 1) * part_tokens) return t0 + p0 + 16;
    return t0 + tile < t_end ? t0 + tile + part * part_tokens : t0 + p0;
}

}  // namespace obc
