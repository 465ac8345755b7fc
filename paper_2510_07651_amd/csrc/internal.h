// Internal declarations shared by the translation units of libobcache (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "obcache.h"

namespace obc {

// True lengths travel to the kernels by value (kernel-argument memory), so the
// library needs no device allocation and no host-to-device copy of its own.
template <int kMost>
struct SeqLensOf {
    int32_t len[kMost];
};
using SeqLens = SeqLensOf<OBC_MAX_RAGGED_BATCH>;
// Kernels take the lengths as a template type.  Half a KB of kernel arguments costs the host 1.7 us per launch (4.5 us
// against 2.8 us), as much as everything else, so equal lengths and batches of up to kFewLens travel in 32 bytes.
constexpr int kFewLens = 8;
template <typename Launch>
inline hipError_t with_lens(int ragged, int B, const SeqLens &lens, Launch &&launch) {
    if (ragged && B > kFewLens) return launch(lens);
    SeqLensOf<kFewLens> few = {};
    for (int b = 0; ragged && b < B; ++b) few.len[b] = lens.len[b];
    return launch(few);
}

// An eviction step closes the gap in pieces of 32 KB of rows and of 2048 scores, each by a workgroup of its own.  The last row
// of a piece moves up from the first place of the next one, which that one's workgroup overwrites: the scoring kernels
// put those rows and scores aside.
constexpr int kEvictPiece = 2048;     // 16-byte words of K or V, scores
struct EvictEdges {
    uint4 *rows;                      // [B*Hkv][K, V][evict_row_pieces][row]: rows that begin a piece
    float *scores;                    // [B*Hkv][evict_score_pieces]: scores that do
};
__host__ __device__ constexpr int evict_piece_rows(int d) { return kEvictPiece / (d / 8); }        // (bf16)
__host__ __device__ inline int evict_row_pieces(int N, int d) { return (N + evict_piece_rows(d) - 1) / evict_piece_rows(d); }
__host__ __device__ inline int evict_score_pieces(int N) { return (N + kEvictPiece - 1) / kEvictPiece; }

struct ScoreArgs {
    const void *q, *k, *v;
    float *scores;
    int B, N, W, Hq, Hkv, d, G;
    int variant;      // obc_variant_t
    int dtype;        // obc_dtype_t
    int ragged;       // 0: every sequence has length N
    int stage_mask;   // OBC_STAGE_* bits to run
    int accumulate;   // 1: add to the scores already in `scores` (positions beyond the true length untouched)
    int find_lowest;  // 1 (decode path only): every wave reports its lowest-scored token among evict_first <= p < len - evict_tail
    int evict_first, evict_tail;
    EvictEdges edges; // with find_lowest: what the decode kernels leave for launch_evict_pieces
    SeqLens lens;     // valid for b < B when ragged
};

// Workspace carve-up for obc_score; offsets in bytes from a 256-byte aligned base.
struct ScoreWorkspace {
    size_t out_bf16;   // bf16  [2][B*Hkv*m_pad*d]  o_i as two bf16 pieces (high, residual); rows of a KV head padded to a multiple of 32
    size_t row_const;  // float [B*Hkv*m_pad*4]  per padded row: 2*(max + log2 sum) in log2 units, ||o||^2, last visible key, spare
    size_t part_ml;    // float [Hkv*records*m_pad*4]  per sequence split: row max (raw q.k), row sum, spare x2
    size_t special;    // float [B*Hkv*m_pad*4]  per padded row: separately scored top key (token or -1) and its value/key/joint terms
    size_t part_o;     // float [Hkv*records*m_pad*d]  per sequence split: unnormalised output
    size_t planes;     // float [n_chunks*nv*B*Hkv*N]   per row-chunk partial scores (only when n_chunks > 1)
    size_t total;
    int m_pad;         // padded rows per KV head (multiple of 32)
    int n_chunks;      // row chunks of 128 rows per KV head
    int splits;        // sequence splits in the first sweep
    int records;       // splits of all sequences together there is room for
    int split_len;     // tokens per split (multiple of 64)
    int range_len;     // tokens per workgroup in the second sweep (multiple of 64)
    int use_mfma;      // 1: bf16 matrix-core path, 0: general path
    size_t z;          // float [B*Hkv*rows*z_stride]  raw q.k, kept by the first sweep when keep_z
    int keep_z, z_stride;
    int once1, once2;  // 1: the first, the second sweep marks K and V as read once (see reads_once)
    int use_wide;      // 1: the second sweep runs in its register-blocked form (score_mfma_wide.hip)
    int solo;          // 1: there the last chunk has at most 64 rows and goes to mfma_sweep2_solo, in ranges of range_solo
    int range_solo;
    // General path: see score_plain.hip.  One piece of the work is `pl_heads` KV heads x `pl_rows` window rows x
    // `pl_seg` tokens; its buffers are reused by the next one.
    size_t pl_z;       // float [heads*rows*seg]     scaled logits
    size_t pl_best;    // float2 [heads*rows*ranges] largest visible logit of a token range, lowest token attaining it
    size_t pl_records; // RowRecord [heads*rows]
    size_t pl_out;     // float [heads*rows*d]       o_i = sum_p A_ip v_p
    size_t pl_o_digits;  // int8 [heads*rows][5][d]  o_i in fixed point (score_fixed.h)
    size_t pl_part_l;  // float [heads*splits*rows]  sum of exp(z - max) of a split, without the row's top token; with pl_digits float4: the
                       // split's own largest logit, the sum without its own top token, that token
    size_t pl_part_o;  // float [heads*splits*rows*d]  unnormalised output of a split, likewise
    int pl_heads, pl_rows, pl_seg, pl_z_stride, pl_short, pl_digits;
    int pl_sweep_rows; // with pl_digits: rows of a workgroup of digit_sweep, 64 or 128
    int pl_range, pl_ranges;   // tokens per range, ranges
    int pl_split, pl_splits;   // tokens per split (a multiple of 64), splits
    // Decode path (one window row per query head): see score_decode.hip.
    size_t dec_z;      // float [B*Hkv*N*dec_rows]  scaled logits, token-major
    size_t dec_head;   // float4 [B*Hkv*dec_splits*dec_rows]  per-range partial records, their vectors below
    size_t dec_vec;    // float [B*Hkv*dec_splits*dec_rows*2d]
    size_t dec_lowest; // uint64 [B*Hkv*dec_lowest_per_head]  evict_candidates of the scoring kernel's waves
    int dec_lowest_per_head;
    size_t dec_edges, dec_edge_scores;   // EvictEdges, last: a call that evicts nothing does without them
    size_t score_need; // bytes such a call needs
    size_t dec_final;  // float [B*Hkv*dec_rows*(2d+4)]  merged row records
    int use_decode;    // 1: decode path (takes precedence over the other two)
    int dec_rows;      // query heads per KV head, padded to 1, 2, 4 or 8
    int dec_range;     // tokens per workgroup (multiple of 32)
    int dec_splits;    // ranges per KV head
    int dec_merge_inline;  // 1: the scoring kernel merges the ranges itself
};

constexpr int kDecodeMaxGroup = 8;   // query heads per KV head the decode path is built for

// Sweep-1 split count and sweep-2 token range forced through obc_set_score_tuning (0: automatic).
int tuned_splits();
int tuned_range();
int tuned_sweep2_form();     // 0: by shape, 1: 32 rows per wave, 2: 64 rows per wave where the variant has a cross term

// `cap`: bytes the plan should stay within where it has a choice (0: what is best).
constexpr size_t kPlainWorkspace = (size_t)96 << 20;      // of the general path, which works in pieces
int plan_score_workspace(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int variant, ScoreWorkspace *ws, size_t cap = 0);
// Adds the general path's buffers to the plan, advancing *off (bytes).
void plain_plan(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int variant, size_t cap, ScoreWorkspace *ws, size_t *off);
// Adds the matrix-core path's buffers to the plan, advancing *off (bytes).
void mfma_plan(int B, int N, int W, int Hq, int Hkv, int d, int variant, ScoreWorkspace *ws, size_t *off);

// Decode path: whether it covers the shape, its buffers (advancing *off), its launcher.
bool decode_path_covers(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int variant, bool any_size);
void decode_plan(int B, int N, int Hq, int Hkv, int d, ScoreWorkspace *ws, size_t *off);
hipError_t launch_score_decode(const ScoreArgs &a, const ScoreWorkspace &ws, char *ws_base, hipStream_t stream);

// Launchers.  Each enqueues on `stream` and returns hipSuccess or the launch error.
hipError_t launch_score_plain(const ScoreArgs &a, const ScoreWorkspace &ws, char *ws_base, hipStream_t stream);
hipError_t launch_score_mfma(const ScoreArgs &a, const ScoreWorkspace &ws, char *ws_base, hipStream_t stream);
// Register-blocked second sweep: whether it serves the variant, and its launcher (same arguments and outputs as the
// 32-rows-per-wave kernel it stands in for).
bool sweep2_wide_covers(int variant);
hipError_t launch_sweep2_wide(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, float *dst, size_t plane_elems,
                              size_t chunk_stride, hipStream_t stream);
hipError_t launch_select(const float *scores, int budget, int32_t *keep_idx, int B, int Hkv, int N, int ragged,
                         const SeqLens &lens, int first, int tail, int radius, void *workspace,
                         size_t workspace_bytes, hipStream_t stream);
size_t select_adaptive_workspace_bytes(int B, int Hkv, int N);
hipError_t launch_select_adaptive(const float *scores, int budget, int n_safe, int cap, int32_t *keep_idx,
                                  int32_t *counts, int B, int Hkv, int N, int ragged, const SeqLens &lens,
                                  void *workspace, hipStream_t stream);
size_t select_workspace_bytes(int B, int Hkv, int N, bool pooled);
bool select_prefers_slices(int B, int Hkv, int N);
hipError_t launch_compact(const void *k, const void *v, const int32_t *keep_idx, void *k_out, void *v_out, int B,
                          int Hkv, int N, int budget, int row_bytes, hipStream_t stream);
hipError_t launch_compact_in_place(void *k, void *v, float *scores, const int32_t *keep_idx, int B, int Hkv, int N,
                                   int budget, int row_bytes, hipStream_t stream);
// Evict-one of a decoding step: the lowest-scored token of each (sequence, KV head) among first <= p < len - tail (ties:
// the highest index) leaves k, v and scores, the gap is closed, and its position goes to `evicted` if that is not NULL.
// `lowest` [B*Hkv]: scratch for the candidates.
hipError_t launch_evict_one(void *k, void *v, float *scores, int32_t *evicted, unsigned long long *lowest, int B, int Hkv, int N,
                            int ragged, const SeqLens &lens, int first, int tail, int row_bytes, hipStream_t stream);
// The same after the decode kernels, which have left the candidates and the pieces' edges.  bf16 rows.
hipError_t launch_evict_pieces(void *k, void *v, float *scores, int32_t *evicted, const unsigned long long *lowest, int n_lowest,
                               const EvictEdges &edges, int B, int Hkv, int N, int ragged, const SeqLens &lens, int row_bytes,
                               hipStream_t stream);
hipError_t launch_gather_scores(const float *in, const int32_t *keep_idx, float *out, int BH, int N, int budget,
                                 int n_out, hipStream_t stream);
hipError_t launch_stream_read(const void *src, size_t bytes, uint32_t *sink, int blocks, hipStream_t stream);

template <typename Lens>
__device__ __forceinline__ int seq_len_of(const Lens &lens, int ragged, int b, int N) {
    return ragged ? lens.len[b] : N;
}

// A token that may be evicted, packed so that one unsigned minimum picks the lowest score and the highest index among
// equals (a protected selection of all but one competing token keeps the lower index).  Scores are ordered as the
// selection kernels order them: -0 folded onto +0, NaN lowest.
__device__ __forceinline__ unsigned long long evict_candidate(float score, int p) {
    uint32_t u = __float_as_uint(score);
    if (u == 0x80000000u) u = 0u;
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    if (score != score) u = 0u;
    return ((unsigned long long)u << 32) | (uint32_t)~p;
}
__device__ __forceinline__ int evict_candidate_token(unsigned long long c) { return (int)~(uint32_t)c; }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t h) {
    return __uint_as_float(((uint32_t)h) << 16);
}

}  // namespace obc
