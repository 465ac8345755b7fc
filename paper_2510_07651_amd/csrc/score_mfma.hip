// Matrix-core scoring path for bf16 caches with head_dim 128 (gfx950, wave64).
//
// The scores of Eq. 4-6 need, for every (window row i, token p) pair, the softmax weight
// A_ip, the logit Z_ip and the cross term v_p . o_i, where A and o_i depend on sums over
// ALL tokens of the row (Section 3).  So the cache is swept twice:
//
//   sweep 1  (mfma_sweep1)   per (KV head, 128-row chunk, sequence split): S^T = K Q^T on
//            the matrix cores, online softmax per row, O^T += V^T P^T on the matrix cores;
//            emits a partial (row max, row sum, unnormalised O) per split.
//   combine  (mfma_combine, mfma_combine_hold)  merges the splits: final sum, o_i as a pair
//            of bf16 pieces, ||o_i||^2, and the constants the second sweep needs per row.
//   sweep 2  (mfma_sweep2)   per (KV head, chunk, token range): Z = Q K^T and the cross
//            terms O V^T on the matrix cores, with tokens on the lane axis of the
//            accumulators so that the sum over window rows and query heads (Eq. 9,
//            Appendix A.5) runs down registers; A^2 = exp2(2 log2e Z - 2 log2(max-shifted
//            sum)) and the three scores are formed in fp32.  The attention-only score
//            of Eq. 8 and its l1-weighted form need Z only and skip the cross terms.
//
// Both sweeps walk their tokens in blocks of 32.  Sweep 1 is software-pipelined inside a
// wave: while the vector ALUs turn block n's accumulators into softmax weights, the matrix
// cores already work on block n+1's K Q^T and on block n-1's P V product; the streams of
// one step are independent, and the instruction scheduler interleaves them.  Sweep 2 exists in
// two forms.  The one in this file gives a wave 32 rows, runs a block's matrix phase and vector
// phase back to back and leaves the overlap to the second wave
// on the SIMD (its stationary operands and row constants leave no registers for a second set of
// accumulators).  The register-blocked forms (score_mfma_wide.hip: 64 rows per wave, stationary
// operands in the accumulator file, the wave pipelined against itself) serve the key, joint and
// all-three variants.  K and V travel
// HBM -> LDS with direct-to-LDS loads: in sweep 1 as 32-token blocks through four-slot rings, three
// batches in flight; in sweep 2 as 64-token tiles, double-buffered here, a four-slot ring there.
//
// Precision.  The matrix cores take bf16 operands, and rows whose attention is
// concentrated on a few keys are sensitive to that rounding (the scores of those keys
// depend on v_p - o_i, a difference of nearly equal vectors).  Two operands are therefore
// fed as an exact-enough pair of bf16 pieces (high part + residual, 16 significant bits):
// the softmax weights P in O^T += V^T P^T, and o_i in the cross term O V^T.  Both pieces
// reuse the same LDS operand, so the cost is matrix-core issue slots only.
// ||v_p - o_i||^2 is evaluated as ||v_p||^2 - 2 v_p.o^_i + ||o^_i||^2 with o^_i the
// two-piece value used by the matrix cores in BOTH the cross term and the norm, so the
// expression is the exact squared distance to o^_i.
//
// Rows dominated by one key (an attention sink, the token's own key) would still lose
// v_p - o_i of that key to cancellation: o_i is then v_p plus a small remainder.  The first
// sweep therefore keeps, per row, the one key that may end up dominant out of its sums (a new
// running maximum that clears the old one by ln 9: no other key can reach a share of 0.9), and the
// combine step forms v_p - o_i = (1 - A_ip)(v_p - mean of the others) for that key directly.
// The (row, key) pair is scored there in fp32 when its share is large, and the second sweep
// skips it.  One pass serves every input: nothing is rescanned for rows that turn out dominated.
//
// A and Z never touch HBM.  All sums have a fixed order: results are bit-reproducible.
#include <algorithm>
#include <cfloat>

#include "internal.h"
#include "mfma_util.h"
#include "wave_util.h"

#include <type_traits>

namespace obc {
using namespace mfma;
namespace {

// ------------------------------------------------------------------------------------
// Sweep 1
// ------------------------------------------------------------------------------------
// Where a head's partial records start: every sequence has as many slots per head as it has live splits.
template <typename Lens>
__device__ __forceinline__ int split_slot(const Lens &lens, int ragged, int b, int g, int N, int Hkv, int split_len) {
    int before = 0, own = (N + split_len - 1) / split_len;
    if (ragged) {
        for (int i = 0; i < b; ++i) before += (lens.len[i] + split_len - 1) / split_len;
        own = (lens.len[b] + split_len - 1) / split_len;
    } else {
        before = b * own;
    }
    return before * Hkv + g * own;
}

struct Sweep1Regs {
    bf16x8 q[8];          // stationary B operand: this lane's query row, pieces 2 kk + half
    f32x16 oacc[4];       // O^T accumulators: head_dim block x 16 registers
    f32x16 s_cur;         // raw q.k of the block whose softmax is due
    PiecePair phi[2], plo[2];   // two-piece softmax weights of the previous block, per k-step
    float p[16];          // the same weights in fp32, from the step that formed them to the step that packs them
    float m_ref, m_true;  // reference of the running sums (raw q.k units, see kLazyRescale); true running max
    float lsum;           // this lane's share of the running sum
    float alpha;          // rescale of oacc still owed from the previous step (1 = none)
    bool rescale;         // uniform: some row of the wave owes a rescale
    // With kNeedO only: the row's candidate for a dominant key, kept out of lsum and oacc.
    float cand_val;       // its raw q.k (-inf: none yet)
    int cand_tok;         // its token (-1: none yet)
    int n_ev;             // former candidates parked in this lane's LDS list, to be added back at the end
};

// A key can end up with more than a share s of a row's attention only if its logit exceeds every
// other one by ln(s / (1 - s)); a new running maximum that clears the old one by less can never
// get there and stays an ordinary key.  The margin below is the one for s = 0.9: rows without a held
// key have no key above that share, which bounds the cancellation in v_p - o_i to a factor 10.
constexpr float kCandMargin = 2.1972245773362196f / kInvSqrtD;   // ln(0.9 / 0.1), in raw q.k units
constexpr float kSeparateShare = 0.5f;   // a candidate holding at least this share of its row is scored by the combine step
constexpr int kEvents = 4;               // former candidates a lane can park

// Adds a former candidate (token `tok`, raw logit `val`) back into this lane's sums: weight
// exp2((val - ref_l) c2) into lsum (one half-wave only, the halves are added at the end) and
// exp2((val - ref_o) c2) v_tok into the lane's 64 entries of O^T.
__device__ __forceinline__ void add_back_fetch(uint2 (&x)[16], const char *vh, int tok, int half) {
    const char *vrow = vh + (size_t)tok * kRowBytes;
#pragma unroll
    for (int ddb = 0; ddb < 4; ++ddb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) x[ddb * 4 + r4] = *(const uint2 *)(vrow + (ddb * 32 + 8 * r4 + 4 * half) * 2);
}

__device__ __forceinline__ void add_back_apply(Sweep1Regs &R, const uint2 (&x)[16], float val, float ref_l, float ref_o,
                                               int half) {
    const float c2 = kLog2e * kInvSqrtD;
    const float w_o = __builtin_amdgcn_exp2f((val - ref_o) * c2);
    if (half == 0) R.lsum += __builtin_amdgcn_exp2f((val - ref_l) * c2);
#pragma unroll
    for (int ddb = 0; ddb < 4; ++ddb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const uint2 w = x[ddb * 4 + r4];
            R.oacc[ddb][4 * r4 + 0] = fmaf(w_o, __uint_as_float(w.x << 16), R.oacc[ddb][4 * r4 + 0]);
            R.oacc[ddb][4 * r4 + 1] = fmaf(w_o, __uint_as_float(w.x & 0xffff0000u), R.oacc[ddb][4 * r4 + 1]);
            R.oacc[ddb][4 * r4 + 2] = fmaf(w_o, __uint_as_float(w.y << 16), R.oacc[ddb][4 * r4 + 2]);
            R.oacc[ddb][4 * r4 + 3] = fmaf(w_o, __uint_as_float(w.y & 0xffff0000u), R.oacc[ddb][4 * r4 + 3]);
        }
}

__device__ __forceinline__ void add_back(Sweep1Regs &R, const char *vh, int tok, float val, float ref_l, float ref_o,
                                         int half) {
    uint2 x[16];
    add_back_fetch(x, vh, tok, half);
    add_back_apply(R, x, val, ref_l, ref_o, half);
}

// P = hi + lo for the matrix cores: hi keeps the top 16 bits of the fp32 weight (a bf16 by truncation), lo is the
// exact remainder rounded to bf16.  The remainders come from a dot product of the packed pair with (-1, 0) and (0, -1), exact like
// the subtraction of one unpacked piece and one instruction less each.
__device__ __forceinline__ void pack_weights(Sweep1Regs &R) {
    union { uint32_t u; bf16x2 h; } first, second, pair;
    first.u = 0x0000bf80u;
    second.u = 0xbf800000u;
    asm("" : "+s"(first.u), "+s"(second.u));       // (in registers: written as the inline constant -1.0 the pair comes out as (0, -1))
#pragma unroll
    for (int sx = 0; sx < 2; ++sx)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p0 = R.p[8 * sx + 2 * e], p1 = R.p[8 * sx + 2 * e + 1];
            pair.u = __builtin_amdgcn_perm(__float_as_uint(p1), __float_as_uint(p0), 0x07060302u);     // {p0 >> 16, p1 >> 16}
            R.phi[sx].u[e] = pair.u;
            R.plo[sx].u[e] = pack_bf16(__builtin_amdgcn_fdot2_f32_bf16(pair.h, first.h, p0, false),
                                       __builtin_amdgcn_fdot2_f32_bf16(pair.h, second.h, p1, false));
        }
}

// The blocks a wave fetches one after the other from one tensor: two transfers of 1 KB each, rows 8 wave .. 8 wave + 7.  The second
// one's instruction offset moves its LDS and its memory address along, which its lane offset takes back, so that the LDS address
// register m0 is written once; kBias keeps the lane offsets from falling below zero.
struct BlockFetch {
    static constexpr int kBias = 1024;
    const char *at;          // kBias bytes ahead of the block that is fetched next (uniform)
    uint32_t off[2];         // per-lane byte offset inside the block (+ kBias, resp. + kBias - 1024)
    __device__ __forceinline__ void start(const char *head, int t0, const uint32_t (&doff)[2]) {
        at = head + (size_t)t0 * kRowBytes - kBias;
        off[0] = doff[0] + kBias;
        off[1] = doff[1];
    }
    // The block fetched from now on has rows 0 .. rmax only: rows past them re-read row rmax.
    __device__ __forceinline__ void cut(int rmax, int wave, int lane) {
        asm volatile("");    // (a branch that is hardly ever taken, not selects in every step)
#pragma unroll
        for (int n = 0; n < 2; ++n) off[n] -= (uint32_t)(max((wave * 2 + n) * 4 + (lane >> 4) - rmax, 0) * kRowBytes);
    }
    template <bool kOnce>
    __device__ __forceinline__ void fetch(uint32_t lds, bool more) {         // `more`: another block follows this one
        if constexpr (kOnce)
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %3 nt\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024 nt" ::"{m0}"(lds), "v"(off[0]), "v"(off[1]), "s"(at) : "memory");
        else
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\tglobal_load_lds_dwordx4 %2, %3 offset:1024" ::"{m0}"(lds), "v"(off[0]), "v"(off[1]), "s"(at) : "memory");
        at += more ? kBlkBytes : 0;
    }
};

// One pipeline step n of sweep 1 (PH = n mod 4 fixes every LDS slot at compile time):
//   matrix cores: O^T += V^T P^T of block n-1, S^T = K Q^T of block n+1
//   vector ALUs : online softmax of block n
// Every step first waits for the two blocks it reads, meets the other waves at a barrier and
// starts the loads of the blocks three steps ahead.
//
// With kNeedO (Eq. 5, 6) every row keeps its candidate for a dominant key (see kCandMargin) out of
// its sums.  The step is then cut in two: K Q^T and the block's row maxima first; a vote whether
// some row of the wave meets a new candidate in block n, and (rarely) the branch that deals with
// it; then V^T P^T and the weights.  Without kNeedO only the branch of the masks divides it.
template <int PH, bool kNeedO, bool kStoreZ, bool kOnce>
__device__ __forceinline__ void sweep1_step(Sweep1Regs &R, const char *smem, uint32_t lds0, int n, int t_begin,
                                            int t_end, int n_last, int n_cut, int rmax, int vis, int n_plain, BlockFetch &kf,
                                            BlockFetch &vf, const char *vh,
                                            const int (&koff)[8], const int (&voff)[4], int wave, int lane, bool wave_active,
                                            int2 *events, char *z_split, uint32_t z_off) {
    // K and V blocks live in rings of four 8 KB slots each (block j in slot j mod 4): K block
    // n+1 and V block n-1, both started three steps ago, are waited for here while the two
    // younger batches stay in flight; then K block n+4 and V block n+2 start in the slots
    // the previous step has finished with.  Past block `n_last` every batch has as many transfers, but they fetch
    // that block again, from the L2; nothing past the split's end counts (see mfma_sweep1).
    constexpr int kKBase = ((PH + 1) & 3) * kBlkBytes;                  // block n+1
    constexpr int kVBase = (4 + ((PH + 3) & 3)) * kBlkBytes;            // block n-1
    const float c2 = kLog2e * kInvSqrtD;
    const int half = lane >> 5;

    // (with kStoreZ the wave that has rows also has four stores per step in flight behind the loads of that step: from the
    // third step on the two younger batches are twice as long)
    constexpr int kBatch = kNeedO ? 4 : 2;
    if (kStoreZ && wave_active && n > 1 && n * 32 < t_end - t_begin) wait_async_loads_keep<2 * kBatch + 8>();
    else if (kStoreZ && wave_active && n == 1 && 32 < t_end - t_begin) wait_async_loads_keep<2 * kBatch + 4>();
    else wait_async_loads_keep<2 * kBatch>();
    __syncthreads();
    if (n + 4 == n_cut) kf.cut(rmax, wave, lane);                      // uniform: the sequence's last rows
    kf.fetch<kOnce>(lds0 + PH * kBlkBytes + wave * 2048, n + 4 < n_last);
    if (kNeedO) {
        if (n + 2 == n_cut) vf.cut(rmax, wave, lane);
        vf.fetch<kOnce>(lds0 + (4 + ((PH + 2) & 3)) * kBlkBytes + wave * 2048, n + 2 < n_last);
    }
    if (!wave_active) return;
    if (kStoreZ && n * 32 < t_end - t_begin && z_off != ~0u) {      // raw q.k of block n for score_few_rows
#pragma unroll
        for (int r = 0; r < 16; r += 4)
            *(float4 *)(z_split + n * 128 + 8 * r + z_off) = make_float4(R.s_cur[r], R.s_cur[r + 1], R.s_cur[r + 2], R.s_cur[r + 3]);
    }

    // Blocks that not every row of the wave sees in full.  (A branch in the step, not steps of their own: those were 2000
    // instructions that only the last split of a sequence ran, fetched for the first time at its very end: 3 us of 24 at 8 heads
    // x 8K.)
    if (n >= n_plain) {                                                // uniform
        const int tok0 = t_begin + n * 32 + 4 * half;  // register r holds token tok0 + 8 (r / 4) + r % 4
        const int past = min(vis, t_end - 1) - tok0;   // what lies past it is hidden
#pragma unroll
        for (int r = 0; r < 16; ++r) R.s_cur[r] = 8 * (r >> 2) + (r & 3) > past ? -INFINITY : R.s_cur[r];
    }

    // ---- matrix cores: block n+1 ----
    // (with kNeedO the operand reads of the whole chain are issued up front, so that one LDS latency is exposed
    // instead of one per pair of matrix ops, and the first value operands follow them ahead of the vote below)
    f32x16 s_next = zero16();
    bf16x8 ka[8], va0[4];
    if (kNeedO) {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) ka[kk] = lds_read16(smem + kKBase + koff[kk]);
#pragma unroll
        for (int ddb = 0; ddb < 4; ++ddb) va0[ddb] = lds_read_vt(smem + kVBase + voff[ddb]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        const bf16x8 a = kNeedO ? ka[kk] : lds_read16(smem + kKBase + koff[kk]);
        s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.q[kk], s_next, 0, 0, 0);
    }
    // ---- vector ALUs: block n-1's weights into operand form, in the shadow of the chain above (the second part of
    // the step, whose matrix ops they feed, has the exponentials of block n for company) ----
    if (kNeedO) {
        pack_weights(R);
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
#pragma unroll
            for (int e = 0; e < 4; ++e) {       // (pinned here: left alone, the packing sinks into the step's second part)
                asm volatile("" : "+v"(R.phi[sx].u[e]));
                asm volatile("" : "+v"(R.plo[sx].u[e]));
            }
#pragma unroll
        for (int i = 0; i < 8; ++i) {           // one matrix op, then its share of the packing
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
        }
    }
    // ---- vector ALUs: block n ----
    f32x16 s = R.s_cur;
    float mx = max3(s[0], s[1], s[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = max3(mx, s[r], s[r + 1]);
    mx = fmaxf(mx, s[15]);
    mx = halves_max(mx);
    if (kNeedO) {
        // Rows whose block maximum clears their running maximum (and the block's other keys) by the margin
        // take the block's first key of that logit as their candidate: its logit becomes -inf before the
        // weights are formed, so it never enters this block's P or sum, and the previous candidate is parked
        // (or, with the list full, added back on the spot).  (-inf + margin = -inf: in a row's first visible
        // block only the block's other keys decide.)
        const float m_true_before = R.m_true;
        if (R.rescale || __any(mx > m_true_before + kCandMargin)) {    // uniform; one branch for both rare events
            // The running max moved in the previous step: bring the accumulated O^T (blocks <= n-2)
            // to the new reference before block n-1, whose weights already use it, is added.
            if (R.rescale) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) R.oacc[i][r] *= R.alpha;
            }
            if (mx > m_true_before + kCandMargin) {
                uint32_t hit = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) hit |= s[r] == mx ? (1u << r) : 0u;
                // (a lane's registers ascend with their tokens: its lowest set bit is its first such key)
                const int rc_own = hit ? __builtin_ctz(hit) : 0;
                const int off_own = hit ? 8 * (rc_own >> 2) + 4 * half + (rc_own & 3) : 64;
                float off_lower, off_upper;
                both_halves(__int_as_float(off_own), off_lower, off_upper);      // (bits only)
                const int off_first = min(__float_as_int(off_lower), __float_as_int(off_upper));
                const int rc = off_own == off_first ? rc_own : -1;              // its register, if in this lane
                // It must clear the other keys of its own block by the margin as well.
                float others = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r) others = fmaxf(others, r == rc ? -INFINITY : s[r]);
                others = halves_max(others);
                if (mx > others + kCandMargin) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[r] = r == rc ? -INFINITY : s[r];
                    if (R.cand_tok >= 0) {                             // the previous candidate is an ordinary key after all
                        if (R.n_ev < kEvents) {
                            events[R.n_ev] = make_int2(R.cand_tok, __float_as_int(R.cand_val));
                            R.n_ev += 1;
                        } else {
                            // (sum and O^T both stand at the current reference: the owed rescale was applied above)
                            add_back(R, vh, R.cand_tok, R.cand_val, R.m_ref, R.m_ref, half);
                        }
                    }
                    R.cand_tok = t_begin + n * 32 + off_first;
                    R.cand_val = mx;
                }
            }
        }
        // ---- matrix cores: block n-1 ----
#pragma unroll
        for (int sx = 0; sx < 2; ++sx)
#pragma unroll
            for (int ddb = 0; ddb < 4; ++ddb) {
                const bf16x8 a = sx == 0 ? va0[ddb] : lds_read_vt(smem + kVBase + 16 * kRowBytes + voff[ddb]);
                R.oacc[ddb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.phi[sx].v, R.oacc[ddb], 0, 0, 0);
                R.oacc[ddb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.plo[sx].v, R.oacc[ddb], 0, 0, 0);
            }
    }
    // The reference may follow a candidate's logit: it only has to bound the weights from above.
    R.m_true = fmaxf(R.m_true, mx);
    const bool moved = mx > R.m_ref + kLazyRescale;                    // also true for the first visible key
    const float m_new = moved ? mx : R.m_ref;
    const float alpha = __builtin_amdgcn_exp2f((R.m_ref - m_new) * c2);      // 1 when the reference stays, 0 with the first visible key
    const float mref = m_new * c2;
    R.m_ref = m_new;
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        R.p[r] = __builtin_amdgcn_exp2f(fmaf(s[r], c2, -mref));
        psum += R.p[r];
    }
    R.lsum = fmaf(R.lsum, alpha, psum);
    if (kNeedO) {
        R.alpha = alpha;
        R.rescale = __any(moved);      // uniform and rare once the running max has settled
    }
    R.s_cur = s_next;
    if (kNeedO) {
        // second part: the remaining value operands first, then one matrix op per three vector ops (the exponentials go along)
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
    } else {
        interleave_hint<8, 12, 1>();
    }
}

// Grid: see sweep_part (a part is a sequence split).
// With kNeedO every row keeps its candidate for a dominant key (see kCandMargin) out of its sums and
// reports it with the partial record; the combine step then forms v_cand - o_i without
// cancellation for every row, and no row ever needs a second pass.
//
// Past its split's end the ring fetches the last block again: the next split's rows are three K and two V blocks from memory for
// nothing, a third of what a split of 256 tokens reads.  But splits of up to four blocks fetch on, to the sequence's end, where wide
// second sweeps follow: the kernel takes 12.2 us with the last block again and 11.5 so among whole calls (8 heads x 128 rows x 2048;
// alone, its keys in cache, 11.2 and 11.4).  Whole calls, joint, the last block again / on, us (sixteen loads of either build, each at an
// address of its own, which alone moves a call by up to 3 %):
//   four blocks   128 rows, 8 heads x 2048 27.2 / 25.6, x 4096 30.4 / 30.2   100 rows, 8 heads x 2049 29.0 / 27.9   112 rows, 4 heads x 4096 27.7 / 26.6
//                  64 rows, 8 heads x 4096 24.2 / 24.9                        64 rows, 4 heads x 8192 24.1 / 24.7
//   more          128 rows, 8 heads x 16384 52.7 / 52.8, 4 x 8 heads x 32K 256 / 255
constexpr int kFetchOnBlocks = 4, kFetchOnRows = 65;
template <bool kNeedO, bool kStoreZ, bool kOnce, typename Lens>
__global__ __launch_bounds__(kThreads, 2) void mfma_sweep1(const uint16_t *__restrict__ q,
                                                           const uint16_t *__restrict__ k,
                                                           const uint16_t *__restrict__ v, int N, int W, int Hq,
                                                           int Hkv, int ragged, Lens lens, int split_len,
                                                           int n_chunks, int m_pad, float *__restrict__ part_ml,
                                                           float *__restrict__ part_o, float *__restrict__ z, int z_stride) {
    __shared__ __attribute__((aligned(1024))) char smem[kLdsTiles];
    __shared__ int2 ev_list[kNeedO ? kThreads * kEvents : 1];   // per lane: parked former candidates (token, logit bits)
    int2 *events = ev_list + (kNeedO ? threadIdx.x * kEvents : 0);

    const SweepPart part = sweep_part(lens, ragged, N, Hkv, n_chunks, split_len);
    const int b = part.b, g = part.g, bg = b * Hkv + g, chunk = part.chunk, split = part.part, G = Hq / Hkv, M = G * W, len = part.len;
    const int t_begin = split * split_len;
    const int t_end = min(t_begin + split_len, len);
    const int n_blk = (t_end - t_begin + 31) / 32;
    const int n_fetch = kNeedO && M >= kFetchOnRows && n_blk <= kFetchOnBlocks ? (len - t_begin + 31) / 32 : n_blk;
    const int t_last = t_begin + (n_fetch - 1) * 32;             // the last block that is fetched

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int rb = chunk * 4 + wave;                             // row block of this wave
    const int row = rb * 32 + (lane & 31);                       // window row (i) owned by this lane
    const bool wave_active = rb * 32 < M;                        // uniform
    const bool row_valid = row < M;
    // Last key the row may see (Eq. 9 window rows are causal).  Padded rows carry a zero
    // query and see everything: they stay finite and are discarded later.
    const int vis = row_valid ? len - W + (row % W) : len - 1;
    // What the wave's first row sees, or with a multiple of W among its rows the least any row sees.
    const int phase = rb * 32 % W;
    const int vis_min = min(len - W + (phase + min(M - 1 - rb * 32, 31) >= W ? 0 : phase), t_end - 1);

    const char *kh = (const char *)k + (size_t)bg * N * kRowBytes;
    const char *vh = (const char *)v + (size_t)bg * N * kRowBytes;
    const uint32_t lds0 = lds_offset_of(smem);

    int koff[8], voff[4];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) koff[kk] = row_piece_offset(lane, kk);
#pragma unroll
    for (int ddb = 0; ddb < 4; ++ddb) voff[ddb] = vt_piece_offset(lane, ddb);

    Sweep1Regs R;
    {
        const char *qrow = (const char *)q + (((size_t)b * Hq + (size_t)g * G) * W + row) * kRowBytes;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            if (row_valid) R.q[kk] = *(const bf16x8 *)(qrow + (2 * kk + half) * 16);
            else R.q[kk] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) R.oacc[i] = zero16();
#pragma unroll
    for (int sx = 0; sx < 2; ++sx)
#pragma unroll
        for (int e = 0; e < 4; ++e) { R.phi[sx].u[e] = 0; R.plo[sx].u[e] = 0; }
#pragma unroll
    for (int r = 0; r < 16; ++r) R.p[r] = 0.f;
    R.m_ref = -FLT_MAX;              // (finite: a row may meet nothing visible in its first blocks)
    R.m_true = -INFINITY;
    R.lsum = 0.f;
    R.alpha = 1.0f;
    R.rescale = false;
    R.cand_val = -INFINITY;
    R.cand_tok = -1;
    R.n_ev = 0;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) settle(R.q[kk]);

    // Prologue.  Step 0 multiplies zero weights with whatever "V block -1" (slot 3 of the V ring)
    // holds, so that slot is cleared.  K blocks 0..3 and V blocks 0..1 are started (the batches
    // the steps -4..-1 would have started), K block 0 is waited for and block 0's S^T formed.
    uint32_t kdoff[2], vdoff[2];
    block_lane_offsets<kXor16>(kdoff, wave, lane);
    block_lane_offsets<kRot4>(vdoff, wave, lane);
    for (int e = threadIdx.x; e < kBlkBytes / 16; e += kThreads) ((uint4 *)(smem + 7 * kBlkBytes))[e] = make_uint4(0, 0, 0, 0);
    block_load_async<kXor16, kOnce>(kh, t_begin, len - 1, lds0, wave, lane, kdoff);
    block_load_async<kXor16, kOnce>(kh, min(t_begin + 32, t_last), len - 1, lds0 + kBlkBytes, wave, lane, kdoff);
    block_load_async<kXor16, kOnce>(kh, min(t_begin + 64, t_last), len - 1, lds0 + 2 * kBlkBytes, wave, lane, kdoff);
    if (kNeedO) block_load_async<kRot4, kOnce>(vh, t_begin, len - 1, lds0 + 4 * kBlkBytes, wave, lane, vdoff);
    block_load_async<kXor16, kOnce>(kh, min(t_begin + 96, t_last), len - 1, lds0 + 3 * kBlkBytes, wave, lane, kdoff);
    if (kNeedO) block_load_async<kRot4, kOnce>(vh, min(t_begin + 32, t_last), len - 1, lds0 + 5 * kBlkBytes, wave, lane, vdoff);
    wait_async_loads_keep<kNeedO ? 10 : 6>();         // everything after K block 0 may still be in flight
    __syncthreads();
    R.s_cur = zero16();
    if (wave_active) {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const bf16x8 a = lds_read16(smem + koff[kk]);
            R.s_cur = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.q[kk], R.s_cur, 0, 0, 0);
        }
    }

    const int n_total = (n_blk + 3) & ~3;
    const int n_plain = max(vis_min + 1 - t_begin, 0) / 32;   // leading blocks every row of this wave sees in full
    // What the steps fetch: K from block 4, V from block 2 on.  A last block with rows past the sequence's end (row rmax) is cut
    // where it comes up, block n_cut, or here.
    const int rmax = len - 1 - t_last, n_cut = rmax < 31 ? n_fetch - 1 : -1;
    BlockFetch kf, vf;
    kf.start(kh, min(t_begin + 4 * 32, t_last), kdoff);
    vf.start(vh, min(t_begin + 2 * 32, t_last), vdoff);
    if (n_cut >= 0 && n_cut < 4) kf.cut(rmax, wave, lane);
    if (n_cut >= 0 && n_cut < 2) vf.cut(rmax, wave, lane);
    // (kStoreZ: at most 32 rows, so they are the first wave's)
    char *z_split = (char *)(z + (size_t)bg * M * z_stride + t_begin);
    const uint32_t z_off = kStoreZ && row_valid ? (uint32_t)row * z_stride * 4 + 16 * half : ~0u;
#define OBC_S1_ARGS smem, lds0, n, t_begin, t_end, n_fetch - 1, n_cut, rmax, vis, n_plain, kf, vf, vh, koff, voff, wave, lane, wave_active, events, z_split, z_off
    for (int n = 0; n < n_total; n += 4) {
        sweep1_step<0, kNeedO, kStoreZ, kOnce>(R, OBC_S1_ARGS); ++n;
        sweep1_step<1, kNeedO, kStoreZ, kOnce>(R, OBC_S1_ARGS); ++n;
        sweep1_step<2, kNeedO, kStoreZ, kOnce>(R, OBC_S1_ARGS); ++n;
        sweep1_step<3, kNeedO, kStoreZ, kOnce>(R, OBC_S1_ARGS); n -= 3;
    }
#undef OBC_S1_ARGS
    // A final candidate that holds less than half of its own split's weight cannot dominate the
    // row; it joins the parked former candidates, which are ordinary keys and are added back below, now that
    // the reference is final.  The first one's value row is fetched ahead of the waits that follow.
    uint2 first_row[16];
    int2 first_ev = make_int2(-1, 0);
    if (kNeedO && wave_active) {
        const float c2 = kLog2e * kInvSqrtD;
        const float l_rest = halves_sum(R.lsum);
        if (R.cand_tok >= 0 && __builtin_amdgcn_exp2f((R.cand_val - R.m_ref) * c2) < l_rest) {
            if (R.n_ev < kEvents) {
                events[R.n_ev] = make_int2(R.cand_tok, __float_as_int(R.cand_val));
                R.n_ev += 1;
                R.cand_tok = -1;
            }
        }
        if (R.n_ev > 0) {
            first_ev = events[0];
            add_back_fetch(first_row, vh, first_ev.x, half);
        }
    }
    wait_async_loads();        // the blocks fetched past the end must have landed before the LDS is given back
    if (kNeedO && wave_active) {      // drain: P V of the last block (n_total - 1, in slot 3 of the V ring)
        pack_weights(R);
        if (R.rescale) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) R.oacc[i][r] *= R.alpha;
        }
#pragma unroll
        for (int ddb = 0; ddb < 4; ++ddb)
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                const bf16x8 a = lds_read_vt(smem + 7 * kBlkBytes + 16 * sx * kRowBytes + voff[ddb]);
                R.oacc[ddb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.phi[sx].v, R.oacc[ddb], 0, 0, 0);
                R.oacc[ddb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, R.plo[sx].v, R.oacc[ddb], 0, 0, 0);
            }
        if (first_ev.x >= 0) add_back_apply(R, first_row, __int_as_float(first_ev.y), R.m_ref, R.m_ref, half);
        for (int e = 1; e < kEvents; ++e) {
            if (!__any(e < R.n_ev)) break;       // uniform
            if (e < R.n_ev) {
                const int2 ev = events[e];
                add_back(R, vh, ev.x, __int_as_float(ev.y), R.m_ref, R.m_ref, half);
            }
        }
    }
    if (kNeedO) __syncthreads();      // every wave is done with the rings: their space now stages the output rows
    if (!wave_active) return;
    const float lrow = halves_sum(R.lsum);
    if (R.m_ref == -FLT_MAX && lrow == 0.f) R.m_ref = -INFINITY;
    const size_t prow0 = (size_t)(split_slot(lens, ragged, b, g, N, Hkv, split_len) + split) * m_pad + rb * 32;     // the wave's first row
    if (half == 0)                    // reference in raw q.k units (-inf when the split holds no visible key), sum, candidate
        *(float4 *)(part_ml + (prow0 + (lane & 31)) * 4) =
            make_float4(R.m_ref, lrow, kNeedO ? R.cand_val : R.m_true, __int_as_float(kNeedO ? R.cand_tok : 0));
    if (kNeedO) {
        // A lane holds 64 scattered entries of its row: written straight out, every store would touch 64 rows' worth of
        // cache lines 16 bytes at a time.  The wave's 32 rows pass through its own 16 KB of LDS instead (16-byte slot c
        // of row r at slot c ^ r: conflict-free both ways) and leave as whole rows, 1 KB per store.
        char *stage = smem + wave * (32 * kD * 4);
        const int r = lane & 31;
#pragma unroll
        for (int ddb = 0; ddb < 4; ++ddb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int c = ddb * 8 + 2 * r4 + half;
                *(float4 *)(stage + r * (kD * 4) + ((c ^ r) << 4)) =
                    make_float4(R.oacc[ddb][4 * r4], R.oacc[ddb][4 * r4 + 1], R.oacc[ddb][4 * r4 + 2], R.oacc[ddb][4 * r4 + 3]);
            }
        // (a wave's LDS operations complete in order: its reads below see its writes above; no other wave touches them)
        float *dst = part_o + prow0 * kD;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row_i = 2 * i + half, c = lane & 31;
            const f32x4 x = *(const f32x4 *)(stage + row_i * (kD * 4) + ((c ^ row_i) << 4));
            // (streaming store: the partials are read once, by the combine step, and 35 MB of them kept dirty in the
            // L2 would all be written back when the kernel ends)
            __builtin_nontemporal_store(x, (f32x4 *)(dst + row_i * kD + 4 * c));
        }
    }
}

// ------------------------------------------------------------------------------------
// Combine
// ------------------------------------------------------------------------------------
// Variants that need no o_i (Eq. 4, Eq. 8 and its l1-weighted form): the splits' row sums are merged into the
// one constant per row the second sweep turns logits into weights with.  Grid: y = (b, KV head); 16 lanes per row, one split
// each (with one lane per row that took sixteen splits at a time, 64 splits of 8 heads x 32K took 18.2 us; now 5.2).
template <typename Lens>
__global__ __launch_bounds__(256) void mfma_combine(const float *__restrict__ part_ml, int N, int W, int Hq, int Hkv,
                                                    int ragged, Lens lens, int split_len, int m_pad,
                                                    float *__restrict__ row_const, float *__restrict__ special) {
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15, bg = blockIdx.y;      // (m_pad: a multiple of 32)
    const int b = bg / Hkv, G = Hq / Hkv, M = G * W;
    const int len = seq_len_of(lens, ragged, b, N);
    const float4 *ml = (const float4 *)part_ml + (size_t)split_slot(lens, ragged, b, bg % Hkv, N, Hkv, split_len) * m_pad + row;
    const int live_splits = (len + split_len - 1) / split_len;
    const float c2 = kLog2e * kInvSqrtD;
    constexpr int kOwn = 4;                           // splits a lane holds at a time
    // The running sum follows the running max of the raw dot products; a split's sum is relative to its own reference.
    float m_raw = -INFINITY, l = 0.f;
    for (int s0 = 0; s0 < live_splits; s0 += 16 * kOwn) {
        float4 x[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
            const int s = s0 + 16 * j + sub;
            x[j] = s < live_splits ? ml[(size_t)s * m_pad] : make_float4(-INFINITY, 0.f, -INFINITY, 0.f);
        }
        float m_new = m_raw;
#pragma unroll
        for (int j = 0; j < kOwn; ++j) m_new = fmaxf(m_new, x[j].z);
        m_new = row16_reduce<MaxOp>(m_new);
        l *= m_raw == -INFINITY ? 0.f : exp2f((m_raw - m_new) * c2);
#pragma unroll
        for (int j = 0; j < kOwn; ++j) l = fmaf(x[j].x == -INFINITY ? 0.f : exp2f((x[j].x - m_new) * c2), x[j].y, l);
        m_raw = m_new;
    }
    l = row16_reduce<SumOp>(l);
    if (sub != 0) return;
    const size_t crow = (size_t)bg * m_pad + row;
    special[crow * 4 + 0] = __int_as_float(-1);       // no separately scored (row, token) pair
    // A_ip^2 = exp2(2 log2e Z_ip - the first); padded rows are weightless in the second sweep
    ((float4 *)row_const)[crow] = row < M ? make_float4(2.0f * (m_raw * c2 + log2f(l)), 0.f, __int_as_float(len - W + (row % W)), 0.f)
                                          : make_float4(1e30f, 0.f, __int_as_float(-1), 0.f);
}

// Variants that need o_i (Eq. 5, 6).  Every split reports, per row, its sums without its
// candidate key and the candidate itself.  The candidate with the largest logit (the first split on
// ties) stays held out; the others are ordinary keys and are added back from the value cache.  With
// l' and O' the sums over every key but that one, relative to a common reference T,
//     w = exp2((z_cand - T) c2),   A_cand = w / (w + l'),
//     v_cand - o_i = l' / (w + l') * (v_cand - O' / l'),      o_i = v_cand - (v_cand - o_i)
// without cancellation however much of the row's attention the candidate holds.  A candidate that
// holds a large share is scored here from these (`special`) and skipped by the second sweep.
//
// Grid: y = (b, KV head).  32 lanes take a row's elements, four each, and kBatch splits in one memory round trip.  With
// kGroups == 1 a workgroup has four rows.  With more, it has one row, and its kGroups groups of 32 lanes take kBatch
// splits each: a long head alone on the chip is cut into up to 128 splits, which one group would fetch in eight round
// trips (4 heads x 128K, 112 rows: 47 us, 14 us in eight groups).
template <int kGroups, int kBatch, typename Lens>
__global__ __launch_bounds__(kGroups == 1 ? 128 : 32 * kGroups) void mfma_combine_hold(
    const uint16_t *__restrict__ v, const float *__restrict__ part_ml, const float *__restrict__ part_o, int N, int W, int M,
    int Hkv, int ragged, Lens lens, int split_len, int splits, int m_pad, uint16_t *__restrict__ out_bf16, float *__restrict__ row_const,
    float *__restrict__ special) {
    const int group = threadIdx.x >> 5, row = kGroups == 1 ? blockIdx.x * 4 + group : blockIdx.x, bg = blockIdx.y;
    const int first = kGroups == 1 ? 0 : group * kBatch;  // this group's first split
    constexpr int kStride = kBatch * kGroups;
    // (Equal lengths: every head has `splits`.  The quotients that ragged ones take are some 25 instructions each ahead of the first
    // load: 1.9 of the kernel's 6.4 us, 8 heads x 128 rows x 8192, with them and with 64-bit addresses per load; 1.45 of 6.0 so.)
    int len = N, live_splits = splits, slot0 = bg * splits;
    if (ragged) {
        const int b = bg / Hkv;
        len = lens.len[b];
        live_splits = (len + split_len - 1) / split_len;
        slot0 = split_slot(lens, ragged, b, bg % Hkv, N, Hkv, split_len);
    }
    const int sub = threadIdx.x & 31, dd = sub * 4;   // this lane's elements dd .. dd + 3
    const size_t crow = (size_t)bg * m_pad + row;
    const size_t lo_plane = (size_t)gridDim.y * m_pad * kD;
    const bool live = row < M;                        // the same for the 32 lanes of a row
    // Records of the row: byte offsets from the head's first one, a record's sums 32 times as far as its four words.  Splits past
    // the last one re-read it.
    const char *ml_head = (const char *)part_ml + (size_t)slot0 * m_pad * 16, *po_head = (const char *)part_o + (size_t)slot0 * m_pad * (kD * 4);
    const uint32_t split_bytes = (uint32_t)m_pad * 16, row_at = (uint32_t)row * 16, last_at = row_at + (uint32_t)(live_splits - 1) * split_bytes;
    auto record_at = [&](int s0, int j) { return min(row_at + (uint32_t)s0 * split_bytes + j * split_bytes, last_at); };
    auto record = [&](uint32_t at) { return *(const float4 *)(ml_head + at); };
    auto sums = [&](uint32_t at) { return *(const float4 *)(po_head + (size_t)at * 32 + sub * 16); };
    const float c2 = kLog2e * kInvSqrtD;
    const uint16_t *vg = v + (size_t)bg * N * kD;
    // First the common reference T (no sum lies more than the lazy-rescale slack above its own
    // reference, so the largest reference or candidate logit will do) and the winning candidate.
    // The first splits' records and sums are fetched in one go and stay in registers.
    float T = -INFINITY, c_val = -INFINITY;
    int c_tok = -1, s_star = -1;
    // What bounds the kernel is these trips to memory one after the other: records, the values that they name, sums.  Records are
    // asked for first and every candidate's value as soon as they are there, before the groups agree on the winner and while
    // the sums are still on their way; the winner's then comes from the group that has it.  Kernel, us, records and sums in
    // turn and values after the agreement / so: 8 heads x 128 rows x 8192 7.9 / 7.3; 4 x 8 heads x 32768, 4 rows 6.3 / 5.5.  Where
    // the sums' bytes are the limit (4 heads x 448 rows x 128K) nothing changes: 10.3 / 10.4.
    float4 ml[kBatch], po[kBatch];
    uint2 vo[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) ml[j] = record(record_at(first, j));
    asm volatile("" ::: "memory");                    // (else the sums are asked for between the records)
#pragma unroll
    for (int j = 0; j < kBatch; ++j) po[j] = sums(record_at(first, j));
    auto candidate_values = [&](int s0) {             // (padded rows: zero queries, nothing of theirs is used)
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int tok = __float_as_int(ml[j].w);
            vo[j] = live && s0 + j < live_splits && tok >= 0 ? *(const uint2 *)(vg + (size_t)tok * kD + dd) : make_uint2(0u, 0u);
        }
    };
    candidate_values(first);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
        if (first + j >= live_splits) continue;
        T = fmaxf(T, fmaxf(ml[j].x, ml[j].z));
        const int tok = __float_as_int(ml[j].w);
        if (tok >= 0 && ml[j].z > c_val) { c_val = ml[j].z; c_tok = tok; s_star = first + j; }
    }
    for (int s0 = first + kStride; s0 < live_splits; s0 += kStride) {
        float4 mm[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) mm[j] = record(record_at(s0, j));
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (s0 + j >= live_splits) continue;
            T = fmaxf(T, fmaxf(mm[j].x, mm[j].z));
            const int tok = __float_as_int(mm[j].w);
            if (tok >= 0 && mm[j].z > c_val) { c_val = mm[j].z; c_tok = tok; s_star = s0 + j; }
        }
    }
    if constexpr (kGroups > 1) {                      // the groups agree (equal logits: the lowest split)
        __shared__ float4 found[kGroups];
        if (sub == 0) found[group] = make_float4(T, c_val, __int_as_float(c_tok), __int_as_float(s_star));
        __syncthreads();
        T = c_val = -INFINITY;
        c_tok = s_star = -1;
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            const float4 f = found[i];
            T = fmaxf(T, f.x);
            const int tok = __float_as_int(f.z), star = __float_as_int(f.w);
            if (tok >= 0 && (f.y > c_val || (f.y == c_val && star < s_star))) { c_val = f.y; c_tok = tok; s_star = star; }
        }
    }
    if (!live) { c_tok = -1; s_star = -1; }
    uint2 vt_bits = make_uint2(0u, 0u);               // the winning candidate's value, in the group that has its split
    float l = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = first; s0 < live_splits; s0 += kStride) {
        if (s0 > first) {
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {         // (the records are in cache from the pass above)
                ml[j] = record(record_at(s0, j));
                po[j] = sums(record_at(s0, j));
            }
            candidate_values(s0);
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (s0 + j >= live_splits) continue;
            const float w = ml[j].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((ml[j].x - T) * c2);
            l = fmaf(w, ml[j].y, l);
            o[0] = fmaf(w, po[j].x, o[0]);
            o[1] = fmaf(w, po[j].y, o[1]);
            o[2] = fmaf(w, po[j].z, o[2]);
            o[3] = fmaf(w, po[j].w, o[3]);
            if (s0 + j == s_star) vt_bits = vo[j];
            if (live && s0 + j != s_star && __float_as_int(ml[j].w) >= 0) {   // this split's candidate is an ordinary key
                const float wc = __builtin_amdgcn_exp2f((ml[j].z - T) * c2);
                l += wc;
                o[0] = fmaf(wc, __uint_as_float(vo[j].x << 16), o[0]);
                o[1] = fmaf(wc, __uint_as_float(vo[j].x & 0xffff0000u), o[1]);
                o[2] = fmaf(wc, __uint_as_float(vo[j].y << 16), o[2]);
                o[3] = fmaf(wc, __uint_as_float(vo[j].y & 0xffff0000u), o[3]);
            }
        }
    }
    if constexpr (kGroups > 1) {                      // the groups' sums meet in group order
        __shared__ float sum_l[kGroups];
        __shared__ float4 sum_o[kGroups][32];
        __shared__ uint2 vt_s[32];
        if (sub == 0) sum_l[group] = l;
        if (s_star >= 0 && s_star % kStride / kBatch == group) vt_s[sub] = vt_bits;
        sum_o[group][sub] = make_float4(o[0], o[1], o[2], o[3]);
        __syncthreads();
        if (group != 0) return;
        if (s_star >= 0) vt_bits = vt_s[sub];
        for (int i = 1; i < kGroups; ++i) {
            const float4 x = sum_o[i][sub];
            l += sum_l[i];
            o[0] += x.x; o[1] += x.y; o[2] += x.z; o[3] += x.w;
        }
    }
    // (no split may have kept a candidate: then w = 0 and o_i = O' / l' as usual)
    const float wc = c_tok >= 0 ? __builtin_amdgcn_exp2f((c_val - T) * c2) : 0.f;
    const float ltot = wc + l;
    const float inv = 1.0f / ltot;
    const float inv_l = l > 0.f ? 1.0f / l : 0.f;
    const float z = c_val * kInvSqrtD;               // Z of the (row, candidate) pair
    const float vt[4] = {__uint_as_float(vt_bits.x << 16), __uint_as_float(vt_bits.x & 0xffff0000u),
                         __uint_as_float(vt_bits.y << 16), __uint_as_float(vt_bits.y & 0xffff0000u)};
    uint16_t ob[4], olo[4];
    float s_oo = 0.f, s_vv = 0.f, s_dd = 0.f, s_cc = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float diff = (l * inv) * (vt[e] - o[e] * inv_l);     // (v_cand - o_i)[dd + e]
        const float oi = vt[e] - diff;
        const float comb = fmaf(z, diff, vt[e]);                   // ((1+Z) v_cand - Z o_i)[dd + e]
        // o^ = hi + lo, the pair of bf16 pieces the second sweep feeds to the matrix cores.
        ob[e] = (uint16_t)(__float_as_uint(oi) >> 16);
        const float ohi = bf16_bits_to_float(ob[e]);
        olo[e] = (uint16_t)(pack_bf16(oi - ohi, 0.f) & 0xffffu);
        const float of = ohi + bf16_bits_to_float(olo[e]);
        s_oo = fmaf(of, of, s_oo);
        s_vv = fmaf(vt[e], vt[e], s_vv);
        s_dd = fmaf(diff, diff, s_dd);
        s_cc = fmaf(comb, comb, s_cc);
    }
    // A candidate with a small share is scored by the second sweep like any other key (its o_i is exact either
    // way); one that may dominate is scored here and skipped there.
    const float a = wc * inv;
    const bool separate = live && a >= kSeparateShare;
    s_oo = row_sum32(s_oo);
    if (__any(separate)) { s_vv = row_sum32(s_vv); s_dd = row_sum32(s_dd); s_cc = row_sum32(s_cc); }
    uint2 hi_bits, lo_bits;
    hi_bits.x = live ? (uint32_t)cross_operand_bf16(ob[0]) | ((uint32_t)cross_operand_bf16(ob[1]) << 16) : 0u;
    hi_bits.y = live ? (uint32_t)cross_operand_bf16(ob[2]) | ((uint32_t)cross_operand_bf16(ob[3]) << 16) : 0u;
    lo_bits.x = live ? (uint32_t)cross_operand_bf16(olo[0]) | ((uint32_t)cross_operand_bf16(olo[1]) << 16) : 0u;
    lo_bits.y = live ? (uint32_t)cross_operand_bf16(olo[2]) | ((uint32_t)cross_operand_bf16(olo[3]) << 16) : 0u;
    *(uint2 *)(out_bf16 + crow * kD + dd) = hi_bits;
    *(uint2 *)(out_bf16 + lo_plane + crow * kD + dd) = lo_bits;
    if (sub != 0) return;
    if (!live) {                                      // padded row: weightless in the second sweep
        row_const[crow * 4 + 0] = 1e30f;
        row_const[crow * 4 + 1] = 0.f;
        row_const[crow * 4 + 2] = __int_as_float(-1);
        row_const[crow * 4 + 3] = 0.f;
        special[crow * 4 + 0] = __int_as_float(-1);
        return;
    }
    const float a2 = a * a;
    row_const[crow * 4 + 0] = 2.0f * (T * c2 + log2f(ltot));   // A_ip^2 = exp2(2 log2e Z_ip - this)
    row_const[crow * 4 + 1] = s_oo * kCrossScale;              // ||o^_i||^2 / 128
    row_const[crow * 4 + 2] = __int_as_float(len - W + (row % W));
    row_const[crow * 4 + 3] = 0.f;
    special[crow * 4 + 0] = __int_as_float(separate ? c_tok : -1);
    if (separate) {
        special[crow * 4 + 1] = a2 * s_vv;             // Eq. 4 term of the pair
        special[crow * 4 + 2] = a2 * z * z * s_dd;     // Eq. 5 term
        special[crow * 4 + 3] = a2 * s_cc;             // Eq. 6 term (completed square)
    }
}

// ------------------------------------------------------------------------------------
// Sweep 2
// ------------------------------------------------------------------------------------
struct Sweep2Regs {
    bf16x8 q[8], ohi[8], olo[8];   // stationary A operands of this wave's row block
    float c_m2[16], c_oo[16];      // per accumulator register: 2 (max + log2 sum), ||o^||^2 of its row
};

// Adds up, in wave order, the four waves' partial scores of one tile (64 tokens starting at
// `tok0`, staged in LDS as [wave][variant][64]) and writes them out; wave c handles variant c.
template <int kNv>
__device__ __forceinline__ void sweep2_flush(const float *stage, float *out, size_t variant_stride, int tok0,
                                             int t_end, int wave, int lane, bool accumulate) {
    if (wave < kNv && tok0 + lane < t_end) {
        const float *p = stage + wave * 64 + lane;
        float *o = out + wave * variant_stride + tok0 + lane;
        const float sum = (p[0] + p[kNv * 64]) + (p[2 * kNv * 64] + p[3 * kNv * 64]);
        *o = accumulate ? *o + sum : sum;
    }
}

// One step of sweep 2 = one block of 32 tokens (PH = n mod 4 fixes the LDS slot):
//   matrix cores: Z = Q K^T and O V^T of the block (+ ||v||^2 on the dot-product unit)
//   vector ALUs : its scores, summed over this wave's 32 rows, parked in LDS
// The two phases of one wave do not overlap; the second wave on the SIMD runs in the gaps
// (on this hardware a 32x32x16 matrix op blocks most vector-ALU issue anyway).
// Even steps first wait for the tile issued two steps earlier and start the next one.
template <int PH, bool kMasked, int kVariant, bool kOnce>
__device__ __forceinline__ void sweep2_step(Sweep2Regs &R, uint32_t lds0, int n, int n_blk,
                                            int t_begin, int t_end, int last_row, const int *vis_i,
                                            const int *excl_i, const char *kh, const char *vh,
                                            const char *const (&kp)[8], const uint32_t (&kdoff)[4], int wave, int lane,
                                            bool wave_active, float *part, float *out, size_t variant_stride, bool accumulate,
                                            int spec_lo_blk, int spec_hi_blk) {
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    constexpr bool kDoV = kVariant == OBC_VALUE || kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    constexpr bool kDoA = kVariant == OBC_ATTN || kVariant == OBC_VATP;   // Eq. 8 and its l1-weighted form
    constexpr bool kNeedVO = kDoK || kDoJ;
    constexpr int kSlot = PH >> 1, kBlk = PH & 1;
    constexpr int kKBase = (kSlot ? kLdsK1 : kLdsK0) + kBlk * 32 * kRowBytes;
    constexpr int kVBase = (kSlot ? kLdsV1 : kLdsV0) + kBlk * 32 * kRowBytes;
    const int half = lane >> 5;
    const float c2x2 = 2.0f * kLog2e * kInvSqrtD;

    if ((PH & 1) == 0) {
        wait_async_loads();
        __syncthreads();
        const int tn = t_begin + ((n >> 1) + 1) * kTileTok;           // first token of the tile to start now
        if (tn < t_end) {
            tile_load_async<kXor16, kOnce>(kh, tn, last_row, lds0 + (PH == 0 ? kLdsK1 : kLdsK0), wave, lane, kdoff);
            if (kVariant != OBC_ATTN)
                tile_load_async<kXor16, kOnce>(vh, tn, last_row, lds0 + (PH == 0 ? kLdsV1 : kLdsV0), wave, lane, kdoff);
        }
        if (n >= 2) sweep2_flush<kNv>(part + (kSlot ^ 1) * 4 * kNv * 64, out, variant_stride, t_begin + (n - 2) * 32, t_end, wave, lane, accumulate);
    }
    if (n >= n_blk) return;                                            // uniform
    float acc_v = 0.f, acc_k = 0.f, acc_j = 0.f;
    if (wave_active) {
        // ---- matrix cores ----
        f32x16 z = zero16(), vo = zero16();
        float vv = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const bf16x8 kb = lds_read16(kp[kk] + kKBase);
            z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(R.q[kk], kb, z, 0, 0, 0);
        }
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            if (kVariant == OBC_ATTN) break;                           // no use for V at all
            const bf16x8 vb = lds_read16(kp[kk] + kVBase);
            vv = kVariant == OBC_VATP ? sumabs8(vb, vv) : sumsq8(vb, vv);
            if (kNeedVO) {
                vo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(R.ohi[kk], vb, vo, 0, 0, 0);
                vo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(R.olo[kk], vb, vo, 0, 0, 0);
            }
        }
        vv += __shfl_xor(vv, 32);                                         // ||v_p||^2 of this lane's token
        if (!kMasked && kNeedVO && n >= spec_lo_blk && n <= spec_hi_blk) {      // uniform, rare
            // This fully visible block may hold a (row, key) pair that is scored separately: such a pair gets a
            // logit so low that its weight is exactly 0 (and low enough only for that: every product below stays finite).
            const int tokx = t_begin + n * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = wave * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (tokx == excl_i[i]) z[r] = kHiddenLogit;
            }
        }
        // ---- vector ALUs ----
        // vo holds -2 v_p.o^_i / 128 and c_oo holds ||o^_i||^2 / 128 (see kCrossScale), so with
        // w7 = ||v_p - o^_i||^2 / 128 = (||v_p||^2 / 128 + c_oo) + vo and z the raw dot product (Z = z / sqrt(128)):
        //   Eq. 5 term  A^2 Z^2 w = A^2 z^2 w7
        //   Eq. 6 term  A^2 ||(1+Z) v - Z o^||^2 = A^2 (||v||^2 + Z (2 (||v||^2 - v.o^) + Z w))
        //                                        = A^2 (||v||^2 + z (2 ||v||^2 / sqrt(128) + sqrt(128) vo + z w7))
        // Rounding can leave a term a hair below zero; the sums are clamped once at the end.
        const int tok = t_begin + n * 32 + (lane & 31);
        const float vv7 = vv * kCrossScale, vv2s = vv * (2.0f * kInvSqrtD);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // A_ip^2, or A_ip itself (half the exponent) for the attention-only scores
            float a2 = kDoA ? __builtin_amdgcn_exp2f(fmaf(z[r], 0.5f * c2x2, -0.5f * R.c_m2[r]))
                            : __builtin_amdgcn_exp2f(fmaf(z[r], c2x2, -R.c_m2[r]));
            if (kMasked) {
                const int i = wave * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (tok > vis_i[i] || tok >= t_end || tok == excl_i[i]) a2 = 0.f; // hidden, padded, or scored separately
            }
            if (kDoV || kDoA) acc_v += a2;
            if (kNeedVO) {
                const float w7 = (vv7 + R.c_oo[r]) + vo[r];                       // ||v_p - o^_i||^2 / 128
                if (kDoK) acc_k = fmaf(a2 * z[r] * z[r], w7, acc_k);
                if (kDoJ) {
                    const float h = fmaf(z[r], w7, fmaf(vo[r], kSqrtD, vv2s));
                    acc_j = fmaf(a2, fmaf(z[r], h, vv), acc_j);
                }
            }
        }
        if (kDoV || kVariant == OBC_VATP) acc_v *= vv;                 // ||v_p||^2, or ||v_p||_1 for the l1 form
        if (kDoV || kDoA) acc_v += __shfl_xor(acc_v, 32);
        if (kDoK) { acc_k += __shfl_xor(acc_k, 32); acc_k = fmaxf(acc_k, 0.f); }
        if (kDoJ) { acc_j += __shfl_xor(acc_j, 32); acc_j = fmaxf(acc_j, 0.f); }
    }
    if (half == 0) {
        float *pw = part + ((kSlot * 4 + wave) * kNv) * 64 + kBlk * 32 + lane;
        int c = 0;
        if (kDoV || kDoA) pw[64 * c++] = acc_v;
        if (kDoK) pw[64 * c++] = acc_k;
        if (kDoJ) pw[64 * c++] = acc_j;
    }
}

// kVariant: OBC_VALUE / OBC_KEY / OBC_JOINT / OBC_ALL / OBC_ATTN / OBC_VATP.  Grid: see sweep_part.
// With one chunk the scores go straight to `scores`; with several, each chunk writes its
// own plane and mfma_sum_planes adds them in chunk order.
template <int kVariant, bool kOnce, typename Lens>
__global__ __launch_bounds__(kThreads, 2) void mfma_sweep2(const uint16_t *__restrict__ q,
                                                           const uint16_t *__restrict__ k,
                                                           const uint16_t *__restrict__ v, int N, int W, int Hq,
                                                           int Hkv, int heads, int ragged, Lens lens, int range_len,
                                                           int n_chunks, int m_pad, const uint16_t *__restrict__ out_bf16,
                                                           const float *__restrict__ row_const,
                                                           const float *__restrict__ special,
                                                           float *__restrict__ dst, size_t variant_stride,
                                                           size_t chunk_stride, int accumulate_flag) {
    const bool accumulate = accumulate_flag != 0;      // add to what `dst` holds; padded positions stay untouched
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    constexpr bool kNeedVO = kVariant == OBC_KEY || kVariant == OBC_JOINT || kVariant == OBC_ALL;
    // the K and V tiles, then 256 row constants and the staged partial scores of two tiles
    __shared__ __attribute__((aligned(1024))) char smem[kLdsTiles + 256 * sizeof(float) + 2 * 4 * kNv * 64 * sizeof(float)];
    float *vis_s = (float *)(smem + kLdsTiles);                // [128] last visible key of each row of the chunk
    float *excl_s = vis_s + 128;                               // [128] key of the row that is scored separately, or -1
    float *part = excl_s + 128;                                // [2 tiles][4 waves][kNv][64] partial scores

    const SweepPart where = sweep_part(lens, ragged, N, Hkv, n_chunks, range_len);
    const int b = where.b, g = where.g, bg = b * Hkv + g, chunk = where.chunk, G = Hq / Hkv, M = G * W, len = where.len;
    const int t_begin = where.part * range_len;
    float *out = dst + (size_t)chunk * chunk_stride + (size_t)bg * N;
    const int t_end = min(t_begin + range_len, len);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int rb = chunk * 4 + wave;
    const bool wave_active = rb * 32 < M;                      // uniform
    const int arow = rb * 32 + (lane & 31);                    // row whose A-operand pieces this lane holds
    const size_t cbase = (size_t)bg * m_pad;

    const char *kh = (const char *)k + (size_t)bg * N * kRowBytes;
    const char *vh = (const char *)v + (size_t)bg * N * kRowBytes;
    const uint32_t lds0 = lds_offset_of(smem);

    // Tile 0 is started before anything else so that its latency hides behind the loads of
    // this wave's stationary operands; step 0 waits for it.
    uint32_t kdoff[4];
    tile_lane_offsets<kXor16>(kdoff, wave, lane);
    tile_load_async<kXor16, kOnce>(kh, t_begin, len - 1, lds0 + kLdsK0, wave, lane, kdoff);
    if (kVariant != OBC_ATTN) tile_load_async<kXor16, kOnce>(vh, t_begin, len - 1, lds0 + kLdsV0, wave, lane, kdoff);

    // (fetched with the stationary operands below, in one memory round trip; used after them)
    float my_vis = __int_as_float(-1);
    int my_excl = -1;
    if (threadIdx.x < 128) {
        const int i = chunk * 128 + threadIdx.x;
        if (i < m_pad) my_vis = row_const[(cbase + i) * 4 + 2];
        if (kNeedVO && i < m_pad) my_excl = __float_as_int(special[(cbase + i) * 4 + 0]);
    }

    int koff[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) koff[kk] = row_piece_offset(lane, kk);

    const char *kp[8];                                         // LDS address of this lane's operand piece kk in a tile at offset 0
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kp[kk] = smem + koff[kk];

    Sweep2Regs R;
    {
        const bool ok = arow < M;
        const char *qrow = (const char *)q + (((size_t)b * Hq + (size_t)g * G) * W + arow) * kRowBytes;
        const char *orow = (const char *)out_bf16 + (cbase + arow) * kRowBytes;
        const size_t lo_plane = (size_t)heads * m_pad * kRowBytes;
        // One array after the other: the four loads that share a 128-byte line of a row follow each other closely.
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            R.q[kk] = ok ? *(const bf16x8 *)(qrow + (2 * kk + half) * 16) : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        if (kNeedVO) {
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                R.ohi[kk] = ok ? *(const bf16x8 *)(orow + (2 * kk + half) * 16) : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                R.olo[kk] = ok ? *(const bf16x8 *)(orow + lo_plane + (2 * kk + half) * 16) : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
        }
    }
    // Constants of the 16 rows this lane meets in the accumulators: row rb*32 + 8 (r/4) + 4 half + r%4.
    int vis_min = 0x7fffffff;                                  // first key some row of this wave cannot see
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = rb * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        const bool ok = wave_active && i < m_pad;
        const float4 rc = ok ? ((const float4 *)row_const)[cbase + i] : make_float4(1e30f, 0.f, __int_as_float(-1), 0.f);
        R.c_m2[r] = rc.x;                                              // padded rows (1e30) weigh nothing
        R.c_oo[r] = rc.y;
        const int vi = __float_as_int(rc.z);
        if (vi >= 0) vis_min = min(vis_min, vi);
    }
    vis_min = min(vis_min, __shfl_xor(vis_min, 32));
    vis_min = __builtin_amdgcn_readfirstlane(min(vis_min, t_end - 1));
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        settle(R.q[kk]);
        if (kNeedVO) { settle(R.ohi[kk]); settle(R.olo[kk]); }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) { settle(R.c_m2[r]); settle(R.c_oo[r]); }
    // First and last block (of 32 tokens, counted from t_begin) that hold a separately scored (row, key) pair.
    __shared__ int spec_lo, spec_hi;
    if (threadIdx.x == 0) { spec_lo = 0x7fffffff; spec_hi = -1; }
    __syncthreads();
    int mine_special = 0;
    if (threadIdx.x < 128) {
        const int ex = my_excl;
        vis_s[threadIdx.x] = my_vis;
        excl_s[threadIdx.x] = __int_as_float(ex);
        mine_special = ex >= t_begin && ex < t_end;
        if (mine_special) {
            atomicMin(&spec_lo, (ex - t_begin) >> 5);
            atomicMax(&spec_hi, (ex - t_begin) >> 5);
        }
    }
    const int *vis_i = (const int *)vis_s, *excl_i = (const int *)excl_s;
    // Uniform: some (row, key) pair of this chunk and token range is scored separately.
    const bool has_special = __syncthreads_or(mine_special) != 0;

    const int n_blk = (t_end - t_begin + 31) / 32;
    const int n_total = (n_blk + 3) & ~3;
    int n_plain = (vis_min + 1 - t_begin) / 32;       // leading blocks every row of this wave sees in full
    n_plain = max(0, min(n_plain, n_blk)) & ~3;
    // Blocks m_lo .. m_hi span the separately scored pairs of this range (none: an empty span).
    const int m_lo = has_special ? __builtin_amdgcn_readfirstlane(spec_lo) : 1;
    const int m_hi = has_special ? __builtin_amdgcn_readfirstlane(spec_hi) : 0;
#define OBC_S2_ARGS lds0, n, n_blk, t_begin, t_end, len - 1, vis_i, excl_i, kh, vh, kp, kdoff, wave, lane, wave_active, part, out, variant_stride, accumulate, m_lo, m_hi
    int n = 0;
    for (; n < n_plain; n += 4) {
        sweep2_step<0, false, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<1, false, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<2, false, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<3, false, kVariant, kOnce>(R, OBC_S2_ARGS); n -= 3;
    }
    for (; n < n_total; n += 4) {
        sweep2_step<0, true, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<1, true, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<2, true, kVariant, kOnce>(R, OBC_S2_ARGS); ++n;
        sweep2_step<3, true, kVariant, kOnce>(R, OBC_S2_ARGS); n -= 3;
    }
#undef OBC_S2_ARGS
    __syncthreads();
    // The last tile's partial sums (second staging slot: n_total is a multiple of 4), then zeros for the padding.
    sweep2_flush<kNv>(part + 4 * kNv * 64, out, variant_stride, t_begin + (n_total - 2) * 32, t_end, wave, lane, accumulate);
    if (!accumulate) zero_padding<kNv>(where, N, out, variant_stride);
    if (has_special) {
        wait_async_loads();
        add_special_pairs<kVariant>(smem, special + (cbase + chunk * 128) * 4, min(128, m_pad - chunk * 128), t_begin, t_end, out, variant_stride);
    }
}

// Second sweep for at most kFewRows window rows per KV head (a one-row window, typically): the logits were kept by the
// first sweep, so only V is read again.  Grid: x = token range, y = (b, KV head); a wave takes 64 tokens at a time in four
// tiles of 16.
//
// One 16x16x32 matrix op takes 16 tokens and all rows at once: rows 0-7 of its A operand are the high pieces of the
// (scaled) o^_i, rows 8-15 the low ones, so their products meet in lanes l and l ^ 32.  V goes from memory straight into
// the B operand (a tile's instruction reads 64 bytes of each of 16 rows), no LDS.  Bound by the read of V: 4 x 8 x 32768
// tokens, G = 4, joint: 109 us for the second sweep over K and V, 57 us for this.
constexpr int kFewRows = 8;
constexpr int kFewTiles = 4;

template <int kVariant, typename Lens>
__global__ __launch_bounds__(kThreads, 2) void score_few_rows(const uint16_t *__restrict__ v, int N, int M, int Hkv, int ragged,
                                                              Lens lens, int range_len, int m_pad,
                                                              const float *__restrict__ z, int z_stride,
                                                              const uint16_t *__restrict__ out_bf16, size_t lo_plane,
                                                              const float *__restrict__ row_const,
                                                              const float *__restrict__ special,
                                                              float *__restrict__ dst, size_t variant_stride, int accumulate) {
    constexpr bool kDoV = kVariant == OBC_VALUE || kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    constexpr bool kDoA = kVariant == OBC_ATTN || kVariant == OBC_VATP;
    constexpr bool kNeedVO = kDoK || kDoJ, kNeedV = kVariant != OBC_ATTN;
    const float c2x2 = 2.0f * kLog2e * kInvSqrtD;
    const int bg = blockIdx.y, len = seq_len_of(lens, ragged, bg / Hkv, N);
    const int t_begin = blockIdx.x * range_len, t_stop = min(t_begin + range_len, N), t_end = min(t_stop, len);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, j = lane >> 4;
    float *out = dst + (size_t)bg * N;
    if (!accumulate)
        for (int t = max(t_begin, len) + (int)threadIdx.x; t < t_stop; t += kThreads)       // the padding
#pragma unroll
            for (int c = 0; c < (kVariant == OBC_ALL ? 3 : 1); ++c) out[c * variant_stride + t] = 0.f;
    if (t_begin >= t_end) return;                            // uniform

    const uint16_t *vg = v + (size_t)bg * N * kD;
    const size_t cbase = (size_t)bg * m_pad;
    // This lane's two rows, and with them its share of the epilogue.
    const int row0 = 4 * (j & 1) + 2 * (j >> 1);
    const float *z0 = z + ((size_t)bg * M + min(row0, M - 1)) * z_stride, *z1 = z + ((size_t)bg * M + min(row0 + 1, M - 1)) * z_stride;
    bf16x8 vb[2][kFewTiles][4];
    float zz[2][kFewTiles][2];
    auto fetch = [&](int slot, int t0) {
#pragma unroll
        for (int i = 0; i < kFewTiles; ++i) {
            const int t = min(t0 + 16 * i + n, t_end - 1);   // (tokens past the end repeat the last one and are not written)
            if (kNeedV)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) vb[slot][i][kk] = *(const bf16x8 *)(vg + (size_t)t * kD + kk * 32 + j * 8);
            zz[slot][i][0] = z0[t];
            zz[slot][i][1] = z1[t];
        }
    };
    // (From the range's end to its start, where the memory-side cache might still be warm from the first sweep: no difference
    // beyond 1 % either way over 1 to 8 rows and 16K to 128K tokens of 8 heads.)
    constexpr int kStep = kThreads;                          // tokens the workgroup takes at a time
    int t0 = t_begin + wave * 64;
    if (t0 < t_end) fetch(0, t0);

    bf16x8 o[4];
    if (kNeedVO) {
        const int row = n & 7;
        const uint16_t *src = out_bf16 + (n < 8 ? 0 : lo_plane) + (cbase + min(row, M - 1)) * kD + j * 8;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) o[kk] = row < M ? *(const bf16x8 *)(src + kk * 32) : bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    }
    float c_m2[2], c_oo[2], sp[2][3];
    int vis[2], excl[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bool ok = row0 + i < M;
        const float4 rc = ok ? ((const float4 *)row_const)[cbase + row0 + i] : make_float4(1e30f, 0.f, __int_as_float(-1), 0.f);
        const float4 s = ok && kNeedVO ? ((const float4 *)special)[cbase + row0 + i] : make_float4(__int_as_float(-1), 0.f, 0.f, 0.f);
        c_m2[i] = rc.x; c_oo[i] = rc.y; vis[i] = __float_as_int(rc.z);
        excl[i] = __float_as_int(s.x);
        const bool none = excl[i] < 0;                       // (the terms are not written then)
        sp[i][0] = none ? 0.f : s.y; sp[i][1] = none ? 0.f : s.z; sp[i][2] = none ? 0.f : s.w;
    }

    auto score = [&](int slot, int t0) {
        float sum_v = 0.f, sum_k = 0.f, sum_j = 0.f;         // of token t0 + lane
#pragma unroll
        for (int i = 0; i < kFewTiles; ++i) {
            f32x4 vo = {0.f, 0.f, 0.f, 0.f};
            float vv = 0.f;
            if (kNeedV)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    if (kVariant == OBC_VATP) vv = sumabs8(vb[slot][i][kk], vv);
                    else vv = sumsq8(vb[slot][i][kk], vv);
                    if (kNeedVO) vo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o[kk], vb[slot][i][kk], vo, 0, 0, 0);
                }
            if (kNeedV) vv = across_rows<SumOp>(vv);
            const int tok = t0 + 16 * i + n;
            float a_v = 0.f, a_k = 0.f, a_j = 0.f;
            // high and low pieces meet: rows 4 (j & 1) + r
            float w[4];
            if (kNeedVO)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float lo, hi;
                    both_of_pair<32>(vo[r], lo, hi);
                    w[r] = lo + hi;
                }
            const float vv7 = vv * kCrossScale, vv2s = vv * (2.0f * kInvSqrtD);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float x = zz[slot][i][h];
                float a2 = kDoA ? __builtin_amdgcn_exp2f(fmaf(x, 0.5f * c2x2, -0.5f * c_m2[h]))
                                : __builtin_amdgcn_exp2f(fmaf(x, c2x2, -c_m2[h]));
                if (tok > vis[h]) a2 = 0.f;
                const bool apart = kNeedVO && tok == excl[h];          // scored by the combine step
                if (kDoV || kDoA) a_v += apart ? 0.f : a2;
                if (kNeedVO) {                                         // (as in sweep2_step)
                    const float cross = j < 2 ? w[h] : w[2 + h];
                    const float w7 = (vv7 + c_oo[h]) + cross;
                    if (kDoK) a_k += apart ? sp[h][1] : a2 * x * x * w7;
                    if (kDoJ) {
                        const float g = fmaf(x, w7, fmaf(cross, kSqrtD, vv2s));
                        a_j += apart ? sp[h][2] : a2 * fmaf(x, g, vv);
                    }
                }
            }
            if (kDoV || kVariant == OBC_VATP) {
                a_v *= vv;
                if (kDoV && kNeedVO)
#pragma unroll
                    for (int h = 0; h < 2; ++h) a_v += tok == excl[h] ? sp[h][0] : 0.f;
            }
            if (kDoV || kDoA) { a_v = across_rows<SumOp>(a_v); sum_v = j == i ? a_v : sum_v; }
            if (kDoK) { a_k = fmaxf(across_rows<SumOp>(a_k), 0.f); sum_k = j == i ? a_k : sum_k; }
            if (kDoJ) { a_j = fmaxf(across_rows<SumOp>(a_j), 0.f); sum_j = j == i ? a_j : sum_j; }
        }
        const int t = t0 + lane;                             // tile j, token n of it
        if (t < t_end) {
            int c = 0;
            auto put = [&](float x) {
                float *d = out + (c++) * variant_stride + t;
                *d = accumulate ? *d + x : x;
            };
            if (kDoV || kDoA) put(sum_v);
            if (kDoK) put(sum_k);
            if (kDoJ) put(sum_j);
        }
    };
    for (; t0 < t_end; t0 += 2 * kStep) {                    // two buffers, both with constant indices
        if (t0 + kStep < t_end) fetch(1, t0 + kStep);
        score(0, t0);
        if (t0 + kStep >= t_end) break;
        if (t0 + 2 * kStep < t_end) fetch(0, t0 + 2 * kStep);
        score(1, t0 + kStep);
    }
}

// scores[c][idx] = sum over chunks of planes[chunk][c][idx], in chunk order.
__global__ __launch_bounds__(256) void mfma_sum_planes(const float *__restrict__ planes, int n_chunks,
                                                       size_t chunk_stride, size_t total, float *__restrict__ scores,
                                                       int accumulate) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    float s = 0.f;
    for (int c = 0; c < n_chunks; ++c) s += planes[(size_t)c * chunk_stride + i];
    scores[i] = accumulate ? scores[i] + s : s;        // the planes hold 0 beyond the true length
}

template <int kVariant, typename Lens>
hipError_t launch_sweep2(const ScoreArgs &a, const Lens &lens, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    constexpr int nv = kVariant == OBC_ALL ? 3 : 1;
    hipError_t e;      // (the kernels size their LDS statically: nothing to configure before a launch)
    const size_t plane_elems = (size_t)a.B * a.Hkv * a.N;
    float *dst = ws.n_chunks > 1 ? (float *)(base + ws.planes) : a.scores;
    const size_t chunk_stride = ws.n_chunks > 1 ? plane_elems * nv : 0;
    if (ws.keep_z) {
        score_few_rows<kVariant><<<dim3((a.N + ws.range_len - 1) / ws.range_len, a.B * a.Hkv), dim3(kThreads), 0, stream>>>(
            (const uint16_t *)a.v, a.N, a.G * a.W, a.Hkv, a.ragged, lens, ws.range_len, ws.m_pad, (const float *)(base + ws.z),
            ws.z_stride, (const uint16_t *)(base + ws.out_bf16), (size_t)a.B * a.Hkv * ws.m_pad * kD, (const float *)(base + ws.row_const),
            (const float *)(base + ws.special), dst, plane_elems, a.accumulate);
        e = hipGetLastError();
    } else if (ws.use_wide) {
        e = launch_sweep2_wide(a, ws, base, dst, plane_elems, chunk_stride, stream);
    } else {
        auto launch = [&](auto once) {
            mfma_sweep2<kVariant, once.value><<<sweep_grid(a, lens, ws.n_chunks, ws.range_len), dim3(kThreads), 0, stream>>>(
                (const uint16_t *)a.q, (const uint16_t *)a.k, (const uint16_t *)a.v, a.N, a.W, a.Hq, a.Hkv, a.B * a.Hkv, a.ragged, lens,
                ws.range_len, ws.n_chunks, ws.m_pad, (const uint16_t *)(base + ws.out_bf16), (const float *)(base + ws.row_const),
                (const float *)(base + ws.special), dst, plane_elems, chunk_stride,
                ws.n_chunks == 1 ? a.accumulate : 0);
        };
        if (ws.once2) launch(std::true_type{}); else launch(std::false_type{});
        e = hipGetLastError();
    }
    if (e != hipSuccess || ws.n_chunks == 1) return e;
    const size_t total = plane_elems * nv;
    mfma_sum_planes<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream>>>(dst, ws.n_chunks, chunk_stride, total, a.scores,
                                                                                 a.accumulate);
    return hipGetLastError();
}

}  // namespace

// Tokens one workgroup should take of every KV head's sequence.  `heads` workgroups walk each sequence side by side.  Among
// the shortest shares whose workgroups fit one to sixteen times the compute units, the one with the least estimated time is
// taken, counted in the time a workgroup alone on its compute unit spends on a token:
//   start   what it does before its first and after its last token
//   pairs   two workgroups share a compute unit where there are that many.  Each then takes `shared` times as long for a token,
//           but all together at least what the chip takes to read the tokens: `crowd` times as long where 512 are busy.  (Where
//           the compute unit itself is the limit both are the same.)  `crowd_start` is their start
//   record  what the combine step spends on the partial records of every further 256 workgroups
// First sweep, us, workgroups x tokens: 256 x 128 11.0, 256 x 256 15.6, 256 x 512 22.5, 256 x 1024 38.8, 256 x 2048 69.5,
// 256 x 4096 130; 512 x 256 25.7, 512 x 512 38.7, 512 x 1024 65.7, 512 x 2048 121, and 3 us more in the combine step: one
// round of 256 up to some 1800 tokens, from where on the bytes in flight of a second workgroup pay.  Without output sums 256 x 256
// 8.9, 256 x 512 12.9, 256 x 1024 21.9, 256 x 4096 75; 512 x 512 19.0, 512 x 2048 58.
// (With shares of at least 512 tokens, and else all 512 places filled whatever the length, whole calls took: 8 heads x 8K, all
// 47.7 us, now 44.2; 8 x 2K 40.2, now 31.9; 8 x 1000 38.8, now 28.2; 4 heads x 20000, 224 rows, 64.8, now 60.4.)
struct ShareCost { int unit, start; bool pairs; float shared, crowd; int crowd_start, record; };
// Windows of at most eight rows keep one wave of a workgroup busy, and a second workgroup costs the first less: 8 heads, G = 1,
// 4 x 7429 ragged 25.4 us on 224 workgroups, 21.4 on 448; x 60000, G = 4 52.6 on 240, 44.2 on 472.  The kernel after it always
// wants both places: 18.3 us on 240 workgroups and 14.0 on 352.
// Without output sums, and in the second sweep with 32 rows per wave, the memory is the limit of a second workgroup.  8 heads,
// 30 and 128 rows, us on 256 x 1024 / 512 x 512 / 256 x 1920 / 512 x 1024 tokens: first sweep 18.7 / 12.8 / 32.0 / 22.7 and 25.2 /
// 17.5 / 42.8 / 31.5; second sweep, value 29.8 / 26.3 / 48.2 / 45.4 and 32.8 / 28.8 / 52.6 / 49.7, attention 22.6 / 17.3 / 34.7 /
// 26.4 and 24.7 / 21.5 / 39.1 / 32.7, l1 33.3 / 26.9 / 53.9 / 46.3 and 35.9 / 31.7 / 58.8 / 54.1.  (Estimated as if it were
// the compute unit, 32 heads x 5580, 17 rows, value took 256 workgroups of 704 tokens for the second, 23.3 us, now 480 of 384, 16.6.)
constexpr ShareCost kSweep1Cost = {128, 230, true, 1.79f, 1.79f, 330, 85}, kSweep1SumsCost = {128, 240, true, 1.1f, 1.27f, 260, 10},
                    kSweep1FewCost = {128, 330, true, 1.55f, 1.55f, 400, 10}, kFewRowsCost = {256, 300, true, 1.f, 1.f, 300, 0},
                    kSweep2Cost = {64, 470, true, 1.45f, 1.8f, 430, 0}, kSweep2AttnCost = {64, 680, true, 1.2f, 1.4f, 700, 0},
                    kSweep2VatpCost = {64, 410, true, 1.35f, 1.57f, 430, 0}, kSweep2WideCost = {64, 400, false, 0.f, 0.f, 0, 0},
                    kSweep2SoloCost = {128, 400, false, 0.f, 0.f, 0, 0};
constexpr float kLaunchCost = 80.f;            // of a launch behind another one, 2 us
static bool needs_output(int variant) { return variant == OBC_KEY || variant == OBC_JOINT || variant == OBC_ALL; }
static size_t record_bytes(int m_pad, int variant) { return (size_t)(m_pad < 128 ? m_pad : 128) * (16 + (needs_output(variant) ? kD * 4 : 0)); }
// Row chunks of the same split share K and V in a die's L2 if the splits are a multiple of the eight dies, as 512 or 256
// workgroups over the heads' chunks are wherever the split can be cut finely enough.  (4 heads x 63094, 406 rows, joint: 31 splits
// of 2048 tokens 106.6 us, 32 of 1984, half a step of each for nothing, 101.3.)
static ShareCost sweep1_cost(int variant, int rows) {
    ShareCost c = rows <= kFewRows ? kSweep1FewCost : needs_output(variant) ? kSweep1Cost : kSweep1SumsCost;
    if (rows > 128) c.unit = 64;
    return c;
}
// A call with lengths searches anew, for every layer and token, so shares that cannot fit or cannot win are not counted out: a
// sequence takes at least its tokens over the share and less than one workgroup more, and the estimate grows with the share.
// Host time of an accumulating call through the binding, 8 heads, one window row, us: 8 x 64K 17 (25 with every round searched
// from end to end), 32 x 4K 20 (37), 128 x 4K 35 (69); the shares are the same (1.7 million random batches).
// `record_bytes`: of a workgroup's partial records; with more than the fewest workgroups they take at most kMostRecords, so
// that plans that fit the static scratch go on doing so.
constexpr size_t kMostRecords = (size_t)36 << 20;
// `most_records`: workgroups per KV head and chunk there is room for (at least what the plan's own share takes).
static int even_share(const int *len, int B, int N, int heads, const ShareCost &c, size_t record_bytes = 0, float *least_cost = nullptr,
                      int most_records = 0x7fffffff) {
    constexpr int kUnits = 256;                                                // compute units
    long long tokens = (long long)B * N;
    if (len) {
        tokens = 0;
        for (int b = 0; b < B; ++b) tokens += len[b];
    }
    auto workgroups = [&](int share) {
        long long n = 0;
        if (!len) return (long long)heads * B * ((N + share - 1) / share);
        for (int b = 0; b < B; ++b) n += (unsigned)(len[b] + share - 1) / (unsigned)share;
        return n * heads;
    };
    auto cost = [&](int share, int rounds) {                                   // on (rounds - 1) * kUnits + 1 .. rounds * kUnits workgroups
        const float records = (float)c.record * (float)rounds;
        if (c.pairs && rounds > 1) {
            const float turns = (float)((rounds + 1) / 2);
            return std::max(turns * c.shared * share, c.crowd * heads * tokens / (2 * kUnits)) + turns * c.crowd_start + records;
        }
        return (float)rounds * (float)(share + c.start) + records;
    };
    auto rounds_of = [&](int share) { return (int)((workgroups(share) + kUnits - 1) / kUnits); };
    const int most = (N + c.unit - 1) / c.unit, fewest = rounds_of(most * c.unit);
    int best = 0, hi = most;                                                   // (hi: fits)
    float best_cost = 0.f;
    for (int rounds = fewest < 1 ? 1 : fewest; rounds <= 16; ++rounds) {
        // The shortest share that fits; one that fits fewer rounds, too, has been looked at with them.
        // (workgroups per KV head and chunk)
        const long long fit = std::min((long long)rounds * kUnits / heads, (long long)most_records);
        int lo = (int)((tokens + fit * c.unit - 1) / (fit * c.unit));
        if (lo < 1) lo = 1;
        if (fit > B) {                                                         // (a sequence takes less than one more than its tokens over the share)
            const long long enough = (tokens + (fit - B) * c.unit - 1) / ((fit - B) * c.unit);
            if (enough < hi) hi = (int)(enough < lo ? lo : enough);
        }
        auto wins = [&](int units) { return best == 0 || cost(units * c.unit, rounds) < best_cost; };
        int top = hi;
        while (lo < top && wins(lo)) {
            const int mid = (lo + top) / 2;
            if (workgroups(mid * c.unit) <= fit * heads) top = mid; else lo = mid + 1;
        }
        if (lo < top || !wins(lo)) continue;
        const int share = lo * c.unit;
        if (best != 0 && workgroups(share) * record_bytes > kMostRecords) break;
        const float t = cost(share, rounds_of(share));
        if (best == 0 || t < best_cost) { best = share; best_cost = t; }
        if (lo == 1 || fit == most_records) break;
        hi = lo;
    }
    if (!best) { best = most * c.unit; best_cost = cost(best, fewest); }       // more sequences than sixteen rounds: one workgroup each
    if (least_cost) *least_cost = best_cost;
    return best;
}

void mfma_plan(int B, int N, int W, int Hq, int Hkv, int d, int variant, ScoreWorkspace *ws, size_t *off) {
    auto align_up = [](size_t x, size_t a) { return (x + a - 1) / a * a; };
    const int BH = B * Hkv;
    const int nv = variant == OBC_ALL ? 3 : 1;
    const int M = Hq / Hkv * W, form = tuned_sweep2_form();
    ws->n_chunks = (ws->m_pad + 127) / 128;
    ws->split_len = even_share(nullptr, B, N, Hkv * ws->n_chunks, sweep1_cost(variant, M), record_bytes(ws->m_pad, variant));
    if (const int v = tuned_splits(); v >= 1 && v <= (N + 511) / 512)           // obc_set_score_tuning
        ws->split_len = ((N + v - 1) / v + kTileTok - 1) / kTileTok * kTileTok;
    ws->splits = (N + ws->split_len - 1) / ws->split_len;
    ws->use_wide = form != 1 && sweep2_wide_covers(variant) ? 1 : 0;
    ws->solo = ws->use_wide && (M - 1) % 128 < 64 ? 1 : 0;
    ws->z_stride = (N + 31) / 32 * 32;
    const size_t rows = (size_t)BH * ws->m_pad, first = *off, z_bytes = (size_t)BH * M * ws->z_stride * sizeof(float);
    ws->keep_z = 0;
    auto lay_out = [&](int records) {
        size_t at = first;
        const size_t record_rows = (size_t)Hkv * records * ws->m_pad;
        ws->records = records;
        ws->out_bf16 = at;  at = align_up(at + 2 * rows * d * 2, 256);      // high pieces, then residual pieces
        ws->row_const = at; at = align_up(at + rows * 4 * sizeof(float), 256);
        ws->part_ml = at;   at = align_up(at + record_rows * 4 * sizeof(float), 256);
        ws->special = at;   at = align_up(at + rows * 4 * sizeof(float), 256);
        ws->part_o = at;
        if (needs_output(variant)) at = align_up(at + record_rows * d * sizeof(float), 256);
        ws->planes = at;
        if (ws->n_chunks > 1) at = align_up(at + (size_t)ws->n_chunks * nv * BH * N * sizeof(float), 256);
        ws->z = at;
        if (ws->keep_z) at = align_up(at + z_bytes, 256);
        return at;
    };
    *off = lay_out(B * ws->splits);
    // With few rows the first sweep keeps their logits (4 bytes per pair) and the second reads them instead of K (256 bytes
    // per token): beyond eight rows the gain fades.  Only within the static scratch, so that a call has the same plan, and
    // with it the same bits, on either scratch; and not where a form of the second sweep is asked for (obc_set_sweep2_form).
    ws->keep_z = form == 0 && M <= kFewRows && *off + z_bytes <= OBC_STATIC_SCRATCH_BYTES && (long long)M * ws->z_stride < (1LL << 29) ? 1 : 0;    // (32-bit offsets)
    if (ws->keep_z) {
        *off = lay_out(B * ws->splits);
        ws->use_wide = ws->solo = 0;
    }
    // A call's lengths may want two workgroups per compute unit where full ones want one.  Room for those, unless the plan would
    // no longer fit the static scratch.  (With B * splits records: 2 x 8 heads of 42588 and 26618 tokens, 30 rows, all, took
    // splits of 2688 tokens instead of 1152, 59.9 us instead of 49.9 in the first sweep; 3 x 4 of 27688 to 55376, 98 rows, key,
    // 77 and 62; 4 x 8 of 7324 to 16739, 30 rows, l1, 23 and 18.)
    const int unit = sweep1_cost(variant, M).unit;
    const int two_rounds = (int)std::min(512ll / (Hkv * ws->n_chunks), (long long)B * ((N + unit - 1) / unit));
    if (two_rounds > ws->records && tuned_splits() == 0) {
        const size_t fewest = *off;
        *off = lay_out(two_rounds);
        if (*off > OBC_STATIC_SCRATCH_BYTES && fewest <= OBC_STATIC_SCRATCH_BYTES) *off = lay_out(B * ws->splits);
    }
}

// Whether a sweep marks its reads of K and V (of K alone without `with_v`) as non-temporal.  It does where nobody reads them
// again soon: not with several row chunks, whose workgroups meet in a die's L2, and not where the memory-side cache of 256 MB
// holds them for the second sweep.  Time with both sweeps marked over neither, 1200 random calls on inputs that change from call to
// call, geometric means by MB of K and V:
//                                        -20    20-40   40-80  80-150 150-210 210-268 268-350 350-500  500-
//   9 to 64 rows, with outputs          1.091   1.067   1.032   1.026   1.028   1.020   1.008   0.950   0.919
//                 value and l1          1.004   1.012   1.005   1.003   1.005   1.017   1.011   0.957   0.931
//                 attention alone       1.030   1.009   1.006   1.005   1.007   1.002   0.976   0.991   0.963
//   65 to 128 rows, with outputs        1.081   1.051   1.040   1.030   1.016   1.006   0.995   0.996   0.991
//                 value and l1          1.005   1.006   0.993   0.996   1.006   1.037   1.016   0.992   0.961
//                 attention alone       1.029   1.016   0.996   1.008   0.999   1.012   1.013   1.027   0.994
//   more rows, with outputs             1.035   1.021   1.019   1.023   1.033   1.037   1.046   1.008
// Value and l1 read K first: from 210 to 400 MB the first sweep leaves it in the cache and the second one marks its reads, 3 % less than
// neither (101.5 / 97.4 us: 2 x 8 heads x 43904, 128 rows, value).  Attention alone with at most 64 rows, its second sweep bound by the
// read, has the mark from 80 MB of K on: 32 heads x 14080, 49.9 / 48.8 us.  Windows of few rows always have it: the same cache comes again
// for every token (4 rows, same inputs: joint, 268 MB 82 / 89 marked / not; value, 201 MB 44 / 48).
constexpr long long kCachedBytes = 256ll << 20, kCachedBytesValue = 200ll << 20, kCachedBytesAttn = 80ll << 20;
static int reads_once(const ScoreArgs &a, const ScoreWorkspace &ws, bool with_v) {
    const int rows = a.G * a.W;
    if (ws.n_chunks > 1) return 0;
    if (ws.keep_z || rows <= kFewRows) return 1;
    long long tokens = (long long)a.B * a.N;
    if (a.ragged) {
        tokens = 0;
        for (int b = 0; b < a.B; ++b) tokens += a.lens.len[b];
    }
    const long long cached = needs_output(a.variant) ? kCachedBytes : a.variant == OBC_ATTN && rows <= 64 ? kCachedBytesAttn : kCachedBytesValue;
    return tokens * a.Hkv * kRowBytes * (with_v ? 2 : 1) > cached;
}

// The shares of this call's true lengths (the plan knows only N): shorter splits as far as they fit the workspace, whose
// records lie one sequence after the other (see split_slot), and the second sweep's ranges.
static ScoreWorkspace mfma_balance(const ScoreArgs &a, ScoreWorkspace ws) {
    const int *len = a.ragged ? a.lens.len : nullptr;
    if (len && tuned_splits() == 0) {
        ws.split_len = even_share(len, a.B, a.N, a.Hkv * ws.n_chunks, sweep1_cost(a.variant, a.G * a.W), record_bytes(ws.m_pad, a.variant),
                                  nullptr, ws.records);
        ws.splits = 1;
        for (int b = 0; b < a.B; ++b) ws.splits = std::max(ws.splits, (len[b] + ws.split_len - 1) / ws.split_len);
    }
    int full = ws.n_chunks - ws.solo;
    float wide = 0.f, solo = 0.f, padded = 0.f;
    const ShareCost &cost = ws.keep_z ? kFewRowsCost : ws.use_wide ? kSweep2WideCost
                            : a.variant == OBC_ATTN ? kSweep2AttnCost : a.variant == OBC_VATP ? kSweep2VatpCost : kSweep2Cost;
    if (full > 0) ws.range_len = even_share(len, a.B, a.N, a.Hkv * full, cost, 0, &wide);        // (kFewRowsCost: whole steps of its workgroups)
    if (ws.solo) ws.range_solo = even_share(len, a.B, a.N, a.Hkv, kSweep2SoloCost, 0, &solo);
    // A last chunk of at most 64 rows behind full ones: a launch of its own spends 0.7 of the time on a token and a start of its
    // own; on short prompts that start costs more than the empty half of a 128-row chunk.  408 rows, 4 x 4 heads x 3507 ragged,
    // key: 27.9 + 12.7 us, as four chunks 32.1; 168 rows, 4 heads x 20000, all: 21.0 + 16.0, as two 29.8; x 60000, joint: 39.9 +
    // 29.0, as two 66.5.
    if (ws.solo && full > 0) {
        const int range = even_share(len, a.B, a.N, a.Hkv * ws.n_chunks, cost, 0, &padded);
        if (padded < wide + 0.7f * solo + kLaunchCost) { ws.solo = 0; ws.range_len = range; }
    }
    ws.once1 = reads_once(a, ws, needs_output(a.variant));
    ws.once2 = reads_once(a, ws, a.variant != OBC_ATTN);
    if (ws.keep_z) return ws;
    if (const int v = tuned_range(); v >= 64 && v <= 65536 && v % 64 == 0) ws.range_len = ws.range_solo = v;
    return ws;
}

template <typename Lens>
static hipError_t launch_with(const ScoreArgs &a, const Lens &lens, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    const bool need_o = needs_output(a.variant);
    float *part_ml = (float *)(base + ws.part_ml), *part_o = (float *)(base + ws.part_o);
    hipError_t e = hipSuccess;
    if (a.stage_mask & OBC_STAGE_SWEEP1) {
        const dim3 grid = sweep_grid(a, lens, ws.n_chunks, ws.split_len);
#define OBC_SWEEP1(need_o, store_z, once)                                                                              \
    mfma_sweep1<need_o, store_z, once><<<grid, dim3(kThreads), 0, stream>>>(                                                 \
        (const uint16_t *)a.q, (const uint16_t *)a.k, (const uint16_t *)a.v, a.N, a.W, a.Hq, a.Hkv, a.ragged, lens,      \
        ws.split_len, ws.n_chunks, ws.m_pad, part_ml, part_o, (float *)(base + ws.z), ws.z_stride)
        if (need_o && ws.keep_z) OBC_SWEEP1(true, true, true);
        else if (need_o && ws.once1) OBC_SWEEP1(true, false, true);
        else if (need_o) OBC_SWEEP1(true, false, false);
        else if (ws.keep_z) OBC_SWEEP1(false, true, true);
        else if (ws.once1) OBC_SWEEP1(false, false, true);
        else OBC_SWEEP1(false, false, false);
#undef OBC_SWEEP1
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.stage_mask & OBC_STAGE_COMBINE) {
        // (score_few_rows reads nothing of the padded rows; the other second sweeps do)
        const int combine_rows = ws.keep_z ? a.G * a.W : ws.m_pad;
#define OBC_COMBINE(groups, batch, rows)                                                                               \
    mfma_combine_hold<groups, batch><<<dim3((combine_rows + rows - 1) / rows, a.B * a.Hkv), dim3(32 * groups * rows), 0, stream>>>(            \
        (const uint16_t *)a.v, part_ml, part_o, a.N, a.W, a.G * a.W, a.Hkv, a.ragged, lens, ws.split_len, ws.splits, ws.m_pad,         \
        (uint16_t *)(base + ws.out_bf16), (float *)(base + ws.row_const), (float *)(base + ws.special))
        if (need_o && ws.splits <= 16) OBC_COMBINE(1, 16, 4);      // (m_pad: a multiple of 32)
        else if (need_o && ws.splits <= 32) OBC_COMBINE(4, 8, 1);
        else if (need_o && ws.splits <= 64) OBC_COMBINE(8, 8, 1);
        else if (need_o) OBC_COMBINE(8, 16, 1);
#undef OBC_COMBINE
        else
            mfma_combine<<<dim3((combine_rows + 15) / 16, a.B * a.Hkv), dim3(256), 0, stream>>>(
                part_ml, a.N, a.W, a.Hq, a.Hkv, a.ragged, lens, ws.split_len, ws.m_pad, (float *)(base + ws.row_const),
                (float *)(base + ws.special));
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!(a.stage_mask & OBC_STAGE_SWEEP2)) return hipSuccess;
    switch (a.variant) {
        case OBC_VALUE: return launch_sweep2<OBC_VALUE>(a, lens, ws, base, stream);
        case OBC_KEY: return launch_sweep2<OBC_KEY>(a, lens, ws, base, stream);
        case OBC_JOINT: return launch_sweep2<OBC_JOINT>(a, lens, ws, base, stream);
        case OBC_ATTN: return launch_sweep2<OBC_ATTN>(a, lens, ws, base, stream);
        case OBC_VATP: return launch_sweep2<OBC_VATP>(a, lens, ws, base, stream);
        default: return launch_sweep2<OBC_ALL>(a, lens, ws, base, stream);
    }
}

hipError_t launch_score_mfma(const ScoreArgs &a, const ScoreWorkspace &plan, char *base, hipStream_t stream) {
    const ScoreWorkspace ws = mfma_balance(a, plan);
    return with_lens(a.ragged, a.B, a.lens, [&](const auto &lens) { return launch_with(a, lens, ws, base, stream); });
}

}  // namespace obc
