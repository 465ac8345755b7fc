// Second sweep of the matrix-core scoring path, register-blocked form for the variants that need
// the cross term v_p . o_i (Eq. 5, Eq. 6, and all three scores at once).
//
// Same mathematics as mfma_sweep2 (score_mfma.hip): per (window row i, token p) the logit Z_ip
// and -2 v_p.o^_i come off the matrix cores with tokens on the lane axis, A_ip^2 and the terms
// of Eq. 4-6 are formed in fp32, and the sum over window rows and query heads (Eq. 9,
// Appendix A.5) runs down accumulator registers.  What differs is the blocking:
//
//   * One workgroup per compute unit, one wave per SIMD.  A wave owns 64 window rows (two
//     32-row sets, A and B) and one 32-token block of every 64-token tile, so each K/V operand
//     piece read from LDS feeds two matrix ops instead of one, and ||v_p||^2 is formed once
//     per 64 rows instead of once per 32.
//   * The wave's 192 registers of stationary operands (Q and the two bf16 pieces of o_i for
//     its 64 rows) live in the accumulator half of the register file.  The matrix ops read
//     them from there directly (inline assembly: the compiler would otherwise copy each
//     operand into the other half before every matrix op), and so they do with the streamed
//     K pieces, leaving the architectural registers to accumulators, row constants and the
//     streamed V pieces.
//   * With one wave per SIMD the overlap of matrix cores and vector ALUs comes from a
//     software pipeline inside the wave: while the matrix cores form set A's logits and
//     cross terms of block n, the vector ALUs score set B of block n-1; then the roles swap.
//     The two streams are interleaved slot by slot (one matrix op, then a slice of the vector
//     work) and the compiler's scheduler is kept from moving anything across a slot boundary.
//   * K and V tiles travel HBM -> LDS through a ring of four 32 KB slots, three tiles in
//     flight per compute unit.
//
// What bounds it: no one thing.  4 x 8 heads x 32K, 128 rows, joint, us, leaving parts out: as it is 131.7; transfers served
// from the L2 130.0; no transfers 113.1; no matrix ops 91.2; no vector tasks 115.3; neither 91.8, what the ring takes to read
// the cache.  Cycles of a wave per block, of 3608: phase 1 1496, phase 2 1001 (768 of each are matrix ops), between them 327,
// bookkeeping and flush 334, tail 283, barrier 115, wait for the ring 44.  The eight transfers cost their issue in phase 1, and
// the matrix cores idle outside the phases.
//
// Blocks that hold a causally hidden (row, key) pair, the ragged end of a sequence or a
// separately scored pair run the same pipeline with the masks applied to every pair.
// All sums have a fixed order: results are bit-reproducible.
#include "internal.h"
#include "mfma_util.h"
#include "wave_util.h"

#include <type_traits>

namespace obc {
using namespace mfma;
namespace {

typedef const __attribute__((address_space(3))) char *lds_ptr;

constexpr int kSlots = 4;                       // tiles in the ring
constexpr int kSlotBytes = 2 * kTileBytes;      // 32 KB: a K tile, then the V tile of the same 64 tokens
constexpr int kRing = kSlots * kSlotBytes;      // 128 KB
constexpr int kTilePerWave = 8;                 // direct-to-LDS transfers a wave issues per tile (4 K + 4 V)

// acc = A * B (first op of a chain) and acc += A * B, with the 16-byte A operand in four accumulator-file registers.  B is
// there, too, where it is a piece of K, which only matrix ops read; a piece of V is in architectural ones, as its norm is formed
// from it.  (With K in those as well mfma_sweep2_solo ran out of them and fetched 7 to 8 values per block back from the
// accumulator file for the joint score and all three, which no time showed: 4 x 8 heads x 32K, 64 rows, joint, 90.8 us then and
// 91.2 now, all 99.)
__device__ __forceinline__ void mma_k_first(f32x16 &acc, const f32x4 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "a"(a), "a"(b));
}
__device__ __forceinline__ void mma_k_next(f32x16 &acc, const f32x4 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "a"(a), "a"(b));
}
__device__ __forceinline__ void mma_v_first(f32x16 &acc, const f32x4 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "a"(a), "v"(b));
}
__device__ __forceinline__ void mma_v_next(f32x16 &acc, const f32x4 &a, const bf16x8 &b) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "a"(a), "v"(b));
}
// Reads a 16-byte operand from LDS into the accumulator file, where it stays: parked() ties it there, which lets the compiler
// load it in place and makes it wait for the load.  (One instruction each: through architectural registers it were five, in a
// part of the kernel where every instruction is fetched for the first time.)
template <int kOffset>
__device__ __forceinline__ void park(f32x4 &x, lds_ptr p) {
    static_assert(kOffset >= 0 && kOffset < 65536, "16 bits of offset");
    x = *(const __attribute__((address_space(3))) f32x4 *)(p + kOffset);
}
__device__ __forceinline__ void parked(f32x4 &x) { asm volatile("" : "+a"(x)); }
// The matrix ops above are opaque to the compiler, which therefore cannot count the cycles a
// vector instruction must keep away from a matrix op's result (the last pass of a 32x32x16 op
// lands ten issue slots after the op).  Wherever vector code may follow a matrix op closely,
// this spends those slots explicitly.
__device__ __forceinline__ void matrix_results_land() { asm volatile("s_nop 7\n\ts_nop 4" ::: "memory"); }

// Ties a value to this point of the instruction stream (no instruction is emitted): the compiler's passes would
// otherwise gather the vector work that is spread between the matrix ops next to its first use.  The value only goes in:
// were it also an output, the compiler would put a wait slot in front of an instruction that reads it next (it cannot see
// what kind of write the assembly is), 45 of them per block.
__device__ __forceinline__ void stay(float x) { asm volatile("" ::"v"(x)); }

__device__ __forceinline__ bf16x8 lds_piece(lds_ptr p, int imm) {
    return *(const __attribute__((address_space(3))) bf16x8 *)(p + imm);
}

// Constants of a row set S, one pair per accumulator register: 2 (max + log2 sum) and ||o^||^2 / 128 of register r's row.
// They stay in registers: read from LDS as they are needed they took 16 reads and as many waits of the block's 660
// instructions, and a lone wave pays for each the same.
struct RowConsts { float m2[2][16], oo[2][16]; };
// From the rows' row_const in LDS; `p`: the lane's first row.
__device__ __forceinline__ RowConsts row_consts(lds_ptr p) {
    typedef const __attribute__((address_space(3))) float *lds_float_ptr;
    RowConsts c;
#pragma unroll
    for (int S = 0; S < 2; ++S)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const lds_float_ptr x = (lds_float_ptr)(p + (32 * S + 8 * (r >> 2) + (r & 3)) * 16);
            c.m2[S][r] = x[0];
            c.oo[S][r] = x[1];
        }
    return c;
}

struct Stationary {          // per 32-row set S: Q, high and residual pieces of -2 o^ (accumulator file)
    f32x4 q[2][8], hi[2][8], lo[2][8];
    __device__ __forceinline__ void tie() {
#pragma unroll
        for (int S = 0; S < 2; ++S)
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) { parked(q[S][kk]); parked(hi[S][kk]); parked(lo[S][kk]); }
    }
};

struct WideState {
    f32x16 zA, voA, zB, voB;             // logits and cross terms of the two row sets
    bf16x8 kreg[8], vreg[8];             // this lane's operand pieces of the current block (K: accumulator file)
    lds_ptr kp[8];                       // LDS address of operand piece kk of this lane's block in the tile read next
    RowConsts rc;
    float sv, sk, sj;                    // set A's sums of the block whose set B is still due
    float vv_prev;                       // ||v_p||^2 (or ||v_p||_1) of that block's token
    bool pend;                           // uniform: set B of the previous block is still due
};

// The vector work for one accumulator register (one (row, token) pair per lane), cut into three tasks of about equal
// cost so that it can be dealt evenly over the slots between the matrix ops.  With z the raw dot product
// (Z = z / sqrt(128)), vo = -2 v_p.o^_i / 128 and oo = ||o^_i||^2 / 128 (see kCrossScale):
//   task 0   A^2 = exp2(2 log2e Z - m2)
//   task 1   w7 = ||v_p - o^_i||^2 / 128 = (||v_p||^2 / 128 + oo) + vo,   sg = 2 ||v_p||^2 / sqrt(128) + sqrt(128) vo
//   task 2   Eq. 5 term  A^2 Z^2 w = A^2 z^2 w7
//            Eq. 6 term  A^2 ||(1+Z) v - Z o^||^2 = A^2 (||v||^2 + z (sg + z w7))
struct TokenConsts { float vv, vv7, vv2s; };      // ||v_p||^2, that / 128, 2 ||v_p||^2 / sqrt(128)
__device__ __forceinline__ TokenConsts token_consts(float vv) { return {vv, vv * kCrossScale, vv * (2.0f * kInvSqrtD)}; }
struct PairWork { float a2, w7, sg; };
template <int kVariant>
__device__ __forceinline__ void pair_task(int task, PairWork &p, float z, float vo, float m2, float oo, const TokenConsts &t,
                                          float &acc_v, float &acc_k, float &acc_j) {
    constexpr bool kDoV = kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    if (task == 0) {
        p.a2 = __builtin_amdgcn_exp2f(fmaf(z, 2.0f * kLog2e * kInvSqrtD, -m2));
        stay(p.a2);
    } else if (task == 1) {
        p.w7 = (t.vv7 + oo) + vo;
        stay(p.w7);
        if (kDoJ) { p.sg = fmaf(vo, kSqrtD, t.vv2s); stay(p.sg); }
    } else {
        if (kDoV) { acc_v += p.a2; stay(acc_v); }
        if (kDoK) { acc_k = fmaf(p.a2 * z * z, p.w7, acc_k); stay(acc_k); }
        if (kDoJ) { acc_j = fmaf(p.a2, fmaf(z, fmaf(z, p.w7, p.sg), t.vv), acc_j); stay(acc_j); }
    }
}

// Adds the two row sets' sums of one block, folds the wave's halves (lanes l and l + 32 hold the same token) and
// parks the wave's 32 partial scores in the staging slot of the block's tile: [row half][variant][64 tokens].
template <int kVariant>
__device__ __forceinline__ void park_block(float *stage_slot, int rh, int th, int lane, float vv, float av, float ak,
                                           float aj, float bv, float bk, float bj) {
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    constexpr bool kDoV = kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    float sv = 0.f, sk = 0.f, sj = 0.f;
    if (kDoV) sv = halves_sum((av + bv) * vv);
    if (kDoK) sk = fmaxf(halves_sum(ak + bk), 0.f);      // (rounding can leave a sum a hair below zero)
    if (kDoJ) sj = fmaxf(halves_sum(aj + bj), 0.f);
    if (lane < 32) {
        float *pw = stage_slot + rh * kNv * 64 + th * 32 + lane;
        int c = 0;
        if (kDoV) pw[64 * c++] = sv;
        if (kDoK) pw[64 * c++] = sk;
        if (kDoJ) pw[64 * c++] = sj;
    }
}

// Adds the two row halves' partial scores of one tile (64 tokens from `tok0`) and writes them out; wave c handles
// variant c.
template <int kNv>
__device__ __forceinline__ void flush_tile(const float *stage_slot, float *out, size_t variant_stride, int tok0,
                                           int t_end, int wave, int lane, bool accumulate) {
    if (wave < kNv && tok0 + lane < t_end) {
        const float *p = stage_slot + wave * 64 + lane;
        float *o = out + wave * variant_stride + tok0 + lane;
        const float sum = p[0] + p[kNv * 64];
        *o = accumulate ? *o + sum : sum;
    }
}

// Vector work of one row set of one block outside the pipeline (the last block's second set).
template <int kVariant>
__device__ __forceinline__ void score_set(const f32x16 &z, const f32x16 &vo, const RowConsts &c, int S, float vv, float &av,
                                          float &ak, float &aj) {
    const TokenConsts t = token_consts(vv);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        PairWork p;
#pragma unroll
        for (int task = 0; task < 3; ++task) pair_task<kVariant>(task, p, z[r], vo[r], c.m2[S][r], c.oo[S][r], t, av, ak, aj);
    }
}

// The 24 matrix ops of row set S on the block held in (kreg, vreg): slot j issues op j, then runs `work(j)`.
template <int S, typename Work>
__device__ __forceinline__ void matrix_phase(const Stationary &A, f32x16 &z, f32x16 &vo, const bf16x8 (&kreg)[8],
                                             const bf16x8 (&vreg)[8], Work &&work) {
#pragma unroll
    for (int j = 0; j < 24; ++j) {
        if (j == 0) mma_k_first(z, A.q[S][0], kreg[0]);
        else if (j < 8) mma_k_next(z, A.q[S][j], kreg[j]);
        else if (j == 8) mma_v_first(vo, A.hi[S][0], vreg[0]);
        else if (j & 1) mma_v_next(vo, A.lo[S][(j - 8) >> 1], vreg[(j - 8) >> 1]);
        else mma_v_next(vo, A.hi[S][(j - 8) >> 1], vreg[(j - 8) >> 1]);
        work(j);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Pairs that must not count (causally hidden, past the sequence's end, or scored separately) get a logit so low that
// their weight is exactly 0, and low enough only for that: every product formed from it stays finite.  Applied to the
// logits of row set S of one block (lane's token `tok`) between the matrix ops that formed them and their scoring.
__device__ __forceinline__ void hide_pairs(f32x16 &z, int S, int tok, int t_end, int rh, int half, const int *vis_i,
                                           const int *excl_i) {
    typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int i0 = rh * 64 + 32 * S + 8 * g + 4 * half;             // four consecutive rows of the 128-row chunk
        const i32x4 vis = *(const i32x4 *)(vis_i + i0), excl = *(const i32x4 *)(excl_i + i0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (tok > vis[e] || tok >= t_end || tok == excl[e]) z[4 * g + e] = kHiddenLogit;
    }
}

// Blocks of 32 tokens (counted from the workgroup's first) that hold a separately scored pair, one bit each, folded at
// kSpecialWords * 32 blocks: a block that is taken for one of them without need only costs its masks.  (With needles all
// over a long context nearly every block lies between the first and the last such pair of a range.)
constexpr int kSpecialWords = 32;
__device__ __forceinline__ int special_word(int blk) { return blk >> 5 & (kSpecialWords - 1); }
__device__ __forceinline__ bool special_bit(uint32_t word, int blk) {
    return __builtin_amdgcn_readfirstlane((int)word) >> (blk & 31) & 1;
}

// Sum of squares of dwords 2 q and 2 q + 1 (four bf16 values) of a 16-byte operand piece.
__device__ __forceinline__ float sumsq_quarter(const bf16x8 x, int q, float acc) {
    union { bf16x8 v; bf16x2 h[4]; } u;
    u.v = x;
    acc = __builtin_amdgcn_fdot2_f32_bf16(u.h[2 * q], u.h[2 * q], acc, false);
    return __builtin_amdgcn_fdot2_f32_bf16(u.h[2 * q + 1], u.h[2 * q + 1], acc, false);
}

// What a wave needs to start one of its eight transfers of the tile that is fetched during a step.  Transfers of one
// tensor lie 1 KB apart in LDS: the instruction's offset moves their memory address along, which the lane's offset takes
// back, so that the LDS address register m0 is written once per tensor (a write, its wait slot and the addition that makes the
// address, for every transfer, were 24 instructions per block).  Every transfer names m0 as its operand and brings the wait
// slot that a write just before it would need; the compiler leaves out the writes that change nothing.  kBias keeps the lane
// offsets from falling below zero.
constexpr int kBias = 4096;
struct TileFetch {
    const char *k_base, *v_base;     // kBias bytes ahead of the tile's first row in K and in V (uniform)
    uint32_t voff[4];                // per-lane byte offset of transfer n inside the tile + kBias - 1024 n (rows past the end clamped)
    uint32_t lds;                    // LDS byte address of the ring slot (K tile; the V tile follows), this wave's first transfer
};
template <int kSlot, bool kOnce>
__device__ __forceinline__ void transfer_at(const char *sbase, uint32_t voff, uint32_t lds) {
    if constexpr (kOnce) asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3 nt" ::"{m0}"(lds), "v"(voff), "s"(sbase), "n"(kSlot * 1024) : "memory");
    else asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" ::"{m0}"(lds), "v"(voff), "s"(sbase), "n"(kSlot * 1024) : "memory");
}
template <bool kOnce>
__device__ __forceinline__ void fetch_one(const TileFetch &f, int n) {       // n = 0..3: K, 4..7: V, in this order
    const char *base = n < 4 ? f.k_base : f.v_base;
    const uint32_t lds = f.lds + (n < 4 ? 0 : kTileBytes);
    switch (n & 3) {
        case 0: return transfer_at<0, kOnce>(base, f.voff[0], lds);
        case 1: return transfer_at<1, kOnce>(base, f.voff[1], lds);
        case 2: return transfer_at<2, kOnce>(base, f.voff[2], lds);
        default: return transfer_at<3, kOnce>(base, f.voff[3], lds);
    }
}
// All four transfers a wave issues for 64 rows from row `row0` of `rows`; rows past `last` (>= row0) re-read it.  `lds`: this
// wave's first one.  Short code: what a kernel runs once costs its instructions' way from memory (see mfma_sweep2_wide).
template <bool kOnce>
__device__ __forceinline__ void load_64_rows(const char *rows, int row0, int last, uint32_t lds, const uint32_t (&moff)[4], int wave, int lane) {
    const char *base = rows + (size_t)row0 * kRowBytes - kBias;
    uint32_t voff[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) voff[n] = moff[n] - (uint32_t)(max((wave * 4 + n) * 4 + (lane >> 4) - (last - row0), 0) * kRowBytes);
    transfer_at<0, kOnce>(base, voff[0], lds);
    transfer_at<1, kOnce>(base, voff[1], lds);
    transfer_at<2, kOnce>(base, voff[2], lds);
    transfer_at<3, kOnce>(base, voff[3], lds);
}
// Zeros for rows `from` .. 63 of a 64-row tile in LDS, whatever its swizzle (256 threads).
__device__ __forceinline__ void zero_rows(char *tile, int from) {
#pragma unroll 1
    for (int e = max(from, 0) * (kRowBytes / 16) + (int)threadIdx.x; e < kTileBytes / 16; e += kThreads) ((uint4 *)tile)[e] = make_uint4(0, 0, 0, 0);
}

// The pipelined work of one wave on one block (32 tokens, lane's token `tok`), operands already in registers:
//   phase 1: matrix cores on set A of this block, vector ALUs on set B of the block before;
//   phase 2: matrix cores on set B of this block, vector ALUs on set A of it; each operand piece is replaced by the
//            next block's (R.kp points into the next tile) as soon as its last matrix op has been issued.
// A phase has 24 slots (one matrix op each) and 48 vector tasks (three per accumulator register): slot j runs tasks
// 2 j and 2 j + 1.  Phase 1 also forms ||v_p||^2 of this block (two dot-product ops in each of the first 16 slots) and
// starts the wave's eight transfers of the tile three steps ahead (one in each of the last eight slots).
// `hidden`: some (row, key) pair of this block is causally hidden or past the sequence's end; `special`: the bits of its
// group of 32 blocks (see special_word).
template <int kVariant, bool kOnce>
__device__ __forceinline__ void pipelined_block(WideState &R, const Stationary &A, const TileFetch &fetch, float *stage_prev,
                                                int tok, int t_end, int rh, int th, int wave, int lane, int blk, bool hidden,
                                                uint32_t special, const int *vis_i, const int *excl_i) {
    const int half = lane >> 5;
    float vvn = 0.f, bv = 0.f, bk = 0.f, bj = 0.f;
    const TokenConsts tp = token_consts(R.vv_prev);
    PairWork pw[16];
    matrix_phase<0>(A, R.zA, R.voA, R.kreg, R.vreg, [&](int j) __attribute__((always_inline)) {
        if (j < 16) { vvn = sumsq_quarter(R.vreg[j >> 1], j & 1, vvn); stay(vvn); }
        else fetch_one<kOnce>(fetch, j - 16);
#pragma unroll
        for (int t = 2 * j; t < 2 * j + 2; ++t) {
            const int r = t / 3;
            pair_task<kVariant>(t % 3, pw[r], R.zB[r], R.voB[r], R.rc.m2[1][r], R.rc.oo[1][r], tp, bv, bk, bj);
        }
    });
    // (unconditional, so that the vector work above stays where it is: with no block before, `stage_prev` is a spare slot)
    park_block<kVariant>(stage_prev, rh, th, lane, tp.vv, R.sv, R.sk, R.sj, bv, bk, bj);
    const bool masks = hidden || special_bit(special, blk);
    if (masks) {                                               // uniform for the wave, rare
        matrix_results_land();
        hide_pairs(R.zA, 0, tok, t_end, rh, half, vis_i, excl_i);
    }
    const TokenConsts tc = token_consts(halves_sum(vvn));
    float av = 0.f, ak = 0.f, aj = 0.f;
    matrix_phase<1>(A, R.zB, R.voB, R.kreg, R.vreg, [&](int j) __attribute__((always_inline)) {
        if (j < 8) R.kreg[j] = lds_piece(R.kp[j], 0);
        else if (j & 1) R.vreg[(j - 8) >> 1] = lds_piece(R.kp[(j - 8) >> 1], kTileBytes);
#pragma unroll
        for (int t = 2 * j; t < 2 * j + 2; ++t) {
            const int r = t / 3;
            pair_task<kVariant>(t % 3, pw[r], R.zA[r], R.voA[r], R.rc.m2[0][r], R.rc.oo[0][r], tc, av, ak, aj);
        }
    });
    if (masks) {
        matrix_results_land();
        hide_pairs(R.zB, 1, tok, t_end, rh, half, vis_i, excl_i);
    }
    R.sv = av; R.sk = ak; R.sj = aj;
    R.vv_prev = tc.vv;
    R.pend = true;
}

// The workgroups of a launch walk their token ranges in step, and ranges start at multiples of a large power of two:
// walking every range front to back would send all compute units to the same few memory channels at any moment.
// Each workgroup therefore starts at its own tile and wraps around (the order of tokens is free: every token's score
// is a sum over rows).  Tile visited at position t of the walk (t may run past the end: the ring prefetches ahead).
__device__ __forceinline__ int tile_at(int t, int first, int n_tiles) {
    int a = t + first;
    while (a >= n_tiles) a -= n_tiles;      // uniform; at most a few rounds
    return a;
}
__device__ __forceinline__ int next_tile(int a, int n_tiles) { return a + 1 == n_tiles ? 0 : a + 1; }

// One tile step of a wave: this block's operands are in registers already; the next tile (ring slot (s+1) mod 4,
// where R.kp points) is read during the step.
template <int kVariant, bool kOnce>
__device__ __forceinline__ void wide_step(WideState &R, const Stationary &A, const uint32_t lds0, int s, int tile,
                                          int tile_fetch, int tile_flush, int t_begin,
                                          int t_end, int last_row, const int *vis_i, const int *excl_i, const char *kh,
                                          const char *vh, const uint32_t (&moff)[4], int wave, int lane, int vis_min,
                                          const uint32_t *special_s, float *stage, float *out, size_t variant_stride,
                                          bool accumulate) {
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    const int rh = wave & 1, th = wave >> 1;

    // Tile s+1 has landed once at most the two younger tiles' transfers are in flight; the barrier also tells that
    // every wave is done with tile s, whose slot the tile fetched during this step reuses.  (The walk wraps around, so
    // the ring also prefetches past its end: every step waits for the same number of transfers.  One row of K and of V instead of those
    // tiles: joint, 128 rows, us, so / one row, 8 heads x 8192 37.4 / 37.6, x 10000 40.2 / 40.5, 4 x 8 heads x 32K 257.4 / 258.4.)
    wait_async_loads_keep<2 * kTilePerWave>();
    __syncthreads();
    TileFetch fetch;
    {
        const int tn = t_begin + tile_fetch * kTileTok;                          // (<= last_row: the tile exists)
        fetch.k_base = kh + (size_t)tn * kRowBytes - kBias;
        fetch.v_base = vh + (size_t)tn * kRowBytes - kBias;
        fetch.lds = lds0 + ((s + 3) & 3) * kSlotBytes + wave * 4096;          // (the slot of tile s)
        const int rmax = last_row - tn;                                    // last row of the tile that exists
#pragma unroll
        for (int n = 0; n < 4; ++n) fetch.voff[n] = moff[n];
        if (rmax < kTileTok - 1) {                                         // uniform, rare: rows past the end re-read the last one
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const int Rn = (wave * 4 + n) * 4 + (lane >> 4);
                fetch.voff[n] -= (uint32_t)(max(Rn - rmax, 0) * kRowBytes);
            }
        }
    }
    if (s >= 2) flush_tile<kNv>(stage + ((s - 2) & 3) * 2 * kNv * 64, out, variant_stride, t_begin + tile_flush * kTileTok, t_end, wave, lane, accumulate);

    const int tok0 = t_begin + tile * kTileTok + th * 32;                // this wave's block
    const int blk = 2 * tile + th;
    // Blocks every row of the wave sees in full and that hold no separately scored pair need no masks.
    const bool hidden = !(tok0 + 31 <= vis_min);                         // uniform for the wave
    float *stage_prev = stage + (R.pend ? (s - 1) & 3 : kSlots) * 2 * kNv * 64;      // (slot 4: never flushed)
    pipelined_block<kVariant, kOnce>(R, A, fetch, stage_prev, tok0 + (lane & 31), t_end, rh, th, wave, lane, blk, hidden, special_s[special_word(blk)], vis_i, excl_i);
    // On to the slot of tile s+2 (the ring wraps after slot 3).
    const int hop = ((s + 1) & 3) == 0 ? -(kSlots - 1) * kSlotBytes : kSlotBytes;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) R.kp[kk] += hop;
}

// kVariant: OBC_KEY / OBC_JOINT / OBC_ALL.  Grid: see sweep_part.
template <int kVariant, bool kOnce, typename Lens>
__global__ __launch_bounds__(kThreads, 1) void mfma_sweep2_wide(const uint16_t *__restrict__ q,
                                                                const uint16_t *__restrict__ k,
                                                                const uint16_t *__restrict__ v, int N, int W, int Hq,
                                                                int Hkv, int heads, int ragged, Lens lens, int range_len, int n_chunks, int m_pad,
                                                                const uint16_t *__restrict__ out_bf16,
                                                                const float *__restrict__ row_const,
                                                                const float *__restrict__ special,
                                                                float *__restrict__ dst, size_t variant_stride,
                                                                size_t chunk_stride, int accumulate_flag) {
    const bool accumulate = accumulate_flag != 0;
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    // the ring of K/V tiles, the records of the chunk's rows, the staged partial scores of four tiles (+ a spare slot)
    constexpr int kStageBytes = 5 * 2 * kNv * 64 * sizeof(float);
    __shared__ __attribute__((aligned(1024))) char smem[kRing + 4096 + 256 * sizeof(int) + kStageBytes];
    float4 *rc_s = (float4 *)(smem + kRing);                   // [128] row_const of each row of the chunk
    const float4 *sp_s = rc_s + 128;                           // [128] its `special`
    int *vis_i = (int *)(rc_s + 256);                          // [128] last visible key
    int *excl_i = vis_i + 128;                                 // [128] key of the row that is scored separately, or -1
    float *stage = (float *)(excl_i + 128);                    // [4 tiles + 1][2 row halves][kNv][64]

    const SweepPart part = sweep_part(lens, ragged, N, Hkv, n_chunks, range_len);
    const int b = part.b, g = part.g, bg = b * Hkv + g, chunk = part.chunk, G = Hq / Hkv, M = G * W, len = part.len;
    const int t_begin = part.part * range_len;
    float *out = dst + (size_t)chunk * chunk_stride + (size_t)bg * N;
    const int t_end = min(t_begin + range_len, len);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int rh = wave & 1, th = wave >> 1;
    const int row0 = chunk * 128 + rh * 64;                    // first of this wave's 64 rows
    const size_t cbase = (size_t)bg * m_pad;

    const char *kh = (const char *)k + (size_t)bg * N * kRowBytes;
    const char *vh = (const char *)v + (size_t)bg * N * kRowBytes;
    const uint32_t lds0 = lds_offset_of(smem);

    // Everything from here to the loop runs once, and what it costs is its instructions' way into the instruction cache, from
    // memory after a sweep that has filled the L2: written out (two forms of every tile load, operands parked through
    // architectural registers, a lane exchange per step of a minimum) it was 1700 instructions and took 9.5 to 13.5 us of a
    // launch; in loops and with loads into the accumulator file, 7 to 10, most of that the transfers themselves.  Kernel, us,
    // before and after: 8 heads x 8K, joint 19.2 / 16.2, all 20.3 / 17.4; 4 x 8 x 32K, joint 135 / 132; 4 x 128K, 448 rows,
    // all (both kernels) 274 / 269.
    // (workgroups start their walks all over the range: see tile_at)
    const int n_tiles = (t_end - t_begin + kTileTok - 1) / kTileTok;
    const int first = (int)__umulhi((blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) * 0x9e3779b1u, (unsigned)n_tiles);
    uint32_t moff[4];
    tile_lane_offsets<kXor16>(moff, wave, lane);
#pragma unroll
    for (int n = 0; n < 4; ++n) moff[n] += kBias - 1024 * n;
    // Tile t of the walk lives in ring slot (t + 3) mod 4.  Slots 0 to 2 first serve as a staging area for the stationary
    // operands of the chunk's 128 rows: Q, then the high and the residual pieces of o_i, each as two 64-row tiles in the K
    // tiles' layout, brought in by the same coalesced direct-to-LDS transfers (per-lane loads of 16-byte pieces from 32 rows
    // each would take ten times as long).  The first tile follows them to slot 3.  The rows' records come the same way,
    // one transfer per wave: ordinary loads of theirs, ahead of the transfers or behind them, are waited for with all of them.
    {
        const char *q_rows = (const char *)q + ((size_t)b * Hq + (size_t)g * G) * W * kRowBytes;      // the KV head's M rows
        const char *o_rows = (const char *)out_bf16 + cbase * kRowBytes;                             // its m_pad rows
        const char *o_low = o_rows + (size_t)heads * m_pad * kRowBytes;
        const char *records = (const char *)((wave < 2 ? row_const : special) + cbase * 4);
        transfer_at<0, false>(records, (uint32_t)min(chunk * 128 + rh * 64 + lane, m_pad - 1) * 16, lds0 + kRing + wave * 1024);
#pragma unroll 1
        for (int t = 0; t < 6; ++t) {              // (rows past the last one re-read it)
            const char *rows = t < 2 ? q_rows : t < 4 ? o_rows : o_low;
            const int from = chunk * 128 + (t & 1) * 64, last = t < 2 ? M - 1 : m_pad - 1;
            load_64_rows<false>(rows, min(from, last), last, lds0 + t * kTileBytes + wave * 4096, moff, wave, lane);
        }
#pragma unroll 1
        for (int t = 6; t < 8; ++t) {
            const int from = t_begin + first * kTileTok;
            load_64_rows<kOnce>(t < 7 ? kh : vh, min(from, len - 1), len - 1, lds0 + t * kTileBytes + wave * 4096, moff, wave, lane);
        }
    }

    WideState R;
    // LDS address of this lane's operand piece kk of its block (tokens 32 th .. 32 th + 31 of a tile) in ring slot 3,
    // where the first tile lands; the V tile of a slot is reached with an immediate offset, the other slots by moving
    // the addresses.
    lds_ptr base = (lds_ptr)smem;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) R.kp[kk] = base + 3 * kSlotBytes + th * 32 * kRowBytes + row_piece_offset(lane, kk);
    __shared__ uint32_t special_s[kSpecialWords];
    if (threadIdx.x < kSpecialWords) special_s[threadIdx.x] = 0;
    wait_async_loads_keep<kTilePerWave>();                     // the staged operands and the records have landed
    __syncthreads();
    if (chunk * 128 + 128 > M) {                               // uniform: rows past the last one have a Q of zeros
        zero_rows(smem, M - chunk * 128);
        zero_rows(smem + kTileBytes, M - chunk * 128 - 64);
        __syncthreads();
    }
    // Stationary operands: rows row0 + 32 S + (lane % 32), pieces 2 kk + half, parked in the accumulator file.
    Stationary A;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        const lds_ptr piece = base + rh * kTileBytes + row_piece_offset(lane, kk);
        park<0>(A.q[0][kk], piece);
        park<32 * kRowBytes>(A.q[1][kk], piece);
        park<kSlotBytes>(A.hi[0][kk], piece);
        park<kSlotBytes + 32 * kRowBytes>(A.hi[1][kk], piece);
        park<0>(A.lo[0][kk], piece + 2 * kSlotBytes);
        park<32 * kRowBytes>(A.lo[1][kk], piece + 2 * kSlotBytes);
    }
    // First key some valid row of this wave cannot see (lane l looks at row l of its 64; -1, a padded row, is above every key).
    const bool wave_row = row0 + lane < m_pad;
    const uint32_t vis_least = wave_reduce<MinOp>(wave_row ? (uint32_t)__float_as_int(rc_s[rh * 64 + lane].z) : 0xffffffffu);
    const int vis_min = __builtin_amdgcn_readfirstlane((int)min(vis_least, (uint32_t)(t_end - 1)));
    int mine_special = 0;
    if (threadIdx.x < 128) {
        const bool row = chunk * 128 + (int)threadIdx.x < m_pad;
        const int ex = row ? __float_as_int(sp_s[threadIdx.x].x) : -1;
        vis_i[threadIdx.x] = row ? __float_as_int(rc_s[threadIdx.x].z) : -1;
        excl_i[threadIdx.x] = ex;
        if (!row) rc_s[threadIdx.x] = make_float4(1e30f, 0.f, 0.f, 0.f);      // (weighs nothing)
        mine_special = ex >= t_begin && ex < t_end;
        if (mine_special) atomicOr(&special_s[special_word((ex - t_begin) >> 5)], 1u << ((ex - t_begin) >> 5 & 31));
    }
    A.tie();
    const bool has_special = __syncthreads_or(mine_special) != 0;

    // Every wave has its stationary operands (the barrier above): the staging slots take the next three tiles.
#pragma unroll 1
    for (int t = 0; t < 6; ++t)
        load_64_rows<kOnce>(t & 1 ? vh : kh, t_begin + tile_at((t >> 1) + 1, first, n_tiles) * kTileTok, len - 1, lds0 + t * kTileBytes + wave * 4096, moff, wave, lane);
    wait_async_loads_keep<3 * kTilePerWave>();                 // the first tile has landed
    __syncthreads();
    // The first block's operand pieces (slot 3).
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        R.kreg[kk] = lds_piece(R.kp[kk], 0);
        R.vreg[kk] = lds_piece(R.kp[kk], kTileBytes);
        R.kp[kk] -= 3 * kSlotBytes;                            // step 0 reads the second tile (slot 0)
    }
    R.zA = zero16(); R.voA = zero16(); R.zB = zero16(); R.voB = zero16();
    R.sv = R.sk = R.sj = 0.f;
    R.vv_prev = 0.f;
    R.pend = false;
    R.rc = row_consts(base + kRing + (rh * 64 + 4 * half) * 16);

    // Positions of the walk: the tile worked on, the one fetched during the step (four ahead), the one flushed (two back).
    int tile = first, tile_fetch = tile_at(4, first, n_tiles), tile_flush = tile_at(2 * n_tiles - 2, first, n_tiles);
    for (int s = 0; s < n_tiles; ++s, tile = next_tile(tile, n_tiles), tile_fetch = next_tile(tile_fetch, n_tiles), tile_flush = next_tile(tile_flush, n_tiles))
        wide_step<kVariant, kOnce>(R, A, lds0, s, tile, tile_fetch, tile_flush, t_begin, t_end, len - 1, vis_i, excl_i, kh, vh, moff, wave, lane, vis_min,
                            special_s, stage, out, variant_stride, accumulate);
    if (R.pend) {                                              // set B of the last block
        matrix_results_land();
        float bv = 0.f, bk = 0.f, bj = 0.f;
        score_set<kVariant>(R.zB, R.voB, R.rc, 1, R.vv_prev, bv, bk, bj);
        park_block<kVariant>(stage + ((n_tiles - 1) & 3) * 2 * kNv * 64, rh, th, lane, R.vv_prev, R.sv, R.sk, R.sj, bv, bk, bj);
    }
    wait_async_loads();        // the tiles fetched past the end must have landed before the LDS is given back
    __syncthreads();
    if (n_tiles >= 2) flush_tile<kNv>(stage + ((n_tiles - 2) & 3) * 2 * kNv * 64, out, variant_stride, t_begin + tile_at(n_tiles - 2, first, n_tiles) * kTileTok, t_end, wave, lane, accumulate);
    flush_tile<kNv>(stage + ((n_tiles - 1) & 3) * 2 * kNv * 64, out, variant_stride, t_begin + tile_at(n_tiles - 1, first, n_tiles) * kTileTok, t_end, wave, lane, accumulate);
    if (!accumulate) zero_padding<kNv>(part, N, out, variant_stride);
    if (has_special) add_special_pairs<kVariant>(smem, special + (cbase + chunk * 128) * 4, min(128, m_pad - chunk * 128), t_begin, t_end, out, variant_stride);
}

// ------------------------------------------------------------------------------------
// The last 64 window rows or fewer of a KV head: every wave by itself
// ------------------------------------------------------------------------------------
// With at most 64 rows one wave holds all of them, and the four waves of a workgroup share nothing but the rows: each
// takes its own 32-token blocks (block 4 g + wave of the range), brings them in with its own transfers through its own
// ring of two 16 KB slots, and writes finished sums.  No barrier, no staging of partial sums; a block's transfers have a
// whole step to land.  Bound by the read of K and V: 4 x 8 heads x 32K, 64 rows, joint: 153 us with 32 rows per wave, 98 us
// here (32 rows: 105 and 97).
constexpr int kSoloTok = 32;
constexpr int kSoloSlot = 2 * kBlkBytes;          // 16 KB: a block's K rows, then its V rows
constexpr int kSoloTransfers = 16;                // direct-to-LDS transfers a wave issues per block (8 K + 8 V)

struct SoloFetch {
    const char *k_base, *v_base;     // first row of the block in K and in V (uniform)
    uint32_t voff[8];                // per-lane byte offset of transfer n inside the block (rows past the end clamped)
    uint32_t lds;                    // LDS byte address of the slot
};
template <bool kOnce>
__device__ __forceinline__ void solo_fetch_one(const SoloFetch &f, int n) {       // n = 0..7: K, 8..15: V
    dma16_based<kOnce>(n < 8 ? f.k_base : f.v_base, f.voff[n & 7], f.lds + (n < 8 ? 0 : kBlkBytes) + (n & 7) * 1024);
}
__device__ __forceinline__ SoloFetch solo_fetch(const char *kh, const char *vh, int t0, int last_row, uint32_t lds, const uint32_t (&doff)[8], int lane) {
    SoloFetch f;
    const int row = min(t0, last_row), rmax = last_row - row;
    f.k_base = kh + (size_t)row * kRowBytes;
    f.v_base = vh + (size_t)row * kRowBytes;
    f.lds = lds;
#pragma unroll
    for (int n = 0; n < 8; ++n) f.voff[n] = doff[n];
    if (rmax < kSoloTok - 1) {                                             // uniform, rare: rows past the end re-read the last one
#pragma unroll
        for (int n = 0; n < 8; ++n) f.voff[n] -= (uint32_t)(max(4 * n + (lane >> 4) - rmax, 0) * kRowBytes);
    }
    return f;
}

// A whole block at once, in short code (for the prologue); rows past the end re-read the last one.
template <bool kOnce>
__device__ __forceinline__ void load_block(const char *kh, const char *vh, int t0, int last_row, uint32_t lds, int lane) {
    const int row = min(t0, last_row);
    const char *k_base = kh + (size_t)row * kRowBytes, *v_base = vh + (size_t)row * kRowBytes;
#pragma unroll 1
    for (int n = 0; n < 8; ++n) {
        const int Rn = 4 * n + (lane >> 4);
        const uint32_t voff = (uint32_t)(min(Rn, last_row - row) * kRowBytes + piece_of(kXor16, Rn, lane & 15) * 16);
        transfer_at<0, kOnce>(k_base, voff, lds + n * 1024);
        transfer_at<0, kOnce>(v_base, voff, lds + kBlkBytes + n * 1024);
    }
}

// One block of a wave, in the two phases of pipelined_block: its operands are in registers, the previous block's set B is
// still due, and the next block lies in slot kNext of the wave's ring from the end of phase 1 on.
template <int kVariant, int kNext, bool kOnce>
__device__ __forceinline__ void solo_block(WideState &R, const Stationary &A, const SoloFetch &fetch, float *out,
                                           size_t variant_stride, int tok, int tok_prev, int t_end, int lane, int blk, bool hidden,
                                           uint32_t special, const int *vis_i, const int *excl_i, bool accumulate) {
    constexpr bool kDoV = kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    const int half = lane >> 5;
    float vvn = 0.f, bv = 0.f, bk = 0.f, bj = 0.f;
    const TokenConsts tp = token_consts(R.vv_prev);
    PairWork pw[16];
    matrix_phase<0>(A, R.zA, R.voA, R.kreg, R.vreg, [&](int j) __attribute__((always_inline)) {
        if (j < 16) { vvn = sumsq_quarter(R.vreg[j >> 1], j & 1, vvn); stay(vvn); }
        if (j >= 8) solo_fetch_one<kOnce>(fetch, j - 8);
#pragma unroll
        for (int t = 2 * j; t < 2 * j + 2; ++t) {
            const int r = t / 3;
            pair_task<kVariant>(t % 3, pw[r], R.zB[r], R.voB[r], R.rc.m2[1][r], R.rc.oo[1][r], tp, bv, bk, bj);
        }
    });
    // Everything older than the transfers just started: the next block has landed.
    wait_async_loads_keep<kSoloTransfers>();
    {
        float sv = 0.f, sk = 0.f, sj = 0.f;
        if (kDoV) sv = halves_sum((R.sv + bv) * tp.vv);
        if (kDoK) sk = fmaxf(halves_sum(R.sk + bk), 0.f);      // (rounding can leave a sum a hair below zero)
        if (kDoJ) sj = fmaxf(halves_sum(R.sj + bj), 0.f);
        if (half == 0 && tok_prev < t_end) {
            float *o = out + tok_prev;
            auto put = [&](float x) { *o = accumulate ? *o + x : x; o += variant_stride; };
            if (kDoV) put(sv);
            if (kDoK) put(sk);
            if (kDoJ) put(sj);
        }
    }
    const bool masks = hidden || special_bit(special, blk);
    if (masks) {                                               // uniform for the wave, rare
        matrix_results_land();
        hide_pairs(R.zA, 0, tok, t_end, 0, half, vis_i, excl_i);
    }
    const TokenConsts tc = token_consts(halves_sum(vvn));
    float av = 0.f, ak = 0.f, aj = 0.f;
    matrix_phase<1>(A, R.zB, R.voB, R.kreg, R.vreg, [&](int j) __attribute__((always_inline)) {
        if (j < 8) R.kreg[j] = lds_piece(R.kp[j], kNext * kSoloSlot);
        else if (j & 1) R.vreg[(j - 8) >> 1] = lds_piece(R.kp[(j - 8) >> 1], kNext * kSoloSlot + kBlkBytes);
#pragma unroll
        for (int t = 2 * j; t < 2 * j + 2; ++t) {
            const int r = t / 3;
            pair_task<kVariant>(t % 3, pw[r], R.zA[r], R.voA[r], R.rc.m2[0][r], R.rc.oo[0][r], tc, av, ak, aj);
        }
    });
    if (masks) {
        matrix_results_land();
        hide_pairs(R.zB, 1, tok, t_end, 0, half, vis_i, excl_i);
    }
    R.sv = av; R.sk = ak; R.sj = aj;
    R.vv_prev = tc.vv;
    // The operand reads above have arrived: the next step's transfers may overwrite the slot they came from.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// kVariant: OBC_KEY / OBC_JOINT / OBC_ALL.  Grid: see sweep_part; rows row0 .. row0 + 63 of the head.
template <int kVariant, bool kOnce, typename Lens>
__global__ __launch_bounds__(kThreads, 1) void mfma_sweep2_solo(const uint16_t *__restrict__ q,
                                                                const uint16_t *__restrict__ k,
                                                                const uint16_t *__restrict__ v, int N, int W, int Hq,
                                                                int Hkv, int heads, int ragged, Lens lens, int range_len,
                                                                int m_pad, int row0, const uint16_t *__restrict__ out_bf16,
                                                                const float *__restrict__ row_const,
                                                                const float *__restrict__ special,
                                                                float *__restrict__ dst, size_t variant_stride,
                                                                int accumulate_flag) {
    const bool accumulate = accumulate_flag != 0;
    constexpr int kNv = kVariant == OBC_ALL ? 3 : 1;
    // the four waves' rings, then the rows' records
    __shared__ __attribute__((aligned(1024))) char smem[4 * 2 * kSoloSlot + 64 * sizeof(float4) + 128 * sizeof(int)];
    float4 *rc_s = (float4 *)(smem + 4 * 2 * kSoloSlot);       // [64] row_const of each row
    int *vis_i = (int *)(rc_s + 64);                           // [64] last visible key of each row
    int *excl_i = vis_i + 64;                                  // [64] key of the row that is scored separately, or -1

    const SweepPart part = sweep_part(lens, ragged, N, Hkv, 1, range_len);
    const int b = part.b, g = part.g, bg = b * Hkv + g, G = Hq / Hkv, M = G * W, len = part.len;
    const int t_begin = part.part * range_len;
    float *out = dst + (size_t)bg * N;
    const int t_end = min(t_begin + range_len, len);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const size_t cbase = (size_t)bg * m_pad + row0;
    const char *kh = (const char *)k + (size_t)bg * N * kRowBytes;
    const char *vh = (const char *)v + (size_t)bg * N * kRowBytes;
    const uint32_t lds0 = lds_offset_of(smem), ring = lds0 + wave * 2 * kSoloSlot;

    // The walk: groups of 128 tokens, from this workgroup's own first group around (see tile_at).
    const int n_groups = (t_end - t_begin + 4 * kSoloTok - 1) / (4 * kSoloTok);
    int group = (int)((13u * (blockIdx.x + gridDim.x * blockIdx.z)) % (unsigned)n_groups);
    auto block_of = [&](int grp) { return t_begin + (4 * grp + wave) * kSoloTok; };       // first token of the wave's block
    uint32_t doff[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int Rn = 4 * n + (lane >> 4);
        doff[n] = (uint32_t)(Rn * kRowBytes + piece_of(kXor16, Rn, lane & 15) * 16);
    }
    // The wave's first block goes to slot 0; the second slots of waves 0, 1 and 2 first stage the stationary operands:
    // Q, the high and the residual pieces of o_i, one 64-row tile each, brought in by all four waves.
    load_block<kOnce>(kh, vh, block_of(group), len - 1, ring, lane);
    {
        uint32_t moff[4];
        tile_lane_offsets<kXor16>(moff, wave, lane);
#pragma unroll
        for (int n = 0; n < 4; ++n) moff[n] += kBias - 1024 * n;
        const char *q_rows = (const char *)q + (((size_t)b * Hq + (size_t)g * G) * W + row0) * kRowBytes;
        const char *o_rows = (const char *)out_bf16 + cbase * kRowBytes;
        const size_t lo_plane = (size_t)heads * m_pad * kRowBytes;
#pragma unroll 1
        for (int t = 0; t < 3; ++t)                            // (rows past the last one re-read it, and are zeroed below)
            load_64_rows<false>(t == 0 ? q_rows : t == 1 ? o_rows : o_rows + lo_plane, 0, M - row0 - 1, lds0 + (2 * t + 1) * kSoloSlot + wave * 4096, moff, wave, lane);
    }
    float4 my_rc = make_float4(1e30f, 0.f, __int_as_float(-1), 0.f);   // rows past the last one (1e30) weigh nothing
    int my_excl = -1;
    if (row0 + lane < M) {                                     // (every wave looks at row `lane`, the first one stores)
        my_rc = ((const float4 *)row_const)[cbase + lane];
        my_excl = __float_as_int(special[(cbase + lane) * 4]);
    }
    const bool mine_special = my_excl >= t_begin && my_excl < t_end;
    const bool has_special = __any(mine_special);              // (the same in every wave)
    uint32_t vis_least = wave_reduce<MinOp>((uint32_t)__float_as_int(my_rc.z));     // (-1, no such row, is above every key)
    const int vis_min = __builtin_amdgcn_readfirstlane((int)min(vis_least, (uint32_t)(t_end - 1)));
    __shared__ uint32_t special_s[kSpecialWords];
    if (threadIdx.x < 64) {
        if (lane < kSpecialWords) special_s[lane] = 0;
        if (mine_special) atomicOr(&special_s[special_word((my_excl - t_begin) >> 5)], 1u << ((my_excl - t_begin) >> 5 & 31));
        rc_s[lane] = my_rc;
        vis_i[lane] = __float_as_int(my_rc.z);
        excl_i[lane] = my_excl;
    }

    WideState R;
    lds_ptr base = (lds_ptr)smem;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) R.kp[kk] = base + wave * 2 * kSoloSlot + row_piece_offset(lane, kk);
    wait_async_loads();
    __syncthreads();
    if (row0 + 64 > M) {                                       // uniform: rows past the last one are zeros
#pragma unroll
        for (int t = 0; t < 3; ++t) zero_rows(smem + (2 * t + 1) * kSoloSlot, M - row0);
        __syncthreads();
    }
    Stationary A;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        const lds_ptr piece = base + kSoloSlot + row_piece_offset(lane, kk);
        park<0>(A.q[0][kk], piece);
        park<32 * kRowBytes>(A.q[1][kk], piece);
        park<2 * kSoloSlot>(A.hi[0][kk], piece);
        park<2 * kSoloSlot + 32 * kRowBytes>(A.hi[1][kk], piece);
        park<0>(A.lo[0][kk], piece + 4 * kSoloSlot);
        park<32 * kRowBytes>(A.lo[1][kk], piece + 4 * kSoloSlot);
    }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        R.kreg[kk] = lds_piece(R.kp[kk], 0);
        R.vreg[kk] = lds_piece(R.kp[kk], kBlkBytes);
    }
    A.tie();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // (the first block's operands, too)
    __syncthreads();                                           // every wave has its stationary operands: the slots are free
    group = next_tile(group, n_groups);
    load_block<kOnce>(kh, vh, block_of(group), len - 1, ring + kSoloSlot, lane);
    R.zA = zero16(); R.voA = zero16(); R.zB = zero16(); R.voB = zero16();
    R.sv = R.sk = R.sj = 0.f;
    R.vv_prev = 0.f;
    R.rc = row_consts(base + 4 * 2 * kSoloSlot + 4 * half * 16);

    int here = group == 0 ? n_groups - 1 : group - 1;          // the group worked on; `group` is the one after it
    int tok_prev = 0x7fffffff;
    int s = 0;
    auto step = [&](auto slot) __attribute__((always_inline)) {        // slot: of the block worked on
        const int after = next_tile(group, n_groups), tok0 = block_of(here), blk = 4 * here + wave;
        // (Past the walk's end one row of K and of V, for the number of transfers.  So / the blocks that the walk comes to there, joint, 64
        // rows, us: 8 heads x 8192 30.1 / 30.8, x 16384 40.8 / 42.4, 4 x 8 heads x 32K 195.8 / 198.4.)
        const SoloFetch f = solo_fetch(kh, vh, block_of(after), s + 2 < n_groups ? len - 1 : min(block_of(after), len - 1), ring + slot.value * kSoloSlot, doff, lane);
        const bool hidden = !(tok0 + 31 <= vis_min);
        const int tok = tok0 + (lane & 31);
        solo_block<kVariant, 1 - slot.value, kOnce>(R, A, f, out, variant_stride, tok, tok_prev, t_end, lane, blk, hidden, special_s[special_word(blk)], vis_i, excl_i, accumulate);
        tok_prev = tok;
        here = group;
        group = after;
    };
    while (s < n_groups) {
        step(std::integral_constant<int, 0>{});
        if (++s == n_groups) break;
        step(std::integral_constant<int, 1>{});
        ++s;
    }
    matrix_results_land();                                     // set B of the last block
    {
        float bv = 0.f, bk = 0.f, bj = 0.f;
        score_set<kVariant>(R.zB, R.voB, R.rc, 1, R.vv_prev, bv, bk, bj);
        const float sv = halves_sum((R.sv + bv) * R.vv_prev), sk = fmaxf(halves_sum(R.sk + bk), 0.f), sj = fmaxf(halves_sum(R.sj + bj), 0.f);
        if (half == 0 && tok_prev < t_end) {
            float *o = out + tok_prev;
            auto put = [&](float x) { *o = accumulate ? *o + x : x; o += variant_stride; };
            if (kVariant == OBC_ALL) put(sv);
            if (kVariant == OBC_KEY || kVariant == OBC_ALL) put(sk);
            if (kVariant == OBC_JOINT || kVariant == OBC_ALL) put(sj);
        }
    }
    wait_async_loads();        // the blocks fetched past the end must have landed before the LDS is given back
    if (!accumulate) zero_padding<kNv>(part, N, out, variant_stride);
    if (has_special) add_special_pairs<kVariant>(smem, special + cbase * 4, min(64, M - row0), t_begin, t_end, out, variant_stride);     // uniform
}

}  // namespace

bool sweep2_wide_covers(int variant) { return variant == OBC_KEY || variant == OBC_JOINT || variant == OBC_ALL; }

template <int kVariant>
static hipError_t launch_wide(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, float *dst, size_t plane_elems,
                              size_t chunk_stride, hipStream_t stream) {
    const uint16_t *q = (const uint16_t *)a.q, *k = (const uint16_t *)a.k, *v = (const uint16_t *)a.v, *o = (const uint16_t *)(base + ws.out_bf16);
    const float *row_const = (const float *)(base + ws.row_const), *special = (const float *)(base + ws.special);
    const int accumulate = ws.n_chunks == 1 ? a.accumulate : 0, BH = a.B * a.Hkv, full = ws.n_chunks - ws.solo;
    return with_lens(a.ragged, a.B, a.lens, [&](const auto &lens) {
        auto launch = [&](auto once) {
            if (full > 0)
                mfma_sweep2_wide<kVariant, once.value><<<sweep_grid(a, lens, full, ws.range_len), dim3(kThreads), 0, stream>>>(
                    q, k, v, a.N, a.W, a.Hq, a.Hkv, BH, a.ragged, lens, ws.range_len, full, ws.m_pad, o, row_const, special, dst, plane_elems,
                    chunk_stride, accumulate);
            if (ws.solo)
                mfma_sweep2_solo<kVariant, once.value><<<sweep_grid(a, lens, 1, ws.range_solo), dim3(kThreads), 0, stream>>>(
                    q, k, v, a.N, a.W, a.Hq, a.Hkv, BH, a.ragged, lens, ws.range_solo, ws.m_pad, full * 128, o, row_const, special,
                    dst + full * chunk_stride, plane_elems, accumulate);
        };
        if (ws.once2) launch(std::true_type{}); else launch(std::false_type{});
        return hipGetLastError();
    });
}

hipError_t launch_sweep2_wide(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, float *dst, size_t plane_elems,
                              size_t chunk_stride, hipStream_t stream) {
    switch (a.variant) {
        case OBC_KEY: return launch_wide<OBC_KEY>(a, ws, base, dst, plane_elems, chunk_stride, stream);
        case OBC_JOINT: return launch_wide<OBC_JOINT>(a, ws, base, dst, plane_elems, chunk_stride, stream);
        case OBC_ALL: return launch_wide<OBC_ALL>(a, ws, base, dst, plane_elems, chunk_stride, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace obc
