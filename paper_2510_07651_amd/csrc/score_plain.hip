// General scoring path: fp32 inputs, bf16 with head_dim 64, and anything pinned to it (obc_set_score_path).
// Logits are accumulated in fp64 on the matrix cores, attention outputs in fp32 there, cross terms in fp64; calls with
// more window rows per KV head form both from pieces on faster units where that is as good (score_fixed.h).
//
// Four kernels over a group of KV heads (Section 3 of the paper, then Eq. 4-6 summed over the window, Eq. 9, and the
// query heads of the KV head, Appendix A.5):
//   plain_logits   Z = Q K^T / sqrt(d): fp64 dot products rounded once to fp32 and stored, and per row the largest
//                  visible logit of every token range with the lowest token that attains it.
//   plain_weights  the row's maximum over all ranges; weights exp(z - max), their sum and P V per sequence split.
//   plain_merge    per row: sums of the splits, the attention output o_i and the constants the scores need.
//   plain_score    V O^T in fp64, A and Z from the stored logits, the three closed forms, summed over the rows.
// Every logit is computed once: a group is as many KV heads as leave their logits within the workspace plan (they
// then pass through the caches between the kernels).  Where even one head's rows do not fit, the rows, and beyond that
// the tokens, are taken in pieces and the logits of a piece recomputed when they are needed again.
//
// Cancellation guard.  When one key takes almost all of a row's attention, o_i is almost v_p and fp32 cannot hold their
// difference.  Each row therefore keeps its top-logit token p* out of the running sums: with
// l' = sum_{q != p*} exp(z_q - z_p*) and o' = sum_{q != p*} exp(z_q - z_p*) v_q / l',
//     v_p* - o_i = (l' / (1 + l')) (v_p* - o')        (exact, no cancellation)
//     o_i        = v_p* - (v_p* - o_i)
// and the (row, p*) pair is scored from the first identity, in the merge kernel.  For every other pair ||v_p - o_i||^2
// and ||v_p + Z (v_p - o_i)||^2 are formed from ||v_p||^2, ||o_i||^2 and v_p.o_i in fp64: their cancellation costs bits
// far below the fp32 of o_i itself.
//
// What bounds it, up to 32 rows: the two fp64 contractions, 2 * 2 d flop per (row, token) pair at the 79 TFLOP/s of the
// fp64 matrix cores (a wave's 16 x 16 x 4 op occupies its SIMD's matrix core for 64 cycles, so operands from LDS, the
// conversion of fp32 to fp64 and the exponentials ride in its shadow), then P V on the fp32 matrix cores (twice that rate).
// The vector-ALU kernels this replaced took one fp64 multiply-add per element and lane with a block per query head.
// More rows: see score_fixed.h, and sweeps_digits for which.  Short sequences: launches, see short_partial.
// Sums run in a fixed order, so results are bit-reproducible.
#include <algorithm>
#include <climits>

#include "internal.h"
#include "plain_layout.h"
#include "wave_util.h"

namespace obc {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;        // tokens per tile; each of the four waves owns 16 of them
constexpr int kThreads = 256;    // 4 waves
constexpr int kPlainRows = 16;   // up to so many the kernels of this file take a call, beyond 32 those of score_fixed.h (sweeps_digits)
// Rows of a workgroup of score_fixed.h, but for digit_sweep: 64 where the last 128 would be half empty.
constexpr int fixed_rows(int rows) { return (rows + 63) / 64 % 2 != 0 ? 64 : 128; }
constexpr int kMaxRanges = 64;   // token ranges with a row maximum of their own, at most
constexpr int kMaxSplits = 32;   // sequence splits of P V, at most
constexpr int kSweepSplits = 64; // of digit_sweep
constexpr int kMergeEach = 8;    // splits of a row that a wave of the merge has on the way together
constexpr int kResident = 1024;  // workgroups the chip holds at four per CU: a launch is cut into about this many
constexpr int kCus = 256;
// Time of a workgroup of digit_sweep, in hundredths of a tile with 128 rows: its tiles and what it takes beside them (its rows' digits,
// its record).
constexpr int sweep_time(int dtype, int rows, int tiles) {
    return rows == 128 ? 100 * tiles + 200 : dtype == OBC_F32 ? 60 * tiles + 200 : 65 * tiles + 160;
}
constexpr int kNoToken = 0x7fffffff;

// Constants of one row, written by plain_weights or fixed_weights (m, top) and plain_merge (the rest; all with digit_sweep).
struct RowRecord {
    float m;                     // largest visible logit
    int top;                     // lowest token that attains it
    float inv_l;                 // 1 / sum of exp(z - m)
    float top_dk, top_dj;        // ||v - o||^2 and ||v + Z (v - o)||^2 of the top token
    int last;                    // last token the row sees
    double oo;                   // ||o_i||^2
    double unit;                 // of o_i's digits (score_fixed.h)
};

template <typename T> __device__ __forceinline__ float load_as_float(const T *p);
template <> __device__ __forceinline__ float load_as_float<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float load_as_float<uint16_t>(const uint16_t *p) { return bf16_bits_to_float(*p); }

// exp(x) for x <= 0.  The product x log2(e) is carried as a pair, so that the argument of exp2 keeps full fp32 accuracy
// however large |x| is: exp(x) = 2^t (1 + ln2 r) with t + r = x log2(e).  Results below 2^-126 become 0, also that of
// -inf and of an x whose pair would not be finite; not a number stays that.
__device__ __forceinline__ float exp_nonpositive(float x) {
    x = __builtin_elementwise_maximum(x, -200.f);
    const float log2e = 1.44269504f, log2e_rest = 1.925963033500e-8f;      // log2(e) = 1.44269504 (as fp32) + the rest
    const float t = x * log2e;
    const float r = fmaf(x, log2e_rest, fmaf(x, log2e, -t));
    const float e = __builtin_amdgcn_exp2f(t);
    return fmaf(e, r * 0.693147181f, e);
}

// A norm that rounding has taken below 0 is 0; not a number stays that (fmaxf would make a 0 of it).
__device__ __forceinline__ float at_least_0(float x) { return __builtin_elementwise_maximum(x, 0.f); }

// (max, lowest token attaining it) merged across the lanes whose index differs in the bits of `below`.
template <int kLanes>
__device__ __forceinline__ void lanes_best(float &m, int &at) {
    static_assert(kLanes == 4 || kLanes == 8 || kLanes == 16, "inside a row of 16 lanes");
    auto step = [&](float om, uint32_t oat) {
        const bool take = om > m || (om == m && (int)oat < at);
        m = take ? om : m;
        at = take ? (int)oat : at;
    };
    step(dpp_pair<0xB1>(m), dpp_pair<0xB1>((uint32_t)at));
    step(dpp_pair<0x4E>(m), dpp_pair<0x4E>((uint32_t)at));
    if (kLanes >= 8) step(dpp_pair<0x141>(m), dpp_pair<0x141>((uint32_t)at));
    if (kLanes == 16) step(dpp_pair<0x140>(m), dpp_pair<0x140>((uint32_t)at));
}

// ------------------------------------------------------------------------------------
// Tiles: `kRows` rows of D values, in LDS as fp32 with row stride D + 4 (16-byte pieces of 16 consecutive rows then
// start in different banks).  Global memory is read in 16-byte pieces through registers, so that a tile can be in
// flight while the one before it is worked on.
// ------------------------------------------------------------------------------------
template <int D> constexpr int kStride = D + 4;

template <typename T, int D, int kRows>
struct TileRegs {
    static constexpr int kPieces = D * (int)sizeof(T) / 16;          // 16-byte pieces per row
    static constexpr int kCount = (kRows * kPieces + kThreads - 1) / kThreads;
    uint4 x[kCount];

    // Rows at or beyond `limit` become zeros; their memory is never read.
    __device__ __forceinline__ void load(const T *__restrict__ base, int row0, int limit) {
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            const int e = (int)threadIdx.x + i * kThreads, r = e / kPieces, c = e % kPieces;
            const bool ok = r < kRows && row0 + r < limit;
            x[i] = ok ? *(const uint4 *)((const char *)(base + (size_t)(row0 + r) * D) + c * 16) : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    __device__ __forceinline__ void store(float *__restrict__ lds) const {
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            const int e = (int)threadIdx.x + i * kThreads, r = e / kPieces, c = e % kPieces;
            if (kRows * kPieces % kThreads != 0 && r >= kRows) continue;
            float *dst = lds + r * kStride<D>;
            if (sizeof(T) == 4) {
                *(uint4 *)(dst + 4 * c) = x[i];
            } else {
                *(uint4 *)(dst + 8 * c) = make_uint4(x[i].x << 16, x[i].x & 0xffff0000u, x[i].y << 16, x[i].y & 0xffff0000u);
                *(uint4 *)(dst + 8 * c + 4) = make_uint4(x[i].z << 16, x[i].z & 0xffff0000u, x[i].w << 16, x[i].w & 0xffff0000u);
            }
        }
    }
};

// One row of a tile in the registers of the four lanes that share it (lane = row % 16 + 16 j): the 16-byte pieces
// 4 j .. 4 j + 3 of every sixteen elements, as fp32.
template <typename T, int D>
struct RowRegs {
    f32x4 x[D / 16];
    // (a row at or beyond `limit` becomes zeros; its memory is never read)
    __device__ __forceinline__ void load(const T *__restrict__ base, int row, int limit, int j) {
        const T *src = base + (size_t)row * D + 4 * j;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            if (sizeof(T) == 4) {
                x[s] = row < limit ? *(const f32x4 *)(src + 16 * s) : f32x4{0.f, 0.f, 0.f, 0.f};
            } else {
                const uint2 h = row < limit ? *(const uint2 *)(src + 16 * s) : make_uint2(0u, 0u);
                x[s] = f32x4{__uint_as_float(h.x << 16), __uint_as_float(h.x & 0xffff0000u), __uint_as_float(h.y << 16),
                             __uint_as_float(h.y & 0xffff0000u)};
            }
        }
    }
};

// fp64 dot products of 16 kRt rows in LDS and this wave's 16 tokens: acc[rt][r] is row 16 rt + 4 r + lane / 16, token
// lane % 16.  The four k values of a matrix op are components c of the four lane groups' 16-byte pieces: any assignment
// of elements to k will do as long as both operands use the same, and this one reads 16 bytes at a time.
// kTokensDown: the transpose, acc[rt][r] is the token of lane 4 r + lane / 16 (among 16) and row 16 rt + lane % 16.
template <typename T, int D, int kRt, bool kTokensDown = false>
__device__ __forceinline__ void tile_dots(const float *rows, const RowRegs<T, D> &tok, int lane, f64x4 (&acc)[kRt]) {
    const float *rp = rows + (lane & 15) * kStride<D> + 4 * (lane >> 4);
    asm volatile("" ::: "memory");                           // (the row operands are not to be kept across calls)
    f32x4 a[2][kRt];
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt) a[0][rt] = *(const f32x4 *)(rp + rt * 16 * kStride<D>);
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
        if (s + 1 < D / 16)
#pragma unroll
            for (int rt = 0; rt < kRt; ++rt) a[(s + 1) & 1][rt] = *(const f32x4 *)(rp + rt * 16 * kStride<D> + 16 * (s + 1));
        __builtin_amdgcn_sched_barrier(0);                   // (one step's operands ahead, no more: registers)
        f32x4 t = tok.x[s];
        asm volatile("" : "+v"(t));                          // (nor its fp64 form, which is twice as large)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int rt = 0; rt < kRt; ++rt) {
                const double x = a[s & 1][rt][c], y = t[c];
                acc[rt] = kTokensDown ? __builtin_amdgcn_mfma_f64_16x16x4f64(y, x, acc[rt], 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[rt], 0, 0, 0);
            }
    }
}

// ------------------------------------------------------------------------------------
// Logits.  Grid: x = token range of the piece, y = chunk of 16 kRt rows, z = KV head.
// ------------------------------------------------------------------------------------
template <typename T, int D, int kRt, typename Lens>
__global__ __launch_bounds__(kThreads, 4) void plain_logits(const T *__restrict__ q, const T *__restrict__ k, int N, int W,
                                                            int Hq, int Hkv, int ragged, Lens lens, Piece w,
                                                            int range_len, int n_ranges, float *__restrict__ z,
                                                            float2 *__restrict__ range_best) {
    constexpr int kRows = 16 * kRt;
    __shared__ __attribute__((aligned(16))) float rows_s[kRows * kStride<D>];
    __shared__ float2 best_s[4][kRows];
    __shared__ int last_s[kRows];                            // last token each row sees; -1: no such row

    const int hl = blockIdx.z, bg = w.bg0 + hl, b = bg / Hkv, g = bg % Hkv, M = Hq / Hkv * W;
    const int len = seq_len_of(lens, ragged, b, N);
    const int range = w.s0 / range_len + blockIdx.x;
    const int t_begin = range * range_len, t_end = min(min(t_begin + range_len, w.s1), len);
    if (t_begin >= t_end) return;                            // uniform: nothing of this range is live
    const int row0 = blockIdx.y * kRows;                     // first row of the chunk inside the piece
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    const T *kg = k + (size_t)bg * N * D;
    RowRegs<T, D> tok;
    tok.load(kg, t_begin + wave * 16 + (lane & 15), t_end, lane >> 4);
    {
        TileRegs<T, D, kRows> qr;
        qr.load(q + ((size_t)b * Hq * W + (size_t)g * M + w.r0) * D, row0, w.nr);
        qr.store(rows_s);
    }
    if ((int)threadIdx.x < kRows) {
        const int row = row0 + threadIdx.x;
        last_s[threadIdx.x] = row < w.nr ? len - W + (w.r0 + row) % W : -1;
    }
    float m[kRt * 4];
    int at[kRt * 4];
#pragma unroll
    for (int i = 0; i < kRt * 4; ++i) { m[i] = -INFINITY; at[i] = kNoToken; }
    __syncthreads();
    for (int t0 = t_begin; t0 < t_end; t0 += kTile) {
        const int p = t0 + wave * 16 + (lane & 15);
        f64x4 acc[kRt];
#pragma unroll
        for (int rt = 0; rt < kRt; ++rt) acc[rt] = f64x4{0.0, 0.0, 0.0, 0.0};
        tile_dots<T, D, kRt>(rows_s, tok, lane, acc);
        if (t0 + kTile < t_end) tok.load(kg, p + kTile, t_end, lane >> 4);
        float *zp = z + ((size_t)hl * w.nr + row0) * w.z_stride + (p - w.s0);
#pragma unroll
        for (int rt = 0; rt < kRt; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * rt + 4 * r + (lane >> 4), i = rt * 4 + r;
                const float x = (float)(acc[rt][r] * (1.0 / sqrt((double)D)));   // scaled logit: the only rounding
                const bool seen = p < t_end && p <= last_s[row];             // (what a row does not see is never read)
                if (seen) zp[(size_t)row * w.z_stride] = x;
                const bool better = seen && x > m[i];                        // (tokens ascend: strict keeps the lowest)
                m[i] = better ? x : m[i];
                at[i] = better ? p : at[i];
            }
    }
#pragma unroll
    for (int i = 0; i < kRt * 4; ++i) {
        lanes_best<16>(m[i], at[i]);
        if ((lane & 15) == 0) best_s[wave][16 * (i >> 2) + 4 * (i & 3) + (lane >> 4)] = make_float2(m[i], __int_as_float(at[i]));
    }
    __syncthreads();
    const int row = threadIdx.x;
    if (row < kRows && row0 + row < w.nr) {
        float2 best = best_s[0][row];
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            const float2 o = best_s[c][row];
            if (o.x > best.x || (o.x == best.x && __float_as_int(o.y) < __float_as_int(best.y))) best = o;
        }
        range_best[((size_t)hl * w.nr + row0 + row) * n_ranges + range] = best;
    }
}

// ------------------------------------------------------------------------------------
// Weights.  Grid: x = split of the piece, y = chunk of 16 kRt rows, z = KV head.  Without kNeedO (Eq. 4, 8 and the
// l1 form) only the sums are formed.
// ------------------------------------------------------------------------------------
template <typename T, int D, int kRt, bool kNeedO, typename Lens>
__global__ __launch_bounds__(kThreads, 2) void plain_weights(const T *__restrict__ v, int N, int W, int Hkv,
                                                             int ragged, Lens lens, Piece w, int range_len, int n_ranges,
                                                             int split_len, int n_splits, const float *__restrict__ z,
                                                             const float2 *__restrict__ range_best,
                                                             RowRecord *__restrict__ records, float *__restrict__ part_l,
                                                             float *__restrict__ part_o) {
    // Tiles of 32 tokens, two of each in LDS: while the matrix cores take one, the weights of the next are formed.
    constexpr int kRows = 16 * kRt, kTok = 32, kPs = kTok + 4;
    constexpr int kCt = D / 64;                              // 16-column tiles of V per wave
    __shared__ __attribute__((aligned(16))) float p_s[2][kNeedO ? kRows * kPs : 4], v_s[2][kNeedO ? kTok * kStride<D> : 4];
    __shared__ float m_s[kRows];
    __shared__ int top_s[kRows];

    const int hl = blockIdx.z, bg = w.bg0 + hl, b = bg / Hkv;
    const int len = seq_len_of(lens, ragged, b, N);
    const int split = w.s0 / split_len + blockIdx.x;
    const int t_begin = split * split_len, t_end = min(min(t_begin + split_len, w.s1), len);
    if (t_begin >= t_end) return;                            // uniform
    const int row0 = blockIdx.y * kRows;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    const T *vg = v + (size_t)bg * N * D;
    TileRegs<T, D, kTok> next;
    if (kNeedO) next.load(vg, t_begin, t_end);
    {
        // the row's maximum over its ranges: kThreads / kRows lanes per row
        constexpr int kSub = kThreads / kRows;
        const int row = threadIdx.x / kSub, live = (len + range_len - 1) / range_len;
        float m = -INFINITY;
        int at = kNoToken;
        if (row0 + row < w.nr)
#pragma unroll 4
            for (int i = threadIdx.x % kSub; i < live; i += kSub) {
                const float2 o = range_best[((size_t)hl * w.nr + row0 + row) * n_ranges + i];
                if (o.x > m || (o.x == m && __float_as_int(o.y) < at)) { m = o.x; at = __float_as_int(o.y); }
            }
        lanes_best<kSub>(m, at);
        if (threadIdx.x % kSub == 0) {
            m_s[row] = row0 + row < w.nr ? m : 0.f;
            top_s[row] = at;
            if (split == 0 && row0 + row < w.nr) {
                RowRecord *rec = records + (size_t)hl * w.nr + row0 + row;
                rec->m = m;
                rec->top = at;
            }
        }
    }
    __syncthreads();
    constexpr int kMine = kRows / 8;                         // this thread's rows: first, first + 8, ...
    const int first = 2 * wave + (lane >> 5), col = lane & 31;
    float m[kMine], sum[kMine], x[kMine];
    int top[kMine], last[kMine];
    const float *zp[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int row = first + 8 * i;
        m[i] = m_s[row];
        top[i] = top_s[row];
        last[i] = row0 + row < w.nr ? min(len - W + (w.r0 + row0 + row) % W, t_end - 1) : -1;     // last token it sees here
        sum[i] = 0.f;
        zp[i] = z + ((size_t)hl * w.nr + row0 + row) * w.z_stride - w.s0;
    }
    auto fetch = [&](int t0) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) x[i] = t0 + col <= last[i] ? zp[i][t0 + col] : 0.f;
    };
    auto weigh = [&](int t0, int slot) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const float e = t0 + col <= last[i] && t0 + col != top[i] ? exp_nonpositive(x[i] - m[i]) : 0.f;
            sum[i] += e;
            if (kNeedO) p_s[slot][(first + 8 * i) * kPs + col] = e;
        }
        if (kNeedO) next.store(v_s[slot]);
    };
    f32x4 acc[kRt][kCt];
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};

    fetch(t_begin);
    weigh(t_begin, 0);
    if (t_begin + kTok < t_end) {
        fetch(t_begin + kTok);
        if (kNeedO) next.load(vg, t_begin + kTok, t_end);
    }
    for (int t0 = t_begin, slot = 0; t0 < t_end; t0 += kTok, slot ^= 1) {
        if (kNeedO) {
            __syncthreads();                                 // this tile is in LDS, the one before it has been read
            // P V: this wave's 16 kCt columns of every row.  k value j of a matrix op is token 4 j + c of sixteen.
#pragma unroll
            for (int s = 0; s < kTok / 16; ++s) {
                f32x4 a[kRt];
#pragma unroll
                for (int rt = 0; rt < kRt; ++rt)
                    a[rt] = *(const f32x4 *)(p_s[slot] + (16 * rt + (lane & 15)) * kPs + 16 * s + 4 * (lane >> 4));
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int ct = 0; ct < kCt; ++ct) {
                        const float vv = v_s[slot][(16 * s + 4 * (lane >> 4) + c) * kStride<D> + (wave * kCt + ct) * 16 + (lane & 15)];
#pragma unroll
                        for (int rt = 0; rt < kRt; ++rt)
                            acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt][c], vv, acc[rt][ct], 0, 0, 0);
                    }
            }
        }
        if (t0 + kTok < t_end) {
            weigh(t0 + kTok, slot ^ 1);
            if (t0 + 2 * kTok < t_end) {
                fetch(t0 + 2 * kTok);
                if (kNeedO) next.load(vg, t0 + 2 * kTok, t_end);
            }
        }
    }
    const size_t out_row = ((size_t)hl * n_splits + split) * w.nr + row0;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        float s = sum[i];
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (col == 0 && row0 + first + 8 * i < w.nr) part_l[out_row + first + 8 * i] = s;
    }
    if (!kNeedO) return;
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * rt + 4 * (lane >> 4) + r;
                if (row0 + row < w.nr) part_o[(out_row + row) * D + (wave * kCt + ct) * 16 + (lane & 15)] = acc[rt][ct][r];
            }
}

#include "score_fixed.h"

// ------------------------------------------------------------------------------------
// Merge.  `spread` waves per row, D / 64 consecutive elements per lane.  Grid: x = 4 / spread rows of the piece, z = KV head.
// The output is left in fp32, with kFixed also as digits.  kOwn: every split has its own reference and has left out a token of its
// own (digit_sweep): the largest reference's split stays as it is, the others are brought to it and get their tokens back.
// What bounds it: loads that wait for one another (heads, then the values that the heads name), each a few us from another die's
// memory, so a wave asks for all of its splits at once.  Calls of 8 heads x 48 rows, 32 splits, us: a loop over the splits in one wave
// 56.1, four waves with eight each 47.7; of 32 heads x 128 rows, 8 splits: one wave 49.2, four 54.0.
// A single split is taken as it is: calls of 128 heads x 192 rows x 109 tokens, with the eight loads / so, 55.3 / 44.0 us (bf16, d = 64; of
// that 4 by this), of x 212 rows x 56 52.6 / 45.6 (fp32, d = 64).  (A branch around every load instead costs full merges 1.6 us of 6.2.)
template <typename T, int D, bool kNeedO, bool kFixed, bool kOwn, typename Lens>
__global__ __launch_bounds__(kThreads) void plain_merge(const T *__restrict__ v, int N, int W, int Hkv, int ragged, Lens lens,
                                                        Piece w, int split_len, int n_splits, int spread,
                                                        const float *__restrict__ part_l, const float4 *__restrict__ part_head,
                                                        const float *__restrict__ part_o, RowRecord *__restrict__ records,
                                                        float *__restrict__ out, int8_t *__restrict__ out_digits) {
    constexpr int kE = D / 64, kWaves = kThreads / 64, kEach = kMergeEach;
    static_assert(kSweepSplits <= 64, "a split per lane");
    __shared__ float o_s[kWaves - 1][D];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = wave % spread, lane = threadIdx.x & 63;
    const int hl = blockIdx.z, bg = w.bg0 + hl, row = min((int)blockIdx.x * (kWaves / spread) + wave / spread, w.nr - 1);
    const int len = seq_len_of(lens, ragged, bg / Hkv, N);
    const int live = (len + split_len - 1) / split_len;
    RowRecord *rec = records + (size_t)hl * w.nr + row;
    auto part_row = [&](int s) { return ((size_t)hl * n_splits + s) * w.nr + row; };
    float os[kEach][kE], o[kE];
    auto load_outputs = [&](int s0) {
        if (live == 1) {                                     // uniform
#pragma unroll
            for (int e = 0; e < kE; ++e) os[0][e] = part_o[part_row(0) * D + lane * kE + e];
            return;
        }
#pragma unroll
        for (int i = 0; i < kEach; ++i)
#pragma unroll
            for (int e = 0; e < kE; ++e) os[i][e] = part_o[part_row(min(s0 + part + i * spread, live - 1)) * D + lane * kE + e];
    };
    const T *vl = v + (size_t)bg * N * D + lane * kE;        // this lane's elements of a value
    int top, best = 0, tok = 0;
    float m, l, wt = 1.f, vt[kE];
    bool back = false;                                       // this lane's split gets its token back
    auto load_top = [&]() {
#pragma unroll
        for (int e = 0; e < kE; ++e) vt[e] = kNeedO ? load_as_float(vl + (size_t)top * D + e) : 0.f;
    };
    // (what has an address is on the way before the first of it is waited for)
    if constexpr (kOwn) {
        const float4 h = lane < live ? part_head[part_row(lane)] : make_float4(-INFINITY, 0.f, __int_as_float(kNoToken), 0.f);
        if (kNeedO) load_outputs(0);
        m = wave_reduce<MaxOp>(h.x);
        best = __ffsll(__ballot(h.x == m)) - 1;              // the first split attaining the maximum holds the lowest such token
        tok = min(__float_as_int(h.z), len - 1);             // (logits that are not numbers have no largest one)
        top = __builtin_amdgcn_readlane(tok, best);
        load_top();
        // (a split without a visible logit above -infinity weighs nothing: exp(-inf); what is not a number stays that)
        wt = lane == best ? 1.f : lane < live ? exp_nonpositive(h.x - m) : 0.f;
        back = lane != best && h.x != -INFINITY;
        l = wave_reduce<SumOp>(lane < live ? fmaf(wt, h.y, back ? wt : 0.f) : 0.f);
    } else {
        top = min(rec->top, len - 1);
        m = rec->m;
        l = lane < live ? part_l[part_row(lane)] : 0.f;
        if (kNeedO) load_outputs(0);
        load_top();
        for (int s = lane + 64; s < live; s += 64) l += part_l[part_row(s)];       // (a row's tokens taken in segments)
        l = wave_reduce<SumOp>(l);
    }
#pragma unroll
    for (int e = 0; e < kE; ++e) o[e] = 0.f;
    if (kNeedO && live == 1) {                               // uniform: its own reference and token are the row's
#pragma unroll
        for (int e = 0; e < kE; ++e) o[e] = part == 0 ? os[0][e] : 0.f;
    } else if (kNeedO) {
        for (int s0 = 0; s0 < live; s0 += kEach * spread) {
            if (s0 > 0) load_outputs(s0);
            if constexpr (kOwn) {
                float vs[kEach][kE];
#pragma unroll
                for (int i = 0; i < kEach; ++i) {
                    const int t = __builtin_amdgcn_readlane(tok, min(s0 + part + i * spread, live - 1));
#pragma unroll
                    for (int e = 0; e < kE; ++e) vs[i][e] = load_as_float(vl + (size_t)t * D + e);
                }
#pragma unroll
                for (int i = 0; i < kEach; ++i) {
                    const int s = min(s0 + part + i * spread, 63);
                    const float ws = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wt), s));
                    const bool again = __builtin_amdgcn_readlane((int)back, s) != 0;
#pragma unroll
                    for (int e = 0; e < kE; ++e) o[e] = s0 + part + i * spread < live ? fmaf(ws, os[i][e] + (again ? vs[i][e] : 0.f), o[e]) : o[e];
                }
            } else {
#pragma unroll
                for (int i = 0; i < kEach; ++i)
#pragma unroll
                    for (int e = 0; e < kE; ++e) o[e] += s0 + part + i * spread < live ? os[i][e] : 0.f;
            }
        }
        if (spread > 1) {                                    // uniform
            if (part > 0)
#pragma unroll
                for (int e = 0; e < kE; ++e) o_s[wave - 1][lane * kE + e] = o[e];
            __syncthreads();
            if (part == 0)
                for (int i = 0; i < spread - 1; ++i)
#pragma unroll
                    for (int e = 0; e < kE; ++e) o[e] += o_s[wave + i][lane * kE + e];
        }
    }
    if (part > 0) return;
    const float frac = l / (1.0f + l);                       // 1 - A_{i,top}; the top token's own weight is exp(0) = 1
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    double oo = 0.0, dk = 0.0, dj = 0.0;
    double unit = 0.0;
    if (kNeedO) {
        float oi[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const float diff = frac * (vt[e] - o[e] * inv);  // v_top - o_i
            oi[e] = vt[e] - diff;
            const float comb = fmaf(m, diff, vt[e]);         // (1+Z) v_top - Z o_i
            oo += (double)oi[e] * oi[e];
            dk += (double)diff * diff;
            dj += (double)comb * comb;
        }
        const size_t at = (size_t)hl * w.nr + row;
        if constexpr (kFixed) {
            const float f[4] = {oi[0], kE > 1 ? oi[kE - 1] : 0.f, 0.f, 0.f};
            const double x[4] = {f[0], f[1], 0.0, 0.0};
            const int oe = max_exponent(wave_reduce<MaxBitsOp>(max_abs(f)));
            unit = row_unit(oe);
            uint32_t p[kRowDigits];
            digits_of<kRowDigits>(x, oe, p);
#pragma unroll
            for (int k = 0; k < kRowDigits; ++k) {
                int8_t *dst = out_digits + digit_address<kRowDigits, D>((size_t)hl * ((w.nr + 15) / 16) + row / 16, k, row, lane * kE);
                if constexpr (kE == 2) *(uint16_t *)dst = (uint16_t)p[k];
                else *dst = (int8_t)p[k];
            }
        }
#pragma unroll
        for (int e = 0; e < kE; ++e) out[at * D + lane * kE + e] = oi[e];
        oo = wave_reduce<SumOp>(oo);
        dk = wave_reduce<SumOp>(dk);
        dj = wave_reduce<SumOp>(dj);
    }
    if (lane == 0) {
        if (kOwn) { rec->m = m; rec->top = top; }
        rec->last = len - W + (w.r0 + row) % W;
        rec->inv_l = 1.0f / (1.0f + l);
        rec->top_dk = (float)dk;
        rec->top_dj = (float)dj;
        rec->oo = oo;
        rec->unit = unit;
    }
}

// ------------------------------------------------------------------------------------
// Short sequences in two launches.  short_partial: logits, weights and P V of one tile of 64 tokens, relative to the tile's
// own maximum and without its top token (and once more with it: the merge wants only the row's top token left out).
// plain_score<.., kShort> merges the tiles' records itself before it scores.  Grid: x = tile, z = KV head.
// What bounds a call this small is launches and the latency of dependent loads: fp32, one head, d = 64, 512 tokens, all
// three scores took 17 us in four launches (logits 5.6, weights 4.8, merge 2.8, scores 5.0).
// ------------------------------------------------------------------------------------
constexpr int kShortTiles = 16;      // most tiles of a short sequence

template <typename T, int D, int kRt, bool kNeedO, typename Lens>
__global__ __launch_bounds__(kThreads) void short_partial(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
                                                          int N, int W, int Hkv, int ragged, Lens lens, Piece w,
                                                          float *__restrict__ z, float4 *__restrict__ heads, float *__restrict__ part_o) {
    constexpr int kRows = 16 * kRt, kPs = kTile + 4, kCt = D / 64;
    __shared__ __attribute__((aligned(16))) float rows_s[kRows * kStride<D>], v_s[kNeedO ? kTile * kStride<D> : 4], p_s[kRows * kPs];
    __shared__ float2 best_s[4][kRows];
    __shared__ float l_s[4][kRows];
    const int hl = blockIdx.z, b = hl / Hkv, M = w.nr, n_tiles = gridDim.x;
    const int len = seq_len_of(lens, ragged, b, N), t0 = blockIdx.x * kTile;
    if (t0 >= len) return;                                   // uniform
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, p = t0 + wave * 16 + (lane & 15);
    RowRegs<T, D> tok;
    tok.load(k + (size_t)hl * N * D, p, len, lane >> 4);
    {
        TileRegs<T, D, kRows> qr;
        qr.load(q + (size_t)hl * M * D, 0, M);
        TileRegs<T, D, kTile> vr;
        if (kNeedO) vr.load(v + (size_t)hl * N * D, t0, len);
        qr.store(rows_s);
        if (kNeedO) vr.store(v_s);
    }
    __syncthreads();
    f64x4 acc[kRt];
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt) acc[rt] = f64x4{0.0, 0.0, 0.0, 0.0};
    tile_dots<T, D, kRt>(rows_s, tok, lane, acc);
    float x[kRt * 4];
#pragma unroll
    for (int i = 0; i < kRt * 4; ++i) {
        const int row = 4 * i + (lane >> 4);
        x[i] = (float)(acc[i >> 2][i & 3] * (1.0 / sqrt((double)D)));            // scaled logit: the only rounding
        const bool seen = row < M && p < len && p <= len - W + row % W;
        if (seen) z[((size_t)hl * M + row) * w.z_stride + p] = x[i];
        float m = seen && x[i] > -INFINITY ? x[i] : -INFINITY;
        int at = seen && x[i] > -INFINITY ? p : kNoToken;
        lanes_best<16>(m, at);
        if ((lane & 15) == 0) best_s[wave][row] = make_float2(m, __int_as_float(at));
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRt * 4; ++i) {
        const int row = 4 * i + (lane >> 4);
        float m = best_s[0][row].x;
        int top = __float_as_int(best_s[0][row].y);
#pragma unroll
        for (int c = 1; c < 4; ++c)                          // (tokens ascend with the wave: strict keeps the lowest)
            if (best_s[c][row].x > m) { m = best_s[c][row].x; top = __float_as_int(best_s[c][row].y); }
        const bool seen = row < M && p < len && p <= len - W + row % W;
        const float e = seen && p != top ? exp_nonpositive(x[i] - m) : 0.f;
        p_s[row * kPs + wave * 16 + (lane & 15)] = e;
        const float l = row16_reduce<SumOp>(e);
        if ((lane & 15) == 0) l_s[wave][row] = l;
        if (wave == 0 && (lane & 15) == 0) best_s[0][row] = make_float2(m, __int_as_float(top));     // (read by this wave alone so far)
    }
    __syncthreads();
    const size_t record = ((size_t)hl * n_tiles + blockIdx.x) * M;
    if ((int)threadIdx.x < M) {
        const int row = threadIdx.x;
        heads[record + row] = make_float4(best_s[0][row].x, (l_s[0][row] + l_s[1][row]) + (l_s[2][row] + l_s[3][row]), best_s[0][row].y, 0.f);
    }
    if (!kNeedO) return;
    f32x4 o[kRt][kCt];
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt)
#pragma unroll
        for (int ct = 0; ct < kCt; ++ct) o[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kTile / 16; ++s) {
        f32x4 a[kRt];
#pragma unroll
        for (int rt = 0; rt < kRt; ++rt) a[rt] = *(const f32x4 *)(p_s + (16 * rt + (lane & 15)) * kPs + 16 * s + 4 * (lane >> 4));
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const float vv = v_s[(16 * s + 4 * (lane >> 4) + c) * kStride<D> + (wave * kCt + ct) * 16 + (lane & 15)];
#pragma unroll
                for (int rt = 0; rt < kRt; ++rt) o[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rt][c], vv, o[rt][ct], 0, 0, 0);
            }
    }
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * rt + 4 * (lane >> 4) + r;
            if (row >= M) continue;
            const int top = __float_as_int(best_s[0][row].y);
#pragma unroll
            for (int ct = 0; ct < kCt; ++ct) {
                const int col = (wave * kCt + ct) * 16 + (lane & 15);
                float *dst = part_o + (record + row) * 2 * D + col;
                dst[0] = o[rt][ct][r];
                dst[D] = o[rt][ct][r] + (top != kNoToken ? v_s[(top - t0) * kStride<D> + col] : 0.f);
            }
        }
}

// The rows' outputs (into LDS as fp32) and records from the tiles' partial ones; the barrier after it is the caller's.
template <typename T, int D, int kRt, bool kNeedO>
__device__ __forceinline__ void merge_short(const T *__restrict__ vg, int len, int W, int M, int hl, int n_tiles,
                                            const float4 *__restrict__ heads, const float *__restrict__ part_o, float *rows_s,
                                            RowRecord *rec_s) {
    constexpr int kRows = 16 * kRt, kSub = kThreads / kRows, kOwn = kShortTiles / kSub, kE = D / 64;
    __shared__ float w_s[kRows][kShortTiles], l_s[kRows];         // the tiles' weights; the sum without the top token
    const int live = (len + kTile - 1) / kTile;
    {
        const int row = threadIdx.x / kSub, sub = threadIdx.x % kSub;
        float hm[kOwn], hl_[kOwn];
        float m = -INFINITY;
        int top = kNoToken;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int s = sub + i * kSub;
            const float4 h = row < M && s < live ? heads[((size_t)hl * n_tiles + s) * M + row] : make_float4(-INFINITY, 0.f, __int_as_float(kNoToken), 0.f);
            hm[i] = h.x;
            hl_[i] = h.y;
            if (h.x > m || (h.x == m && __float_as_int(h.z) < top)) { m = h.x; top = __float_as_int(h.z); }
        }
        lanes_best<kSub>(m, top);
        top = min(top, len - 1);                             // (logits that are not numbers have no largest one)
        float l = 0.f;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int s = sub + i * kSub;
            const float wt = hm[i] > -INFINITY ? exp_nonpositive(hm[i] - m) : 0.f;
            w_s[row][s] = wt;
            l += fmaf(wt, hl_[i], s != top / kTile ? wt : 0.f);          // (other tiles count their top token)
        }
#pragma unroll
        for (int off = kSub / 2; off > 0; off >>= 1) l += __shfl_xor(l, off);
        if (sub == 0) {
            RowRecord &rec = rec_s[row];
            rec.m = m;
            rec.top = top;
            rec.inv_l = 1.0f / (1.0f + l);
            rec.last = len - W + row % W;
            l_s[row] = l;
        }
    }
    __syncthreads();
    if (!kNeedO) return;
    // Sixteen lanes per row, 16-byte pieces: short code matters where every instruction is fetched for the first time.
    const int sub = threadIdx.x & 15;
#pragma unroll 1
    for (int row = threadIdx.x >> 4; row < kRows; row += 16) {
        const int rc = min(row, M - 1), top = rec_s[rc].top;
        f32x4 vt[kE], o[kE];
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const T *src = vg + (size_t)top * D + (sub + 16 * e) * 4;
            vt[e] = f32x4{load_as_float(src), load_as_float(src + 1), load_as_float(src + 2), load_as_float(src + 3)};
            o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int s0 = 0; s0 < live; s0 += 8)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int s = min(s0 + u, live - 1);
                const float wt = s0 + u < live ? w_s[rc][s] : 0.f;
                const float *src = part_o + ((((size_t)hl * n_tiles + s) * M + rc) * 2 + (s != top / kTile ? 1 : 0)) * D + sub * 4;
#pragma unroll
                for (int e = 0; e < kE; ++e) o[e] += wt * *(const f32x4 *)(src + 64 * e);
            }
        const float l = l_s[rc], m = rec_s[rc].m;
        const float frac = l / (1.0f + l);                   // 1 - A_{i,top}; the top token's own weight is exp(0) = 1
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        double oo = 0.0, dk = 0.0, dj = 0.0;
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            f32x4 oi;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float diff = frac * (vt[e][c] - o[e][c] * inv);    // v_top - o_i
                oi[c] = vt[e][c] - diff;
                const float comb = fmaf(m, diff, vt[e][c]);  // (1+Z) v_top - Z o_i
                oo += (double)oi[c] * oi[c];
                dk += (double)diff * diff;
                dj += (double)comb * comb;
            }
            *(f32x4 *)(rows_s + row * kStride<D> + (sub + 16 * e) * 4) = oi;
        }
        oo = row16_reduce<SumOp>(oo);
        dk = row16_reduce<SumOp>(dk);
        dj = row16_reduce<SumOp>(dj);
        if (sub == 0) {
            rec_s[row].oo = oo;
            rec_s[row].top_dk = (float)dk;
            rec_s[row].top_dj = (float)dj;
        }
    }
}

// ------------------------------------------------------------------------------------
// Scores.  Grid: x = `n_tiles` tiles of 64 tokens of the piece, z = KV head.  `add`: on top of what `scores` holds (the
// caller's running scores, or the rows of an earlier piece).
// ------------------------------------------------------------------------------------
template <typename T, int D, int kRt, int kVariant, bool kShort, typename Lens>
__global__ __launch_bounds__(kThreads, kShort ? 2 : 4) void plain_score(const T *__restrict__ v, int N, int W, int Hkv,
                                                           int ragged, Lens lens, Piece w, int n_tiles,
                                                           const float *__restrict__ z,
                                                           const RowRecord *__restrict__ records,
                                                           const float *__restrict__ out, const float4 *__restrict__ heads,
                                                           const float *__restrict__ part_o, float *__restrict__ scores,
                                                           size_t variant_stride, int add) {
    constexpr int kRows = 16 * kRt;
    constexpr bool kAttnLike = kVariant == OBC_ATTN || kVariant == OBC_VATP;
    constexpr bool kNeedO = kVariant == OBC_KEY || kVariant == OBC_JOINT || kVariant == OBC_ALL;
    constexpr bool kNeedV = kVariant != OBC_ATTN;
    __shared__ __attribute__((aligned(16))) float rows_s[kNeedO ? kRows * kStride<D> : 4];
    __shared__ __attribute__((aligned(16))) RowRecord rec_s[kRows];

    const int hl = blockIdx.z, bg = w.bg0 + hl, b = bg / Hkv;
    const int len = seq_len_of(lens, ragged, b, N);
    const int t_begin = w.s0 + blockIdx.x * n_tiles * kTile, t_end = min(t_begin + n_tiles * kTile, w.s1);
    const int t_live = min(t_end, len);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, j = lane >> 4;
    const T *vg = v + (size_t)bg * N * D;

    for (int t0 = t_begin; t0 < t_end; t0 += kTile) {
        const int p = t0 + wave * 16 + (lane & 15);
        float acc_v = 0.f, acc_k = 0.f, acc_j = 0.f;
        if (t0 < t_live) {                                   // uniform
            RowRegs<T, D> tok;
            double vv = 0.0;
            float l1 = 0.f;
            if (kNeedV) {                                    // ||v_p||^2 (and ||v_p||_1): four lanes per token
                tok.load(vg, p, t_live, j);
#pragma unroll
                for (int s = 0; s < D / 16; ++s)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        vv += (double)tok.x[s][c] * tok.x[s][c];
                        l1 += fabsf(tok.x[s][c]);
                    }
                vv += __shfl_xor(vv, 16);
                vv += __shfl_xor(vv, 32);
                l1 += __shfl_xor(l1, 16);
                l1 += __shfl_xor(l1, 32);
            }
            for (int row0 = 0; row0 < w.nr; row0 += kRows) {
                TileRegs<float, D, kRows> orow;
                if (kNeedO && !kShort) orow.load(out + (size_t)hl * w.nr * D, row0, w.nr);
                float x[kRt * 4];
#pragma unroll
                for (int i = 0; i < kRt * 4; ++i) {
                    const int row = row0 + 4 * i + j;
                    x[i] = p < t_live && row < w.nr ? z[((size_t)hl * w.nr + row) * w.z_stride + (p - w.s0)] : 0.f;
                }
                __syncthreads();                             // the rows before these have been read
                if (kShort) merge_short<T, D, kRt, kNeedO>(vg, len, W, w.nr, hl, gridDim.x, heads, part_o, rows_s, rec_s);
                if (kNeedO && !kShort) orow.store(rows_s);
                if (!kShort && (int)threadIdx.x < kRows && row0 + (int)threadIdx.x < w.nr)
                    rec_s[threadIdx.x] = records[(size_t)hl * w.nr + row0 + threadIdx.x];
                __syncthreads();
                f64x4 acc[kRt];
#pragma unroll
                for (int rt = 0; rt < kRt; ++rt) acc[rt] = f64x4{0.0, 0.0, 0.0, 0.0};
                if (kNeedO) tile_dots<T, D, kRt>(rows_s, tok, lane, acc);
#pragma unroll
                for (int i = 0; i < kRt * 4; ++i) {
                    __builtin_amdgcn_sched_barrier(0);       // (one row's constants at a time: registers)
                    const int row = row0 + 4 * i + j;
                    const RowRecord &r = rec_s[4 * i + j];
                    if (row >= w.nr || p > r.last) continue;
                    const float a = exp_nonpositive(x[i] - r.m) * r.inv_l;
                    if (kAttnLike) {                         // Eq. 8: only the weight itself is summed
                        acc_v += a;
                        continue;
                    }
                    const float a2 = a * a;
                    acc_v = fmaf(a2, (float)vv, acc_v);
                    if (kNeedO) {
                        const double vo = acc[i >> 2][i & 3], zd = x[i];
                        const double d2 = (vv + r.oo) - 2.0 * vo;                        // ||v_p - o_i||^2
                        const bool is_top = p == r.top;
                        if (kVariant != OBC_JOINT)
                            acc_k = fmaf(a2 * x[i] * x[i], is_top ? r.top_dk : at_least_0((float)d2), acc_k);
                        if (kVariant != OBC_KEY) {
                            const double dj = vv + zd * (2.0 * (vv - vo) + zd * d2);     // ||v_p + Z (v_p - o_i)||^2
                            acc_j = fmaf(a2, is_top ? r.top_dj : at_least_0((float)dj), acc_j);
                        }
                    }
                }
            }
            if (kVariant == OBC_VATP) acc_v *= l1;
            acc_v += __shfl_xor(acc_v, 16);                  // the four lanes of a token held different rows
            acc_v += __shfl_xor(acc_v, 32);
            acc_k += __shfl_xor(acc_k, 16);
            acc_k += __shfl_xor(acc_k, 32);
            acc_j += __shfl_xor(acc_j, 16);
            acc_j += __shfl_xor(acc_j, 32);
        }
        if (j == 0 && p < t_end) {
            float *dst = scores + (size_t)bg * N + p;
            const float s[3] = {acc_v, acc_k, acc_j};
            constexpr int kFirst = kVariant == OBC_ALL || kAttnLike ? 0 : kVariant, kCount = kVariant == OBC_ALL ? 3 : 1;
#pragma unroll
            for (int c = 0; c < kCount; ++c) {
                float *d = dst + c * variant_stride;
                if (!add) *d = p < len ? s[kFirst + c] : 0.f;
                else if (p < len) *d += s[kFirst + c];       // running scores: the padding is left alone
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// Host
// ------------------------------------------------------------------------------------
// f with the variant as a constant.
template <typename F>
void with_variant(int variant, F &&f) {
    switch (variant) {
        case OBC_VALUE: return f(std::integral_constant<int, OBC_VALUE>());
        case OBC_KEY: return f(std::integral_constant<int, OBC_KEY>());
        case OBC_JOINT: return f(std::integral_constant<int, OBC_JOINT>());
        case OBC_ATTN: return f(std::integral_constant<int, OBC_ATTN>());
        case OBC_VATP: return f(std::integral_constant<int, OBC_VATP>());
        default: return f(std::integral_constant<int, OBC_ALL>());
    }
}

// Short sequences: see short_partial.
template <typename T, int D, int kRt, typename Lens>
hipError_t run_short(const ScoreArgs &a, const Lens &lens, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    const T *q = (const T *)a.q, *k = (const T *)a.k, *v = (const T *)a.v;
    float *z = (float *)(base + ws.pl_z), *part_o = (float *)(base + ws.pl_part_o);
    float4 *heads = (float4 *)(base + ws.pl_part_l);
    const bool need_o = a.variant == OBC_KEY || a.variant == OBC_JOINT || a.variant == OBC_ALL;
    Piece w;
    w.bg0 = w.r0 = w.s0 = 0; w.nr = a.G * a.W; w.s1 = a.N; w.z_stride = ws.pl_z_stride;
    const dim3 grid(ws.pl_splits, 1, a.B * a.Hkv);
    if (a.stage_mask & OBC_STAGE_SWEEP1) {
        if (need_o)
            short_partial<T, D, kRt, true><<<grid, dim3(kThreads), 0, stream>>>(q, k, v, a.N, a.W, a.Hkv, a.ragged, lens, w, z, heads, part_o);
        else
            short_partial<T, D, kRt, false><<<grid, dim3(kThreads), 0, stream>>>(q, k, v, a.N, a.W, a.Hkv, a.ragged, lens, w, z, heads, part_o);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    if (!(a.stage_mask & OBC_STAGE_SWEEP2)) return hipSuccess;
    with_variant(a.variant, [&](auto which) {
        plain_score<T, D, kRt, decltype(which)::value, true><<<grid, dim3(kThreads), 0, stream>>>(
            v, a.N, a.W, a.Hkv, a.ragged, lens, w, 1, z, nullptr, nullptr, heads, part_o, a.scores, (size_t)a.B * a.Hkv * a.N, a.accumulate);
    });
    return hipGetLastError();
}

template <typename T, int D, int kRt, typename Lens>
hipError_t run_with(const ScoreArgs &a, const Lens &lens, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    const T *q = (const T *)a.q, *k = (const T *)a.k, *v = (const T *)a.v;
    float *z = (float *)(base + ws.pl_z), *part_l = (float *)(base + ws.pl_part_l), *part_o = (float *)(base + ws.pl_part_o);
    float *out = (float *)(base + ws.pl_out);
    float2 *best = (float2 *)(base + ws.pl_best);
    RowRecord *rec = (RowRecord *)(base + ws.pl_records);
    int8_t *o_digits = (int8_t *)(base + ws.pl_o_digits);
    // score_fixed.h, 64 or 128 rows per workgroup.
    constexpr bool fixed = kRt == 4 || kRt == 8;
    constexpr int kRb = kRt == 8 ? 8 : 4;
    const bool need_o = a.variant == OBC_KEY || a.variant == OBC_JOINT || a.variant == OBC_ALL;
    const int BH = a.B * a.Hkv, M = a.G * a.W;
    const size_t variant_stride = (size_t)BH * a.N;
    const bool one_piece = ws.pl_heads >= BH && ws.pl_rows >= M && ws.pl_seg >= a.N;
    // A piece's buffers hold nothing of the other pieces: with several, a later stage repeats the earlier ones.
    const int mask = one_piece ? a.stage_mask : a.stage_mask & OBC_STAGE_SWEEP2 ? (int)OBC_STAGE_ALL
                     : a.stage_mask & OBC_STAGE_COMBINE ? OBC_STAGE_SWEEP1 | OBC_STAGE_COMBINE : a.stage_mask;
    const int segs = (a.N + ws.pl_seg - 1) / ws.pl_seg;
    const bool with_digits = fixed && ws.pl_digits;
    constexpr bool kOwnOnly = fixed && sizeof(T) == 2;       // (sweeps_digits)
    if (kOwnOnly && !with_digits) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    for (int bg0 = 0; bg0 < BH; bg0 += ws.pl_heads)
        for (int r0 = 0; r0 < M; r0 += ws.pl_rows) {
            Piece w;
            w.bg0 = bg0; w.r0 = r0; w.nr = std::min(ws.pl_rows, M - r0); w.z_stride = ws.pl_z_stride;
            const unsigned heads = std::min(ws.pl_heads, BH - bg0), chunks = (w.nr + 16 * kRt - 1) / (16 * kRt);
            auto segment = [&](int i) { w.s0 = i * ws.pl_seg; w.s1 = std::min(w.s0 + ws.pl_seg, a.N); };
            const unsigned row_chunks = (w.nr + 16 * kRb - 1) / (16 * kRb);         // (score_fixed.h)
            auto logits = [&]() {
                const unsigned ranges = (w.s1 - w.s0 + ws.pl_range - 1) / ws.pl_range;
                if constexpr (!fixed)
                    plain_logits<T, D, kRt><<<dim3(ranges, chunks, heads), dim3(kThreads), 0, stream>>>(
                        q, k, a.N, a.W, a.Hq, a.Hkv, a.ragged, lens, w, ws.pl_range, ws.pl_ranges, z, best);
                else if constexpr (!kOwnOnly)
                    blocked_logits<T, D><<<dim3(heads, ranges, (w.nr + kLogitRows - 1) / kLogitRows), dim3(kThreads), 0, stream>>>(
                        q, k, a.N, a.W, a.Hq, a.Hkv, a.ragged, lens, w, ws.pl_range, ws.pl_ranges, z, best);
                e = hipGetLastError();
                return e == hipSuccess;
            };
            auto weights = [&](auto with_output) {           // (with digits: from the keys on)
                constexpr bool kNeedO = decltype(with_output)::value;
                const unsigned splits = (w.s1 - w.s0 + ws.pl_split - 1) / ws.pl_split;
                if constexpr (fixed)
                    if (with_digits) {
                        auto sweep = [&](auto row_blocks) {
                            constexpr int kRows = 16 * decltype(row_blocks)::value;
                            digit_sweep<T, D, decltype(row_blocks)::value, kNeedO><<<dim3(heads, splits, (w.nr + kRows - 1) / kRows), dim3(kWeightThreads), 0, stream>>>(
                                q, k, v, a.N, a.W, a.Hq, a.Hkv, a.ragged, lens, w, ws.pl_split, ws.pl_splits, z, (float4 *)part_l, part_o);
                        };
                        if (ws.pl_sweep_rows == 64) sweep(std::integral_constant<int, 4>());
                        else sweep(std::integral_constant<int, 8>());
                    }
                if constexpr (!fixed)
                    plain_weights<T, D, kRt, kNeedO><<<dim3(splits, chunks, heads), dim3(kThreads), 0, stream>>>(
                        v, a.N, a.W, a.Hkv, a.ragged, lens, w, ws.pl_range, ws.pl_ranges, ws.pl_split, ws.pl_splits, z, best, rec,
                        part_l, part_o);
                else if constexpr (!kOwnOnly)
                    if (!with_digits)
                        fixed_weights<T, D, kRb, kNeedO><<<dim3(heads, splits, row_chunks), dim3(kWeightThreads), 0, stream>>>(
                            v, a.N, a.W, a.Hkv, a.ragged, lens, w, ws.pl_range, ws.pl_ranges, ws.pl_split, ws.pl_splits, z, best, rec,
                            part_l, part_o);
            };
            if (mask & OBC_STAGE_SWEEP1) {
                for (int i = 0; i < segs && !with_digits; ++i) {               // every range's maximum first
                    segment(i);
                    if (!logits()) return e;
                }
                for (int i = 0; i < segs; ++i) {
                    segment(i);
                    if (segs > 1 && !logits()) return e;
                    if (need_o) weights(std::true_type());
                    else weights(std::false_type());
                    if ((e = hipGetLastError()) != hipSuccess) return e;
                }
            }
            if (mask & OBC_STAGE_COMBINE) {
                const int spread = ws.pl_splits <= kMergeEach ? 1 : ws.pl_splits <= 2 * kMergeEach ? 2 : 4;
                const dim3 grid((w.nr * spread + 3) / 4, 1, heads);
                auto merge = [&](auto with_output, auto own) {
                    constexpr bool kNeedO = decltype(with_output)::value;
                    plain_merge<T, D, kNeedO, kNeedO && fixed, decltype(own)::value><<<grid, dim3(kThreads), 0, stream>>>(
                        v, a.N, a.W, a.Hkv, a.ragged, lens, w, ws.pl_split, ws.pl_splits, spread, part_l, (const float4 *)part_l, part_o, rec, out, o_digits);
                };
                auto merge_own = [&](auto own) {
                    if (need_o) merge(std::true_type(), own);
                    else merge(std::false_type(), own);
                };
                if constexpr (fixed)
                    if (with_digits) merge_own(std::true_type());
                if constexpr (!kOwnOnly)
                    if (!with_digits) merge_own(std::false_type());
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            if (!(mask & OBC_STAGE_SWEEP2)) continue;
            for (int i = 0; i < segs; ++i) {
                segment(i);
                if (segs > 1 && !logits()) return e;
                const int add = a.accumulate || r0 > 0;
                auto score = [&](auto which) {
                    constexpr int kVariant = decltype(which)::value;
                    if constexpr (fixed) {
                        constexpr int kTok = kFixedTile<D>;
                        const int tiles = (w.s1 - w.s0 + kTok - 1) / kTok;
                        const int n_tiles = (int)std::min((tiles * (long long)heads + kResident / 2 - 1) / (kResident / 2), kScoreTokens / kTok + 0ll);
                        fixed_score<T, D, kRb, kVariant><<<dim3(heads, (tiles + n_tiles - 1) / n_tiles), dim3(kFixedThreads), 0, stream>>>(
                            v, a.N, a.Hkv, a.ragged, lens, w, n_tiles, z, rec, out, o_digits, a.scores, variant_stride, add);
                    } else {
                        const int tiles = (w.s1 - w.s0 + kTile - 1) / kTile;
                        const int n_tiles = (int)((tiles * (long long)heads + kResident - 1) / kResident);
                        plain_score<T, D, kRt, kVariant, false><<<dim3((tiles + n_tiles - 1) / n_tiles, 1, heads), dim3(kThreads), 0, stream>>>(
                            v, a.N, a.W, a.Hkv, a.ragged, lens, w, n_tiles, z, rec, out, nullptr, nullptr, a.scores, variant_stride, add);
                    }
                };
                with_variant(a.variant, score);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
    return hipSuccess;
}

template <typename T, int D, int kRt>
hipError_t run(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    return with_lens(a.ragged, a.B, a.lens, [&](const auto &lens) {
        if constexpr (kRt <= 2)
            if (ws.pl_short) return run_short<T, D, kRt>(a, lens, ws, base, stream);
        if constexpr (kRt == 2 && sizeof(T) == 2) return hipErrorInvalidValue;          // (digit_sweep takes the others: sweeps_digits)
        else return run_with<T, D, kRt>(a, lens, ws, base, stream);
    });
}

template <typename T, int D>
hipError_t run_rows(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    // 16-row tiles of a workgroup.
    const int rows = std::min(ws.pl_rows, a.G * a.W);
    if (rows <= 16) return run<T, D, 1>(a, ws, base, stream);
    if (rows <= 32 && !(ws.pl_digits && rows > kPlainRows)) return run<T, D, 2>(a, ws, base, stream);
    if (fixed_rows(rows) == 64) return run<T, D, 4>(a, ws, base, stream);
    return run<T, D, 8>(a, ws, base, stream);
}

}  // namespace

// Two launches instead of three or four where every tile of a head may merge all of the head's records (short_partial): as long
// as that reads less than 32 MB, some 5 us, and the buffers fit the static scratch (on either scratch the same kernels).
bool fits_short(int heads, int M, int d, long long tiles) {
    const size_t rows = (size_t)heads * ((M + 15) / 16 * 16);
    return M <= 32 && tiles <= kShortTiles && (size_t)heads * tiles * tiles * M * d * 4 <= (size_t)32 << 20 &&
           rows * (tiles * (kTile * 4 + 8 * d + 16)) <= (size_t)OBC_STATIC_SCRATCH_BYTES - 7 * 256;
}

// Which calls digit_sweep takes.  Time without it over time with it, whole calls one after the other, geometric means over 8500 random
// shapes (1 to 160 heads, 17 to 512 rows, inputs that change from call to call), with outputs (key, joint, all) / without:
//   17 to 32 rows, up to 16 tiles of 64 tokens (short_partial): tiles      1-2         3-4         5-8        9-16
//     bf16, d =  64                                                  0.96 / 0.90 0.99 / 0.91 1.02 / 0.93 1.13 / 0.95
//     fp32, d =  64                                                  0.89 / 0.87 0.90 / 0.88 0.93 / 0.88 1.01 / 0.89
//     fp32, d = 128                                                  0.88 / 0.84 0.91 / 0.85 0.94 / 0.84 0.99 / 0.84
//   17 to 32 rows, longer: heads               1-2         3-5        6-11       12-23       24-47        48-
//     bf16, d =  64                        1.31 / 1.45 1.26 / 1.41 1.23 / 1.35 1.19 / 1.28 1.15 / 1.23 1.09 / 1.18
//     fp32, d =  64                        1.19 / 1.31 1.13 / 1.28 1.08 / 1.20 0.99 / 1.09 0.98 / 1.04 0.91 / 1.00
//     fp32, d = 128                        1.13 / 1.22 1.07 / 1.17 1.04 / 1.12 0.99 / 1.04 1.00 / 1.01 0.96 / 1.02
//   over 32 rows: tiles x 128-row chunks      -63         64-95      96-127      128-159     160-191     192-255     256-383      384-
//     bf16, d =  64                        1.01 / 1.06 1.01 / 1.04 1.03 / 1.12 1.03 / 1.09 1.06 / 1.13 1.10 / 1.16 1.12 / 1.16 1.19 / 1.28
//     fp32, d =  64                        0.99 / 1.03 0.98 / 1.02 1.00 / 1.05 1.00 / 1.06 1.04 / 1.07 1.08 / 1.08 1.05 / 1.09 1.10 / 1.11
//     fp32, d = 128                        0.92 / 0.90 0.91 / 0.89 0.98 / 0.94 0.96 / 0.95 1.02 / 1.02 1.08 / 1.05 1.05 / 1.05 1.13 / 1.14
// (over 32 rows with 128-row workgroups where digit_sweep takes 64 now, which it gains by).  So: of calls that short_partial would take
// only bf16 ones with outputs, from five tiles up; else bf16 always; of up to 32 fp32 rows, which leave half of its waves without any,
// only few heads (the kernels for up to 32 rows need many to fill the chip); beyond, fp32 from 128 and 160 tiles up.  (The line counts
// every head of the call, so which kernel forms a sequence's logits, and with it their last bit now and then, depends on the batch.)
int sweeps_digits(int dtype, bool outputs, int heads, int M, int d, long long tiles) {
    if (M <= kPlainRows) return 0;
    if (fits_short(heads, M, d, tiles)) return dtype != OBC_F32 && outputs && tiles > 4;
    if (dtype != OBC_F32) return 1;
    if (M <= 32) return heads < (outputs ? 12 : 24);
    return tiles * heads * ((M + 127) / 128) >= (d == 128 ? 160 : 128);
}

// Pieces.  `cap` bounds the workspace: as many KV heads at a time as fit (which leaves every sum as it is), then as many
// rows of one head, then as many tokens (which does not).  Within it a launch should fill the chip once (kResident; whole turns of
// kCus workgroups for digit_sweep), so that no workgroup pays a prologue more than needed and no last turn is nearly empty; a row has at most kMaxRanges
// maxima, which every workgroup of the weight kernel reads.
static void plan_with(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int digits, size_t cap, ScoreWorkspace *ws, size_t *off) {
    auto align_up = [](size_t x, size_t a) { return (x + a - 1) / a * a; };
    const int BH = B * Hkv, M = Hq / Hkv * W;
    const long long tiles = (N + kTile - 1) / kTile, logit_chunks = (long long)BH * ((M + 31) / 32);
    ws->pl_digits = digits;
    const bool fixed = M > 32 || ws->pl_digits;
    const long long chunks = fixed ? (long long)BH * ((M + 127) / 128) : logit_chunks, resident = fixed ? kResident / 2 : kResident;
    const long long logit_tiles = (tiles * logit_chunks + kResident - 1) / kResident;
    const long long range_tiles = std::max((tiles + kMaxRanges - 1) / kMaxRanges, logit_tiles);
    ws->pl_range = (int)(std::min(range_tiles, tiles) * kTile);
    ws->pl_ranges = (N + ws->pl_range - 1) / ws->pl_range;
    auto split_in = [&](long long splits) {
        splits = std::max<long long>(1, std::min<long long>(splits, tiles));
        ws->pl_split = (int)align_up((N + splits - 1) / splits, kTile);
        ws->pl_splits = (N + ws->pl_split - 1) / ws->pl_split;
    };
    // digit_sweep has a workgroup per CU: as many splits as make whole turns of the chip of what a launch takes, and 64 or 128 rows
    // each.  Random calls of over 64 rows, time with 128 rows over time with 64, geometric means by 64-row chunks times tiles: up to
    // 256 1.09 (bf16, d = 64), 1.03 (fp32, d = 64), 1.05 (fp32, d = 128); 4096 and more 0.95, 0.92, 0.94.  The better of the two by
    // sweep_time is within 0.1, 0.2 and 0.2 % of the faster one in the mean, of 870, 790 and 840 calls; 64 rows where the last 128 would be
    // half empty, and 128 else, lost 4.6, 2.1 and 2.9 %.
    auto split_turns = [&](int heads) {
        const unsigned n = (unsigned)tiles, most = std::min<unsigned>(kSweepSplits, n);         // (a 32-bit division takes half the host's time)
        unsigned best = 1;
        long long least = LLONG_MAX;
        for (const int rows : {64, 128}) {
            const unsigned workgroups = (unsigned)heads * ((M + rows - 1) / rows);               // (heads whose logits fit the workspace: thousands)
            for (unsigned s = 1; s <= most; ++s) {
                const long long time = (long long)((workgroups * s + kCus - 1) / kCus) * sweep_time(dtype, rows, (int)((n + s - 1) / s));
                if (time < least) { least = time; best = s; ws->pl_sweep_rows = rows; }
            }
        }
        split_in(best);
    };
    const long long usual_splits = std::min<long long>(kMaxSplits, (resident / 2 + chunks - 1) / chunks);
    split_in(usual_splits);
    auto best_bytes = [&]() { return ws->pl_digits ? 0 : ws->pl_ranges * sizeof(float2); };
    auto row_bytes = [&]() {                                 // of one row, beside its logits
        return best_bytes() + sizeof(RowRecord) + (size_t)d * (fixed ? 9 : 4) + (size_t)ws->pl_splits * (d + (ws->pl_digits ? 4 : 1)) * 4;
    };
    auto per_row = [&]() { return row_bytes() + (size_t)align_up(N, kTile) * 4; };
    const size_t alignment = 7 * 256;                        // of the buffers
    // As many heads as fit, in as many launches of about the same size.
    auto heads_in = [&](size_t bytes) {
        const int heads = (int)std::min<size_t>(BH, (bytes - alignment) / (per_row() * align_up(M, 16)));
        const int launches = heads > 0 ? (BH + heads - 1) / heads : 0;
        return heads > 0 ? (BH + launches - 1) / launches : 0;
    };
    if (ws->pl_digits) {                                     // of what a launch takes in the default workspace: the same sums in any
        int heads = heads_in(kPlainWorkspace);
        do split_turns(std::max(heads, 1));
        while (heads_in(kPlainWorkspace) < heads && --heads > 0);              // (more splits need more room)
    }
    ws->pl_seg = N;
    ws->pl_rows = M;
    ws->pl_heads = heads_in(cap);
    cap -= alignment;
    if (ws->pl_heads < 1) {
        ws->pl_heads = 1;
        ws->pl_rows = (int)std::min<size_t>(M, cap / per_row() / 16 * 16);
        if (ws->pl_digits && ws->pl_rows <= kPlainRows) {    // so few rows at a time are not digit_sweep's
            ws->pl_digits = 0;
            split_in(usual_splits);
            ws->pl_rows = (int)std::min<size_t>(kPlainRows, cap / per_row() / 16 * 16);
        }
        if (ws->pl_rows < 1) {
            // One tile of rows at a time and as many tokens as fit, in whole splits (here also the ranges).
            ws->pl_rows = std::min(M, 16);
            ws->pl_split = ws->pl_range = (int)align_up((N + 1023) / 1024, kTile);
            ws->pl_splits = ws->pl_ranges = (N + ws->pl_split - 1) / ws->pl_split;
            const size_t room = cap / ws->pl_rows / 4, taken = row_bytes() / 4;
            const size_t seg = room > taken ? (room - taken) / ws->pl_split * ws->pl_split : 0;
            ws->pl_seg = (int)std::min<size_t>(align_up(N, ws->pl_split), std::max<size_t>(seg, ws->pl_split));
        }
    }
    auto take = [&](size_t *at, size_t bytes) { *at = *off; *off = align_up(*off + bytes, 256); };
    size_t rows = BH * align_up(M, 16);                      // (whole blocks are written)
    ws->pl_short = !fixed && fits_short(BH, M, d, tiles);
    if (ws->pl_short) {
        ws->pl_heads = BH;
        ws->pl_rows = M;
        ws->pl_split = ws->pl_range = kTile;
        ws->pl_splits = (int)tiles;
        ws->pl_z_stride = (int)tiles * kTile;
        take(&ws->pl_z, rows * ws->pl_z_stride * 4);
        take(&ws->pl_part_l, rows * tiles * sizeof(float4));
        take(&ws->pl_part_o, rows * tiles * 2 * d * 4);
        return;
    }
    rows = ws->pl_heads * align_up(ws->pl_rows, 16);
    ws->pl_z_stride = (int)align_up(ws->pl_seg, kTile);       // (whole tiles are written)
    take(&ws->pl_z, rows * ws->pl_z_stride * 4);
    take(&ws->pl_best, rows * best_bytes());
    take(&ws->pl_records, rows * sizeof(RowRecord));
    take(&ws->pl_out, rows * d * 4);
    if (fixed) take(&ws->pl_o_digits, rows * d * 5);
    take(&ws->pl_part_l, rows * ws->pl_splits * (ws->pl_digits ? sizeof(float4) : sizeof(float)));
    take(&ws->pl_part_o, rows * ws->pl_splits * d * 4);
}

void plain_plan(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int variant, size_t cap, ScoreWorkspace *ws, size_t *off) {
    const bool outputs = variant == OBC_KEY || variant == OBC_JOINT || variant == OBC_ALL;
    const long long tiles = (N + kTile - 1) / kTile;
    const int M = Hq / Hkv * W, digits = sweeps_digits(dtype, outputs, B * Hkv, M, d, tiles), other = sweeps_digits(dtype, !outputs, B * Hkv, M, d, tiles);
    const size_t begin = *off;
    plan_with(B, N, W, Hq, Hkv, d, dtype, digits, cap, ws, off);
    if (other == digits) return;
    // One workspace serves every score of a shape, whichever of them its size was asked for.
    ScoreWorkspace of_other = *ws;
    size_t end = begin;
    plan_with(B, N, W, Hq, Hkv, d, dtype, other, cap, &of_other, &end);
    *off = std::max(*off, end);
}

hipError_t launch_score_plain(const ScoreArgs &a, const ScoreWorkspace &ws, char *ws_base, hipStream_t stream) {
    if (a.dtype == OBC_F32) {
        if (a.d == 64) return run_rows<float, 64>(a, ws, ws_base, stream);
        if (a.d == 128) return run_rows<float, 128>(a, ws, ws_base, stream);
    } else {
        if (a.d == 64) return run_rows<uint16_t, 64>(a, ws, ws_base, stream);
        if (a.d == 128) return run_rows<uint16_t, 128>(a, ws, ws_base, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace obc
