// Per-head top-`budget` selection (Section 3 "Cache Eviction"; Appendix E, Algorithm 2:
// topk followed by an ascending sort of the kept indices).
//
// The budget-th largest score of a head is found by a most-significant-digit-first radix
// select over order-preserving 32-bit keys: a histogram of the leading digit over all keys picks
// the digit class that holds the threshold, the class's keys (a percent or so of the head) are
// collected into a list, and two more digits over the list fix the threshold.  A final ordered
// sweep emits, in index order, every token above it plus the first tokens equal to it until the
// budget is filled -- which is both the lowest-index tie-break and the ascending output
// order.  Integer-only bookkeeping: results are exact and reproducible.
//
// Heads of up to 32768 tokens: one workgroup per head (select_topk).  Longer heads, given a
// workspace, and the ranking of all heads of a layer together (head-adaptive budgets): slices of
// a head on separate workgroups, in three short kernels (slices_*).
//
// Protected regions (Appendix E, Algorithm 2: only positions below the cutoff compete and the
// recent tail is always kept; Appendix C: leading attention-sink tokens are always kept):
// tokens p < first or p >= len - tail get the key 0xffffffff, which no score maps to, so
// they outrank every competitor and the same select keeps them all when the budget is
// first + heavy hitters + tail.
//
// Pooling (Appendix C, SnapKV paragraph: average pooling of the scores, kernel size 5, before
// eviction): with radius r > 0 a competing token is ranked by the fp32 sum of the scores in
// its centred window of 2r+1 positions, taken in ascending position order, positions
// outside the competing range counting as zero.  The sum orders tokens as the average does
// and needs no division.
//
// select_topk reads heads of up to 65536 tokens from memory once (128-bit loads) and keeps their
// keys in registers; longer heads without a workspace are streamed again in every pass.
#include <type_traits>

#include "internal.h"
#include "wave_util.h"

namespace obc {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kItems = 4;                              // consecutive scores per thread and chunk
constexpr int kChunk = kSelThreads * kItems;           // 4096 scores per chunk

// Monotone map float -> uint32: larger float <=> larger key.  -0.0 is folded onto +0.0,
// every NaN maps to 1 (below -inf, whose key is 0x007fffff).  No score maps to 0: that key marks
// positions that do not exist (past a sequence's length), which therefore rank below every token
// and never reach a threshold as long as the budget does not exceed the length.  (Six instructions; eight with the sign
// and the zero tested apart.  A select_topk of 32K tokens forms 32 keys per thread and is bound by its instructions, four waves
// to a SIMD: with the kept keys counted per chunk before they are packed, 15.8 -> 15.3 us, 4 x 8 heads.)
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);           // (-0.0 + 0.0 is +0.0)
    const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    return f != f ? 1u : key;
}

// The same for a pooled sum.  (The shorter form above made select_topk 0.4 us slower there, 32 heads x 14.7K.)
__device__ __forceinline__ uint32_t pooled_key(float f) {
    uint32_t u = __float_as_uint(f);
    if (f != f) return 1u;
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kMaxRadius = 7;                           // largest pooling window: 15 scores

constexpr int kMaxRegChunks = 16;                       // chunks a block can keep in registers (64K scores)
constexpr int kList = 4096;                             // keys of the threshold's class that fit the LDS list

// Digits, from the top.  Scores crowd into a few binades, and LDS atomics of a wave to one counter take turns: a block
// that sees 32 keys per thread spreads its first digit over 13 bits (counting and picking it: 5.0 -> 3.4 us at 32K), where few keys per thread
// would not pay for the larger table.
template <int kFirstBits>
struct Digits {
    static constexpr int kBits0 = kFirstBits, kBits1 = kFirstBits == 13 ? 10 : 11, kBits2 = 32 - kBits0 - kBits1;
    static constexpr int kShift0 = 32 - kBits0, kShift1 = kBits2;
    static constexpr int kBins0 = 1 << kBits0, kBins1 = 1 << kBits1, kBins2 = 1 << kBits2;
};
constexpr int kSliceBits = 11;                          // first digit of the sliced kernels
constexpr int kSliceBins = 1 << kSliceBits;

struct PickShared {
    int wave_tot[kSelWaves];
    uint32_t digit;
    int remaining, in_digit;
};

template <int kFirstBits>
struct SelectShared {
    using D = Digits<kFirstBits>;
    int hist0[D::kBins0], hist1[D::kBins1], hist2[D::kBins2];
    uint32_t list[kList];
    int n_list;
    PickShared pick;
    // ordered emission of a register-resident head: per (chunk, wave) the packed counts, then the
    // numbers of greater / equal keys that come before that (chunk, wave)
    int cw_tot[kMaxRegChunks * kSelWaves];
    int cw_gt[kMaxRegChunks * kSelWaves], cw_eq[kMaxRegChunks * kSelWaves];
};

template <int kCount>
__device__ __forceinline__ void clear_counters(int *h) {     // (kCount: a multiple of 4)
    for (int i = threadIdx.x * 4; i < kCount; i += kSelThreads * 4) *(int4 *)(h + i) = make_int4(0, 0, 0, 0);
}

// Inclusive scan of one int per lane over the wave, register to register: four data-parallel-primitive steps inside
// each row of 16 lanes (shifts by 1, 2, 4, 8, lanes outside the row reading zero), then the totals of the rows on the
// far side, read from their end lanes.  kSuffix: lane l gets the sum over lanes >= l; otherwise over lanes <= l.
template <bool kSuffix>
__device__ __forceinline__ int wave_scan(int x, int lane) {
    constexpr int kShift = kSuffix ? 0x100 : 0x110;        // row_shl : row_shr
    x += __builtin_amdgcn_update_dpp(0, x, kShift + 1, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kShift + 2, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kShift + 4, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, kShift + 8, 0xf, 0xf, true);
    const int row = lane >> 4;
    if (kSuffix) {
        const int t1 = __builtin_amdgcn_readlane(x, 16), t2 = __builtin_amdgcn_readlane(x, 32), t3 = __builtin_amdgcn_readlane(x, 48);
        x += row == 0 ? t1 + t2 + t3 : row == 1 ? t2 + t3 : row == 2 ? t3 : 0;
    } else {
        const int t0 = __builtin_amdgcn_readlane(x, 15), t1 = __builtin_amdgcn_readlane(x, 31), t2 = __builtin_amdgcn_readlane(x, 47);
        x += row == 3 ? t0 + t1 + t2 : row == 2 ? t0 + t1 : row == 1 ? t0 : 0;
    }
    return x;
}

// Which digit of a histogram of kBins counters holds the element of rank `remaining` (from the top), that element's rank
// inside the digit, and how many elements the digit has.  All threads get the same answer.  Call when the histogram is
// complete but before a barrier; the shared results are not written again before the barrier of the next call.
template <int kBins>
__device__ __forceinline__ void pick_digit(const int *hist, PickShared &sh, uint32_t *digit, int *remaining, int *in_digit) {
    constexpr int kOwn = kBins >= kSelThreads ? kBins / kSelThreads : 1;       // consecutive counters of a thread
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __syncthreads();
    int c[kOwn], mine = 0;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        c[i] = tid * kOwn < kBins ? hist[tid * kOwn + i] : 0;
        mine += c[i];
    }
    const int incl = wave_scan<true>(mine, lane);          // inclusive suffix scan inside the wave (towards higher lanes)
    if (lane == 0) sh.wave_tot[wave] = incl;
    __syncthreads();
    int above = incl - mine;                               // elements in digits of higher threads
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w)
        if (w > wave) above += sh.wave_tot[w];
    if (above < *remaining && *remaining <= above + mine) {      // exactly one thread satisfies this
#pragma unroll
        for (int i = kOwn - 1; i >= 0; --i) {
            if (above < *remaining && *remaining <= above + c[i]) {
                sh.digit = (uint32_t)(tid * kOwn + i);
                sh.remaining = *remaining - above;
                sh.in_digit = c[i];
            }
            above += c[i];
        }
    }
    __syncthreads();
    *digit = sh.digit;
    *remaining = sh.remaining;
    *in_digit = sh.in_digit;
}

// The threshold inside a digit class from the class's keys.  `visit(f)` calls f(key) for this thread's share of them;
// the two histograms are cleared.  `prefix`: the class's digit in place.  Leaves the threshold in `prefix`, how many keys
// equal to it are kept in `remaining`, how many there are in `n_equal`.
template <typename D, typename Visit>
__device__ __forceinline__ void finish_class(int *hist1, int *hist2, PickShared &sh, Visit &&visit, uint32_t *prefix, int *remaining,
                                             int *n_equal) {
    uint32_t digit;
    visit([&](uint32_t key) { atomicAdd(&hist1[(key >> D::kShift1) & (D::kBins1 - 1)], 1); });
    pick_digit<D::kBins1>(hist1, sh, &digit, remaining, n_equal);
    const uint32_t middle = digit;
    visit([&](uint32_t key) {
        if (((key >> D::kShift1) & (D::kBins1 - 1)) == middle) atomicAdd(&hist2[key & (D::kBins2 - 1)], 1);
    });
    pick_digit<D::kBins2>(hist2, sh, &digit, remaining, n_equal);
    *prefix |= (middle << D::kShift1) | digit;
}

// Ordered emission of one chunk: position = #greater before + min(#equal before, need_eq).
__device__ __forceinline__ void emit_chunk(int *wave_tot, const uint32_t (&key)[kItems], int i0, int len,
                                           uint32_t thr, int need_eq, int budget, int &gt_base, int &eq_base,
                                           int32_t *out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool gt[kItems], eq[kItems];
    int packed = 0;                     // low 16 bits: #equal, high 16 bits: #greater (both <= 4096 per chunk)
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
        gt[e] = i0 + e < len && key[e] > thr;
        eq[e] = i0 + e < len && key[e] == thr;
        packed += (gt[e] ? 0x10000 : 0) + (eq[e] ? 1 : 0);
    }
    const int incl = wave_scan<false>(packed, lane);       // inclusive scan inside the wave
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int before = incl - packed, total = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        const int t = wave_tot[w];
        if (w < wave) before += t;
        total += t;
    }
    int gt_before = gt_base + (before >> 16), eq_before = eq_base + (before & 0xffff);
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
        if (gt[e] || (eq[e] && eq_before < need_eq)) {
            const int pos = gt_before + min(eq_before, need_eq);
            if (pos < budget) out[pos] = i0 + e;          // always true; guards the store
        }
        gt_before += gt[e] ? 1 : 0;
        eq_before += eq[e] ? 1 : 0;
    }
    gt_base += total >> 16;
    eq_base += total & 0xffff;
    __syncthreads();
}

// Ordered emission of a head whose keys all sit in registers: the same positions as emit_chunk chunk after
// chunk, with three barriers in all.  Every wave scans its 256 keys of every chunk; the first wave then
// scans the (chunk, wave) totals in emission order; every thread places its keys.
template <int kRegChunks, typename Shared>
__device__ __forceinline__ void emit_resident(Shared &sh, const uint32_t (&keys)[kRegChunks][kItems], int n_chunks,
                                              uint32_t thr, int need_eq, int budget, int32_t *out) {
    static_assert(kRegChunks <= kMaxRegChunks, "cw_tot is sized for kMaxRegChunks chunks");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int before[kRegChunks];                     // packed counts: low 16 bits #equal, high 16 bits #greater (<= 256 per wave)
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        // Counts over the lower lanes and over the wave from the lane masks of the comparisons (no shuffles).
        int gt_lower = 0, eq_lower = 0, gt_wave = 0, eq_wave = 0;
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            // (no range checks: positions past the length and chunks past the head hold key 0 < thr)
            const unsigned long long mg = __ballot(keys[c][e] > thr), me = __ballot(keys[c][e] == thr);
            gt_lower += __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0));
            eq_lower += __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0));
            gt_wave += __popcll(mg);
            eq_wave += __popcll(me);
        }
        if (lane == 0) sh.cw_tot[c * kSelWaves + wave] = (gt_wave << 16) | eq_wave;
        before[c] = (gt_lower << 16) | eq_lower;
    }
    __syncthreads();
    if (wave == 0) {
        // entries in emission order: j = chunk * kSelWaves + wave; lane l owns kPer consecutive ones
        constexpr int kPer = kRegChunks * kSelWaves / 64 > 0 ? kRegChunks * kSelWaves / 64 : 1;
        constexpr int kEntries = kRegChunks * kSelWaves;
        int gt[kPer], eq[kPer], gsum = 0, esum = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int j = lane * kPer + u;
            const int t = j < kEntries ? sh.cw_tot[j] : 0;
            gt[u] = t >> 16; eq[u] = t & 0xffff;
            gsum += gt[u]; esum += eq[u];
        }
        const int ginc = wave_scan<false>(gsum, lane), einc = wave_scan<false>(esum, lane);
        int g = ginc - gsum, q = einc - esum;       // exclusive
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int j = lane * kPer + u;
            if (j < kEntries) { sh.cw_gt[j] = g; sh.cw_eq[j] = q; }
            g += gt[u]; q += eq[u];
        }
    }
    __syncthreads();
    // (the comparisons are taken again rather than kept: 128 lane masks would not fit the scalar registers)
    uint32_t thr_again = thr;
    asm volatile("" : "+v"(thr_again));
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        if (c >= n_chunks) continue;              // uniform
        const int i0 = c * kChunk + tid * kItems;
        int gt_before = sh.cw_gt[c * kSelWaves + wave] + (before[c] >> 16);
        int eq_before = sh.cw_eq[c * kSelWaves + wave] + (before[c] & 0xffff);
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            const bool gt = keys[c][e] > thr_again, eq = keys[c][e] == thr_again;
            if (gt || (eq && eq_before < need_eq)) {
                const int pos = gt_before + min(eq_before, need_eq);
                if (pos < budget) out[pos] = i0 + e;          // always true; guards the store
            }
            gt_before += gt ? 1 : 0;
            eq_before += eq ? 1 : 0;
        }
    }
}

// The same when every key equal to the threshold is kept (no tie is cut: the usual case): a key is kept iff it is
// >= the threshold.  A thread keeps at most 4 keys per chunk and a wave 256, so one wave scan carries three chunks.
template <int kRegChunks, typename Shared>
__device__ __forceinline__ void emit_resident_uncut(Shared &sh, const uint32_t (&keys)[kRegChunks][kItems],
                                                    int n_chunks, uint32_t thr, int budget, int32_t *out) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kPacks = (kRegChunks + 2) / 3;
    int before[kPacks];                         // kept keys of the wave's lower lanes, 10 bits per chunk
#pragma unroll
    for (int g = 0; g < kPacks; ++g) {
        int mine = 0;
#pragma unroll
        for (int c = 3 * g; c < 3 * g + 3 && c < kRegChunks; ++c) {
            int of_chunk = 0;
#pragma unroll
            for (int e = 0; e < kItems; ++e) of_chunk += keys[c][e] >= thr ? 1 : 0;
            mine += of_chunk << (10 * (c - 3 * g));
        }
        const int incl = wave_scan<false>(mine, lane);
        before[g] = incl - mine;
        if (lane == 63) {
#pragma unroll
            for (int c = 3 * g; c < 3 * g + 3 && c < kRegChunks; ++c)
                sh.cw_tot[c * kSelWaves + wave] = (incl >> (10 * (c - 3 * g))) & 1023;
        }
    }
    __syncthreads();
    if (wave == 0) {
        constexpr int kPer = kRegChunks * kSelWaves / 64 > 0 ? kRegChunks * kSelWaves / 64 : 1;
        constexpr int kEntries = kRegChunks * kSelWaves;
        int n[kPer], sum = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int j = lane * kPer + u;
            n[u] = j < kEntries ? sh.cw_tot[j] : 0;
            sum += n[u];
        }
        int g = wave_scan<false>(sum, lane) - sum;  // exclusive
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int j = lane * kPer + u;
            if (j < kEntries) sh.cw_gt[j] = g;
            g += n[u];
        }
    }
    __syncthreads();
    uint32_t thr_again = thr;                       // (compared again rather than kept: the lane masks would not fit)
    asm volatile("" : "+v"(thr_again));
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        if (c >= n_chunks) continue;                // uniform
        const int i0 = c * kChunk + tid * kItems;
        int pos = sh.cw_gt[c * kSelWaves + wave] + ((before[c / 3] >> (10 * (c % 3))) & 1023);
#pragma unroll
        for (int e = 0; e < kItems; ++e) {
            const bool keep = keys[c][e] >= thr_again;
            if (keep && pos < budget) out[pos] = i0 + e;      // (pos < budget always holds; it guards the store)
            pos += keep ? 1 : 0;
        }
    }
}

// Sum over the 2R+1 scores around each of four consecutive positions, in ascending position order, from aligned loads.
template <int R>
__device__ __forceinline__ void pooled_four(const float *__restrict__ s, int i0, uint32_t (&keys)[kItems]) {
    constexpr int kSide = (R + kItems - 1) / kItems;          // groups of four on either side
    float w[(2 * kSide + 1) * kItems];
#pragma unroll
    for (int g = 0; g < 2 * kSide + 1; ++g) {
        const float4 f = *(const float4 *)(s + i0 + (g - kSide) * kItems);
        w[g * kItems] = f.x; w[g * kItems + 1] = f.y; w[g * kItems + 2] = f.z; w[g * kItems + 3] = f.w;
    }
#pragma unroll
    for (int e = 0; e < kItems; ++e) {
        float sum = w[kSide * kItems + e - R];
#pragma unroll
        for (int j = 1; j <= 2 * R; ++j) sum = __fadd_rn(sum, w[kSide * kItems + e - R + j]);
        keys[e] = pooled_key(sum);
    }
}

// Keys of chunks c0 .. c0 + kRegChunks - 1 of one head (128-bit loads where possible).
template <int kRegChunks>
__device__ __forceinline__ void load_batch(uint32_t (&keys)[kRegChunks][kItems], const float *__restrict__ s, int c0,
                                           int n_chunks, int len, bool vec_ok, int first, int cutoff, int radius,
                                           bool keys_in = false) {
    if (radius == 0 && !keys_in && vec_ok) {              // uniform: plain scores of an aligned head, the usual case
        // Every load of the batch goes out before any key is formed: one memory round trip, not one per chunk.
        float4 f[kRegChunks];
#pragma unroll
        for (int c = 0; c < kRegChunks; ++c) {
            const int i0 = (c0 + c) * kChunk + (int)threadIdx.x * kItems;
            f[c] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c0 + c < n_chunks) {                      // uniform
                if (i0 + kItems <= len) {
                    f[c] = *(const float4 *)(s + i0);
                } else {                                  // the head's last, partial group of four
                    if (i0 < len) f[c].x = s[i0];
                    if (i0 + 1 < len) f[c].y = s[i0 + 1];
                    if (i0 + 2 < len) f[c].z = s[i0 + 2];
                }
            }
        }
#pragma unroll
        for (int c = 0; c < kRegChunks; ++c) {
            if (c0 + c < n_chunks) {                      // uniform
                const int i0 = (c0 + c) * kChunk + (int)threadIdx.x * kItems;
                keys[c][0] = order_key(f[c].x); keys[c][1] = order_key(f[c].y);
                keys[c][2] = order_key(f[c].z); keys[c][3] = order_key(f[c].w);
                if (i0 + kItems > len) {                  // positions past the length
#pragma unroll
                    for (int e = 0; e < kItems; ++e)
                        if (i0 + e >= len) keys[c][e] = 0u;
                }
                if (i0 < first || i0 + kItems > cutoff) { // some of these tokens are protected
#pragma unroll
                    for (int e = 0; e < kItems; ++e)
                        if (i0 + e < first || (i0 + e >= cutoff && i0 + e < len)) keys[c][e] = 0xffffffffu;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c) {
        if (c0 + c < n_chunks) {                          // uniform
            const int i0 = (c0 + c) * kChunk + (int)threadIdx.x * kItems;
            if (radius > 0 && vec_ok && i0 - 2 * kItems >= first && i0 + 3 * kItems <= cutoff) {     // pooled, away from every edge
                switch (radius) {                         // uniform
                    case 1: pooled_four<1>(s, i0, keys[c]); break;
                    case 2: pooled_four<2>(s, i0, keys[c]); break;
                    case 3: pooled_four<3>(s, i0, keys[c]); break;
                    case 4: pooled_four<4>(s, i0, keys[c]); break;
                    case 5: pooled_four<5>(s, i0, keys[c]); break;
                    case 6: pooled_four<6>(s, i0, keys[c]); break;
                    default: pooled_four<7>(s, i0, keys[c]); break;
                }
            } else if (radius > 0) {                      // uniform: pooled ranking
                float w[kItems + 2 * kMaxRadius];
#pragma unroll
                for (int j = 0; j < kItems + 2 * kMaxRadius; ++j) {
                    const int idx = i0 - radius + j;
                    const bool ok = j < kItems + 2 * radius && idx >= first && idx < cutoff;
                    w[j] = ok ? s[idx] : 0.f;
                }
#pragma unroll
                for (int e = 0; e < kItems; ++e) {
                    float sum = w[e];
#pragma unroll
                    for (int j = 1; j <= 2 * kMaxRadius; ++j)
                        if (j <= 2 * radius) sum = __fadd_rn(sum, w[e + j]);
                    keys[c][e] = i0 + e < len ? pooled_key(sum) : 0u;
                }
            } else if (keys_in) {                         // uniform: the input already holds order-preserving keys
                const uint32_t *kin = (const uint32_t *)s;
                if (vec_ok && i0 + kItems <= len) {
                    const uint4 u = *(const uint4 *)(kin + i0);
                    keys[c][0] = u.x; keys[c][1] = u.y; keys[c][2] = u.z; keys[c][3] = u.w;
                } else
#pragma unroll
                for (int e = 0; e < kItems; ++e) keys[c][e] = i0 + e < len ? kin[i0 + e] : 0u;
            } else if (vec_ok && i0 + kItems <= len) {
                const float4 f = *(const float4 *)(s + i0);
                keys[c][0] = order_key(f.x); keys[c][1] = order_key(f.y);
                keys[c][2] = order_key(f.z); keys[c][3] = order_key(f.w);
            } else {
#pragma unroll
                for (int e = 0; e < kItems; ++e) keys[c][e] = i0 + e < len ? order_key(s[i0 + e]) : 0u;
            }
            if (!keys_in && (i0 < first || i0 + kItems > cutoff)) {     // some of these tokens are protected
#pragma unroll
                for (int e = 0; e < kItems; ++e)
                    if (i0 + e < first || (i0 + e >= cutoff && i0 + e < len)) keys[c][e] = 0xffffffffu;
            }
        }
    }
}

// kResident: the head has at most kRegChunks * 4096 tokens; its keys are loaded once and
// live in registers.  Otherwise every pass streams the head in batches of kRegChunks
// chunks (all loads of a batch are issued before any is used).
template <int kRegChunks, bool kResident, typename Lens>
__global__ __launch_bounds__(kSelThreads) void select_topk(const float *__restrict__ scores, int N, int budget,
                                                           int Hkv, int ragged, Lens lens, int first, int tail,
                                                           int radius, int32_t *__restrict__ keep_idx) {
    constexpr int kFirstBits = kRegChunks >= 8 ? 13 : 11;
    using D = Digits<kFirstBits>;
    __shared__ __attribute__((aligned(16))) SelectShared<kFirstBits> sh;
    const int bg = blockIdx.x;
    const int len = seq_len_of(lens, ragged, bg / Hkv, N);
    const int cutoff = len - tail;                        // tokens at or beyond it are always kept
    const float *s = scores + (size_t)bg * N;
    int32_t *out = keep_idx + (size_t)bg * budget;
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_chunks = (len + kChunk - 1) / kChunk;
    const bool vec_ok = ((size_t)s & 15) == 0;            // the head starts on a 16-byte boundary

    clear_counters<D::kBins0>(sh.hist0);
    clear_counters<D::kBins1>(sh.hist1);
    clear_counters<D::kBins2>(sh.hist2);
    if (tid == 0) sh.n_list = 0;
    uint32_t keys[kRegChunks][kItems];
#pragma unroll
    for (int c = 0; c < kRegChunks; ++c)
#pragma unroll
        for (int e = 0; e < kItems; ++e) keys[c][e] = 0u;
    if (kResident) load_batch<kRegChunks>(keys, s, 0, n_chunks, len, vec_ok, first, cutoff, radius);
    __syncthreads();

    // f(key) for this thread's keys; positions past the length hold key 0: they land in the lowest class and never
    // reach the threshold.
    auto visit_all = [&](auto &&f) {
        for (int c0 = 0; c0 < (kResident ? 1 : n_chunks); c0 += kRegChunks) {
            if (!kResident) load_batch<kRegChunks>(keys, s, c0, n_chunks, len, vec_ok, first, cutoff, radius);
#pragma unroll
            for (int c = 0; c < kRegChunks; ++c) {
                if (c0 + c < n_chunks) {                  // uniform
#pragma unroll
                    for (int e = 0; e < kItems; ++e) f(keys[c][e]);
                }
            }
        }
    };
    visit_all([&](uint32_t key) { atomicAdd(&sh.hist0[key >> D::kShift0], 1); });
    uint32_t digit;
    int remaining = budget, n_equal;    // rank (1-based, from the top) still to resolve inside the class
    pick_digit<D::kBins0>(sh.hist0, sh.pick, &digit, &remaining, &n_equal);
    uint32_t thr = digit << D::kShift0;
    const uint32_t first_digit = digit;
    if (n_equal <= kList) {
        // The class's keys into the list, in any order: one place per wave and its lanes' counts before it.
        int mine = 0;
        visit_all([&](uint32_t key) { mine += (key >> D::kShift0) == first_digit ? 1 : 0; });
        const int incl = wave_scan<false>(mine, lane);
        int base = 0;
        if (lane == 63 && incl > 0) base = atomicAdd(&sh.n_list, incl);
        int at = __builtin_amdgcn_readlane(base, 63) + incl - mine;
        visit_all([&](uint32_t key) {
            if ((key >> D::kShift0) == first_digit) sh.list[at++] = key;
        });
        __syncthreads();
        const int n_list = n_equal;
        finish_class<D>(sh.hist1, sh.hist2, sh.pick, [&](auto &&f) {
            for (int j = tid; j < n_list; j += kSelThreads) f(sh.list[j]);
        }, &thr, &remaining, &n_equal);
    } else {
        finish_class<D>(sh.hist1, sh.hist2, sh.pick, [&](auto &&f) {
            visit_all([&](uint32_t key) { if ((key >> D::kShift0) == first_digit) f(key); });
        }, &thr, &remaining, &n_equal);
    }
    const int need_eq = remaining;      // how many tokens equal to the threshold are kept (lowest indices first)

    // ---- ordered sweep ----
    if constexpr (kResident) {
        if (need_eq == n_equal) emit_resident_uncut<kRegChunks>(sh, keys, n_chunks, thr, budget, out);
        else emit_resident<kRegChunks>(sh, keys, n_chunks, thr, need_eq, budget, out);
    } else {
        int gt_base = 0, eq_base = 0;
        for (int c0 = 0; c0 < n_chunks; c0 += kRegChunks) {
            load_batch<kRegChunks>(keys, s, c0, n_chunks, len, vec_ok, first, cutoff, radius);
#pragma unroll
            for (int c = 0; c < kRegChunks; ++c)
                if (c0 + c < n_chunks)
                    emit_chunk(sh.pick.wave_tot, keys[c], (c0 + c) * kChunk + tid * kItems, len, thr, need_eq, budget, gt_base, eq_base, out);
        }
    }
}

// ------------------------------------------------------------------------------------
// Slices of long heads on separate workgroups: a group (one head, or all heads of a sequence when they are ranked
// together) is cut into slices of whole chunks, a slice never spans two heads, and three kernels do the select:
//   slices_count    histogram of the first digit per slice
//   slices_collect  sum of the group's histograms -> the threshold's class; the slice's keys in it -> its list; how many
//                   of the slice's keys lie above the class
//   slices_emit     the class's keys from all lists -> threshold; ordered emission of the slice, starting at what the
//                   slices before it keep
// No global atomics and nothing to clear; every workgroup of a group repeats the integer sums.  Bound by the launches
// and their memory round trips (a 4 x 128K selection reads 2 MB): five kernels with a histogram of the whole slice per
// digit took 52 us there, these three take 21, of which 6.6 to collect (7.3 with counters of 32 bits).
// ------------------------------------------------------------------------------------
struct SliceState {      // of a group, written by slices_collect
    uint32_t digit;      // first digit of the threshold
    int remaining;       // its rank inside that class
};

// Shape of a sliced selection and its buffers in the workspace.
struct Slices {
    int groups, group0, heads;       // in all, first of the launch; heads per group
    int per_head, chunks;            // slices per head, chunks of 4096 scores per slice
    int key_stride;                  // keys between the heads of `keys`: N rounded up to 4
    int list_stride;                 // keys between the slices of `list`: the most a slice has
    int *hist;                       // [groups][slices][kSliceBins]
    uint32_t *list;                  // [groups][slices][list_stride]
    int *above, *count;              // [groups][slices] keys above the class, keys in the list
    SliceState *state;               // [groups]
    uint32_t *keys;                  // [heads of all groups][key_stride]; NULL: the keys are formed from the scores each time
};

constexpr int kPackedChunks = 8;         // chunks of a slice whose counters stay below 2^16
constexpr int kMaxGroupSlices = 1024;    // of a group whose bookkeeping fits LDS; larger ones (that many heads) read it where it lies

// Where a workgroup of the sliced kernels works: blockIdx.x = slice of the group, blockIdx.y = group of the launch's.
struct SlicePlace {
    int slice, group, head, in_head;         // head: of all groups
    int c0, c1, len;                         // chunks of the head, its true length
    template <typename Lens>
    __device__ __forceinline__ SlicePlace(const Slices &S, int N, int Hkv, int ragged, const Lens &lens) {
        slice = blockIdx.x;
        group = S.group0 + blockIdx.y;
        head = group * S.heads + slice / S.per_head;
        in_head = slice % S.per_head;
        len = seq_len_of(lens, ragged, head / Hkv, N);
        c0 = in_head * S.chunks;
        c1 = min(c0 + S.chunks, (len + kChunk - 1) / kChunk);
    }
    __device__ __forceinline__ size_t flat() const { return (size_t)group * gridDim.x + slice; }
};

// The slice's keys, kBatch chunks at a time: f(keys, first chunk).  From the scores, or from S.keys once those hold them.
// `prepare` runs once, after the first batch has been loaded: what it needs from memory was asked for before the call, so
// both are one round trip.
template <int kBatch, typename P, typename F>
__device__ __forceinline__ void for_batches(const Slices &S, const SlicePlace &at, const float *__restrict__ scores, int N, int first,
                                            int tail, int radius, bool from_keys, P &&prepare, F &&f) {
    const float *s = from_keys ? (const float *)(S.keys + (size_t)at.head * S.key_stride) : scores + (size_t)at.head * N;
    const bool vec_ok = ((size_t)s & 15) == 0;
    uint32_t keys[kBatch][kItems];
    auto load = [&](int c) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int e = 0; e < kItems; ++e) keys[i][e] = 0u;
        load_batch<kBatch>(keys, s, c, at.c1, at.len, vec_ok, first, at.len - tail, from_keys ? 0 : radius, from_keys);
    };
    load(at.c0);                             // (a slice past the length loads nothing)
    prepare();
    for (int c = at.c0; c < at.c1; c += kBatch) {
        if (c != at.c0) load(c);
        f(keys, c);
    }
}

__device__ __forceinline__ void store_keys(const Slices &S, const SlicePlace &at, int i0, const uint32_t (&key)[kItems]) {
    if (i0 < at.len)       // (rows are padded to whole groups of four)
        *(uint4 *)(S.keys + (size_t)at.head * S.key_stride + i0) = make_uint4(key[0], key[1], key[2], key[3]);
}

// kPacked: counters of 16 bits, two neighbours to a word (slices of at most kPackedChunks chunks).
template <int kBatch, bool kPacked, typename Lens>
__global__ __launch_bounds__(kSelThreads) void slices_count(const float *__restrict__ scores, int N, int Hkv, int ragged, Lens lens,
                                                            int first, int tail, int radius, Slices S) {
    __shared__ __attribute__((aligned(16))) int hist[kSliceBins];
    const SlicePlace at(S, N, Hkv, ragged, lens);
    clear_counters<kSliceBins>(hist);
    for_batches<kBatch>(S, at, scores, N, first, tail, radius, false, [&]() { __syncthreads(); }, [&](uint32_t (&keys)[kBatch][kItems], int c) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (c + i >= at.c1) continue;                    // uniform
            const int i0 = (c + i) * kChunk + (int)threadIdx.x * kItems;
#pragma unroll
            for (int e = 0; e < kItems; ++e)
                if (i0 + e < at.len) atomicAdd(&hist[keys[i][e] >> (32 - kSliceBits)], 1);
            if (S.keys) store_keys(S, at, i0, keys[i]);
        }
    });
    __syncthreads();
    const int2 two = *(const int2 *)(hist + 2 * threadIdx.x);
    if constexpr (kPacked) ((uint32_t *)S.hist)[at.flat() * (kSliceBins / 2) + threadIdx.x] = (uint32_t)two.x | (uint32_t)two.y << 16;
    else *(int2 *)(S.hist + at.flat() * kSliceBins + 2 * threadIdx.x) = two;
}

// Sum of a group's `n` histograms in LDS, fetched ahead of what follows and added up later; the whole workgroup.
template <bool kPacked>
struct HistogramSum {
    // A thread has 16 bytes of a histogram, so kParts slices are read side by side.
    static constexpr int kOwn = kPacked ? 8 : 4, kParts = kSelThreads * kOwn / kSliceBins;
    static constexpr int kAhead = 32 / kParts;               // slices of a part in flight at once
    uint4 h[kAhead];
    __device__ __forceinline__ void fetch(const int *__restrict__ hist, int n, int s0) {      // hist: of the group
        const int part = threadIdx.x / (kSliceBins / kOwn), piece = threadIdx.x % (kSliceBins / kOwn);
        const uint4 *src = (const uint4 *)hist + piece;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const int sl = s0 + kParts * i + part;
            h[i] = make_uint4(0u, 0u, 0u, 0u);
            if (sl < n) h[i] = src[(size_t)sl * (kSliceBins / kOwn)];
        }
    }
    // The first slices have been fetched.  Leaves the sums in parts[0]; a barrier has to follow.
    __device__ __forceinline__ void sum(const int *__restrict__ hist, int n, int (&parts)[kParts][kSliceBins]) {
        const int part = threadIdx.x / (kSliceBins / kOwn), piece = threadIdx.x % (kSliceBins / kOwn);
        int c[kOwn] = {};
        for (int s0 = 0; s0 < n; s0 += kParts * kAhead) {
            if (s0 > 0) fetch(hist, n, s0);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                const uint32_t w[4] = {h[i].x, h[i].y, h[i].z, h[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (kPacked) { c[2 * j] += w[j] & 0xffff; c[2 * j + 1] += w[j] >> 16; }
                    else c[j] += w[j];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kOwn; j += 4) *(int4 *)(&parts[part][piece * kOwn + j]) = make_int4(c[j], c[j + 1], c[j + 2], c[j + 3]);
        __syncthreads();
        int2 t = make_int2(0, 0);
#pragma unroll
        for (int i = 0; i < kParts; ++i) {
            const int2 x = *(const int2 *)(&parts[i][2 * threadIdx.x]);
            t.x += x.x;
            t.y += x.y;
        }
        *(int2 *)(&parts[0][2 * threadIdx.x]) = t;           // (read by this thread alone so far)
    }
};

template <int kBatch, bool kPacked, typename Lens>
__global__ __launch_bounds__(kSelThreads) void slices_collect(const float *__restrict__ scores, int N, int budget, int Hkv, int ragged,
                                                              Lens lens, int first, int tail, int radius, Slices S) {
    using Sum = HistogramSum<kPacked>;
    __shared__ __attribute__((aligned(16))) int hist[Sum::kParts][kSliceBins];
    __shared__ PickShared pick;
    __shared__ int n_list, n_above;
    const SlicePlace at(S, N, Hkv, ragged, lens);
    const int tid = threadIdx.x, lane = tid & 63, n = gridDim.x;
    if (tid == 0) { n_list = 0; n_above = 0; }
    const int *src = S.hist + (size_t)at.group * n * (kPacked ? kSliceBins / 2 : kSliceBins);
    Sum histograms;
    uint32_t digit;
    auto pick_class = [&]() {
        histograms.sum(src, n, hist);
        int remaining = budget, in_digit;
        pick_digit<kSliceBins>(hist[0], pick, &digit, &remaining, &in_digit);
        if (at.slice == 0 && tid == 0) S.state[at.group] = SliceState{digit, remaining};
    };
    histograms.fetch(src, n, 0);
    uint32_t *list = S.list + at.flat() * S.list_stride;
    for_batches<kBatch>(S, at, scores, N, first, tail, radius, S.keys != nullptr, pick_class, [&](uint32_t (&keys)[kBatch][kItems], int c) {
        int mine = 0;                                        // low 16 bits: in the class, high 16 bits: above it
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const bool in = c + i < at.c1 && (c + i) * kChunk + tid * kItems + e < at.len;
                const uint32_t d = keys[i][e] >> (32 - kSliceBits);
                mine += in && d == digit ? 1 : in && d > digit ? 0x10000 : 0;
            }
        const int incl = wave_scan<false>(mine, lane);
        int base = 0;
        if (lane == 63 && incl != 0) {
            base = atomicAdd(&n_list, incl & 0xffff);
            atomicAdd(&n_above, incl >> 16);
        }
        int pos = __builtin_amdgcn_readlane(base, 63) + ((incl - mine) & 0xffff);
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const bool in = c + i < at.c1 && (c + i) * kChunk + tid * kItems + e < at.len;
                if (in && (keys[i][e] >> (32 - kSliceBits)) == digit) list[pos++] = keys[i][e];
            }
    });
    __syncthreads();
    if (tid == 0) { S.count[at.flat()] = n_list; S.above[at.flat()] = n_above; }
}

// The threshold of a group, and what of it lies where relative to a slice.
struct SliceShared {
    using D = Digits<kSliceBits>;
    int hist1[D::kBins1], hist2[D::kBins2];
    uint32_t list[kList];
    int count[kMaxGroupSlices], offset[kMaxGroupSlices + 1];
    PickShared pick;
    int head_gt_before, head_gt, eq_before_head, eq_before, eq_head;
};

struct SliceThreshold {
    uint32_t thr;
    int need_eq, n_equal;    // keys equal to it: kept (the first ones of the group), all
    int gt_before, gt_head;  // keys above it: in the head's earlier slices, in the head
    int eq_before_head, eq_before, eq_head;    // keys equal to it: in earlier heads of the group, in earlier slices of the group, in the head
};

// What slice_threshold needs first, asked for ahead of it.
struct SliceAhead {
    SliceState state;
    int count;               // of the slice with this thread's index
    __device__ __forceinline__ SliceAhead(const Slices &S, const SlicePlace &at) {
        state = S.state[at.group];
        count = (int)gridDim.x <= kMaxGroupSlices && threadIdx.x < gridDim.x ? S.count[(size_t)at.group * gridDim.x + threadIdx.x] : 0;
    }
};

__device__ __forceinline__ SliceThreshold slice_threshold(SliceShared &sh, const Slices &S, const SlicePlace &at, const SliceAhead &ahead) {
    using D = Digits<kSliceBits>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = gridDim.x;
    const int head0 = at.slice - at.in_head, head1 = head0 + S.per_head;       // the head's slices
    const SliceState st = ahead.state;
    clear_counters<D::kBins1>(sh.hist1);
    clear_counters<D::kBins2>(sh.hist2);
    if (tid == 0) sh.head_gt_before = sh.head_gt = sh.eq_before_head = sh.eq_before = sh.eq_head = 0;
    const int *counts = S.count + (size_t)at.group * n, *aboves = S.above + (size_t)at.group * n;
    const bool few = n <= kMaxGroupSlices;                   // uniform
    if (few && tid < n) sh.count[tid] = ahead.count;
    __syncthreads();
    if (few && wave == 0) {                                  // offsets of the slices' lists laid end to end
        int base = 0;
        for (int s0 = 0; s0 < n; s0 += 64) {
            const int c = s0 + lane < n ? sh.count[s0 + lane] : 0;
            const int incl = wave_scan<false>(c, lane);
            if (s0 + lane < n) sh.offset[s0 + lane] = base + incl - c;
            base += __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) sh.offset[n] = base;
    } else if (wave == 1) {                                  // keys above the class in the head
        int before = 0, all = 0;
        for (int sl = head0 + lane; sl < head1; sl += 64) {
            const int a = aboves[sl];
            all += a;
            before += sl < at.slice ? a : 0;
        }
        before = (int)wave_reduce<SumOp>((uint32_t)before);
        all = (int)wave_reduce<SumOp>((uint32_t)all);
        if (lane == 0) { atomicAdd(&sh.head_gt_before, before); atomicAdd(&sh.head_gt, all); }
    }
    __syncthreads();
    const int n_list = few ? sh.offset[n] : 0;
    const bool in_lds = few && n_list <= kList;              // uniform
    const uint32_t *lists = S.list + (size_t)at.group * n * S.list_stride;
    // f(key, slice) over the lists where they lie: a wave per slice
    auto visit_global = [&](auto &&f) {
        for (int sl = wave; sl < n; sl += kSelWaves) {
            const uint32_t *src = lists + (size_t)sl * S.list_stride;
            const int c = few ? sh.count[sl] : counts[sl];
            for (int i = lane; i < c; i += 64) f(src[i], sl, i);
        }
    };
    if (in_lds) {
        visit_global([&](uint32_t key, int sl, int i) { sh.list[sh.offset[sl] + i] = key; });
        __syncthreads();
    }
    SliceThreshold t;
    t.thr = st.digit << (32 - kSliceBits);
    t.need_eq = st.remaining;
    finish_class<D>(sh.hist1, sh.hist2, sh.pick, [&](auto &&f) {
        if (in_lds) for (int j = tid; j < n_list; j += kSelThreads) f(sh.list[j]);
        else visit_global([&](uint32_t key, int, int) { f(key); });
    }, &t.thr, &t.need_eq, &t.n_equal);
    // class keys above and at the threshold, by where they lie
    int gt_before = 0, gt_head = 0, eq_first = 0, eq_before = 0, eq_head = 0;
    const int p_head0 = few ? sh.offset[head0] : 0, p_slice = few ? sh.offset[at.slice] : 0, p_head1 = few ? sh.offset[head1] : 0;
    auto tally = [&](uint32_t key, bool before_head, bool before_slice, bool in_head) {
        // (branches here became sums through selected addresses, in scratch memory)
        const int gt = key > t.thr ? 1 : 0, eq = key == t.thr ? 1 : 0;
        gt_head += in_head ? gt : 0;
        gt_before += in_head & before_slice ? gt : 0;
        eq_first += before_head ? eq : 0;
        eq_before += before_slice ? eq : 0;
        eq_head += in_head ? eq : 0;
    };
    if (in_lds) for (int j = tid; j < n_list; j += kSelThreads) tally(sh.list[j], j < p_head0, j < p_slice, j >= p_head0 && j < p_head1);
    else visit_global([&](uint32_t key, int sl, int) { tally(key, sl < head0, sl < at.slice, sl >= head0 && sl < head1); });
    auto add = [&](int *to, int x) {
        if (__ballot(x != 0) == 0ull) return;                // uniform
        x = (int)wave_reduce<SumOp>((uint32_t)x);
        if (lane == 0) atomicAdd(to, x);
    };
    add(&sh.head_gt_before, gt_before);
    add(&sh.head_gt, gt_head);
    add(&sh.eq_before_head, eq_first);
    add(&sh.eq_before, eq_before);
    add(&sh.eq_head, eq_head);
    __syncthreads();
    t.gt_before = sh.head_gt_before;
    t.gt_head = sh.head_gt;
    t.eq_before_head = sh.eq_before_head;
    t.eq_before = sh.eq_before;
    t.eq_head = sh.eq_head;
    return t;
}

// `counts` == NULL: keep_idx [heads][room], every list full.  Otherwise the heads of a group share the budget: counts
// [heads] receives how many each one keeps, and its list of `room` is filled up with -1.
template <int kBatch, typename Lens>
__global__ __launch_bounds__(kSelThreads) void slices_emit(const float *__restrict__ scores, int N, int room, int Hkv, int ragged,
                                                           Lens lens, int first, int tail, int radius, Slices S,
                                                           int32_t *__restrict__ keep_idx, int32_t *__restrict__ counts) {
    __shared__ __attribute__((aligned(16))) SliceShared sh;
    const SlicePlace at(S, N, Hkv, ragged, lens);
    const SliceAhead ahead(S, at);
    SliceThreshold t;
    int32_t *out = keep_idx + (size_t)at.head * room;
    int eq_skip, gt_base, eq_base;
    for_batches<kBatch>(S, at, scores, N, first, tail, radius, S.keys != nullptr, [&]() {
        t = slice_threshold(sh, S, at, ahead);
        // kept keys equal to the threshold are the first need_eq of the group; positions count inside the head
        eq_skip = min(t.eq_before_head, t.need_eq);
        gt_base = t.gt_before - eq_skip;
        eq_base = t.eq_before;
    }, [&](uint32_t (&keys)[kBatch][kItems], int c) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (c + i < at.c1)
                emit_chunk(sh.pick.wave_tot, keys[i], (c + i) * kChunk + (int)threadIdx.x * kItems, at.len, t.thr, t.need_eq, room, gt_base,
                           eq_base, out);
    });
    if (!counts) return;
    const int kept = min(t.gt_head + min(t.eq_before_head + t.eq_head, t.need_eq) - eq_skip, room);
    if (at.in_head == 0 && threadIdx.x == 0) counts[at.head] = kept;
    for (int j = kept + at.in_head * kSelThreads + threadIdx.x; j < room; j += S.per_head * kSelThreads) out[j] = -1;
}

// ------------------------------------------------------------------------------------
// Head-adaptive budgets (Appendix C, AdaKV paragraph): the layer's budget is spread over the
// KV heads by ranking all (head, token) scores of a sequence together, after each head's own
// top n_safe tokens (the safeguard) have been put beyond competition.  slices_count and
// slices_collect find every head's class for n_safe; the kernel below finishes that selection and
// turns the slice's scores into the keys of the second one (live tokens >= 1, 0 for positions
// beyond the true length, 0xffffffff for the safeguard), with their histogram; then
// slices_collect and slices_emit run over all heads of a sequence as one group.  For many heads or long ones, and where the
// safeguard is the whole budget; the others take the three kernels after these.
// ------------------------------------------------------------------------------------
template <int kBatch, typename Lens>
__global__ __launch_bounds__(kSelThreads) void slices_safeguard(const float *__restrict__ scores, int N, int n_safe, int Hkv, int ragged,
                                                                Lens lens, Slices S, uint32_t *__restrict__ keys_out,
                                                                int *__restrict__ hist_out) {
    __shared__ __attribute__((aligned(16))) SliceShared sh;
    __shared__ __attribute__((aligned(16))) int hist[kSliceBins];
    const SlicePlace at(S, N, Hkv, ragged, lens);            // (a group is one head here)
    clear_counters<kSliceBins>(hist);
    const SliceAhead ahead(S, at);           // (not used without a safeguard: nothing has written it then)
    SliceThreshold t = {};
    int eq_base = 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for_batches<kBatch>(S, at, scores, N, 0, 0, 0, false, [&]() {
        if (n_safe > 0) t = slice_threshold(sh, S, at, ahead);
        else __syncthreads();
        eq_base = t.eq_before;
    }, [&](uint32_t (&keys)[kBatch][kItems], int c) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (c + i >= at.c1) continue;                    // uniform
            const int i0 = (c + i) * kChunk + (int)threadIdx.x * kItems;
            int eq_before = 0;
            if (n_safe > 0 && t.need_eq < t.n_equal) {       // uniform: the first need_eq of the equal keys are safe
                int mine = 0;
#pragma unroll
                for (int e = 0; e < kItems; ++e) mine += i0 + e < at.len && keys[i][e] == t.thr ? 1 : 0;
                const int incl = wave_scan<false>(mine, lane);
                __syncthreads();
                if (lane == 63) sh.pick.wave_tot[wave] = incl;
                __syncthreads();
                eq_before = eq_base + incl - mine;
#pragma unroll
                for (int w = 0; w < kSelWaves; ++w) {
                    if (w < wave) eq_before += sh.pick.wave_tot[w];
                    eq_base += sh.pick.wave_tot[w];
                }
            } else {
                eq_before = -0x40000000;                     // all of them
            }
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const bool live = i0 + e < at.len, eq = keys[i][e] == t.thr;
                const bool safe = n_safe > 0 && live && (keys[i][e] > t.thr || (eq && eq_before < t.need_eq));
                eq_before += eq ? 1 : 0;
                keys[i][e] = !live ? 0u : safe ? 0xffffffffu : keys[i][e];
                if (live) atomicAdd(&hist[keys[i][e] >> (32 - kSliceBits)], 1);
            }
            if (i0 < at.len)
                *(uint4 *)(keys_out + (size_t)at.head * S.key_stride + i0) = make_uint4(keys[i][0], keys[i][1], keys[i][2], keys[i][3]);
        }
    });
    __syncthreads();
    int *dst = hist_out + at.flat() * kSliceBins;
    *(int2 *)(dst + 2 * threadIdx.x) = *(const int2 *)(hist + 2 * threadIdx.x);
}

// ------------------------------------------------------------------------------------
// The same for few heads, without a first selection.  A head keeps max(n_safe, its keys above the common threshold T), so T
// is the largest value at which the sum of those maxima over the heads reaches the budget, and the histograms of
// slices_count give T's class.  By the class, a head
//   has its safeguard above it: it keeps its keys above T;
//   falls short of its safeguard even with the whole class: it keeps its own top n_safe and stands apart;
//   holds the end of its safeguard in the class: the safeguard's keys there are kept in any case and do not compete.
// adaptive_collect leaves one class of every head, the common one or, apart, the one its own n_safe-th key is in;
// adaptive_emit finishes both kinds from the lists.  Three kernels where the selection of the safeguard first takes five;
// bound, as they are, by launches and round trips: 2 x 8 heads of up to 24001 scores, budget 1024, 38.4 -> 24.3 us on the device
// (count 4.7, collect 10.1, emit 9.5), and with the copying of the rows 48.6 -> 33.8; 8 heads of 90K, budget 4096, 77.8 ->
// 51.7; 4 x 32 heads of 4000, budget 400, 103 -> 101.
// ------------------------------------------------------------------------------------
// Most heads (a workgroup finishes a safeguard per wave, the bookkeeping is a lane per head); the gain has shrunk to a
// few percent there, as every workgroup goes through all heads' histograms one by one.
constexpr int kFewHeads = 32;

struct HeadState {       // written by adaptive_collect
    uint32_t digit;      // class of the head's list
    int above;           // keys of the head above it
    int safe_rank;       // rank of the safeguard's last key inside it (0: the safeguard lies above)
    int apart;
};

// Sums of the heads' histograms, two counters per thread, and how many of their keys lie in the counters of higher threads,
// for kHeads heads at a time.
template <int kHeads>
struct HeadSuffix {
    // Slices of each head in flight at once: as many loads of eight heads are, and a head of fewer slices repeats its last one.
    // Selections with 2 / 6 / 12, us: 4 x 32 heads of one slice 28.4 / 31.5 / (uniform scores) 58.6 / 62.0 / 97.0; 8 heads of two
    // 18.2 / 19.1; of six 22.1 / 22.1; of twenty-two, in slices of four chunks, 30.2 / 29.8.
    static constexpr int kAhead = 2;
    int2 c[kHeads];
    int above[kHeads];
    uint32_t x[kAhead][kHeads];
    // hist: of the first head.  (A head too many reads the last one's: no branch between the loads.)
    __device__ __forceinline__ void fetch(const uint32_t *__restrict__ hist, int heads, int per_head, int s0) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
#pragma unroll
            for (int h = 0; h < kHeads; ++h) {
                const int sl = min(h, heads - 1) * per_head + min(s0 + i, per_head - 1);
                x[i][h] = hist[(size_t)sl * (kSliceBins / 2) + threadIdx.x];
            }
    }
    // The first slices have been fetched.
    __device__ __forceinline__ void sum(const uint32_t *__restrict__ hist, int heads, int per_head) {
#pragma unroll
        for (int h = 0; h < kHeads; ++h) c[h] = make_int2(0, 0);
        for (int s0 = 0; s0 < per_head; s0 += kAhead) {
            if (s0 > 0) fetch(hist, heads, per_head, s0);
#pragma unroll
            for (int i = 0; i < kAhead; ++i) {
                if (s0 + i >= per_head) continue;            // uniform
#pragma unroll
                for (int h = 0; h < kHeads; ++h) { c[h].x += x[i][h] & 0xffff; c[h].y += x[i][h] >> 16; }
            }
        }
    }
    __device__ __forceinline__ void scan(int (&tot)[kHeads][kSelWaves]) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        __syncthreads();                                     // (the totals of the heads before these have been read)
#pragma unroll
        for (int h = 0; h < kHeads; ++h) {
            const int mine = c[h].x + c[h].y, incl = wave_scan<true>(mine, lane);
            above[h] = incl - mine;
            if (lane == 0) tot[h][wave] = incl;
        }
        __syncthreads();
        static_assert(kHeads <= kSelWaves && kSelWaves == 16, "a wave per head, its totals in one row of lanes");
        if (wave < kHeads) {                                 // totals -> totals of the higher waves
            const int x = lane < kSelWaves ? tot[wave][lane] : 0, incl = wave_scan<true>(x, lane);
            if (lane < kSelWaves) tot[wave][lane] = incl - x;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < kHeads; ++h) above[h] += tot[h][wave];
    }
};

// Grid: x = slice of the sequence's heads, y = sequence.
template <int kBatch, typename Lens>
__global__ __launch_bounds__(kSelThreads) void adaptive_collect(const float *__restrict__ scores, int N, int budget, int n_safe,
                                                                int Hkv, int ragged, Lens lens, Slices S,
                                                                HeadState *__restrict__ states) {
    constexpr int kHeads = 8;
    __shared__ int tot[kHeads][kSelWaves];
    __shared__ uint32_t common, own_class;
    __shared__ int safe_rank_s;
    __shared__ HeadState own;
    __shared__ int n_list, n_above;
    const SlicePlace at(S, N, Hkv, ragged, lens);
    const int tid = threadIdx.x, lane = tid & 63, own_head = at.slice / S.per_head;
    if (tid == 0) { n_list = 0; n_above = 0; }
    const uint32_t *hist = (const uint32_t *)S.hist + (size_t)at.group * gridDim.x * (kSliceBins / 2);
    HeadSuffix<kHeads> hs;
    hs.fetch(hist, S.heads, S.per_head, 0);
    auto classes = [&]() {
        // F(d) = sum over the heads of max(n_safe, keys with a first digit >= d), at the thread's two digits and past them
        long long f0 = 0, f1 = 0, f2 = 0;
        int own_above = 0;
        int2 own_c = make_int2(0, 0);
        for (int h0 = 0; h0 < S.heads; h0 += kHeads) {
            const uint32_t *first = hist + (size_t)h0 * S.per_head * (kSliceBins / 2);
            if (h0 > 0) hs.fetch(first, S.heads - h0, S.per_head, 0);
            hs.sum(first, S.heads - h0, S.per_head);
            hs.scan(tot);
#pragma unroll
            for (int h = 0; h < kHeads; ++h) {
                if (h0 + h >= S.heads) continue;             // uniform
                const int a2 = hs.above[h], a1 = a2 + hs.c[h].y, a0 = a1 + hs.c[h].x;
                f2 += max(n_safe, a2);
                f1 += max(n_safe, a1);
                f0 += max(n_safe, a0);
                if (h0 + h == own_head) { own_above = a2; own_c = hs.c[h]; }
            }
        }
        const long long total = (long long)S.heads * budget;
        if (f2 < total && f0 >= total) common = 2 * tid + (f1 >= total ? 1 : 0);         // exactly one thread
        if (own_above < n_safe && n_safe <= own_above + own_c.y + own_c.x) {              // likewise, with a safeguard
            const bool upper = n_safe <= own_above + own_c.y;
            own_class = 2 * tid + (upper ? 1 : 0);
            safe_rank_s = n_safe - own_above - (upper ? 0 : own_c.y);
        }
        __syncthreads();
        const uint32_t cls = common;
        if ((int)(cls >> 1) == tid) {
            const int above = own_above + ((cls & 1) ? 0 : own_c.y), in_class = (cls & 1) ? own_c.y : own_c.x;
            if (above + in_class < n_safe) own = HeadState{own_class, n_safe - safe_rank_s, safe_rank_s, 1};
            else own = HeadState{cls, above, max(n_safe - above, 0), 0};
            if (at.in_head == 0) states[at.head] = own;
        }
        __syncthreads();
    };
    uint32_t *list = S.list + at.flat() * S.list_stride;
    for_batches<kBatch>(S, at, scores, N, 0, 0, 0, false, classes, [&](uint32_t (&keys)[kBatch][kItems], int c) {
        const uint32_t digit = own.digit;
        int mine = 0;                                        // low 16 bits: in the class, high 16 bits: above it
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const bool in = c + i < at.c1 && (c + i) * kChunk + tid * kItems + e < at.len;
                const uint32_t d = keys[i][e] >> (32 - kSliceBits);
                mine += in && d == digit ? 1 : in && d > digit ? 0x10000 : 0;
            }
        const int incl = wave_scan<false>(mine, lane);
        int base = 0;
        if (lane == 63 && incl != 0) {
            base = atomicAdd(&n_list, incl & 0xffff);
            atomicAdd(&n_above, incl >> 16);
        }
        int pos = __builtin_amdgcn_readlane(base, 63) + ((incl - mine) & 0xffff);
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
            for (int e = 0; e < kItems; ++e) {
                const bool in = c + i < at.c1 && (c + i) * kChunk + tid * kItems + e < at.len;
                if (in && (keys[i][e] >> (32 - kSliceBits)) == digit) list[pos++] = keys[i][e];
            }
    });
    __syncthreads();
    if (tid == 0) { S.count[at.flat()] = n_list; S.above[at.flat()] = n_above; }
}

constexpr int kAdaptiveList = 14336;     // keys of all heads' lists that fit LDS beside the counters, two workgroups to a compute unit

struct AdaptiveShared {
    using D = Digits<kSliceBits>;
    int hist1[D::kBins1], hist2[D::kBins2];
    uint32_t list[kAdaptiveList];
    int count[kMaxGroupSlices], offset[kMaxGroupSlices + 1];
    HeadState head[kFewHeads];
    uint32_t safe_thr[kFewHeads];        // of the heads whose safeguard ends inside the common class: its last key
    int safe_eq[kFewHeads];              // and how many keys equal to that belong to it
    PickShared pick;
    int above_before, gt_before, gt_head, eq_before_heads, eq_before, eq_head;
};

// The key of rank *rank among the keys of a class: three digits of 7 bits over what is left of a key below its first digit.
constexpr int kRankBits = 7;
static_assert(3 * kRankBits == 32 - kSliceBits, "three digits below the first one");

// One digit, by one wave, from its 128 counters: into *key, and into *rank what is left of it among the keys with that digit.
__device__ __forceinline__ void wave_digit(const int *hist, int shift, uint32_t *key, int *rank) {
    const int lane = threadIdx.x & 63;
    const int2 c = *(const int2 *)(hist + 2 * lane);
    const int incl = wave_scan<true>(c.x + c.y, lane), above = incl - c.x - c.y;
    const unsigned long long at = __ballot(above < *rank && *rank <= incl);      // one lane
    const bool upper = *rank <= above + c.y;
    const int from = at ? __ffsll(at) - 1 : 0;
    const int digit = __shfl(2 * lane + (upper ? 1 : 0), from), less = __shfl(above + (upper ? 0 : c.y), from);
    *key |= (uint32_t)digit << shift;
    *rank -= less;
}

// All three by one wave.  visit(f) calls f(key) for the lane's share.  hist: 128 counters of the wave's own.  Leaves in *rank
// how many keys equal to it there are down to that rank.
template <typename Visit>
__device__ __forceinline__ uint32_t wave_select(int *hist, uint32_t key, int *rank, Visit &&visit) {
    const int lane = threadIdx.x & 63;
    auto ordered = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
#pragma unroll
    for (int shift = 2 * kRankBits; shift >= 0; shift -= kRankBits) {
        *(int2 *)(hist + 2 * lane) = make_int2(0, 0);
        ordered();
        visit([&](uint32_t k) { if ((k ^ key) >> (shift + kRankBits) == 0) atomicAdd(&hist[(k >> shift) & 127], 1); });
        ordered();
        wave_digit(hist, shift, &key, rank);
    }
    return key;
}

// What adaptive_emit needs of a slice: the threshold its head's keys are kept by, how many equal to it, and what lies before.
struct HeadThreshold { uint32_t thr; int need_eq, gt_before, eq_before, kept; };

__device__ __forceinline__ HeadThreshold head_threshold(AdaptiveShared &sh, const Slices &S, const SlicePlace &at, int n_safe, int budget) {
    using D = Digits<kSliceBits>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = gridDim.x, own_head = at.slice / S.per_head;
    const int head0 = own_head * S.per_head, head1 = head0 + S.per_head;
    clear_counters<D::kBins1>(sh.hist1);
    clear_counters<D::kBins2>(sh.hist2);
    if (tid == 0) sh.above_before = sh.gt_before = sh.gt_head = sh.eq_before_heads = sh.eq_before = sh.eq_head = 0;
    __syncthreads();
    const HeadState own = sh.head[own_head];
    // The lists that count: of the head alone where it stands apart, else of all heads that do not.
    if (wave == 0) {
        int base = 0;
        for (int s0 = 0; s0 < n; s0 += 64) {
            const int sl = s0 + lane;
            int c = 0;
            if (sl < n && (own.apart ? sl >= head0 && sl < head1 : sh.head[sl / S.per_head].apart == 0)) c = sh.count[sl];
            if (sl < n) sh.count[sl] = c;
            const int incl = wave_scan<false>(c, lane);
            if (sl < n) sh.offset[sl] = base + incl - c;
            base += __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) sh.offset[n] = base;
    } else if (wave == 1) {                                  // keys above the class in the head's earlier slices
        int before = 0;
        for (int sl = head0 + lane; sl < at.slice; sl += 64) before += S.above[(size_t)at.group * n + sl];
        before = (int)wave_reduce<SumOp>((uint32_t)before);
        if (lane == 0) sh.above_before = before;
    }
    // What the lists decide between themselves (the budget less what the heads keep in any case), and whether a safeguard
    // ends inside the common class.
    int remaining = own.safe_rank, n_equal;
    bool any_safe = false;
    if (!own.apart) {
        const bool head = lane < S.heads;
        const HeadState st = sh.head[head ? lane : 0];
        static_assert(kFewHeads <= 64, "a lane per head");
        any_safe = __ballot(head && !st.apart && st.safe_rank > 0) != 0ull;
        const int sure = !head ? 0 : st.apart ? n_safe : st.above + st.safe_rank;       // (at most heads * budget in all)
        remaining = (int)((uint32_t)S.heads * budget - wave_reduce<SumOp>((uint32_t)sure));
    }
    auto safe_of = [&](int h) { return any_safe && sh.head[h].apart == 0 && sh.head[h].safe_rank > 0; };
    __syncthreads();
    const int n_list = sh.offset[n], p_head0 = sh.offset[head0], p_slice = sh.offset[at.slice], p_head1 = sh.offset[head1];
    const bool in_lds = n_list <= kAdaptiveList;             // uniform
    const uint32_t *lists = S.list + (size_t)at.group * n * S.list_stride;
    if (in_lds) {
        constexpr int kAhead = 4;                            // slices of a wave in flight at once
        for (int s0 = wave; s0 < n; s0 += kAhead * kSelWaves) {
            uint32_t key[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int sl = s0 + u * kSelWaves;
                key[u] = sl < n && lane < sh.count[sl] ? lists[(size_t)sl * S.list_stride + lane] : 0u;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int sl = s0 + u * kSelWaves;
                if (sl >= n) continue;                       // uniform
                const int c = sh.count[sl], o = sh.offset[sl];
                if (lane < c) sh.list[o + lane] = key[u];
                for (int i = 64 + lane; i < c; i += 64) sh.list[o + i] = lists[(size_t)sl * S.list_stride + i];
            }
        }
        __syncthreads();
    }
    // f(key, place) over the lists of slices with want(head) where they lie: a wave takes 1024 keys of a slice at a time, several
    // waves the same slice where there are fewer than sixteen.  (With one load in flight, and a wave per head for the safeguards,
    // crowded classes made the selection slower than the five kernels are.  2 x 8 heads x 24001 scores, budget 1024, us, five
    // kernels / so / now: uniform 57 / 82 / 47, all in one class 221 / 308 / 135; 8 x 90000 141 / 191 / 88 and 808 / 1133 / 464;
    // 4 x 32 x 4000, uniform 45 / 62 / 51.)
    const int by = 31 - __builtin_clz(max(kSelWaves / n, 1));                    // 2^by waves per slice
    auto visit_global = [&](auto &&want, auto &&f) {
        constexpr int kLoads = 4;                            // (of four keys per lane, in flight together)
        const int uwave = __builtin_amdgcn_readfirstlane(wave);
        for (int sl = uwave >> by; sl < n; sl += kSelWaves >> by) {
            const int c = __builtin_amdgcn_readfirstlane(sh.count[sl]);
            if (c == 0 || !want(sl / S.per_head)) continue;  // uniform in the wave
            const uint32_t *src = lists + (size_t)sl * S.list_stride;            // (lists start at multiples of four keys)
            const int last = (c - 1) / 4 * 4, o = __builtin_amdgcn_readfirstlane(sh.offset[sl]);
            for (int i0 = (uwave & ((1 << by) - 1)) * 256 * kLoads; i0 < c; i0 += 256 * kLoads << by) {
                uint4 key[kLoads];
#pragma unroll
                for (int u = 0; u < kLoads; ++u) key[u] = *(const uint4 *)(src + min(i0 + 256 * u + 4 * lane, last));
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    const int i = i0 + 256 * u + 4 * lane;
                    if (i0 + 256 * u >= c) break;            // uniform
                    const uint32_t k[4] = {key[u].x, key[u].y, key[u].z, key[u].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (i + e < c) f(k[e], o + i + e);
                }
            }
        }
    };
    // Safeguards that end inside the common class; their keys leave the competition: as 0, which no key is, but for those
    // equal to the last one.  A wave per head; where the lists do not fit LDS, whose space is free then, all heads at a time.
    if (any_safe && in_lds) {                                // uniform
        static_assert(D::kBins1 == kSelWaves * 128, "counters of wave_select");
        for (int h = wave; h < S.heads; h += kSelWaves) {
            if (!safe_of(h)) continue;                       // uniform in the wave
            const int j0 = sh.offset[h * S.per_head], j1 = sh.offset[(h + 1) * S.per_head];
            int rank = sh.head[h].safe_rank;
            const uint32_t thr = wave_select(sh.hist1 + 128 * wave, sh.head[h].digit << (32 - kSliceBits), &rank, [&](auto &&f) {
#pragma unroll 4
                for (int j = j0 + lane; j < j1; j += 64) f(sh.list[j]);
            });
            if (lane == 0) { sh.safe_thr[h] = thr; sh.safe_eq[h] = rank; }
            for (int j = j0 + lane; j < j1; j += 64)
                if (sh.list[j] > thr) sh.list[j] = 0u;
        }
        __syncthreads();
        clear_counters<D::kBins1>(sh.hist1);
        __syncthreads();
    } else if (__builtin_expect(any_safe, false)) {
        static_assert(kFewHeads * 128 <= kAdaptiveList, "counters of a digit for every head");
        int *const counters = (int *)sh.list;
        if (tid < S.heads && safe_of(tid)) { sh.safe_thr[tid] = sh.head[tid].digit << (32 - kSliceBits); sh.safe_eq[tid] = sh.head[tid].safe_rank; }
#pragma unroll 1
        for (int shift = 2 * kRankBits; shift >= 0; shift -= kRankBits) {
            for (int i = tid; i < S.heads * 128; i += kSelThreads) counters[i] = 0;
            __syncthreads();
            uint32_t prefix;
            int *of_head;
            visit_global([&](int h) {
                if (!safe_of(h)) return false;
                prefix = sh.safe_thr[h];
                of_head = counters + 128 * h;
                return true;
            }, [&](uint32_t key, int) { if ((key ^ prefix) >> (shift + kRankBits) == 0) atomicAdd(&of_head[(key >> shift) & 127], 1); });
            __syncthreads();
            for (int h = wave; h < S.heads; h += kSelWaves) {
                if (!safe_of(h)) continue;                   // uniform in the wave
                uint32_t thr = sh.safe_thr[h];
                int rank = sh.safe_eq[h];
                wave_digit(counters + 128 * h, shift, &thr, &rank);
                if (lane == 0) { sh.safe_thr[h] = thr; sh.safe_eq[h] = rank; }
            }
            __syncthreads();
        }
    }
    // keys equal to a safeguard's last one that belong to it, taken off a digit's counters
    auto take_off = [&](int *hist, int shift, uint32_t bins, auto &&counted) {
        if (!any_safe) return;                               // uniform
        __syncthreads();
        if (tid < S.heads && safe_of(tid) && counted(sh.safe_thr[tid])) atomicSub(&hist[(sh.safe_thr[tid] >> shift) & (bins - 1)], sh.safe_eq[tid]);
    };
    // visit(f): f(key, place) over the lists; key 0: of a safeguard
    HeadThreshold t;
    uint32_t common;
    bool safe_only;
    int gt_before = 0, gt_head = 0, eq_heads = 0, eq_before = 0, eq_head = 0;
    auto settle = [&](auto &&visit) {
        uint32_t digit;
        visit([&](uint32_t key, int) { if (key) atomicAdd(&sh.hist1[(key >> D::kShift1) & (D::kBins1 - 1)], 1); });
        take_off(sh.hist1, D::kShift1, D::kBins1, [](uint32_t) { return true; });
        pick_digit<D::kBins1>(sh.hist1, sh.pick, &digit, &remaining, &n_equal);
        const uint32_t middle = digit;
        auto in_middle = [&](uint32_t key) { return ((key >> D::kShift1) & (D::kBins1 - 1)) == middle; };
        visit([&](uint32_t key, int) { if (key && in_middle(key)) atomicAdd(&sh.hist2[key & (D::kBins2 - 1)], 1); });
        take_off(sh.hist2, 0, D::kBins2, in_middle);
        pick_digit<D::kBins2>(sh.hist2, sh.pick, &digit, &remaining, &n_equal);
        common = (own.digit << (32 - kSliceBits)) | (middle << D::kShift1) | digit;
        // The head keeps its safeguard alone where that ends below the threshold.
        safe_only = safe_of(own_head) && sh.safe_thr[own_head] < common;
        t.thr = safe_only ? sh.safe_thr[own_head] : common;
        visit([&](uint32_t key, int j) {
            const bool in_head = j >= p_head0 && j < p_head1;    // (no branches: as in slice_threshold)
            const int gt = in_head & (key == 0u || key > t.thr) ? 1 : 0, eq = in_head & (key == t.thr) ? 1 : 0;
            gt_head += gt;
            eq_head += eq;
            gt_before += j < p_slice ? gt : 0;
            eq_before += j < p_slice ? eq : 0;
            eq_heads += (j < p_head0) & (key == common) ? 1 : 0;
        });
    };
    if (__builtin_expect(in_lds, true)) {
        settle([&](auto &&f) { for (int j = tid; j < n_list; j += kSelThreads) f(sh.list[j], j); });
    } else {
        settle([&](auto &&f) {
            uint32_t most;
            visit_global([&](int h) { most = safe_of(h) ? sh.safe_thr[h] : 0xffffffffu; return true; },
                         [&](uint32_t key, int j) { f(key > most ? 0u : key, j); });
        });
    }
    auto add = [&](int *to, int x) {
        if (__ballot(x != 0) == 0ull) return;                // uniform
        x = (int)wave_reduce<SumOp>((uint32_t)x);
        if (lane == 0) atomicAdd(to, x);
    };
    add(&sh.gt_before, gt_before);
    add(&sh.gt_head, gt_head);
    add(&sh.eq_before_heads, eq_heads);
    add(&sh.eq_before, eq_before);
    add(&sh.eq_head, eq_head);
    if (any_safe && tid < own_head && safe_of(tid) && sh.safe_thr[tid] == common) atomicSub(&sh.eq_before_heads, sh.safe_eq[tid]);
    __syncthreads();
    if (safe_only) {
        t.need_eq = sh.safe_eq[own_head];
    } else {                                                 // the safeguard's first, then as many as earlier heads leave
        const int safe = safe_of(own_head) && sh.safe_thr[own_head] == common ? sh.safe_eq[own_head] : 0;
        t.need_eq = safe + min(max(remaining - sh.eq_before_heads, 0), sh.eq_head - safe);
    }
    t.gt_before = sh.above_before + sh.gt_before;
    t.eq_before = sh.eq_before;
    t.kept = own.above + sh.gt_head + t.need_eq;
    return t;
}

template <int kBatch, typename Lens>
__global__ __launch_bounds__(kSelThreads) void adaptive_emit(const float *__restrict__ scores, int N, int budget, int n_safe, int room,
                                                             int Hkv, int ragged, Lens lens, Slices S,
                                                             const HeadState *__restrict__ states, int32_t *__restrict__ keep_idx,
                                                             int32_t *__restrict__ counts) {
    __shared__ __attribute__((aligned(16))) AdaptiveShared sh;
    const SlicePlace at(S, N, Hkv, ragged, lens);
    const int tid = threadIdx.x, n = gridDim.x;
    const int count = tid < n ? S.count[(size_t)at.group * n + tid] : 0;      // (n <= kMaxGroupSlices: the host's choice)
    if (tid < S.heads) sh.head[tid] = states[(size_t)at.group * S.heads + tid];
    HeadThreshold t;
    int32_t *out = keep_idx + (size_t)at.head * room;
    int gt_base, eq_base;
    for_batches<kBatch>(S, at, scores, N, 0, 0, 0, false, [&]() {
        if (tid < n) sh.count[tid] = count;
        t = head_threshold(sh, S, at, n_safe, budget);
        gt_base = t.gt_before;
        eq_base = t.eq_before;
    }, [&](uint32_t (&keys)[kBatch][kItems], int c) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (c + i < at.c1)
                emit_chunk(sh.pick.wave_tot, keys[i], (c + i) * kChunk + tid * kItems, at.len, t.thr, t.need_eq, room, gt_base, eq_base, out);
    });
    const int kept = min(t.kept, room);
    if (at.in_head == 0 && tid == 0) counts[at.head] = kept;
    for (int j = kept + at.in_head * kSelThreads + tid; j < room; j += S.per_head * kSelThreads) out[j] = -1;
}

}  // namespace

static size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// Slices of about 4096 scores, longer ones where a group would have more than 64 of them (every workgroup sums the
// group's histograms, 8 KB per slice); 256 from 16K scores per slice on, where that is little beside the slice itself.
static int slice_chunks(int heads, int N) {
    int chunks = 1;
    auto per_head = [&]() { return (N + (long long)chunks * kChunk - 1) / ((long long)chunks * kChunk); };
    while (per_head() > 1 && heads * per_head() > (chunks < 4 ? 64 : 256)) chunks = chunks == 1 ? 4 : chunks * 2;
    return chunks;
}

// Carves the buffers of a sliced selection out of `base` (nullptr: sizes only); returns the bytes.
static size_t plan_slices(Slices *S, char *base, int groups, int heads, int N, bool own_keys) {
    S->groups = groups;
    S->group0 = 0;
    S->heads = heads;
    S->chunks = slice_chunks(heads, N);
    S->per_head = (int)((N + (long long)S->chunks * kChunk - 1) / ((long long)S->chunks * kChunk));
    S->key_stride = (N + 3) / 4 * 4;
    S->list_stride = S->per_head == 1 ? S->key_stride : S->chunks * kChunk;
    const size_t slices = (size_t)groups * heads * S->per_head;
    size_t off = 0;
    auto take = [&](size_t bytes) { char *p = base + off; off += up256(bytes); return p; };
    S->hist = (int *)take(slices * kSliceBins * sizeof(int));
    S->list = (uint32_t *)take(slices * S->list_stride * sizeof(uint32_t));
    S->above = (int *)take(slices * sizeof(int));
    S->count = (int *)take(slices * sizeof(int));
    S->state = (SliceState *)take((size_t)groups * sizeof(SliceState));
    S->keys = own_keys ? (uint32_t *)take((size_t)groups * heads * S->key_stride * sizeof(uint32_t)) : nullptr;
    return off;
}

// f(shape, grid) for launches of as many groups as the grid's y takes: one, but for tens of thousands of heads.  (One launch
// with all slices along x cost a division ahead of the first loads, with the groups along y and z another round trip for the
// grid's size: 0.1 us per kernel.)
template <typename F>
static void over_groups(Slices S, F &&f) {
    constexpr int kMost = 65535;
    for (S.group0 = 0; S.group0 < S.groups; S.group0 += kMost) {
        const int left = S.groups - S.group0;
        f(S, dim3((unsigned)S.heads * S.per_head, left < kMost ? left : kMost));
    }
}

template <typename F>
static hipError_t with_batch(const Slices &S, F &&f) {
    return S.chunks == 1 ? f(std::integral_constant<int, 1>()) : f(std::integral_constant<int, 4>());
}

// Only the pooled ranking reads keys; scores are turned into them as quickly as keys are read.
size_t select_workspace_bytes(int B, int Hkv, int N, bool pooled) {
    Slices S;
    return plan_slices(&S, nullptr, B * Hkv, 1, N, pooled);
}

// Long heads take the sliced path: one workgroup per head keeps a 32K-token head in registers, but beyond that it
// spills or re-streams the head in every pass (53 us at 64K, 390 us at 128K measured).
bool select_prefers_slices(int B, int Hkv, int N) {
    return N > 8 * kChunk && (long long)B * Hkv <= 65535;
}

static hipError_t launch_select_sliced(const float *scores, int budget, int32_t *keep_idx, int B, int Hkv, int N, int ragged,
                                       const SeqLens &lens, int first, int tail, int radius, void *workspace, hipStream_t stream) {
    Slices S;
    plan_slices(&S, (char *)workspace, B * Hkv, 1, N, radius > 0);
    const dim3 block(kSelThreads);
    return with_lens(ragged, B, lens, [&](const auto &few) {
        return with_batch(S, [&](auto batch) {
            constexpr int kBatch = decltype(batch)::value;
            over_groups(S, [&](const Slices &S, dim3 grid) {
                if (S.chunks <= kPackedChunks) {
                    slices_count<kBatch, true><<<grid, block, 0, stream>>>(scores, N, Hkv, ragged, few, first, tail, radius, S);
                    slices_collect<kBatch, true><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, S);
                } else {
                    slices_count<kBatch, false><<<grid, block, 0, stream>>>(scores, N, Hkv, ragged, few, first, tail, radius, S);
                    slices_collect<kBatch, false><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, S);
                }
                slices_emit<kBatch><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, S, keep_idx,
                                                                (int32_t *)nullptr);
            });
            return hipGetLastError();
        });
    });
}

// The per-head selection of the safeguard and the selection over a sequence's heads cut heads into the same slices.
static size_t plan_adaptive(Slices *safe, Slices *all, char *base, int B, int Hkv, int N) {
    size_t off = plan_slices(all, base, B, Hkv, N, true);
    *safe = *all;
    safe->groups = B * Hkv;
    safe->heads = 1;
    safe->keys = nullptr;                    // (formed from the scores; the second selection's keys are written beside)
    const size_t slices = (size_t)B * Hkv * all->per_head;
    safe->hist = (int *)(base + off);
    off += up256(slices * kSliceBins * sizeof(int));
    safe->state = (SliceState *)(base + off);
    off += up256((size_t)B * Hkv * sizeof(SliceState));
    return off;
}

size_t select_adaptive_workspace_bytes(int B, int Hkv, int N) {
    Slices a, b;
    return plan_adaptive(&a, &b, nullptr, B, Hkv, N);
}

hipError_t launch_select_adaptive(const float *scores, int budget, int n_safe, int cap, int32_t *keep_idx,
                                  int32_t *counts, int B, int Hkv, int N, int ragged, const SeqLens &lens,
                                  void *workspace, hipStream_t stream) {
    Slices safe, all;
    plan_adaptive(&safe, &all, (char *)workspace, B, Hkv, N);
    const dim3 block(kSelThreads);
    return with_lens(ragged, B, lens, [&](const auto &few) {
        return with_batch(all, [&](auto batch) {
            constexpr int kBatch = decltype(batch)::value;
            if (Hkv <= kFewHeads && Hkv * all.per_head <= kMaxGroupSlices && all.chunks <= kPackedChunks && n_safe < budget) {
                HeadState *states = (HeadState *)safe.hist;              // (a second set of histograms is not needed)
                safe.hist = all.hist;
                over_groups(safe, [&](const Slices &S, dim3 grid) {
                    slices_count<kBatch, true><<<grid, block, 0, stream>>>(scores, N, Hkv, ragged, few, 0, 0, 0, S);
                });
                over_groups(all, [&](const Slices &S, dim3 grid) {
                    adaptive_collect<kBatch><<<grid, block, 0, stream>>>(scores, N, budget, n_safe, Hkv, ragged, few, S, states);
                    adaptive_emit<kBatch><<<grid, block, 0, stream>>>(scores, N, budget, n_safe, cap, Hkv, ragged, few, S, states, keep_idx, counts);
                });
                return hipGetLastError();
            }
            over_groups(safe, [&](const Slices &S, dim3 grid) {
                if (n_safe > 0) {
                    slices_count<kBatch, false><<<grid, block, 0, stream>>>(scores, N, Hkv, ragged, few, 0, 0, 0, S);
                    slices_collect<kBatch, false><<<grid, block, 0, stream>>>(scores, N, n_safe, Hkv, ragged, few, 0, 0, 0, S);
                }
                slices_safeguard<kBatch><<<grid, block, 0, stream>>>(scores, N, n_safe, Hkv, ragged, few, S, all.keys, all.hist);
            });
            over_groups(all, [&](const Slices &S, dim3 grid) {
                slices_collect<kBatch, false><<<grid, block, 0, stream>>>(scores, N, Hkv * budget, Hkv, ragged, few, 0, 0, 0, S);
                slices_emit<kBatch><<<grid, block, 0, stream>>>(scores, N, cap, Hkv, ragged, few, 0, 0, 0, S, keep_idx, counts);
            });
            return hipGetLastError();
        });
    });
}

hipError_t launch_select(const float *scores, int budget, int32_t *keep_idx, int B, int Hkv, int N, int ragged,
                         const SeqLens &lens, int first, int tail, int radius, void *workspace,
                         size_t workspace_bytes, hipStream_t stream) {
    if (workspace && select_prefers_slices(B, Hkv, N) && workspace_bytes >= select_workspace_bytes(B, Hkv, N, radius > 0))
        return launch_select_sliced(scores, budget, keep_idx, B, Hkv, N, ragged, lens, first, tail, radius, workspace, stream);
    const dim3 grid(B * Hkv), block(kSelThreads);
    return with_lens(ragged, B, lens, [&](const auto &few) {
        if (N <= kChunk)             // (short heads: fewer unrolled chunk bodies to step through)
            select_topk<1, true><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, keep_idx);
        else if (N <= 2 * kChunk)
            select_topk<2, true><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, keep_idx);
        else if (N <= 8 * kChunk)
            select_topk<8, true><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, keep_idx);
        else if (N <= 16 * kChunk)
            select_topk<16, true><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, keep_idx);
        else
            select_topk<8, false><<<grid, block, 0, stream>>>(scores, N, budget, Hkv, ragged, few, first, tail, radius, keep_idx);
        return hipGetLastError();
    });
}

}  // namespace obc
