// Decode-time scoring: a perturbation window of ONE query row per head (W = 1, the setting
// Section 3.2 and Appendix C use while generating), bf16 cache.
//
// With one row per query head a KV head sees only G = Hq/Hkv rows, far too few to fill a
// matrix-core tile, and at the cache sizes of decoding the call is bound by memory round
// trips and dependent instructions, not by bandwidth.  The path is three kernels with 128-bit
// coalesced loads (one token row spread over d/8 lanes), on the vector ALUs but for the sums of P V of five to eight
// rows, in which a workgroup owns a short range of tokens and every lane issues ALL its loads of the range before it computes:
//   decode_partial   per range: scaled logits Z = q.k/sqrt(d) (Section 3), kept in the
//                    workspace so K is read once; range max, sum and unnormalised output
//                    (the range's top-logit token is held out of both sums, see below)
//   decode_merge     per KV head: log-sum-exp merge of the ranges into the row max, 1/sum,
//                    o_i and v_p* - o_i (folded into decode_score when the ranges are few)
//   decode_score     Eq. 4-6 in their direct forms ||v_p||^2, ||v_p - o_i||^2 and
//                    ||v_p + Z (v_p - o_i)||^2 (the completed square of Eq. 6), Eq. 8 and
//                    the l1-weighted variant of Appendix C, summed over the query heads of
//                    the KV head (Appendix A.5), written or added to the running scores; for an
//                    eviction step also every wave's lowest-scored token.
// Ranges are as short as lets all their workgroups run at once and keeps the inline merge possible
// (1, 2 or 4 tokens per lane, sixteen waves): instructions of a lone wave issue one by one, so the count per wave is its
// time.  8 KV heads x 1025 tokens, G = 4, d = 128, joint, per layer: 72 workgroups of 8 tokens per
// lane, four waves each, 26 us for the two kernels; 136 workgroups of one token per lane, sixteen waves, 11 us.
//
// Cancellation guard.  When one key takes almost all of a row's attention, o_i is almost
// v_p* and fp32 cannot hold their difference.  Every range keeps its top-logit token out of
// its sums and reports the output with and without it; the merge takes the sums with it from all
// ranges but the winning one, so with l' and o' the sum and the mean over every key but p*,
//     v_p* - o_i = (l' / (1 + l')) (v_p* - o')        (no cancellation)
//     o_i        = v_p* - (v_p* - o_i)
// and the (row, p*) pair is scored from the first identity.
// Every sum runs in a fixed order: results are bit-reproducible.
#include "internal.h"
#include "wave_util.h"

namespace obc {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxSteps = 4;         // most token rows per lane: a range is 1, 2 or 4 workgroup-wide steps
constexpr int kVectorRows = 4;       // most rows whose sums of P V are vector ops
constexpr int kInlineSplits = 48;    // most ranges per head the scoring kernel merges itself
constexpr int kMergeThreads = 1024;
constexpr int kMergeOwn = 4;         // ranges per merging thread
constexpr int kMaxSplits = kMergeThreads * kMergeOwn;
constexpr int kRecHead = 4;          // floats ahead of the vectors in a final record

__host__ __device__ constexpr int tokens_per_step(int d) { return kWaves * (64 / (d / 8)); }
// Partial record of (KV head, range, row): head {range max, sum without the top token, top token
// (int bits, -1 for an empty range), spare}; vectors {unnormalised output without the top token [d],
// the same with it [d]}, valid unless the range is empty.
// Final record of (KV head, row): {row max, 1/sum, top token (int bits), spare, o_i [d],
// v_p* - o_i [d]}.
__host__ __device__ constexpr int final_stride(int d) { return 2 * d + kRecHead; }

__device__ __forceinline__ void unpack8(const uint4 w, float *x) {
    x[0] = __uint_as_float(w.x << 16); x[1] = __uint_as_float(w.x & 0xffff0000u);
    x[2] = __uint_as_float(w.y << 16); x[3] = __uint_as_float(w.y & 0xffff0000u);
    x[4] = __uint_as_float(w.z << 16); x[5] = __uint_as_float(w.z & 0xffff0000u);
    x[6] = __uint_as_float(w.w << 16); x[7] = __uint_as_float(w.w & 0xffff0000u);
}

// Sum over the `kLanes` (8 or 16) consecutive lanes that share a token; all of them end with the
// same bits.
template <int kLanes>
__device__ __forceinline__ float group_sum(float x) {
    x += dpp_pair<0xB1>(x);
    x += dpp_pair<0x4E>(x);
    x += dpp_pair<0x141>(x);
    if (kLanes == 16) x += dpp_pair<0x140>(x);
    return x;
}
// x of the lane whose index differs in bit 2 alone: the mirror image inside 8 lanes, then inside 4.
__device__ __forceinline__ float xor4(float x) { return dpp_pair<0x1B>(dpp_pair<0x141>(x)); }
// Sums over the lanes that share a token for the kG rows at once: lane `sub` of them ends up with the sum of row own_row(sub),
// and lanes of the same row with the same bits.  Each of the first levels adds two rows across lane pairs with one exchange and
// leaves one of them in each lane of the pair (11 operations for four rows of 16 lanes; 16 with every sum in every lane).
template <int kG>
__device__ __forceinline__ int own_row(int sub) { return sub & (kG - 1); }
template <int kLanes, int kG>
__device__ __forceinline__ float row_sums(float (&x)[kG], int sub) {
    if constexpr (kG >= 2) {
#pragma unroll
        for (int i = 0; i < kG / 2; ++i) {
            const float keep = sub & 1 ? x[2 * i + 1] : x[2 * i], give = sub & 1 ? x[2 * i] : x[2 * i + 1];
            x[i] = keep + dpp_pair<0xB1>(give);
        }
    } else {
        x[0] += dpp_pair<0xB1>(x[0]);
    }
    if constexpr (kG >= 4) {
#pragma unroll
        for (int i = 0; i < kG / 4; ++i) {
            const float keep = sub & 2 ? x[2 * i + 1] : x[2 * i], give = sub & 2 ? x[2 * i] : x[2 * i + 1];
            x[i] = keep + dpp_pair<0x4E>(give);
        }
    } else {
        x[0] += dpp_pair<0x4E>(x[0]);
    }
    if constexpr (kG >= 8) {
        const float keep = sub & 4 ? x[1] : x[0], give = sub & 4 ? x[0] : x[1];
        x[0] = keep + xor4(give);
        if (kLanes == 16) x[0] += dpp_pair<0x128>(x[0]);
    } else if (kLanes == 16) {
        x[0] += dpp_pair<0x128>(x[0]);
        x[0] += dpp_pair<0x124>(x[0]);                  // (the two halves of the row are alike: the lane 4 further is that of bit 2)
    } else {
        x[0] += xor4(x[0]);
    }
    return x[0];
}
typedef __bf16 bf16_pair __attribute__((ext_vector_type(2)));
// Sums over the wave's token slots of a lane's eight channels: row q of 16 lanes gets those of channels 2 q and 2 q + 1.  (Each
// exchange brings two channels together and leaves one of them in either half.)
template <int kLpt>
__device__ __forceinline__ float2 sums_over_slots(const float (&x)[8]) {
    float half[4], two[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[j]), __float_as_uint(x[j + 4]), false, false);
        half[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(half[j]), __float_as_uint(half[j + 2]), false, false);
        two[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        if (kLpt == 8) two[j] += dpp_pair<0x128>(two[j]);
    }
    return make_float2(two[0], two[1]);
}
typedef float f32_quad __attribute__((ext_vector_type(4)));
// acc + the dot product of 8 bf16 values each (exact products, fp32 sums).
__device__ __forceinline__ float dot8(const uint4 a, const uint4 b, float acc) {
    union { uint4 w; bf16_pair h[4]; } x, y;
    x.w = a;
    y.w = b;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_fdot2_f32_bf16(x.h[e], y.h[e], acc, false);
    return acc;
}
// (larger value, lower index on ties) of two candidates.
__device__ __forceinline__ void take_better(float &bm, int &ba, float om, int oa) {
    if (om > bm || (om == bm && oa < ba)) { bm = om; ba = oa; }
}

// Token of step u for this lane: steps interleave the waves so that a step of the workgroup
// covers consecutive rows.
template <int kD>
__device__ __forceinline__ int token_of(int t0, int u, int wave, int slot) {
    return t0 + u * tokens_per_step(kD) + wave * (64 / (kD / 8)) + slot;
}

// The scaled logits of the range, its row maxima and the unnormalised sums around them.  With kEdges, for an eviction step, also
// copies of the rows that begin a piece of evict_pieces; other calls carry none of that.
template <int kG, int kD, int kSteps, bool kNeedO, bool kEdges, typename Lens>
__global__ __launch_bounds__(kThreads) void decode_partial(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, const uint16_t *__restrict__ v, int N, int G,
    int Hkv, int ragged, Lens lens, int splits, float *__restrict__ z_buf, float4 *__restrict__ part_head,
    float *__restrict__ part_vec, uint4 *__restrict__ edge_rows) {
    constexpr int kLpt = kD / 8;        // lanes per token row
    __shared__ float red_m[kWaves * kG];
    __shared__ int red_a[kWaves * kG];
    __shared__ float red_l[kWaves * kG];
    // Sums of P V by matrix op: [wave, and with 8 lanes per token its even or odd tokens][channel j of a lane's 8][lane][row]; the
    // padding between two j takes the closing sum's reads to as many banks.
    constexpr int kHalves = 16 / kLpt, kChannel = kLpt * kG + 8, kPartSums = kWaves * kHalves;
    constexpr bool kVector = kG <= kVectorRows;     // sums of P V by vector ops: [wave][row][channel]
    __shared__ __attribute__((aligned(16))) float red_o[!kNeedO ? 4 : kVector ? kWaves * kG * kD : kPartSums * 8 * kChannel];
    __shared__ float top_v[kNeedO ? kG * kD : 1];   // V rows of the top tokens

    const int bh = blockIdx.x, b = bh / Hkv, split = blockIdx.y;
    const int len = seq_len_of(lens, ragged, b, N);
    const int t0 = split * kSteps * tokens_per_step(kD);
    const int t1 = min(t0 + kSteps * tokens_per_step(kD), len);
    float4 *head = part_head + ((size_t)bh * splits + split) * kG;
    if (t0 >= len) {                                // nothing of this sequence falls in the range
        if (threadIdx.x < kG) head[threadIdx.x] = make_float4(-INFINITY, 0.f, __int_as_float(-1), 0.f);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane % kLpt, slot = lane / kLpt;
    const float scale = kD == 128 ? 0.088388347648318440550f : 0.125f;
    const uint16_t *kg = k + (size_t)bh * N * kD;
    const uint16_t *vg = v + (size_t)bh * N * kD;

    // Every load of the range up front.
    uint4 qw[kG], kw[kSteps], vw[kSteps];
#pragma unroll
    for (int r = 0; r < kG; ++r) {
        qw[r] = make_uint4(0, 0, 0, 0);
        if (r < G) qw[r] = *(const uint4 *)(q + ((size_t)bh * G + r) * kD + sub * 8);
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        kw[u] = make_uint4(0, 0, 0, 0);
        if (p < t1) kw[u] = *(const uint4 *)(kg + (size_t)p * kD + sub * 8);
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        vw[u] = make_uint4(0, 0, 0, 0);
        if (kNeedO && p < t1) vw[u] = *(const uint4 *)(vg + (size_t)p * kD + sub * 8);
    }

    // Copies of the rows that begin a piece of evict_pieces, at the very end, where nobody waits for them, kept as they came by.  V that
    // the sums do not need is fetched there, in long ranges with the other loads: those workgroups do not all run at once, and
    // the next one waits for this one's last trip (32 heads, value, d = 128, 4117 tokens: 9.5 us without copies, V at the end 11.3).
    // A piece is two steps long: only even steps have any.
    static_assert(evict_piece_rows(kD) == 2 * tokens_per_step(kD), "pieces begin at even steps");
    constexpr bool kEarly = !kNeedO && kSteps == kMaxSteps;
    constexpr int kEdgeSteps = kEdges ? (kSteps + 1) / 2 : 0;
    uint4 edge_v[kEdgeSteps > 0 ? kEdgeSteps : 1];
    if constexpr (kEdges && kEarly) {
#pragma unroll
        for (int i = 0; i < kEdgeSteps; ++i) {
            const int p = token_of<kD>(t0, 2 * i, wave, slot);
            edge_v[i] = make_uint4(0, 0, 0, 0);
            if (p % evict_piece_rows(kD) == 0 && p != 0 && p < t1) edge_v[i] = *(const uint4 *)(vg + (size_t)p * kD + sub * 8);
        }
    }
    auto put_edges_aside = [&]() {
        const int pieces = evict_row_pieces(N, kD);
#pragma unroll
        for (int i = 0; i < kEdgeSteps; ++i) {
            const int p = token_of<kD>(t0, 2 * i, wave, slot);
            if (p % evict_piece_rows(kD) != 0 || p == 0 || p >= t1) continue;        // (nothing moves up from the first row)
            uint4 *to = edge_rows + ((size_t)bh * 2 * pieces + p / evict_piece_rows(kD)) * kLpt + sub;
            to[0] = kw[2 * i];
            to[(size_t)pieces * kLpt] = kEarly ? edge_v[i] : kNeedO ? vw[2 * i] : *(const uint4 *)(vg + (size_t)p * kD + sub * 8);
        }
    };

    // From here on lane `sub` of a token's lanes looks after row own: one logit, one weight, one sum per lane and token.
    const int own = own_row<kG>(sub);
    float z[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        float dot[kG];
#pragma unroll
        for (int r = 0; r < kG; ++r) dot[r] = dot8(qw[r], kw[u], 0.f);
        z[u] = row_sums<kLpt, kG>(dot, sub) * scale;
        if (p < t1 && sub < kG) z_buf[((size_t)bh * N + p) * kG + sub] = z[u];
    }

    // Row maxima of the range and the lowest token attaining each.
    {
        float bm = -INFINITY;
        int ba = 0x7fffffff;
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {          // tokens ascend with u: a strict compare keeps the lowest
            const int p = token_of<kD>(t0, u, wave, slot);
            if (p < t1 && z[u] > bm) { bm = z[u]; ba = p; }
        }
        // over the wave's token slots: the value first, then the lowest token that has it
        const float mine = bm;
        if (kLpt == 8) bm = fmaxf(bm, dpp_pair<0x128>(bm));
        bm = across_rows<MaxOp>(bm);
        uint32_t at = mine == bm ? (uint32_t)ba : 0x7fffffffu;
        if (kLpt == 8) at = MinOp()(at, dpp_pair<0x128>(at));
        at = across_rows<MinOp>(at);
        if (lane < kG) { red_m[lane * kWaves + wave] = bm; red_a[lane * kWaves + wave] = (int)at; }
    }
    __syncthreads();
    // over the waves: one row of 16 lanes per window row (four at a time; fewer rows than four repeat)
    constexpr int kQuads = (kG + 3) / 4;
    float row_m[kQuads];
    int row_top[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) {
        const int e = kG >= 4 ? 4 * i * kWaves + lane : lane % (kG * kWaves);
        const float mine = red_m[e];
        row_m[i] = row16_reduce<MaxOp>(mine);
        row_top[i] = min((int)row16_reduce<MinOp>(mine == row_m[i] ? (uint32_t)red_a[e] : 0x7fffffffu), t1 - 1);   // (no logit was a number: any token)
    }
    float m = 0.f;
    int top = 0;
#pragma unroll
    for (int i = 0; i < kQuads; ++i) {
        const int from = 16 * (own & 3) * 4;
        const float mi = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(row_m[i])));
        const int ti = __builtin_amdgcn_ds_bpermute(from, row_top[i]);
        if (i == 0 || own >= 4 * i) { m = mi; top = ti; }
    }

    // Sums of exp(z - m) and of exp(z - m) v over the range without the top token.  The second one, up to kVectorRows rows: products
    // on the vector ALUs with the weights of a row handed round each four lanes; the sums over the token slots leave two channels in
    // each slot.  Eight rows, whose 64 sums have no registers beside a long range's loads: a matrix op per channel: its first operand's
    // row is a lane's own row, its four k are the wave's token slots, and a lane's channel j is a column of the second; fp32
    // throughout.  With 8 lanes per token a row of 16 lanes has an even and an odd token: rows 0 to 7 are the even ones' weights, 8 to
    // 15 the odd ones', and of the product only what meets its own half counts.
    // (The matrix ops take a wave's step 120 ns however many rows are in use.  A decoding step's three kernels in a graph, 8 heads, d = 128,
    // joint, with every row's weight and sum in every lane and sums by exchanges of whole registers / matrix ops / so, us:
    //   G = 1, 2000 tokens 13.6 / 13.6 / 13.4      G = 4, 1025 tokens 15.0 / 13.7 / 13.5
    //   G = 2, 4000 tokens 18.8 / 18.3 / 17.6      G = 4, 4000 tokens 21.5 / 20.2 / 19.9
    // (with matrix ops 4 x 8 heads, G = 1, 1000 tokens took 16.7, before 15.8, so 15.9).)
    float lsum = 0.f;
    f32_quad acc[8];
    float sums[kVector ? kG : 1][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        acc[j] = f32_quad{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < (kVector ? kG : 1); ++r) sums[r][j] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        const bool is_top = p == top;
        const float w = p < t1 && !is_top ? __expf(z[u] - m) : 0.f;
        lsum += w;
        if (kNeedO) {
            float vv[8];
            unpack8(vw[u], vv);
            if constexpr (kVector) {
                float of_row[4] = {w, w, w, w};     // (lanes r, r + kG, .. of a token's have row r's)
                if (kG >= 2) { of_row[0] = dpp_pair<0x00>(w); of_row[1] = dpp_pair<0x55>(w); }
                if (kG >= 4) { of_row[2] = dpp_pair<0xAA>(w); of_row[3] = dpp_pair<0xFF>(w); }
#pragma unroll
                for (int r = 0; r < kG; ++r)
#pragma unroll
                    for (int j = 0; j < 8; ++j) sums[r][j] = fmaf(of_row[r], vv[j], sums[r][j]);
            } else {
                const float a = sub < kG ? w : 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, vv[j], acc[j], 0, 0, 0);
            }
            if (__any(is_top)) {                    // uniform: the wave holds some row's top token
#pragma unroll
                for (int r = 0; r < kG; ++r) {
                    if (p != __builtin_amdgcn_readlane(row_top[r / 4], 16 * (r % 4))) continue;
                    *(float4 *)(top_v + r * kD + sub * 8) = make_float4(vv[0], vv[1], vv[2], vv[3]);
                    *(float4 *)(top_v + r * kD + sub * 8 + 4) = make_float4(vv[4], vv[5], vv[6], vv[7]);
                }
            }
        }
    }
    if (kLpt == 8) lsum += dpp_pair<0x128>(lsum);
    lsum = across_rows<SumOp>(lsum);
    if (lane < kG) red_l[lane * kWaves + wave] = lsum;
    if constexpr (kNeedO && kVector) {
#pragma unroll
        for (int r = 0; r < kG; ++r) {
            const float2 two = sums_over_slots<kLpt>(sums[r]);
            if (kLpt == 16 || (lane & 8) == 0) *(float2 *)(red_o + (wave * kG + r) * kD + sub * 8 + 2 * (lane >> 4)) = two;
        }
    } else if (kNeedO) {
        // rows 4 (lane / 16) .. + 3 of the product, column lane % 16
        const int quad = lane >> 4, r0 = 4 * (kHalves == 1 ? quad : quad & 1), odd = kHalves == 1 ? 0 : (lane >> 3) & 1;
        if (r0 < kG && (kHalves == 1 || quad >> 1 == odd)) {
            float *to = red_o + (wave * kHalves + odd) * 8 * kChannel + sub * kG + r0;
#pragma unroll
            for (int j = 0; j < 8; ++j) *(f32_quad *)(to + j * kChannel) = acc[j];
        }
    }
    __syncthreads();
    if (wave < kQuads) {                            // one row of 16 lanes per window row again
        const int r = wave * 4 + (lane >> 4);
        const float l = row16_reduce<SumOp>(r < kG ? red_l[r * kWaves + (lane & 15)] : 0.f);
        float mr = row_m[0];
        int tr = row_top[0];
#pragma unroll
        for (int i = 1; i < kQuads; ++i)
            if (wave == i) { mr = row_m[i]; tr = row_top[i]; }
        if ((lane & 15) == 0 && r < kG) head[r] = make_float4(mr, l, __int_as_float(tr), 0.f);
    }
    if (!kNeedO) {
        put_edges_aside();
        return;
    }
    float *vec = part_vec + ((size_t)bh * splits + split) * kG * 2 * kD;
    for (int e = threadIdx.x; e < kG * kD; e += kThreads) {         // (16 channels of each row side by side)
        const int r = (e >> 4) % kG, c = e / (16 * kG) * 16 + (e & 15), at = kVector ? r * kD + c : (c % 8) * kChannel + c / 8 * kG + r;
        float o = red_o[at];
#pragma unroll
        for (int w = 1; w < (kVector ? kWaves : kPartSums); ++w) o += red_o[w * (kVector ? kG * kD : 8 * kChannel) + at];
        vec[r * 2 * kD + c] = o;
        vec[r * 2 * kD + kD + c] = o + top_v[r * kD + c];
    }
    put_edges_aside();
}

// Closing step of a merge for column c of a row: from the sum l_rest and the weighted vector
// sum o_rest over every key but the top one, the final record's entries of that column.
template <int kD>
__device__ __forceinline__ void merge_finish(float l_rest, float o_rest, float v_top, int c, float *rec) {
    const float inv_l = 1.f / (1.f + l_rest);
    const float d_top = l_rest > 0.f ? (l_rest * inv_l) * (v_top - o_rest / l_rest) : 0.f;
    rec[kRecHead + c] = v_top - d_top;
    rec[kRecHead + kD + c] = d_top;
}

// Merge of at most kInlineSplits ranges of one KV head by one workgroup, into final records in LDS.  The vectors of all
// ranges are fetched while the heads are still on their way; only the winning range's two rows wait for them.
template <int kG, int kD, bool kNeedO>
struct MergeFew {
    static constexpr int kFs = final_stride(kD);
    static constexpr int kQuads = kG * kD / 4;                // float4 columns of all rows
    static constexpr int kParts = kThreads / kQuads;          // threads that share one
    static constexpr int kOwn = (kInlineSplits + kParts - 1) / kParts;      // ranges a thread adds up
    static_assert(kQuads <= kThreads, "one column per thread at most");
    float4 h;                                                 // head of range `lane`, row `wave`
    float4 x[kNeedO ? kOwn : 1];                              // this thread's columns of its ranges, top tokens included

    // First in the caller's queue: what follows (the caller's own loads) is not waited for.
    __device__ __forceinline__ void load(const float4 *__restrict__ part_head, const float *__restrict__ part_vec, int splits, int G) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        h = make_float4(-INFINITY, 0.f, __int_as_float(-1), 0.f);
        if (wave < kG && wave < G && lane < splits) h = part_head[(size_t)lane * kG + wave];
        if (!kNeedO) return;
        const int quad = threadIdx.x % kQuads, part = threadIdx.x / kQuads, row = quad * 4 / kD, col = quad * 4 % kD;
        const float *mine = part_vec + (size_t)row * 2 * kD + kD + col;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int s = part + i * kParts;
            x[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s < splits) x[i] = *(const float4 *)(mine + (size_t)s * kG * 2 * kD);
        }
    }
    __device__ __forceinline__ void merge(const float *__restrict__ part_vec, int splits, int G,
                                          const uint16_t *__restrict__ vg, float *fin);
};

template <int kG, int kD, bool kNeedO>
__device__ __forceinline__ void MergeFew<kG, kD, kNeedO>::merge(const float *__restrict__ part_vec, int splits, int G,
                                                                const uint16_t *__restrict__ vg, float *fin) {
    __shared__ float w_s[kG * kInlineSplits];
    __shared__ int best_s[kG];
    __shared__ __attribute__((aligned(16))) float sum_s[kNeedO ? kParts * kG * kD : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quad = threadIdx.x % kQuads, part = threadIdx.x / kQuads, row = quad * 4 / kD, col = quad * 4 % kD;
    const float *mine = part_vec + (size_t)row * 2 * kD + kD + col;         // sums that include the range's top token
    if (wave < kG && wave < G) {                              // one wave per row, one lane per range
        const int r = wave;
        const float bm = wave_reduce<MaxOp>(h.x);
        const int bs = __ffsll((unsigned long long)__ballot(h.x == bm)) - 1;    // the first range attaining the max holds
        const float w = h.x == -INFINITY ? 0.f : __expf(h.x - bm);              // the lowest token that does
        const float l = wave_reduce<SumOp>(fmaf(w, h.y, lane != bs ? w : 0.f));  // (other ranges count their top token)
        if (lane < splits) w_s[r * kInlineSplits + lane] = lane == bs ? 0.f : w;
        if (lane == bs) {
            best_s[r] = bs;
            float *rec = fin + r * kFs;
            rec[0] = bm;
            rec[1] = 1.f / (1.f + l);
            rec[2] = h.z;
            rec[3] = l;
        }
    }
    if (!kNeedO) return;                                      // (the caller meets at a barrier)
    __syncthreads();
    // the winning range's rows: its sums without its top token (weight 1), and that token's own row
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    uint2 vt = make_uint2(0u, 0u);
    const bool live = row < G;
    if (live && part == 0) {
        o = *(const float4 *)(mine - kD + (size_t)best_s[row] * kG * 2 * kD);
        vt = *(const uint2 *)(vg + (size_t)__float_as_int(fin[row * kFs + 2]) * kD + col);
    }
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (live) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const int s = part + i * kParts;
            const float w = s < splits ? w_s[row * kInlineSplits + s] : 0.f;
            if (w != 0.f) {                                   // (an empty range has no vectors)
                t.x = fmaf(w, x[i].x, t.x);
                t.y = fmaf(w, x[i].y, t.y);
                t.z = fmaf(w, x[i].z, t.z);
                t.w = fmaf(w, x[i].w, t.w);
            }
        }
        if (kParts > 1) *(float4 *)(sum_s + part * kG * kD + quad * 4) = t;
    }
    if (kParts > 1) __syncthreads();
    if (live && part == 0) {
#pragma unroll 8                                              // (all 63 of one row of 64 at once do not fit the registers)
        for (int i = 1; i < kParts; ++i) {
            const float4 y = *(const float4 *)(sum_s + i * kG * kD + quad * 4);
            t.x += y.x; t.y += y.y; t.z += y.z; t.w += y.w;
        }
        float *rec = fin + row * kFs;
        const float l = rec[3];
        merge_finish<kD>(l, t.x + o.x, __uint_as_float(vt.x << 16), col, rec);
        merge_finish<kD>(l, t.y + o.y, __uint_as_float(vt.x & 0xffff0000u), col + 1, rec);
        merge_finish<kD>(l, t.z + o.z, __uint_as_float(vt.y << 16), col + 2, rec);
        merge_finish<kD>(l, t.w + o.w, __uint_as_float(vt.y & 0xffff0000u), col + 3, rec);
    }
}

// Merge of many ranges: one workgroup per (row, KV head); up to kMergeOwn ranges per thread for
// the scalar part, then columns x segments of ranges for the vector part; fixed summation order.
template <int kG, int kD, bool kNeedO>
__global__ __launch_bounds__(kMergeThreads) void decode_merge(const uint16_t *__restrict__ v, int N, int splits,
                                                              const float4 *__restrict__ part_head_all,
                                                              const float *__restrict__ part_vec, float *__restrict__ fin) {
    constexpr int kSeg = kMergeThreads / kD;
    constexpr int kMergeWaves = kMergeThreads / 64;
    constexpr int kBatch = 8;
    __shared__ float w_s[kMaxSplits];
    __shared__ int top_s;
    __shared__ float red_m[kMergeWaves];
    __shared__ int red_a[kMergeWaves];
    __shared__ float red_l[kMergeWaves];
    __shared__ float red_o[kSeg * kD];
    const int r = blockIdx.x, bh = blockIdx.y;
    const float4 *part_head = part_head_all + (size_t)bh * splits * kG;
    const float *vec = part_vec + ((size_t)bh * splits * kG + r) * 2 * kD;
    const uint16_t *vg = v + (size_t)bh * N * kD;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    float hm[kMergeOwn], hl[kMergeOwn];
    int ht[kMergeOwn];
#pragma unroll
    for (int i = 0; i < kMergeOwn; ++i) {
        const int s = i * kMergeThreads + threadIdx.x;
        hm[i] = -INFINITY; hl[i] = 0.f; ht[i] = -1;
        if (s < splits) {
            const float4 h = part_head[(size_t)s * kG + r];
            hm[i] = h.x;
            hl[i] = h.y;
            ht[i] = __float_as_int(h.z);
        }
    }
    float bm = -INFINITY;
    int ba = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < kMergeOwn; ++i) take_better(bm, ba, hm[i], i * kMergeThreads + (int)threadIdx.x);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) take_better(bm, ba, __shfl_xor(bm, off), __shfl_xor(ba, off));
    if (lane == 0) { red_m[wave] = bm; red_a[wave] = ba; }
    __syncthreads();
    bm = red_m[0];
    ba = red_a[0];
#pragma unroll
    for (int w = 1; w < kMergeWaves; ++w) take_better(bm, ba, red_m[w], red_a[w]);
    const float m = bm;
    const int s_top = ba;                           // first range attaining the max: lowest token index

    float l = 0.f;
#pragma unroll
    for (int i = 0; i < kMergeOwn; ++i) {
        const int s = i * kMergeThreads + threadIdx.x;
        const float w = hm[i] == -INFINITY ? 0.f : __expf(hm[i] - m);
        if (s < splits) w_s[s] = w;
        if (s == s_top) top_s = ht[i];
        // ranges other than the winning one count their top token
        l += fmaf(w, hl[i], s != s_top ? w : 0.f);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
    if (lane == 0) red_l[wave] = l;
    __syncthreads();
    float l_rest = red_l[0];
#pragma unroll
    for (int x = 1; x < kMergeWaves; ++x) l_rest += red_l[x];
    const int top = top_s;

    const int c = threadIdx.x % kD, seg = threadIdx.x / kD;
    float v_top = 0.f;
    if (kNeedO) {
        if (seg == 0) v_top = bf16_bits_to_float(vg[(size_t)top * kD + c]);
        float o = 0.f;
        for (int s0 = seg; s0 < splits; s0 += kBatch * kSeg) {
            float po[kBatch], pw[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int si = s0 + u * kSeg;
                po[u] = 0.f; pw[u] = 0.f;
                if (si < splits && w_s[si] != 0.f) {
                    pw[u] = w_s[si];
                    po[u] = vec[(size_t)si * kG * 2 * kD + (si != s_top ? kD : 0) + c];
                }
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) o = fmaf(pw[u], po[u], o);
        }
        red_o[seg * kD + c] = o;
    }
    __syncthreads();
    if (seg == 0) {
        float *rec = fin + ((size_t)bh * kG + r) * final_stride(kD);
        if (kNeedO) {
            float o_rest = red_o[c];
#pragma unroll
            for (int x = 1; x < kSeg; ++x) o_rest += red_o[x * kD + c];
            merge_finish<kD>(l_rest, o_rest, v_top, c, rec);
        }
        if (c == 0) {
            rec[0] = m;
            rec[1] = 1.f / (1.f + l_rest);
            rec[2] = __int_as_float(top);
            rec[3] = l_rest;
        }
    }
}

template <int kVariant>
struct DecodeNeeds {
    static constexpr bool o = kVariant == OBC_KEY || kVariant == OBC_JOINT || kVariant == OBC_ALL;
    static constexpr bool v = kVariant != OBC_ATTN;
};

// Scores of the range's tokens from the stored logits, the merged row statistics and V.  With `lowest`, also the
// lowest (score, highest index) among each wave's tokens first <= p < len - tail, as an evict_candidate, and copies of the
// scores that begin a piece of evict_pieces.
template <int kG, int kD, int kSteps, int kVariant, typename Lens>
__global__ __launch_bounds__(kThreads) void decode_score(
    const uint16_t *__restrict__ v, int N, int G, int Hkv, int ragged, Lens lens, int splits,
    const float *__restrict__ z_buf, const float4 *__restrict__ part_head, const float *__restrict__ part_vec,
    const float *__restrict__ fin_global, int merge_here, float *__restrict__ scores, size_t plane_stride, int accumulate,
    unsigned long long *__restrict__ lowest, int first, int tail, float *__restrict__ edge_scores) {
    constexpr int kLpt = kD / 8;
    constexpr bool kNeedO = DecodeNeeds<kVariant>::o;
    constexpr bool kNeedV = DecodeNeeds<kVariant>::v;
    constexpr bool kDoV = kVariant == OBC_VALUE || kVariant == OBC_ALL;
    constexpr bool kDoK = kVariant == OBC_KEY || kVariant == OBC_ALL;
    constexpr bool kDoJ = kVariant == OBC_JOINT || kVariant == OBC_ALL;
    constexpr int kPlanes = kVariant == OBC_ALL ? 3 : 1;
    constexpr int kFs = final_stride(kD);
    __shared__ __attribute__((aligned(16))) float fin[kG * kFs];

    const int bh = blockIdx.x, b = bh / Hkv, split = blockIdx.y;
    const int len = seq_len_of(lens, ragged, b, N);
    const int t0 = split * kSteps * tokens_per_step(kD);
    const int t1 = min(t0 + kSteps * tokens_per_step(kD), N);
    const uint16_t *vg = v + (size_t)bh * N * kD;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = lane % kLpt, slot = lane / kLpt;
    float *out = scores + (size_t)bh * N;

    if (t0 >= len) {                                // only padding here
        if (lowest && threadIdx.x < kWaves) lowest[((size_t)bh * splits + split) * kWaves + threadIdx.x] = ~0ull;
        if (!accumulate) {
            for (int p = t0 + threadIdx.x; p < t1; p += kThreads) {
#pragma unroll
                for (int x = 0; x < kPlanes; ++x) out[x * plane_stride + p] = 0.f;
            }
        }
        return;
    }

    // Every load of the range up front; they are in flight while the ranges are merged.
    MergeFew<kG, kD, kNeedO> few;
    if (merge_here) few.load(part_head + (size_t)bh * splits * kG, part_vec + (size_t)bh * splits * kG * 2 * kD, splits, G);
    uint4 vw[kSteps];
    float z[kSteps][kG], old[kSteps][kPlanes];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        vw[u] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < kG; ++r) z[u][r] = 0.f;
#pragma unroll
        for (int x = 0; x < kPlanes; ++x) old[u][x] = 0.f;
        if (p < len) {
            if (kNeedV) vw[u] = *(const uint4 *)(vg + (size_t)p * kD + sub * 8);
            const float *zp = z_buf + ((size_t)bh * N + p) * kG;
#pragma unroll
            for (int r = 0; r < kG; ++r) z[u][r] = zp[r];
            if (accumulate && sub == 0) {
#pragma unroll
                for (int x = 0; x < kPlanes; ++x) old[u][x] = out[x * plane_stride + p];
            }
        }
    }

    if (merge_here) {
        few.merge(part_vec + (size_t)bh * splits * kG * 2 * kD, splits, G, vg, fin);
    } else {
        const float *src = fin_global + (size_t)bh * kG * kFs;
        for (int e = threadIdx.x; e < G * kFs; e += kThreads) fin[e] = src[e];
    }
    __syncthreads();

    // Rows outside, tokens inside: one row's constants and outputs at a time.
    float vv[kSteps][8], a_sum[kSteps], a2_sum[kSteps], k_sum[kSteps], j_sum[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        if (kNeedV) unpack8(vw[u], vv[u]);
        a_sum[u] = a2_sum[u] = k_sum[u] = j_sum[u] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < kG; ++r) {
        if (r >= G) continue;                                   // uniform
        const float m = fin[r * kFs], inv_l = fin[r * kFs + 1];
        const int top = __float_as_int(fin[r * kFs + 2]);
        float o[8];
        if (kNeedO) {
            const float4 lo = *(const float4 *)(fin + r * kFs + kRecHead + sub * 8), hi = *(const float4 *)(fin + r * kFs + kRecHead + sub * 8 + 4);
            o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w;
            o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
        }
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int p = token_of<kD>(t0, u, wave, slot);
            const float zz = z[u][r];
            const float a = p < len ? __expf(zz - m) * inv_l : 0.f;
            const float a2 = a * a;
            a_sum[u] += a;
            a2_sum[u] += a2;
            if (kNeedO) {
                float dlt[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) dlt[j] = vv[u][j] - o[j];
                if (p == top) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) dlt[j] = fin[r * kFs + kRecHead + kD + sub * 8 + j];
                }
                float dk = 0.f, dj = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (kDoK) dk = fmaf(dlt[j], dlt[j], dk);
                    if (kDoJ) {
                        const float t = fmaf(zz, dlt[j], vv[u][j]);
                        dj = fmaf(t, t, dj);
                    }
                }
                if (kDoK) k_sum[u] = fmaf(a2 * zz * zz, dk, k_sum[u]);
                if (kDoJ) j_sum[u] = fmaf(a2, dj, j_sum[u]);
            }
        }
    }

    unsigned long long low = ~0ull;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int p = token_of<kD>(t0, u, wave, slot);
        float s_v = 0.f, s_k = k_sum[u], s_j = j_sum[u], s_a = 0.f;
        if (kDoV) {
            float n2 = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) n2 = fmaf(vv[u][j], vv[u][j], n2);
            s_v = a2_sum[u] * n2;
        }
        if (kVariant == OBC_VATP) {
            float n1 = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) n1 += fabsf(vv[u][j]);
            s_a = a_sum[u] * n1;
        }
        if (kVariant == OBC_ATTN) s_a = a_sum[u];
        // per-lane pieces cover 8 of the d columns: add the pieces of the lanes sharing the token
        if (kDoV) s_v = group_sum<kLpt>(s_v);
        if (kDoK) s_k = group_sum<kLpt>(s_k);
        if (kDoJ) s_j = group_sum<kLpt>(s_j);
        if (kVariant == OBC_VATP) s_a = group_sum<kLpt>(s_a);
        if (sub == 0 && p < t1 && (p < len || !accumulate)) {   // padding: zeroed by a plain call, left alone by an accumulating one
            if (kVariant == OBC_ALL) {
                out[p] = old[u][0] + s_v;
                out[plane_stride + p] = old[u][kPlanes > 1 ? 1 : 0] + s_k;
                out[2 * plane_stride + p] = old[u][kPlanes > 2 ? 2 : 0] + s_j;
            } else {
                const float sc = kVariant == OBC_VALUE ? s_v : kVariant == OBC_KEY ? s_k
                               : kVariant == OBC_JOINT ? s_j : s_a;
                const float now = old[u][0] + sc;
                out[p] = now;
                if (lowest && p % kEvictPiece == 0) edge_scores[(size_t)bh * evict_score_pieces(N) + p / kEvictPiece] = now;
                if (p >= first && p < len - tail) {
                    const unsigned long long cand = evict_candidate(now, p);
                    low = cand < low ? cand : low;
                }
            }
        }
    }
    if (lowest) {                                               // uniform; one candidate per wave
        if (kLpt == 8) low = min64(low, dpp_pair<0x128>(low));
        low = across_rows<Min64Op>(low);                        // (only lanes with sub == 0 have one: those of lane 0's place)
        if (lane == 0) lowest[((size_t)bh * splits + split) * kWaves + wave] = low;
    }
}

template <int kG, int kD, int kSteps, int kVariant, typename Lens>
hipError_t launch_decode_steps(const ScoreArgs &a, const Lens &lens, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    constexpr bool kNeedO = DecodeNeeds<kVariant>::o;
    const int BH = a.B * a.Hkv;
    float *z_buf = (float *)(base + ws.dec_z);
    float4 *part_head = (float4 *)(base + ws.dec_head);
    float *part_vec = (float *)(base + ws.dec_vec);
    float *fin = (float *)(base + ws.dec_final);
    // (KV head fastest: the workgroups of a head then share an XCD, and its L2 the head's rows and records, where the
    // head count allows)
    const dim3 grid(BH, ws.dec_splits);
    if (ws.dec_splits > kMaxSplits || (long long)ws.dec_splits * kSteps * tokens_per_step(kD) < a.N) return hipErrorInvalidValue;
    if (a.stage_mask & OBC_STAGE_SWEEP1) {
        const auto partial = a.find_lowest ? decode_partial<kG, kD, kSteps, kNeedO, kVariant != OBC_ALL, Lens> : decode_partial<kG, kD, kSteps, kNeedO, false, Lens>;
        partial<<<grid, dim3(kThreads), 0, stream>>>(
            (const uint16_t *)a.q, (const uint16_t *)a.k, (const uint16_t *)a.v, a.N, a.G, a.Hkv, a.ragged, lens,
            ws.dec_splits, z_buf, part_head, part_vec, a.edges.rows);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if ((a.stage_mask & OBC_STAGE_COMBINE) && !ws.dec_merge_inline) {
        decode_merge<kG, kD, kNeedO><<<dim3(a.G, BH), dim3(kMergeThreads), 0, stream>>>((const uint16_t *)a.v, a.N, ws.dec_splits,
                                                                                        part_head, part_vec, fin);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.stage_mask & OBC_STAGE_SWEEP2) {
        decode_score<kG, kD, kSteps, kVariant><<<grid, dim3(kThreads), 0, stream>>>(
            (const uint16_t *)a.v, a.N, a.G, a.Hkv, a.ragged, lens, ws.dec_splits, z_buf, part_head, part_vec, fin,
            ws.dec_merge_inline, a.scores, (size_t)a.B * a.Hkv * a.N, a.accumulate,
            a.find_lowest ? (unsigned long long *)(base + ws.dec_lowest) : nullptr, a.evict_first, a.evict_tail,
            a.edges.scores);
        return hipGetLastError();
    }
    return hipSuccess;
}

template <int kG, int kD, int kVariant>
hipError_t launch_decode_variant(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    return with_lens(a.ragged, a.B, a.lens, [&](const auto &lens) {
        switch (ws.dec_range / tokens_per_step(kD)) {
            case 1: return launch_decode_steps<kG, kD, 1, kVariant>(a, lens, ws, base, stream);
            case 2: return launch_decode_steps<kG, kD, 2, kVariant>(a, lens, ws, base, stream);
            default: return launch_decode_steps<kG, kD, 4, kVariant>(a, lens, ws, base, stream);
        }
    });
}

template <int kG, int kD>
hipError_t launch_decode_rows(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    switch (a.variant) {
        case OBC_VALUE: return launch_decode_variant<kG, kD, OBC_VALUE>(a, ws, base, stream);
        case OBC_KEY: return launch_decode_variant<kG, kD, OBC_KEY>(a, ws, base, stream);
        case OBC_JOINT: return launch_decode_variant<kG, kD, OBC_JOINT>(a, ws, base, stream);
        case OBC_ATTN: return launch_decode_variant<kG, kD, OBC_ATTN>(a, ws, base, stream);
        case OBC_VATP: return launch_decode_variant<kG, kD, OBC_VATP>(a, ws, base, stream);
        default: return launch_decode_variant<kG, kD, OBC_ALL>(a, ws, base, stream);
    }
}

template <int kD>
hipError_t launch_decode_dim(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    switch (ws.dec_rows) {
        case 1: return launch_decode_rows<1, kD>(a, ws, base, stream);
        case 2: return launch_decode_rows<2, kD>(a, ws, base, stream);
        case 4: return launch_decode_rows<4, kD>(a, ws, base, stream);
        default: return launch_decode_rows<8, kD>(a, ws, base, stream);
    }
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

int splits_for(int N, int d, int steps) { return (N + steps * tokens_per_step(d) - 1) / (steps * tokens_per_step(d)); }

}  // namespace

bool decode_path_covers(int B, int N, int W, int Hq, int Hkv, int d, int dtype, int variant, bool any_size) {
    if (dtype != OBC_BF16 || W != 1 || Hq / Hkv > kDecodeMaxGroup || (d != 64 && d != 128)) return false;
    if (splits_for(N, d, kMaxSteps) > kMaxSplits) return false;            // what one merging workgroup takes
    // These kernels win while the call is bound by round trips.  On long caches the direct forms
    // of the norms make them vector-ALU bound and the matrix-core path is faster, the sooner the more rows.  An accumulating call's
    // time there over its time here, 4 x 8 heads:
    //              joint, 49K head-tokens  98K   180K  262K      value, 129K   262K  500K
    //      G = 1          1.60             1.29  1.13  0.92             1.29   0.96  0.95
    //      G = 4          1.27             0.94  0.82  0.69             1.22   0.94  0.91
    //      G = 8          0.98             0.70  0.62  0.53             0.94   0.71  0.68
    // An eviction step there has evict_pick and evict_shift behind it: joint, 98K, 1.41 / 1.14 / 0.92, of one sequence of 8 heads
    // 2.15 / 1.71 / 1.37.  One line for all G and for both, between the two.
    const bool need_o = variant == OBC_KEY || variant == OBC_JOINT || variant == OBC_ALL;
    const long long head_tokens = (long long)B * Hkv * N;
    return any_size || d != 128 || head_tokens <= (need_o ? 98304 : 262144);   // (head_dim 64 has no matrix-core path)
}

void decode_plan(int B, int N, int Hq, int Hkv, int d, ScoreWorkspace *ws, size_t *off) {
    const int G = Hq / Hkv;
    const int BH = B * Hkv;
    // The shortest ranges with at most one workgroup per compute unit, and no shorter ones than the inline merge can take.  Two would
    // fit (decode_partial has 64 registers and 77 KB of LDS at most, decode_score 62 registers up to four rows), but a second one costs more than twice the tokens per lane: a decoding
    // step of 8 heads, d = 128, joint, G = 1 / 4 / 8, us, with one, two and four tokens per lane: 2100 tokens (264 workgroups with one)
    // 16.2 / 19.5 / 27.3, 15.5 / 18.0 / 22.5 and 17.7 / 21.9 / 28.3; 2 x 1900 (480) 18.0 / 21.3 / 29.6, 17.7 / 20.1 / 24.5 and 19.4 / 23.6 / 30.0;
    // within one round 1600 tokens (200) 13.6 / 15.1 / 18.5, 14.3 / 16.7 / 21.1 and 16.6 / 20.7 / 27.1.
    int steps = 1;
    while (steps < kMaxSteps && ((long long)BH * splits_for(N, d, steps) > 256 || splits_for(N, d, steps) > kInlineSplits)) steps *= 2;
    const int splits = splits_for(N, d, steps);
    ws->dec_rows = G <= 1 ? 1 : G <= 2 ? 2 : G <= 4 ? 4 : 8;
    ws->dec_range = steps * tokens_per_step(d);
    ws->dec_splits = splits;
    ws->dec_merge_inline = splits <= kInlineSplits ? 1 : 0;
    const size_t records = (size_t)BH * splits * ws->dec_rows;
    ws->dec_z = *off;      *off = align256(*off + (size_t)BH * N * ws->dec_rows * sizeof(float));
    ws->dec_head = *off;   *off = align256(*off + records * sizeof(float4));
    ws->dec_vec = *off;    *off = align256(*off + records * 2 * d * sizeof(float));
    ws->dec_final = *off;  *off = align256(*off + (size_t)BH * ws->dec_rows * final_stride(d) * sizeof(float));
    ws->dec_lowest = *off; *off = align256(*off + (size_t)BH * splits * kWaves * sizeof(unsigned long long));
    ws->dec_lowest_per_head = splits * kWaves;
    ws->score_need = *off;
    ws->dec_edges = *off;       *off = align256(*off + (size_t)BH * 2 * evict_row_pieces(N, d) * d * sizeof(uint16_t));
    ws->dec_edge_scores = *off; *off = align256(*off + (size_t)BH * evict_score_pieces(N) * sizeof(float));
}

hipError_t launch_score_decode(const ScoreArgs &a, const ScoreWorkspace &ws, char *base, hipStream_t stream) {
    return a.d == 128 ? launch_decode_dim<128>(a, ws, base, stream) : launch_decode_dim<64>(a, ws, base, stream);
}

}  // namespace obc
