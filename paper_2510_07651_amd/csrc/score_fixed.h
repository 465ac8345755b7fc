// Part of score_plain.hip: its kernels for more than 32 window rows per KV head, and for more than 16 where sweeps_digits says so.
//
// The fp64 matrix cores do 79 TFLOP/s and the fp32 ones 157, the 8-bit integer ones 5000 and the bf16 ones 2500, so
// contractions whose accuracy allows it are taken apart into pieces the fast ones multiply exactly.
//
// Logits (digit_sweep).  Rows of q and k as fixed point relative to their largest element, fp32 values 46 bits and a sign in
// six balanced base-256 digits, bf16 values 30 bits in four, which hold their elements exactly down to 2^-23 of the row's
// largest.  Products of digits are summed exactly in 32-bit integers, for the seven highest of the levels (all of four by
// four digits).  Fixed point alone cannot stand in for fp64: where a key has a large element that meets a small one of the
// query, the digits that are left out are those the logit is made of.  So a wave whose 16 x 16 pairs have a dot product that
// the digits may miss by more than 2^-27 of it (its rounding to fp32 is 2^-25 to 2^-24) forms them in fp64 as blocked_logits
// does.  With 2^E for the product of the powers of two just above the rows' largest elements and d <= 128:
//   the levels left out are at most d (4 * 2^14 * 2^24 + 3 * 2^14 * 2^16 + ..) 2^-92 = 2^-45 (fp32 only), what join_seven cuts
//   off is 2^-50: 2^-27.9 of an fp32 dot product from 2^-17 2^E up, 2^-28 of a bf16 one from 2^-22 2^E up (kLeastDot);
//   an fp32 row with an element below 2^-23 of its largest may have it cut off: by up to 2^-47 of the row's power of two per
//   element, 2^-40 2^E per dot product and side, 2^-27 of it from 2^-12 2^E up (kLeastDotCut, for the blocks with such a row
//   in their tile or their window rows).  Normal rows: one in 30000;
//   bf16 rows with such elements, infinities, NaN: fp64 always.
// Rows of zeros, keys as padding leaves them and the zeros past a sequence's end among them, are held exactly and pass the test.
// Of normal keys with channels larger by 8, 0.5 % of the blocks go to fp64.  A block that goes that way does both, and fetches its
// operands from memory again: whole calls, joint, us, ordinary inputs / every block in fp64 (key channels 2^26 larger that meet query
// channels as much smaller) / fp32 keys that are all cut, and with blocked_logits:
//   fp32, d = 128,  8 heads x 128 rows x  8111 tokens    97 / 146 / 112    114      1500 tokens    39.1 / 48.7 / 42.6    40.7
//   fp32, d = 128, 32 heads x 256 rows x  8111 tokens   636 / 987 / 731   1114
//   fp32, d =  64, 16 heads x 160 rows x 16000 tokens   313 / 449 / 366    340
//   bf16, d =  64,  8 heads x 128 rows x 16384 tokens    84 / 130          108      1500 tokens    25.0 / 31.1           31.4
// (a key of zeros among every sixteen cost about the same as the second figures before such rows passed, and next to nothing now: 97.9,
// 40.3, 634, 319, 84.8, 25.3 us).
// (Without the digits while a wave's blocks go to fp64 one after the other, and with four of their loads in flight, such calls took 2
// to 8 % less: what they cost is the fp64 products themselves, at a wave's own pace from memory.)
// Which calls digit_sweep takes: sweeps_digits (score_plain.hip).
//
// v_p . o_i (fixed_score).  Each row of v and o is scaled by a power of two to fixed point, 38 bits and a sign relative to
// the row's largest element (30 for bf16 values, whose elements have 8 significant bits), and written as five (four)
// balanced base-256 digits, |digit| <= 128.  Products of digits are summed exactly in 32-bit integers; pairs of digits
// beyond the fifth level are left out, and the levels are put together in fp64.  With 2^E for the product of the powers of
// two just above the rows' largest elements, the arithmetic in a CPU model is off by 2^-35 2^E (rms, 2^-33 at most over
// millions of pairs: normal elements, channels larger than the others by up to 2^26, elements over 20 binades; there bf16
// values, which keep fewer bits, reach 2^-30).  The norms it goes into are as good as an fp32 rounding where they are above
// 2^-4 2^E; where a pair that counts has a smaller one (a v_p that is nearly o_i), the wave forms its 16 x 16 dot products
// again in fp64 (block_dots), from where on they are what plain_score computes.
// Sums in fp32 cannot stand in for this: with three bf16 pieces each, six products and three accumulators on the bf16 matrix cores the
// kernel took 28 / 32 us instead of 30 / 40 (fp32, d = 128, 8111 tokens / bf16, d = 64, 16384), but where values share a large channel a
// rounding of v . o is 32 times that in a distance just above the line: errors of single distances, some 10^3 tokens that share a channel
// of 2.75 sqrt(d), were 6e-7 rms and 1.3e-6 to 2.9e-6 at most, with digits 1e-7 and 3e-7 to 4e-7.
//
// P V (weights_pv).  Weights and fp32 values as three bf16 pieces each, all nine products (exact, normal numbers), fp32
// accumulation: per 32 tokens nine bf16 ops (three for bf16 values) of 16 cycles replace eight fp32 ones of 32.
// The outputs are as good as those of the fp32 ops: key scores of values that differ by 2^-6 (2^-9) of their norm, where the
// outputs' error is what shows, are off by 1.0e-6 (8.6e-6) in the 2-norm, with plain_weights by 1.1e-6 (8.7e-6); fp32,
// d = 128, 8111 tokens.
//
// What bounds them.  blocked_logits: the fp64 matrix cores, busy 64 % of the kernel.  digit_sweep: vector ALUs and matrix cores, a wave
// using one after the other (some 18 instructions put a pair's levels together, check and scale them, some 9 take an element apart, some
// 20 make its weight and the weight's pieces), all four waves of a SIMD at the same stage, and waits, half of the waves' time: with
// 7 % fewer vector instructions (maxima by blocks of tokens, weights' pieces by dot products) it took as long, as it did without a
// branch per weight and with the matrix phases at a higher wave priority.  fixed_score: the vector ALUs, 75 instructions per 64
// pairs (55 for bf16 values): putting a dot product together about 10, its weight 10, the norms and the closeness test 13, mostly in
// fp64, and taking an element apart about 15 (7 for bf16), paid once per workgroup of up to 128 rows; matrix cores busy 27 %.  The
// blocks in which a row's view ends or its top stands, few, have code of their own: in the others no pair is masked.  With that, the
// token's and the row's share of the closeness test multiplied in fp32, the sums over the rows in half as many steps and a
// record of 40 bytes (eight more instructions per 64 pairs, and banks met twice, before) 38.6 -> 34.7 us (bf16, d = 64, 16384) and
// 29.5 -> 28.2 (fp32, d = 128, 8111).
// Kernel times, 32/8 heads, joint, two sets of inputs in turn, in us: digit_sweep (as two kernels, logits / weights) / merge / scores
//   fp32, d = 128,  8111 tokens   59.9 (37.2 / 28.2) / 8.6 / 28.2
//   bf16, d = 64,  16384 tokens   48.0 (29.3 / 23.3) / 6.0 / 34.7
// Two kernels met between them: the maxima of all ranges first.  Whole calls, blocked_logits and fixed_weights / digit_sweep (with as many
// splits as fill the chip where the calls' heads pass in several launches), joint, inputs that change from call to call, us:
//   fp32, d = 128, 4 x 8 heads x 128 rows x 8000   406 / 317     bf16, d = 64, 8 x 8 heads x 128 rows x 3000   188 / 140
//   fp32, d = 128, 1 head x 128 rows x 60000       194 / 125     bf16, d = 64, 8 heads x 48 rows x 16384      64.1 / 52.1
//   fp32, d =  64, 8 heads x 512 rows x 6000       220 / 177     fp32, d = 128, 8 heads x 128 rows x 8111      115 / 97
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

template <typename T> constexpr int kDigits = sizeof(T) == 4 ? 5 : 4;
constexpr int kRowDigits = 5;                  // of o_i, which is fp32 whatever the inputs are
constexpr int kLevels = 5;
template <typename T> constexpr int kLogitDigits = sizeof(T) == 4 ? 6 : 4;
constexpr int kLogitLevels = 7;
// Least dot products that the digits give, in units of join_seven: of rows that they hold, and of fp32 rows that they cut.
template <typename T> constexpr double kLeastDot = sizeof(T) == 4 ? 0x1p34 : 0x1p29;
constexpr double kLeastDotCut = 0x1p39;

// A wave has 16 window rows: the rows' digits and a block's sums fit 128 registers, so that four waves share a SIMD and hide
// each other's latencies (with 32 rows per wave and two waves weights and scores took 37 and 43 us where 29 and 36 then were
// left: fp32, d = 128, 8111 tokens).
// kRb = 8 puts 128 rows into a workgroup; kRb = 4 puts 64 and gives its waves different parts of a token tile.
constexpr int kFixedThreads = 512, kWeightThreads = 1024;
template <int D> constexpr int kFixedTile = D == 64 ? 64 : 32;           // tokens

// Layouts in memory, such that a wave reads and writes whole kilobytes (a lane has one row; rows side by side in memory would
// make every lane's 16 bytes a line of their own: 64 cache accesses instead of 8).
//   z       z_block (plain_layout.h)
//   digits  [head][row / 16][digit][element / 64][element % 64 / 16][row % 16][element % 16]
template <int K, int D>
__device__ __forceinline__ size_t digit_address(size_t block, int k, int row, int c) {
    return ((block * K + k) * (D / 64) + c / 64) * 1024 + (c % 64 / 16 * 16 + row % 16) * 16 + c % 16;
}

// Largest |x|, as bits: integers order them like the numbers and put what is not a number on top.
struct MaxBitsOp { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; } };
__device__ __forceinline__ uint32_t max_abs(const float (&x)[4]) {
    const float m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(x[0]), fabsf(x[1])),
                                                  __builtin_elementwise_maximum(fabsf(x[2]), fabsf(x[3])));
    return __float_as_uint(m) & 0x7fffffffu;
}
// Exponent e with |x|max < 2^e.
__device__ __forceinline__ int max_exponent(uint32_t amax) { return (int)(amax >> 23) - 126; }
// A row's share of the unit of a dot product, 2^(e - 18); NaN where an element was infinite or not a number.
__device__ __forceinline__ double row_unit(int e) { return e > 128 ? __longlong_as_double(0x7ff8000000000000ll) : ldexp(1.0, e - 18); }
// Its share of the least norm that the digits are good for, 2^-4 2^E (fp32 holds it, as a subnormal number at worst).
__device__ __forceinline__ float least_share(double unit) { return (float)(unit * 0x1p16); }

// The last four planes of digits from four words whose bytes are digits plus 128.
template <int K>
__device__ __forceinline__ void byte_planes(const uint32_t (&w)[4], uint32_t (&plane)[K]) {
    const uint32_t t0 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602), t1 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602);
    const uint32_t u0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400), u1 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400);
    plane[K - 4] = __builtin_amdgcn_perm(t1, t0, 0x07060302) ^ 0x80808080u;
    plane[K - 3] = __builtin_amdgcn_perm(t1, t0, 0x05040100) ^ 0x80808080u;
    plane[K - 2] = __builtin_amdgcn_perm(u1, u0, 0x07060302) ^ 0x80808080u;
    plane[K - 1] = __builtin_amdgcn_perm(u1, u0, 0x05040100) ^ 0x80808080u;
}
// The digits of four elements, most significant first, one byte per element.  The sum with 1.5 * 2^52 rounds to the
// fixed-point integer and leaves it in the low bits; 128 added to every digit makes its bytes the digits plus 128.
template <int K>          // 4, 5 or 6
__device__ __forceinline__ void digits_of(const double (&x)[4], int e, uint32_t (&plane)[K]) {
    const double scale = __hiloint2double((1023 + 8 * K - 2 - e) << 20, 0);
    const double bias = 6755399441055744.0 + (K == 6 ? (double)0x808080808080ll : K == 5 ? (double)0x8080808080ll : (double)0x80808080ll);
    uint32_t w[4], top[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double t = fma(x[i], scale, bias);
        w[i] = (uint32_t)__double2loint(t);
        top[i] = (uint32_t)__double2hiint(t);
    }
    byte_planes<K>(w, plane);
    if (K >= 5)
        plane[K - 5] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(top[3], top[2], 0x0c0c0400),
                                             __builtin_amdgcn_perm(top[1], top[0], 0x0c0c0400), 0x05040100) ^ 0x80808080u;
    if (K == 6)
        plane[0] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(top[3], top[2], 0x0c0c0501),
                                         __builtin_amdgcn_perm(top[1], top[0], 0x0c0c0501), 0x05040100) ^ 0x80808080u;
}

// x . y of the two fixed-point vectors from the level sums, in units of row_unit(ex) row_unit(ey).
__device__ __forceinline__ double join_levels(int l0, int l1, int l2, int l3, int l4) {
    const int hi = (l0 << 8) + l1, lo = (l2 << 8) + l3 + (l4 >> 8);      // (at most 2^27 and 2^31: |digit| <= 128, the first one <= 64)
    return fma((double)hi, 65536.0, (double)lo);
}

// The same from the seven levels of a logit, in units of 2^(E - 51); what is cut off is less than two of them.
template <int K>
__device__ __forceinline__ double join_seven(int l0, int l1, int l2, int l3, int l4, int l5, int l6) {
    const int hi = (l0 << 8) + l1, mid = (l2 << 8) + l3;                 // (at most 2^27 and 2^30, as is lo)
    const int lo = (l4 << 7) + (K == 4 ? ((l5 << 8) + l6) >> 9 : (l5 + (l6 >> 8)) >> 1);
    return fma(fma((double)hi, 65536.0, (double)mid), 32768.0, (double)lo);
}
// Exponents of a row whose elements the digits of a logit cannot hold, and of a row of zeros, whose dot products are 0 exactly
// (with the one: more than kNoExponent / 2, with any other: nothing that ldexp makes of a 0).
constexpr int kNoExponent = 1 << 20, kZeroExponent = -4096;
__device__ __forceinline__ int logit_exponent(uint32_t amax) {
    return amax >= 0x7f800000u ? kNoExponent : amax == 0u ? kZeroExponent : max_exponent(amax);
}
// What four elements below 2^e have below the digits' bits, above zero if anything (but for what falls below fp32's range here:
// 2^-149 of a unit and less).
template <int K>
__device__ __forceinline__ float below_digits(const float (&y)[4], int e, float cut) {
#pragma unroll
    for (int i = 0; i < 4; ++i) cut = fmaxf(cut, __builtin_amdgcn_fractf(__builtin_amdgcn_ldexpf(y[i], 8 * K - 2 - e)));
    return cut;
}
// Digits of elements below 2^e.  bf16 values: as integers of 30 bits, and `cut` is above zero where one has bits below those.
template <typename T, int K>
__device__ __forceinline__ void logit_digits(const float (&y)[4], int e, uint32_t (&plane)[K], float &cut) {
    if constexpr (sizeof(T) == 4) {
        const double yd[4] = {y[0], y[1], y[2], y[3]};
        digits_of<K>(yd, e, plane);
    } else {
        static_assert(K == 4, "30 bits and a sign");
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float t = __builtin_amdgcn_ldexpf(y[i], 30 - e);
            cut = fmaxf(cut, __builtin_amdgcn_fractf(t));
            w[i] = (uint32_t)(int)t + 0x80808080u;
        }
        byte_planes<K>(w, plane);
    }
}

// Rows of digits in LDS, kTok rows x K planes of D bytes.  A row's 16-byte piece c sits at slot c ^ f(row), so that the 16
// lanes of a read (same piece of 16 consecutive rows) touch every bank once.
template <int D, int kTok>
__device__ __forceinline__ int digit_offset(int plane, int row, int c) {
    const int slot = D == 128 ? c ^ (row >> 1 & 7) : c ^ (row >> 2 & 3);
    return (plane * kTok + row) * D + slot * 16;
}

// A span of memory by its bounds: loads beyond its end give zeros.  (One 32-bit address per lane instead of two words per
// load; the workspace's cap keeps a workgroup's span far below 4 GB.)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t span_of(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00027000);
}

// ------------------------------------------------------------------------------------
// Token tiles: kTok rows of k or v on their way from memory into LDS.
// ------------------------------------------------------------------------------------
template <typename T, int D, int kTok, int kTileThreads>
struct TokenTile {
    static constexpr int kPer = 16 / (int)sizeof(T);                     // elements of a 16-byte piece
    static constexpr int kLanes = D / kPer;                              // lanes per row
    static constexpr int kCount = kTok * kLanes / kTileThreads;
    static_assert(kTok * kLanes % kTileThreads == 0, "whole pieces per thread");
    static constexpr int kStep = kTileThreads / kLanes;                  // rows from one piece of a thread to its next
    static_assert(kStep % 16 == 0, "the swizzles repeat every 16 rows");
    uint4 x[kCount];

    // Rows from row t of the span; rows beyond its end become zeros.
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t span, int t) {
        int thread = threadIdx.x;
        asm volatile("" : "+v"(thread));                     // (addresses anew for every tile: registers)
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(span, (t * kLanes + thread + i * kTileThreads) * 16, 0, 0);
            x[i] = make_uint4(u.x, u.y, u.z, u.w);
        }
    }
    __device__ __forceinline__ void unpack(int i, float (&y)[kPer / 4][4]) const {
        if constexpr (sizeof(T) == 4) {
            y[0][0] = __uint_as_float(x[i].x); y[0][1] = __uint_as_float(x[i].y);
            y[0][2] = __uint_as_float(x[i].z); y[0][3] = __uint_as_float(x[i].w);
        } else {
            y[0][0] = __uint_as_float(x[i].x << 16); y[0][1] = __uint_as_float(x[i].x & 0xffff0000u);
            y[0][2] = __uint_as_float(x[i].y << 16); y[0][3] = __uint_as_float(x[i].y & 0xffff0000u);
            y[1][0] = __uint_as_float(x[i].z << 16); y[1][1] = __uint_as_float(x[i].z & 0xffff0000u);
            y[1][2] = __uint_as_float(x[i].w << 16); y[1][3] = __uint_as_float(x[i].w & 0xffff0000u);
        }
    }
    // Over the lanes of a row.
    template <typename Op, typename F>
    static __device__ __forceinline__ F over_row(F v) {
        const Op op;
        v = op(v, dpp_pair<0xB1>(v));
        v = op(v, dpp_pair<0x4E>(v));
        v = op(v, dpp_pair<0x141>(v));
        if (kLanes >= 16) v = op(v, dpp_pair<0x140>(v));
        if (kLanes == 32) {
            F a, b;
            both_of_pair<16>(v, a, b);
            v = op(a, b);
        }
        return v;
    }
    // The digits of digit_sweep and the rows' exponents into LDS; fp32: also whether elements of the wave's rows were cut.
    template <int K>
    __device__ __forceinline__ void store_logit_digits(char *digits, int *exponents, uint8_t *cut_s) const {
        int thread = threadIdx.x;
        asm volatile("" : "+v"(thread));                     // (addresses anew for every tile: registers)
        const int r0 = thread / kLanes, c = thread % kLanes;
        char *dst = digits + digit_offset<D, kTok>(0, r0, c * kPer / 16) + c * kPer % 16;
        bool any_cut = false;                                // uniform
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            __builtin_amdgcn_sched_barrier(0);               // (one piece at a time: registers)
            float y[kPer / 4][4];
            unpack(i, y);
            uint32_t amax = max_abs(y[0]);
            if (kPer == 8) amax = MaxBitsOp()(amax, max_abs(y[kPer / 4 - 1]));
            amax = over_row<MaxBitsOp>(amax);
            uint32_t p[kPer / 4][K];
            float cut = 0.f;
#pragma unroll
            for (int q = 0; q < kPer / 4; ++q) logit_digits<T>(y[q], max_exponent(amax), p[q], cut);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                char *at = dst + (k * kTok + i * kStep) * D;
                if constexpr (kPer == 4) *(uint32_t *)at = p[0][k];
                else *(uint2 *)at = make_uint2(p[0][k], p[1][k]);
            }
            if (c == 0) exponents[r0 + i * kStep] = logit_exponent(amax);
            if constexpr (sizeof(T) == 4) {
                // (elements from 2^(e - 23) up are held; one below that, or a zero, is rare: in 1 of 10000 waves for normal ones)
                const float least = __builtin_elementwise_minimum(__builtin_elementwise_minimum(fabsf(y[0][0]), fabsf(y[0][1])),
                                                                  __builtin_elementwise_minimum(fabsf(y[0][2]), fabsf(y[0][3])));
                const int e = max_exponent(amax);
                if (__builtin_amdgcn_ballot_w64(least < __builtin_amdgcn_ldexpf(1.f, e - 23)) != 0ull)
                    any_cut |= __builtin_amdgcn_ballot_w64(below_digits<K>(y[0], e, 0.f) > 0.f) != 0ull;
            } else if (__builtin_amdgcn_ballot_w64(cut > 0.f) != 0ull) {     // uniform, rare; a row's lanes are in one wave
                if (cut > 0.f) *(volatile int *)(exponents + r0 + i * kStep) = kNoExponent;
            }
        }
        if (sizeof(T) == 4 && threadIdx.x % 64 == 0) cut_s[threadIdx.x / 64] = any_cut;
    }
    // Digits, units and their shares of a closeness test into LDS and, where asked for, the rows' norms: ||v||^2 (2) or ||v||_1 (1).
    template <bool kWithDigits, int kNorm>
    __device__ __forceinline__ void store_digits(char *digits, double *units, float *least, double *norms) const {
        constexpr int K = kDigits<T>;
        int thread = threadIdx.x;
        asm volatile("" : "+v"(thread));                     // (addresses anew for every tile: registers)
        const int r0 = thread / kLanes, c = thread % kLanes;
        char *dst = digits + digit_offset<D, kTok>(0, r0, c * kPer / 16) + c * kPer % 16;
#pragma unroll
        for (int i = 0; i < kCount; ++i) {
            __builtin_amdgcn_sched_barrier(0);               // (one piece at a time: registers)
            float y[kPer / 4][4];
            unpack(i, y);
            double yd[kPer / 4][4];
#pragma unroll
            for (int q = 0; q < kPer / 4; ++q)
#pragma unroll
                for (int k = 0; k < 4; ++k) yd[q][k] = y[q][k];
            if constexpr (kWithDigits) {
                uint32_t amax = max_abs(y[0]);
                if (kPer == 8) amax = MaxBitsOp()(amax, max_abs(y[kPer / 4 - 1]));
                const int e = max_exponent(over_row<MaxBitsOp>(amax));
                uint32_t p[kPer / 4][K];
#pragma unroll
                for (int q = 0; q < kPer / 4; ++q) digits_of<K>(yd[q], e, p[q]);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    char *at = dst + (k * kTok + i * kStep) * D;
                    if constexpr (kPer == 4) *(uint32_t *)at = p[0][k];
                    else *(uint2 *)at = make_uint2(p[0][k], p[1][k]);
                }
                if (c == 0) {
                    units[r0 + i * kStep] = row_unit(e);
                    least[r0 + i * kStep] = least_share(row_unit(e));
                }
            }
            if (kNorm != 0) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < kPer / 4; ++q)
#pragma unroll
                    for (int k = 0; k < 4; ++k) s = kNorm == 2 ? fma(yd[q][k], yd[q][k], s) : s + fabs(yd[q][k]);
                s = over_row<SumOp>(s);
                if (c == 0) norms[r0 + i * kStep] = s;
            }
        }
    }
};

// A wave's 16 rows of digits as a matrix operand: lane = row + 16 g holds bytes 16 g .. 16 g + 15 of every 64.
template <int K, int D>
struct RowDigits {
    i32x4 x[K][D / 64];
    __device__ __forceinline__ void load(const int8_t *__restrict__ digits, int hl, int block, int blocks, int lane) {
        const __amdgpu_buffer_rsrc_t span = span_of(digits + digit_address<K, D>((size_t)hl * blocks, 0, 0, 0), (size_t)blocks * 16 * K * D);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int kk = 0; kk < D / 64; ++kk)
                x[k][kk] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                         span, (int)digit_address<K, D>(block, k, 0, kk * 64) + lane * 16, 0, 0));
    }
    // Digits of a row itself, for digit_sweep; returns the row's exponent.  fp32: `any_cut`, whether elements of the wave's
    // rows were cut.
    template <typename T>
    __device__ __forceinline__ int take(const T *__restrict__ row, int g, bool &any_cut) {
        float y[D / 64][4][4];
#pragma unroll
        for (int kk = 0; kk < D / 64; ++kk) {
            const T *src = row + kk * 64 + 16 * g;
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float4 f = *(const float4 *)(src + 4 * c);
                    y[kk][c][0] = f.x; y[kk][c][1] = f.y; y[kk][c][2] = f.z; y[kk][c][3] = f.w;
                }
            } else {
#pragma unroll
                for (int c = 0; c < 4; c += 2) {
                    const uint4 h = *(const uint4 *)(src + 4 * c);
                    const uint32_t u[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        y[kk][c + i / 2][i % 2 * 2] = __uint_as_float(u[i] << 16);
                        y[kk][c + i / 2][i % 2 * 2 + 1] = __uint_as_float(u[i] & 0xffff0000u);
                    }
                }
            }
        }
        uint32_t amax = 0u;
#pragma unroll
        for (int kk = 0; kk < D / 64; ++kk)
#pragma unroll
            for (int c = 0; c < 4; ++c) amax = MaxBitsOp()(amax, max_abs(y[kk][c]));
        amax = across_rows<MaxBitsOp>(amax);
        float cut = 0.f;
#pragma unroll
        for (int kk = 0; kk < D / 64; ++kk)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t p[K];
                if (sizeof(T) == 4) cut = below_digits<K>(y[kk][c], max_exponent(amax), cut);
                logit_digits<T>(y[kk][c], max_exponent(amax), p, cut);
#pragma unroll
                for (int k = 0; k < K; ++k) x[k][kk][c] = (int)p[k];
            }
        any_cut = sizeof(T) == 4 && __builtin_amdgcn_ballot_w64(cut > 0.f) != 0ull;
        if (sizeof(T) == 2) cut = across_rows<MaxOp>(cut);
        return sizeof(T) == 2 && cut > 0.f ? kNoExponent : logit_exponent(amax);
    }
};

// Level sums of 16 tokens in LDS (accumulator rows) and 16 window rows (lanes).
template <int KR, int KT, int D, int kTok, int L>
__device__ __forceinline__ void level_sums(const RowDigits<KR, D> &rows, const char *digits, int tok, int g, i32x4 (&acc)[L]) {
#pragma unroll
    for (int t = 0; t < L; ++t) acc[t] = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < D / 64; ++kk) {
        if (kk > 0) __builtin_amdgcn_sched_barrier(0);       // (one piece at a time: registers)
        i32x4 b[KT];
#pragma unroll
        for (int k = 0; k < KT; ++k) b[k] = *(const i32x4 *)(digits + digit_offset<D, kTok>(k, tok, 4 * kk + g));
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int i = 0; i < KR && i + k < L; ++i)
                acc[i + k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b[k], rows.x[i][kk], acc[i + k], 0, 0, 0);
    }
}

// fp64 dot products of 16 tokens and 16 rows from memory: lane = row + 16 g, dot[r] that of token 4 g + r.  `tok`: the
// lane's token, 4 (lane % 4) + lane / 4 % 4 of the 16; `row`: row lane % 16.
template <typename T>
__device__ __forceinline__ f32x4 four_elements(const T *x) {
    if constexpr (sizeof(T) == 4) {
        return *(const f32x4 *)x;
    } else {
        const uint2 h = *(const uint2 *)x;
        return f32x4{__uint_as_float(h.x << 16), __uint_as_float(h.x & 0xffff0000u), __uint_as_float(h.y << 16), __uint_as_float(h.y & 0xffff0000u)};
    }
}
template <typename T, int D, typename R>
__device__ __forceinline__ void block_dots(const T *__restrict__ tok, const R *__restrict__ row, int g, double (&dot)[4]) {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int s = 0; s < D / 16; ++s) {
        const f32x4 x = four_elements(tok + 16 * s + 4 * g), y = four_elements(row + 16 * s + 4 * g);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[c], (double)y[c], acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) dot[r] = acc[r];
}

// The larger maximum, or the lower token that has it, of the lanes whose numbers differ in kBit.
template <int kBit>
__device__ __forceinline__ void best_of_pair(float &m, int &at) {
    float m0, m1;
    uint32_t a0, a1;
    both_of_pair<kBit>(m, m0, m1);
    both_of_pair<kBit>((uint32_t)at, a0, a1);
    const bool second = m1 > m0 || (m1 == m0 && a1 < a0);
    m = second ? m1 : m0;
    at = (int)(second ? a1 : a0);
}

// ------------------------------------------------------------------------------------
// Logits, as plain_logits forms them (fp64 dot products, rounded once), into the blocked layout.  For short calls.  Grid: x = KV head
// (neighbours run on different XCDs, whose L2 caches then hold the rows, values and logits of few heads), y = token range
// of the piece, z = chunk of kLogitRows rows.  A wave has 16 tokens of every tile of 64; lane = row + 16 g of every 16 rows,
// with tokens 4 g .. 4 g + 3, which the lanes' order of loading puts there.
// ------------------------------------------------------------------------------------
constexpr int kLogitRows = 32;
template <typename T, int D, typename Lens>
__global__ __launch_bounds__(kThreads, 4) void blocked_logits(const T *__restrict__ q, const T *__restrict__ k, int N, int W, int Hq,
                                                              int Hkv, int ragged, Lens lens, Piece w, int range_len, int n_ranges,
                                                              float *__restrict__ z, float2 *__restrict__ range_best) {
    constexpr int kRt = kLogitRows / 16;
    __shared__ __attribute__((aligned(16))) float rows_s[kLogitRows * kStride<D>];
    __shared__ float2 best_s[4][kLogitRows];
    const int hl = blockIdx.x, bg = w.bg0 + hl, b = bg / Hkv, M = Hq / Hkv * W;
    const int len = seq_len_of(lens, ragged, b, N);
    const int range = w.s0 / range_len + blockIdx.y;
    const int t_begin = range * range_len, t_end = min(min(t_begin + range_len, w.s1), len);
    if (t_begin >= t_end) return;                            // uniform
    const int row0 = blockIdx.z * kLogitRows, blocks = (w.nr + 15) / 16;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4;
    const T *kg = k + (size_t)bg * N * D;
    const int mine = wave * 16 + 4 * (lane & 3) + (lane >> 2 & 3);       // operand row 4 r + g is token 4 g + r
    RowRegs<T, D> tok;
    tok.load(kg, t_begin + mine, t_end, g);
    {
        TileRegs<T, D, kLogitRows> qr;
        qr.load(q + ((size_t)b * Hq * W + (size_t)(bg % Hkv) * M + w.r0) * D, row0, w.nr);
        qr.store(rows_s);
    }
    int last[kRt], at[kRt];
    float m[kRt];
    float *zp[kRt];
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt) {
        const int row = row0 + 16 * rt + (lane & 15);
        last[rt] = row < w.nr ? min(len - W + (w.r0 + row) % W, t_end - 1) : -1;     // last token the row sees here
        m[rt] = -INFINITY;
        at[rt] = kNoToken;
        zp[rt] = z + z_block(w, hl, row0 / 16 + rt, t_begin + wave * 16) + lane * 4;
    }
    __syncthreads();
    for (int t0 = t_begin; t0 < t_end; t0 += kTile) {
        f64x4 acc[kRt];
#pragma unroll
        for (int rt = 0; rt < kRt; ++rt) acc[rt] = f64x4{0.0, 0.0, 0.0, 0.0};
        tile_dots<T, D, kRt, true>(rows_s, tok, lane, acc);
        if (t0 + kTile < t_end) tok.load(kg, t0 + kTile + mine, t_end, g);
#pragma unroll
        for (int rt = 0; rt < kRt; ++rt) {
            float x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[r] = (float)(acc[rt][r] * (1.0 / sqrt((double)D)));    // scaled logit: the only rounding
                const int p = t0 + wave * 16 + 4 * g + r;
                if (p <= last[rt] && x[r] > m[rt]) { m[rt] = x[r]; at[rt] = p; }     // (tokens ascend: strict keeps the lowest)
            }
            if (row0 / 16 + rt < blocks) *(float4 *)(zp[rt] + (t0 - t_begin) * 16) = make_float4(x[0], x[1], x[2], x[3]);   // (room for whole tiles)
        }
    }
#pragma unroll
    for (int rt = 0; rt < kRt; ++rt) {
        best_of_pair<16>(m[rt], at[rt]);
        best_of_pair<32>(m[rt], at[rt]);
        if (g == 0) best_s[wave][16 * rt + lane] = make_float2(m[rt], __int_as_float(at[rt]));
    }
    __syncthreads();
    const int row = threadIdx.x;
    if (row < kLogitRows && row0 + row < w.nr) {
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
// Weights and P V.  Grid: x = KV head, y = split of the piece, z = chunk of 16 kRb rows.  O^T += V^T P^T, 32 tokens
// at a time; lane = row + 16 g.  The parts of a tile (16 / kRb of them) meet in LDS at the
// end: two waves per SIMD are too few to hide the chain logit, weight, product, and more splits would be more traffic.
// ------------------------------------------------------------------------------------
// V pieces in LDS: kP planes of kTok rows of D bf16.  A row's 16-byte piece c sits where the transposing read (32 lanes
// fetch 32 bytes each of eight consecutive tokens) meets every bank once.
template <int D, int kTok>
__device__ __forceinline__ int value_offset(int plane, int tok, int c) {
    const int slot = D == 128 ? (c + 2 * (tok & 7)) & 15 : (c + 2 * (tok >> 1 & 3)) & 7;
    return (plane * kTok + tok) * D * 2 + slot * 16;
}

// Two elements as three bf16 pieces each, rounded to nearest and each remainder exact (9 + 9 + 8 bits and more hold the 24).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void three_pieces(float a, float b, uint32_t (&p)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const bf16x2 r = __builtin_convertvector((f32x2{a, b}), bf16x2);     // v_cvt_pk_bf16_f32
        p[i] = *(const uint32_t *)&r;
        a -= __uint_as_float(p[i] << 16);
        b -= __uint_as_float(p[i] & 0xffff0000u);
    }
}
// Tokens of a tile of values: 32 for every part, or 64 where a tile would have fewer 16-byte pieces than threads.
template <typename T, int D, int kRb>
constexpr int kWeightTile = 16 / kRb * 32 * D * (int)sizeof(T) >= kWeightThreads * 16 ? 16 / kRb * 32 : 16 / kRb * 64;
template <typename T> constexpr int kValuePieces = sizeof(T) == 4 ? 3 : 1;
template <typename T, int D, int kRb> constexpr int kValueBytes = kValuePieces<T> * kWeightTile<T, D, kRb> * D * 2;
template <typename T, int D, int kRb> constexpr int kValueBuffers = kValueBytes<T, D, kRb> <= 64 * 1024 ? 2 : 1;
template <typename T, int D, int kRb>                                    // of LDS: tiles of values, later the parts' sums
constexpr int kWeightBytes = std::max(kValueBuffers<T, D, kRb> * kValueBytes<T, D, kRb>, (16 / kRb - 1) * 16 * kRb * D * 4);

// Weights and P V of tokens t_begin .. t_end - 1 for the wave's 16 rows: O^T += V^T P^T, 32 tokens at a time; lane = row + 16 g.  The
// parts of a tile (16 / kRb of them) meet in LDS at the end: two waves per SIMD are too few to hide the chain logit, weight, product,
// and more splits would be more traffic.  `zg`, `z_at`: where the lane's logits of t_begin lie; `vg`: the values from t_begin on.
// `before` runs while the first loads are on their way, `rows(m, top, last)` gives the lane's row once all waves are through that: the
// reference, the token left out, the last token it sees.  Returns the row's sum, and the sums of P V in `acc`, for the first part.
template <typename T, int D, int kRb, bool kNeedO, typename Before, typename Rows>
__device__ __forceinline__ float weights_pv(char *values, float (*sum_s)[16 * kRb], __amdgpu_buffer_rsrc_t zg, int z_at, __amdgpu_buffer_rsrc_t vg,
                                            int t_begin, int t_end, int rb, int part, int lane, Before &&before, Rows &&rows, f32x4 (&acc)[D / 16]) {
    constexpr int kTok = kWeightTile<T, D, kRb>, kParts = 16 / kRb, kPart = kTok / kParts, kP = kValuePieces<T>,
                  kTileBytes = kValueBytes<T, D, kRb>, kBuf = kValueBuffers<T, D, kRb>;
    const int g = lane >> 4, row_l = rb * 16 + (lane & 15);
    TokenTile<T, D, kTok, kWeightThreads> next;
    if (kNeedO) next.load(vg, 0);
    // This lane's logits of a 32-token step: tokens 4 g + {0..3} and 16 + 4 g + {0..3}, the order of the transposing reads.
    // (What lies beyond the last token's tile is anything, and not used.)
    float4 x[2 * (kPart / 32)];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int i = 0; i < 2 * (kPart / 32); ++i) {
            const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(zg, z_at + (t0 - t_begin + part * kPart + 16 * i) * 64, 0, 0);
            x[i] = make_float4(__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w));
        }
    };
    fetch(t_begin);
    before();
    auto store_values = [&](int slot) {
        int thread = threadIdx.x;
        asm volatile("" : "+v"(thread));                     // (addresses anew for every tile: registers)
        const int c = thread % next.kLanes;
        char *dst = values + slot % kBuf * kTileBytes + value_offset<D, kTok>(0, thread / next.kLanes, c * next.kPer / 8) + c * next.kPer % 8 * 2;
#pragma unroll
        for (int i = 0; i < next.kCount; ++i) {
            char *at = dst + i * next.kStep * D * 2;
            if constexpr (kP == 1) {
                *(uint4 *)at = next.x[i];
            } else {
                float y[1][4];
                next.unpack(i, y);
                uint32_t p[2][3];
                three_pieces(y[0][0], y[0][1], p[0]);
                three_pieces(y[0][2], y[0][3], p[1]);
#pragma unroll
                for (int k = 0; k < 3; ++k) *(uint2 *)(at + k * kTok * D * 2) = make_uint2(p[0][k], p[1][k]);
            }
        }
    };
    if (kNeedO) store_values(0);
    __syncthreads();
    float m;
    int top, last;
    rows(m, top, last);
    if (kNeedO && t_begin + kTok < t_end) next.load(vg, kTok);
#pragma unroll
    for (int d = 0; d < D / 16; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
    int slot = 0;
    // Transposing read: in every 16 lanes four tokens' 16 elements of head_dim block d; two reads make a 32-token operand.
    const int i16 = lane & 15, tok_l = part * kPart + 4 * g + (i16 >> 2), c_l = i16 >> 1 & 1, byte_l = (i16 & 1) * 8;
    for (int t0 = t_begin; t0 < t_end; t0 += kTok, slot ^= 1) {
        if (kNeedO && t0 > t_begin) __syncthreads();         // this tile is in LDS, the one before it has been read
        union Pieces { bf16x8 v; uint32_t u[4]; } p[kPart / 32][3];
#pragma unroll
        for (int s = 0; s < kPart / 32; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 f = x[2 * s + h];
                const float y[4] = {f.x, f.y, f.z, f.w};
                float e4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = t0 + part * kPart + 32 * s + 16 * h + 4 * g + i;
                    e4[i] = t <= last && t != top ? exp_nonpositive(y[i] - m) : 0.f;
                    sum += e4[i];
                }
                uint32_t q[2][3];
                three_pieces(e4[0], e4[1], q[0]);
                three_pieces(e4[2], e4[3], q[1]);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    p[s][k].u[2 * h] = q[0][k];
                    p[s][k].u[2 * h + 1] = q[1][k];
                }
            }
        if (t0 + kTok < t_end) fetch(t0 + kTok);
        if (!kNeedO) continue;
        auto advance = [&]() {
            if (t0 + kTok < t_end) store_values(slot ^ 1);
            if (t0 + 2 * kTok < t_end) next.load(vg, t0 - t_begin + 2 * kTok);
        };
        if (kBuf == 2) advance();
#pragma unroll
        for (int s = 0; s < kPart / 32; ++s)
#pragma unroll
            for (int d = 0; d < D / 16; ++d)
#pragma unroll
                for (int k = 0; k < kP; ++k) {
                    union { bf16x8 v; i16x4 h[2]; } a;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        a.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(
                            values + slot % kBuf * kTileBytes + value_offset<D, kTok>(k, tok_l + 32 * s + 16 * h, 2 * d + c_l) + byte_l));
#pragma unroll
                    for (int j = 0; j < 3; ++j)
                        acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, p[s][j].v, acc[d], 0, 0, 0);
                }
        if (kBuf == 1) {
            __syncthreads();
            advance();
        }
    }
    sum = across_rows<SumOp>(sum);
    if (g == 0) sum_s[part][row_l] = sum;
    __syncthreads();                                         // (also: the last tile has been read)
    float4 *merge = (float4 *)values + (rb * (D / 16)) * 64 + lane;      // [part - 1][row block][element / 16][lane]
    if (kNeedO && part > 0)
#pragma unroll
        for (int d = 0; d < D / 16; ++d)
            merge[((part - 1) * kRb * (D / 16) + d) * 64] = make_float4(acc[d][0], acc[d][1], acc[d][2], acc[d][3]);
    __syncthreads();
    if (part > 0) return sum;
#pragma unroll
    for (int c = 1; c < kParts; ++c) sum += sum_s[c][row_l];
    if (kNeedO)
#pragma unroll
        for (int d = 0; d < D / 16; ++d)
#pragma unroll
            for (int c = 0; c < kParts - 1; ++c) {
                const float4 x = merge[(c * kRb * (D / 16) + d) * 64];
                acc[d][0] += x.x; acc[d][1] += x.y; acc[d][2] += x.z; acc[d][3] += x.w;
            }
    return sum;
}
// The row's sums of P V to memory.
template <int D>
__device__ __forceinline__ void write_output(float *__restrict__ to, const f32x4 (&acc)[D / 16], int g) {
#pragma unroll
    for (int d = 0; d < D / 16; ++d) *(float4 *)(to + d * 16 + 4 * g) = make_float4(acc[d][0], acc[d][1], acc[d][2], acc[d][3]);
}

// ------------------------------------------------------------------------------------
// Weights and P V behind blocked_logits, relative to the row's maximum over all its ranges.  Grid: x = KV head, y = split of the piece,
// z = chunk of 16 kRb rows.
// ------------------------------------------------------------------------------------
template <typename T, int D, int kRb, bool kNeedO, typename Lens>
__global__ __launch_bounds__(kWeightThreads, 4) void fixed_weights(const T *__restrict__ v, int N, int W, int Hkv, int ragged, Lens lens,
                                                                  Piece w, int range_len, int n_ranges, int split_len, int n_splits,
                                                                  const float *__restrict__ z, const float2 *__restrict__ range_best,
                                                                  RowRecord *__restrict__ records, float *__restrict__ part_l,
                                                                  float *__restrict__ part_o) {
    constexpr int kRows = 16 * kRb;
    __shared__ __attribute__((aligned(16))) char values[kNeedO ? kWeightBytes<T, D, kRb> : 16];
    __shared__ float sum_s[16 / kRb][kRows];
    __shared__ float m_s[kRows];
    __shared__ int top_s[kRows];
    const int hl = blockIdx.x, bg = w.bg0 + hl, b = bg / Hkv;
    const int len = seq_len_of(lens, ragged, b, N);
    const int split = w.s0 / split_len + blockIdx.y;
    const int t_begin = split * split_len, t_end = min(min(t_begin + split_len, w.s1), len);
    if (t_begin >= t_end) return;                            // uniform
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int rb = wave % kRb, part = wave / kRb, row0 = blockIdx.z * kRows, row_l = rb * 16 + (lane & 15), row = row0 + row_l;
    const int block = min(row0 / 16 + rb, (w.nr + 15) / 16 - 1);
    const size_t z_head = z_block(w, hl, 0, w.s0);
    f32x4 acc[D / 16];
    const float sum = weights_pv<T, D, kRb, kNeedO>(
        values, sum_s, span_of(z + z_head, z_block(w, 1, 0, w.s0) * 4), (int)(z_block(w, hl, block, t_begin) - z_head) * 4 + lane * 16,
        span_of(v + ((size_t)bg * N + t_begin) * D, (size_t)(t_end - t_begin) * D * sizeof(T)), t_begin, t_end, rb, part, lane,
        [&]() {
            constexpr int kSub = kWeightThreads / kRows;          // the row's maximum over its ranges: kSub lanes per row
            const int row = threadIdx.x / kSub, live = (len + range_len - 1) / range_len;
            float m = -INFINITY;
            int at = kNoToken;
            if (row0 + row < w.nr)
#pragma unroll 8
                for (int i = threadIdx.x % kSub; i < live; i += kSub) {
                    const float2 o = range_best[((size_t)hl * w.nr + row0 + row) * n_ranges + i];
                    if (o.x > m || (o.x == m && __float_as_int(o.y) < at)) { m = o.x; at = __float_as_int(o.y); }
                }
            lanes_best<kSub>(m, at);
            if (threadIdx.x % kSub == 0) {
                m_s[row] = m;
                top_s[row] = at;
                if (split == 0 && row0 + row < w.nr) {
                    RowRecord *rec = records + (size_t)hl * w.nr + row0 + row;
                    rec->m = m;
                    rec->top = at;
                }
            }
        },
        [&](float &m, int &top, int &last) {
            m = row < w.nr ? m_s[row_l] : 0.f;
            top = top_s[row_l];
            last = row < w.nr ? min(len - W + (w.r0 + row) % W, t_end - 1) : -1;       // last token the row sees here
        },
        acc);
    if (part > 0 || row >= w.nr) return;
    const size_t out_row = ((size_t)hl * n_splits + split) * w.nr + row;
    if (lane < 16) part_l[out_row] = sum;
    if (kNeedO) write_output<D>(part_o + out_row * D, acc, lane >> 4);
}

// ------------------------------------------------------------------------------------
// Logits from digits, weights and P V in one kernel, where the call is long enough.  Grid: x = KV head, y = split of the piece, z = chunk
// of 16 kRb rows.  A workgroup first forms the logits of its split (kept, for the scores), then, with the split's own largest logit as
// reference and without the token that has it, their weights: the logits come back from the die's L2, nobody waits for the other
// splits' maxima, and a launch is saved.  plain_merge brings the splits to one reference and puts their tokens back.
// Lane = row + 16 g, registers = tokens 4 g .. 4 g + 3 of the 16 at hand.
// ------------------------------------------------------------------------------------
template <typename T, int D> constexpr int kSweepTile = sizeof(T) == 2 && D == 64 ? 128 : 64;      // tokens of a tile of keys: a piece per thread
template <typename T, int D, int kRb>
constexpr int kSweepBytes = std::max(2 * kLogitDigits<T> * kSweepTile<T, D> * D, kWeightBytes<T, D, kRb>);
template <typename T, int D, int kRb, bool kNeedO, typename Lens>
__global__ __launch_bounds__(kWeightThreads, 4) void digit_sweep(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, int N,
                                                                 int W, int Hq, int Hkv, int ragged, Lens lens, Piece w, int split_len,
                                                                 int n_splits, float *z, float4 *__restrict__ part_head,
                                                                 float *__restrict__ part_o) {
    constexpr int K = kLogitDigits<T>, kTok = kSweepTile<T, D>, kParts = 16 / kRb, kPart = kTok / kParts, kRows = 16 * kRb;
    static_assert(kPart % 16 == 0, "whole blocks of 16 tokens");
    __shared__ __attribute__((aligned(16))) char smem[kSweepBytes<T, D, kRb>];       // digits of two tiles, then tiles of values
    __shared__ __attribute__((aligned(16))) int exponents[2][kTok];
    __shared__ __attribute__((aligned(16))) uint8_t cut_s[2][kWeightThreads / 64];
    __shared__ float2 best_s[kParts][kRows];
    __shared__ float sum_s[kParts][kRows];
    const int hl = blockIdx.x, bg = w.bg0 + hl, b = bg / Hkv, M = Hq / Hkv * W;
    const int len = seq_len_of(lens, ragged, b, N);
    const int split = blockIdx.y, t_begin = split * split_len, t_end = min(t_begin + split_len, len);
    if (t_begin >= t_end) return;                            // uniform
    const int row0 = blockIdx.z * kRows, blocks = (w.nr + 15) / 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rb = wave % kRb, part = wave / kRb, row = row0 + rb * 16 + (lane & 15);
    float m = -INFINITY;
    int at = kNoToken;
    {
        char (&digits)[2][K * kTok * D] = *(char (*)[2][K * kTok * D])smem;
        const bool live = row0 / 16 + rb < blocks;           // uniform in the wave
        const T *kg = k + (size_t)bg * N * D;
        const __amdgpu_buffer_rsrc_t span = span_of(kg + (size_t)t_begin * D, (size_t)(t_end - t_begin) * D * sizeof(T));
        TokenTile<T, D, kTok, kWeightThreads> next;
        next.load(span, 0);
        const T *q_row = q + ((size_t)b * Hq * W + (size_t)(bg % Hkv) * M + w.r0 + min(row, w.nr - 1)) * D;
        RowDigits<K, D> rows;
        bool rows_cut;
        const int row_exponent = rows.template take<T>(q_row, lane >> 4, rows_cut), exponent = row_exponent - 51 - 3;
        const int last = min(len - W + (w.r0 + min(row, w.nr - 1)) % W, t_end - 1);                // last token the row sees here
        const int least = __builtin_amdgcn_readfirstlane((int)row16_reduce<MinOp>((uint32_t)last));      // of the 16 rows
        float *zp = z + z_block(w, hl, min(row0 / 16 + rb, blocks - 1), t_begin) + lane * 4;
        next.template store_logit_digits<K>(digits[0], exponents[0], cut_s[0]);
        if (t_begin + kTok < t_end) next.load(span, kTok);
        int slot = 0;
        for (int t0 = t_begin; t0 < t_end; t0 += kTok, slot ^= 1) {
            __syncthreads();                                 // this tile is in LDS, the one before it has been read
            if (t0 + kTok < t_end) next.template store_logit_digits<K>(digits[slot ^ 1], exponents[slot ^ 1], cut_s[slot ^ 1]);
            if (t0 + 2 * kTok < t_end) next.load(span, t0 - t_begin + 2 * kTok);
            if (!live) continue;
            double least_dot = kLeastDot<T>;
            if (sizeof(T) == 4) {
                const uint4 cut = *(const uint4 *)cut_s[slot];
                if (rows_cut || __builtin_amdgcn_readfirstlane((int)(cut.x | cut.y | cut.z | cut.w)) != 0) least_dot = kLeastDotCut;     // uniform
            }
#pragma unroll 1
            for (int p0 = part * kPart; p0 < (part + 1) * kPart; p0 += 16) {
                if (t0 + p0 >= t_end) break;                 // uniform (what follows is another split's)
                i32x4 acc[kLogitLevels];
                level_sums<K, K, D, kTok>(rows, digits[slot], p0 + (lane & 15), lane >> 4, acc);
                __builtin_amdgcn_sched_barrier(0);
                const int first = t0 + p0 + 4 * (lane >> 4);     // register r has token first + r
                const i32x4 ex = *(const i32x4 *)&exponents[slot][p0 + 4 * (lane >> 4)];
                float x[4];
                bool again = max(max(max(ex[0], ex[1]), ex[2]), ex[3]) + exponent >= kNoExponent / 2, small[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double dot = join_seven<K>(acc[0][r], acc[1][r], acc[2][r], acc[3][r], acc[4][r], acc[5][r], acc[6][r]);
                    small[r] = fabs(dot) < least_dot;
                    if (D == 128) dot *= 0.088388347648318440550 * 8.0;
                    x[r] = __builtin_amdgcn_ldexpf((float)dot, ex[r] + exponent);
                }
                if (__builtin_amdgcn_ballot_w64(again || small[0] || small[1] || small[2] || small[3]) != 0ull)      // uniform, rare
#pragma unroll
                    for (int r = 0; r < 4; ++r)              // (keys of zeros, also those past the end, and such queries are held)
                        again |= small[r] && ex[r] != kZeroExponent && row_exponent != kZeroExponent;
                if (__builtin_amdgcn_ballot_w64(again) != 0ull) {            // uniform
                    double dot[4];
                    block_dots<T, D>(kg + (size_t)min(t0 + p0 + 4 * (lane & 3) + (lane >> 2 & 3), t_end - 1) * D, q_row, lane >> 4, dot);
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = (float)(dot[r] * (1.0 / sqrt((double)D)));
                }
                auto improve = [&](const float (&y)[4]) {
                    const float best = fmaxf(fmaxf(fmaxf(y[0], y[1]), y[2]), y[3]);
                    if (__builtin_amdgcn_ballot_w64(best > m) == 0ull) return;       // uniform, usual once the maxima have settled
#pragma unroll
                    for (int r = 0; r < 4; ++r)                  // (tokens ascend: strict keeps the lowest)
                        if (y[r] > m) { m = y[r]; at = first + r; }
                };
                if (t0 + p0 + 15 > least) {                      // uniform: not every row sees every token
                    float y[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[r] = first + r <= last ? x[r] : -INFINITY;
                    improve(y);
                } else {
                    improve(x);
                }
                *(float4 *)(zp + (t0 - t_begin + p0) * 16) = make_float4(x[0], x[1], x[2], x[3]);      // (room for whole tiles)
            }
        }
    }
    best_of_pair<16>(m, at);
    best_of_pair<32>(m, at);
    if (lane < 16) best_s[part][rb * 16 + lane] = make_float2(m, __int_as_float(at));
    __syncthreads();                                         // (also: the logits are written, the digits have been read)
    const int row_l = rb * 16 + (lane & 15);
    float2 best = best_s[0][row_l];
#pragma unroll
    for (int c = 1; c < kParts; ++c) {
        const float2 o = best_s[c][row_l];
        if (o.x > best.x || (o.x == best.x && __float_as_int(o.y) < __float_as_int(best.y))) best = o;
    }
    // (a row that sees nothing here, or logits of -infinity alone: every weight is 0)
    const float reference = best.x == -INFINITY ? 0.f : best.x;
    const size_t z_head = z_block(w, hl, 0, w.s0);
    f32x4 acc[D / 16];
    const float sum = weights_pv<T, D, kRb, kNeedO>(
        smem, sum_s, span_of(z + z_head, z_block(w, 1, 0, w.s0) * 4),
        (int)(z_block(w, hl, min(row0 / 16 + rb, blocks - 1), t_begin) - z_head) * 4 + lane * 16,
        span_of(v + ((size_t)bg * N + t_begin) * D, (size_t)(t_end - t_begin) * D * sizeof(T)), t_begin, t_end, rb, part, lane, []() {},
        [&](float &ref, int &top, int &last) {
            ref = row < w.nr ? reference : 0.f;
            top = __float_as_int(best.y);
            last = row < w.nr ? min(len - W + (w.r0 + row) % W, t_end - 1) : -1;       // last token the row sees here
        },
        acc);
    if (part > 0 || row >= w.nr) return;
    const size_t out_row = ((size_t)hl * n_splits + split) * w.nr + row;
    if (lane < 16) part_head[out_row] = make_float4(best.x, sum, best.y, 0.f);
    if (kNeedO) write_output<D>(part_o + out_row * D, acc, lane >> 4);
}

// ------------------------------------------------------------------------------------
// Scores of every variant.  Grid: x = KV head, y = `n_tiles` tiles of the piece.  Lane = row + 16 g, registers =
// tokens 4 g .. 4 g + 3 of the 16 at hand.  A workgroup takes its tokens against one chunk of rows after the other.
// ------------------------------------------------------------------------------------
constexpr int kScoreTokens = 512;              // most tokens of a workgroup
// What it needs of a row for every pair (40 bytes: the 16 rows of a read meet every bank once), and what for few of them.
struct ScoreRow {
    float m, inv_l;
    double oo;
    double unit;                 // -2 times the unit of o_i's digits
    float least;                 // the row's share of the closeness test
    int top, last, unused;
};
struct ScoreTop { float dk, dj; };

// Sums of four registers over each row of 16 lanes: lanes 4 i .. 4 i + 3 of the row get that of x_i.  (Eight additions instead of sixteen:
// the first two rounds leave half as many registers each.  The waits are those of a data-parallel read of what was just written.)
__device__ __forceinline__ float four_sums(float x0, float x1, float x2, float x3) {
    asm volatile("s_nop 1\n"
                 "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n"
                 "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n"
                 "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n"
                 "v_add_f32_dpp %1, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n"
                 "s_nop 0\n"
                 "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n"
                 "v_add_f32_dpp %0, %1, %1 row_shr:4 row_mask:0xf bank_mask:0xa\n"
                 "s_nop 1\n"
                 "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n"
                 "s_nop 1\n"
                 "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
                 : "+&v"(x0), "+&v"(x1) : "v"(x2), "v"(x3));
    return x0;
}
template <typename T, int D, int kRb, int kVariant, typename Lens>
__global__ __launch_bounds__(kFixedThreads, 4) void fixed_score(const T *__restrict__ v, int N, int Hkv, int ragged, Lens lens, Piece w,
                                                                int n_tiles, const float *__restrict__ z,
                                                                const RowRecord *__restrict__ records, const float *__restrict__ o,
                                                                const int8_t *__restrict__ o_digits, float *__restrict__ scores,
                                                                size_t variant_stride, int add) {
#pragma clang fp contract(off)                               // (a score has the same bits alone and among all three)
    constexpr int K = kDigits<T>, kTok = kFixedTile<D>, kPart = kTok / (8 / kRb), kRows = 16 * kRb;
    constexpr bool kAttnLike = kVariant == OBC_ATTN || kVariant == OBC_VATP;
    constexpr bool kDoV = kVariant == OBC_ALL || kVariant == OBC_VALUE || kAttnLike, kDoK = kVariant == OBC_ALL || kVariant == OBC_KEY,
                   kDoJ = kVariant == OBC_ALL || kVariant == OBC_JOINT, kNeedO = kDoK || kDoJ, kNeedV = kVariant != OBC_ATTN;
    constexpr int kSums = kVariant == OBC_ALL ? 3 : 1, kNorm = kVariant == OBC_VATP ? 1 : 2;
    constexpr bool kAhead = D == 64 || !kNeedO;
    __shared__ __attribute__((aligned(16))) char digits[2][kNeedO ? K * kTok * D : 16];
    __shared__ __attribute__((aligned(16))) double units[2][kTok];
    __shared__ __attribute__((aligned(16))) double norm_s[2][kTok];
    __shared__ __attribute__((aligned(16))) float least_s[2][kTok];
    __shared__ ScoreRow rec_s[kRows];
    __shared__ ScoreTop top_s[kRows];
    __shared__ __attribute__((aligned(16))) float sum_s[kSums][kRb][kTok];
    __shared__ float run_s[kSums][kScoreTokens];             // sums over the chunks so far
    const int hl = blockIdx.x, bg = w.bg0 + hl, b = bg / Hkv;
    const int len = seq_len_of(lens, ragged, b, N);
    const int t_begin = w.s0 + blockIdx.y * n_tiles * kTok, t_stop = min(t_begin + n_tiles * kTok, w.s1), t_end = min(t_stop, len);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;    // (a scalar: registers)
    const int rb = wave % kRb, part = wave / kRb;
    float *out = scores + (size_t)bg * N;
    if (!add)
        for (int t = max(t_begin, len) + (int)threadIdx.x; t < t_stop; t += kFixedThreads)       // the padding
#pragma unroll
            for (int c = 0; c < kSums; ++c) out[c * variant_stride + t] = 0.f;
    if (t_begin >= t_end) return;                            // uniform
    const __amdgpu_buffer_rsrc_t vg = span_of(v + ((size_t)bg * N + t_begin) * D, (size_t)(t_end - t_begin) * D * sizeof(T));
    const int blocks = (w.nr + 15) / 16;
    for (int row0 = 0; row0 < w.nr; row0 += kRows) {
        TokenTile<T, D, kTok, kFixedThreads> next;
        if (kNeedV) next.load(vg, 0);
        const int block = min(row0 / 16 + rb, blocks - 1);
        RowDigits<kRowDigits, D> rows;
        if (kNeedO) rows.load(o_digits, hl, block, blocks, lane);
        const __amdgpu_buffer_rsrc_t zg = span_of(z + z_block(w, hl, 0, w.s0), z_block(w, 1, 0, w.s0) * 4);
        const int z_at = (int)(z_block(w, 0, block, w.s0) * 4);
        // Of 16 tokens from t on (there is room for whole tiles); those of the next block are on their way, but for scores with
        // outputs and 128 channels: there the fp32 all-in-one kernels spill up to 8 registers over them (8 heads x 128 rows x 1500 41.2 us, with
        // them 41.9), and the others take as long.
        auto logits = [&](int t, int l) { return __builtin_amdgcn_raw_buffer_load_b128(zg, l * 16, z_at + (t - w.s0) * 64, 0); };
        u32x4 ahead;
        if (kAhead) ahead = logits(t_begin + part * kPart, lane);
        __syncthreads();                                     // (the chunk before this one is done with)
        int i = threadIdx.x;
        asm volatile("" : "+v"(i));                          // (addresses anew for every chunk: registers)
        if (i < kRows) {
            const RowRecord r = records[(size_t)hl * w.nr + min(row0 + i, w.nr - 1)];
            rec_s[i] = ScoreRow{r.m, r.inv_l, r.oo, -2.0 * r.unit, least_share(r.unit), r.top, row0 + i < w.nr ? r.last : -1, 0};
            top_s[i] = ScoreTop{r.top_dk, r.top_dj};         // (last -1: no such row, it sees nothing)
        }
        if (kNeedV) next.template store_digits<kNeedO, kNorm>(digits[0], units[0], least_s[0], norm_s[0]);
        if (kNeedV && t_begin + kTok < t_end) next.load(vg, kTok);
        const bool live = row0 / 16 + rb < blocks;           // uniform in the wave
        if (!live && part == 0)                              // (no other wave writes these)
            for (int j = lane; j < kSums * kTok; j += 64) sum_s[j / kTok][rb][j % kTok] = 0.f;
        int slot = 0, least_last = 0;
        for (int t0 = t_begin; t0 < t_end; t0 += kTok, slot ^= 1) {
            __syncthreads();                                 // this tile is in LDS, the one before it has been read
            if (t0 == t_begin)                               // of the wave's rows
                least_last = __builtin_amdgcn_readfirstlane((int)row16_reduce<MinOp>((uint32_t)(rec_s[rb * 16 + (lane & 15)].last + 1))) - 1;
            auto advance = [&]() {
                if (!kNeedV) return;
                if (t0 + kTok < t_end)
                    next.template store_digits<kNeedO, kNorm>(digits[slot ^ 1], units[slot ^ 1], least_s[slot ^ 1], norm_s[slot ^ 1]);
                if (t0 + 2 * kTok < t_end) next.load(vg, t0 - t_begin + 2 * kTok);
            };
            advance();
#pragma unroll 1
            for (int p0 = part * kPart; live && p0 < (part + 1) * kPart; p0 += 16) {
                int l = lane;
                asm volatile("" : "+v"(l));                  // (addresses anew: registers)
                const u32x4 u = kAhead ? ahead : logits(t0 + p0, l);
                float x[4] = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
                i32x4 acc[kLevels];
                if (kNeedO) {
                    level_sums<kRowDigits, K, D, kTok>(rows, digits[slot], p0 + (l & 15), l >> 4, acc);
                    __builtin_amdgcn_sched_barrier(0);       // (the row's record only now: registers)
                }
                if (kAhead) ahead = logits(next_scored(t0, p0, part, kPart, kTok, t_end), l);
                float acc_v[4], acc_k[4], acc_j[4];
                const int tok0 = p0 + 4 * (l >> 4);          // register r has token tok0 + r of the tile
                const ScoreRow rec = rec_s[rb * 16 + (l & 15)];
                // The pairs' terms; returns whether one of them that counts has a norm too small for the digits' error.  kAny: a row
                // may not see a token, or have it as its top.  kExact: v_p . o_i (vo), not the level sums.
                double vo[4];
                auto pairs = [&](auto any, auto exact) {
                    constexpr bool kAny = decltype(any)::value, kExact = decltype(exact)::value;
                    const ScoreTop top = kAny && kNeedO ? top_s[rb * 16 + (l & 15)] : ScoreTop();
                    bool close = false;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (r % (D == 64 ? 2 : 1) == 0) __builtin_amdgcn_sched_barrier(0);
                        const int p = t0 + tok0 + r;
                        float a = exp_nonpositive(x[r] - rec.m) * rec.inv_l;
                        if (kAny && p > rec.last) a = 0.f;
                        const float a2 = a * a;
                        acc_v[r] = kAttnLike ? a : a2;
                        if (!kNeedO) continue;
                        const bool is_top = kAny && p == rec.top;
                        const double vv = norm_s[slot][tok0 + r], with_oo = vv + rec.oo;
                        const double dot = kExact ? vo[r] : join_levels(acc[0][r], acc[1][r], acc[2][r], acc[3][r], acc[4][r]);
                        const double unit = kExact ? -2.0 : units[slot][tok0 + r] * rec.unit;
                        const double d2 = fma(dot, unit, with_oo);                                  // ||v_p - o_i||^2
                        const float least = least_s[slot][tok0 + r] * rec.least;                    // 2^-4 2^E
                        // (what is close and counts: times the pair's weight, so that one of weight 0 is not)
                        if (kDoK) {
                            const float w = a2 * x[r] * x[r], dk = at_least_0((float)d2);
                            acc_k[r] = w * (is_top ? top.dk : dk);
                            close |= !is_top && acc_k[r] < w * least;
                        }
                        if (kDoJ) {
                            const double zd = x[r];          // ||v_p + Z (v_p - o_i)||^2 = vv + Z (2 (v_p - o_i).v_p + Z d2)
                            const float dj = at_least_0((float)fma(zd, fma(zd, d2, fma(dot, unit, vv + vv)), vv));
                            acc_j[r] = a2 * (is_top ? top.dj : dj);
                            close |= !is_top && acc_j[r] < a2 * (least * fabsf(fmaf(x[r], x[r], x[r])));      // (its share of d2's error)
                        }
                    }
                    return close;
                };
                // (Scores without outputs have little to mask: every block on the one path, whose code then comes from memory once.  Value
                // score, 8 heads, us, two paths / one: bf16, d = 64, 128 rows x 300 16.22 / 15.95, 256 rows x 1000 21.16 / 20.73, x 8111
                // 58.0 / 57.8; fp32, d = 128, 128 rows x 300 18.41 / 18.27, x 8111 60.2 / 60.1.)
                const bool any = !kNeedO || t0 + p0 + 15 > least_last || __ballot((uint32_t)(rec.top - (t0 + tok0)) < 4u) != 0ull;      // uniform
                bool close;
                if (any) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) asm volatile("" : "+v"(x[r]));       // (nothing of this ahead of the branch)
                    close = pairs(std::true_type(), std::false_type());
                } else {
                    close = pairs(std::false_type(), std::false_type());
                }
                if (kNeedO && __ballot(close) != 0ull) {     // uniform, rare
                    asm volatile("" : "+v"(l));              // (and here)
                    block_dots<T, D>(v + ((size_t)bg * N + min(t0 + p0 + 4 * (l & 3) + (l >> 2 & 3), t_end - 1)) * D,
                                     o + ((size_t)hl * w.nr + min(block * 16 + (l & 15), w.nr - 1)) * D, l >> 4, vo);
                    pairs(std::true_type(), std::true_type());
                }
                // over the 16 rows; the other row blocks held others
                int n = 0;
                auto put = [&](float (&s)[4]) {
                    const float sums = four_sums(s[0], s[1], s[2], s[3]);
                    if ((l & 3) == 0) sum_s[n][rb][p0 + (l >> 2)] = sums;
                    ++n;
                };
                if (kDoV) put(acc_v);
                if (kDoK) put(acc_k);
                if (kDoJ) put(acc_j);
            }
            __syncthreads();
            int thread = threadIdx.x;
            asm volatile("" : "+v"(thread));                 // (addresses anew for every tile: registers)
            if (thread < kSums * kTok) {                     // (the same thread for a token in every chunk)
                const int c = thread / kTok, tok_l = thread % kTok, p = t0 + tok_l;
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < kRb; ++i) s += sum_s[c][i][tok_l];
                if (kDoV && kNeedV && c == 0) s *= (float)norm_s[slot][tok_l];
                if (row0 > 0) s += run_s[c][p - t_begin];
                if (row0 + kRows < w.nr) run_s[c][p - t_begin] = s;
                else if (p < t_end) {
                    float *d = out + c * variant_stride + p;
                    *d = add ? *d + s : s;
                }
            }
        }
    }
}
