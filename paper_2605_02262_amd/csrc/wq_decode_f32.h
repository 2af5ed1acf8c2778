// a4, matrix-core path of fp32 accuracy: the walkers of caches with one or four groups per head.
// (included by wq_decode_mfma.h, whose body cuts the work and merges it)
//
// Results are as accurate as those of fp32 arithmetic throughout (the figures are below); v_scale_max is not read.  Codes, scales and
// minima are exact, sums are fp32.  What is rounded apart from them:
//
//   query    exact in f16 for entries of at least 2^-28 of the head's largest one, else to within 2^-39 of that one: less than an
//            fp32 sum over the head errs by, unless keys that meet such entries are 2^15 times those that meet the largest ones.
//   weight * scale   two f16 values hold 23 bits: a quarter of the products are rounded, by up to 2^-23 of themselves (root mean
//            square 4.2e-8; an fp32 rounding is 2.4e-8).  Below 2^-29 of the top of their place they are off by up to 2^-52 of that top,
//            2^-46 of what a token at the reference with the group's largest scale has: it counts only where all tokens that
//            weigh anything have scales below 2^-22 of that one.
//
// The quantized classes go through v_mfma_f32_16x16x32_f16 with such operands, in the layout of the walkers
// for two groups (the storage layout is the A operand; columns (g, h) = one group or half of the head x query head):
//
//   logits   A = code - c, an integer (shifted(); c: code_of_zero), B = the query times a
//            power of two.  One product per group of the head (four groups: two sets of two groups' columns), so that scale
//            and minimum come in after the contraction:  s sum(q (code - c)) + (m + c s) sum(q).
//   values   A = code - c, likewise per token and group, B = weight * scale of the token's group, an fp32 number w in two f16 values: hi = w rounded,
//            lo = what is left, 2^12 times as large and in accumulators of its own.  A power of two
//            per group (SplitState::place) keeps w in f16's range; it moves when a scale is larger than those seen so far.
//            The other part of the values, weight * (m + c s), is a sum per lane.
//
// Codes minus a constant, and not the codes themselves, because with them the two parts of a logit or value, which are far larger
// than their sum, would be rounded at their own size.  The instruction's sums are as good as fp32 additions one by one, or
// better (a third of their error over 2048 products).  Errors against 64 bits, relative 2-norm, 16 batches of 196 to 23520 tokens a sequence,
// keys with channel outliers, six draws each: 1.8e-7 to 4.2e-7 (2.4e-7 on average), with fp32 products 2.0e-7 to 4.6e-7 (2.9e-7); a batch's
// is 0.65 to 1.01 times what it was.
//
// Bound by instruction issue: a 32-token block of a head of 128 takes about 370 vector instructions (four groups; 300 with one) of
// four cycles and 32 products of 16; 136 of them unpack codes, 70 split the weights.  Measured, us per call, products in fp32
// on v_mfma_f32_4x4x1 (256 of them, 9.6 cycles each, and a dequantizing instruction per number) -> this: 8 x 12795 tokens, 28 / 4
// heads of 128, group 32: 31.7 -> 21.0, group 128: 31.8 -> 19.2; 4 x 50676, group 32: 53 -> 32; 16 x 6545 tokens, 14 / 2 heads of 64,
// group 64: 14.5 -> 10.6.  (917 us on the vector kernel, the first of these.)
//
// The 16-bit segment keeps fp32 products, on v_mfma_f32_4x4x1_16b_f32: sixteen 4 x 4 products D += a b^T of one contraction
// step each, D's elements the fused multiply-adds that the vector unit computes (bit for bit, subnormals included).  Of its
// 64 A values each meets 4 columns; with the broadcast of one A block to two neighbouring blocks (cbsz = 1, abid = 0 or 1) it
// meets the 8 query heads of a KV head.
//
//   logits   lane (j, m), j = l / 16, m = l % 16, holds quarter j of token m of a 16-token tile: row m % 4 of
//            A block 4j + m / 4.  A step is one channel of every quarter.  B: lane l holds that channel of query l % 8.
//            abid a leaves in D, lane (j, m), element i: token 8 (m / 8) + 4 a + i, query l % 8, the part of quarter j.
//   values   lane (j, m) holds channel 16 ct + m of the tokens 4j .. 4j + 3 of both tiles.  A step is one token of every
//            lane group j.  B: that token's weight for query l % 8.  abid a leaves channel 16 ct + 8 (m / 8) + 4 a + i of
//            query l % 8, the part of lane group j's tokens.
//
// Between them the four quarters' parts are added up and every lane group gets its own tokens, in registers (tokens_of_group);
// at the end of the segment the channels likewise (carry_on).
//
// A wavefront's blocks are a fixed share of its workgroup's range, so that a split count fixes every bit of the result, as it
// does in the vector kernel.
#pragma once

namespace {

// Cost of a 32-token block of the 2-, 4-, 8- and 16-bit class, in the unit of WQ_BLOCK_COST: the quantized classes differ by their
// unpacking and little else.  us per call with these, with those of two groups (100, 130, 230, 500), with 140 for all quantized ones,
// with 250 for the 16-bit class: 8 x 12795 tokens, group 32: 21.0, 24.8, 22.7, 22.4; group 128: 19.1, 22.6, 20.5, 21.3; 4 x 50676,
// group 32: 32.1, 36.3, 33.5, 32.6; 20 ragged ones of up to 15931: 37.5, 46.6, 38.4, 37.6; 16 x 6545, heads of 64: 10.5, 11.6, 10.5, 10.5
constexpr int WQ_BLOCK_COST_F32[4] = {130, 140, 170, 400};
template <int HD, int G>
constexpr int block_cost(int c)
{
    return G != 2 ? WQ_BLOCK_COST_F32[c] : HD == 64 ? WQ_BLOCK_COST_64[c] : WQ_BLOCK_COST[c];
}

template <int HD, int G>
struct F32Smem {
    static constexpr int PITCH = HD + 4;                 // 4 rows apart = 8 banks
    float meta[WQ_WAVES][4][32 * G];                     // per wave: scales and offsets of the current block's K groups, then of its V groups
    uint32_t vzero[WQ_WAVES][16 * G];                    // ... and what is taken off V's codes (f16, tile 0's token and tile 1's)
    __attribute__((aligned(16))) uint16_t vt[WQ_WAVES][32][PITCH];     // per wave: V rows of a 16-bit block, read back one channel per lane
    U4 bq[3][HD / 32][64];                               // query operands of the quantized classes, per lane
    float qx[3][64];                                     // ... their power of two, the sums of set 0's and set 1's group
    // what the body uses (MfmaSmem has the same)
    __attribute__((aligned(16))) float O[WQ_WAVES][WQ_MAX_REP][HD + 4];
    float ml[WQ_WAVES][WQ_MAX_REP][2];
    int expect[64], grown[64];
};

template <int HD>
struct F32State {
    floatx4 O[HD / 16][2];  // [ct][a], element i: channel 16 ct + 8 (m / 8) + 4 a + i of query l % 8, this lane group's tokens
    float m;                // reference of the lane's query (a recent largest logit; the same in all lane groups)
    float l;                // sum of the weights of this lane group's tokens
    float q[HD / 4];        // query l % 8, quarter l / 16
};

template <int A>
__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 1, A, 0);
}

// Vector and matrix instructions don't cross this, others may
__device__ __forceinline__ void apart() { __builtin_amdgcn_sched_barrier(0x3F4); }

// acc0[a] += the products of the A values x0 with the B values y0, acc1[a] those of x1 and y1.  The A values are there before
// the first product: one that follows the vector instruction it needs waits for it (29 cycles per A value in alternation, 24
// in groups of eight).  Four accumulators in turn, so that none waits for its own last product.
__device__ __forceinline__ void mfma_f32_4(const float* x0, const float* y0, floatx4* acc0, const float* x1, const float* y1, floatx4* acc1)
{
    apart();
#pragma unroll
    for (int e = 0; e < 4; e++) {
        acc0[0] = mfma_f32<0>(x0[e], y0[e], acc0[0]);
        acc0[1] = mfma_f32<1>(x0[e], y0[e], acc0[1]);
        acc1[0] = mfma_f32<0>(x1[e], y1[e], acc1[0]);
        acc1[1] = mfma_f32<1>(x1[e], y1[e], acc1[1]);
    }
    apart();
}

// The query of lane l, quarter l / 16 of head l % 8 (zeros beyond the KV head's heads)
template <int HD>
__device__ __forceinline__ void load_q_quarter(const DecodeArgs& a, int b, int kvh, float (&q)[HD / 4])
{
    const int lane = threadIdx.x & 63, h = lane & 7;
    const bool live = h < a.rep;
    const int64_t base = ((int64_t)b * a.Hq + kvh * a.rep + (live ? h : 0)) * HD + (lane >> 4) * (HD / 4);
    if (a.q_dtype == WQ_BF16) {
        const __hip_bfloat16* p = static_cast<const __hip_bfloat16*>(a.q) + base;
#pragma unroll
        for (int k = 0; k < HD / 4; k += 8) wq_ld8(p + k, q + k);
    } else {                                             // (fp32 queries do not come here)
        const __half* p = static_cast<const __half*>(a.q) + base;
#pragma unroll
        for (int k = 0; k < HD / 4; k += 8) wq_ld8(p + k, q + k);
    }
#pragma unroll
    for (int k = 0; k < HD / 4; k++) q[k] = live ? q[k] : 0.f;
}

// Logits of a 16-token tile.  The products of a quarter's channels are added up in two chains, each as long as the vector
// kernel's: a chain's rounding errors grow with its length, and a wide query's logits are the sums of large terms.
struct TileAcc {
    floatx4 v[2][2];        // [chain][a]
};

// From products as the instruction leaves them (a = 0 and 1) to x[i] = the whole sum of row 4j + i, query l % 8, for lane (j, m)
__device__ __forceinline__ void rows_of_group(const floatx4& acc0, const floatx4& acc1, float* x)
{
    const int lane = threadIdx.x & 63;
    const bool own = ((lane >> 3) & 1) == (lane >> 5);   // lane (j, m) has the rows 8 (m / 8) + ..., needs 8 (j / 2) + ...
#pragma unroll
    for (int i = 0; i < 4; i++) {
        // rows 2k and 2k + 1 of 16 lanes: the even one keeps a = 0, the odd one a = 1
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc0[i]), __float_as_uint(acc1[i]), false, false);
        const RowPair h = halves_32(__uint_as_float(r[0]) + __uint_as_float(r[1]));
        const float v = h.even + h.odd, o = ror8(v);
        x[i] = own ? v : o;
    }
}
__device__ __forceinline__ void tokens_of_group(const TileAcc& t, float* x) { rows_of_group(t.v[0][0] + t.v[1][0], t.v[0][1] + t.v[1][1], x); }

// Weights of a block's 8 tokens per lane from their logits (-inf: not there).  A logit of -inf leaves its token out, also
// where all have been -inf so far.
constexpr float F32_SLACK = 3.5f;                  // weights stay below e^3.5 = 2^5.05; the reference moves when a logit is farther up
template <int HD>
__device__ __forceinline__ void softmax_weights(F32State<HD>& st, float* x, float sm_scale, float* p)
{
#pragma unroll
    for (int k = 0; k < 8; k++) x[k] *= sm_scale;
    float lm = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    if (__builtin_amdgcn_ballot_w64(lm > st.m + F32_SLACK) != 0) {
        lm = max_over_rows(lm);
        const float mn = fmaxf(st.m, lm);
        const float alpha = (mn == -INFINITY) ? 1.0f : __expf(st.m - mn);      // 0 on the first block
        st.m = mn;
        st.l *= alpha;
#pragma unroll
        for (int ct = 0; ct < HD / 16; ct++) {
            st.O[ct][0] *= alpha;
            st.O[ct][1] *= alpha;
        }
    }
    const float ref = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        p[k] = __expf(x[k] - ref);
        st.l += p[k];
    }
}

// ---- the quantized classes ----------------------------------------------------------------------------------------
template <int HD, int G>
struct SplitState {
    static constexpr int SETS = G == 4 ? 2 : 1;
    floatx4 O[HD / 16];     // sums of weight * scale * place[set] * (code - c) * 2^-9: row = channel 16 ct + 4 j + i, column = (g, h)
    floatx4 P[HD / 16];     // ... of what the first f16 value left of the weights, 2^12 times as large
    float m;                // reference of head h (a recent largest logit), the same in all lanes of the head
    float l;                // sum of the weights of lane group j's tokens
    float accM[SETS];       // ... of the weights times the offsets of the groups that the lane's column is for
    float place[SETS];      // power of two that brings these groups' weights times scales to at most 2^15
    uint32_t ref;           // the largest magnitude of a scale (its f16 bits) of group j that the places leave room for; 0: none seen
    float own;              // group j's place
};

// The query operands of class CLS, built by one wavefront: lane (j, col) has quarter j of head h = col % 8, times the power of
// two that brings the head's largest entry into [2^14, 2^15): what a 16-bit query holds is exact in f16 then, down to
// 2^-28 of its largest entry, and below that off by no more than 2^-39 of it.  sums[s]: of the scaled query over group 2 s + g (four groups), or over the head (one group).
template <int HD, int CLS, int G>
__device__ __forceinline__ void build_q_split(const DecodeArgs& a, int b, int kvh, U4* Bq, float& unit, float (&sums)[2])
{
    constexpr int QC = HD / 4, NK = HD / 32;
    const int lane = threadIdx.x & 63, g = (lane >> 3) & 1;
    float v[QC];
    load_q_quarter<HD>(a, b, kvh, v);
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < QC; k++) mx = fmaxf(mx, fabsf(v[k]));
    mx = max_over_rows(mx);
    const int eb = (int)((__float_as_uint(mx) >> 23) & 0xFFu), up = min(141 - eb, 126);      // (mx in [2^(eb - 127), 2^(eb - 126)))
    const float scale = __uint_as_float((uint32_t)(127 + up) << 23);
    unit = __uint_as_float((uint32_t)(127 - up) << 23);
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < QC; k++) {
        v[k] *= scale;
        s += v[k];
    }
    const RowPair pair = rows_16(s);                     // the quarters 2 (j / 2) and 2 (j / 2) + 1
    if constexpr (G == 4) {
        const RowPair sets = halves_32(g ? pair.odd : pair.even);
        sums[0] = sets.even;
        sums[1] = sets.odd;
    } else {
        const RowPair halves = halves_32(pair.even + pair.odd);
        sums[0] = halves.even + halves.odd;
        sums[1] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < NK; r++) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            int ch0, ch1, sh;
            k_slot(CLS, r, 2 * e, ch0, sh);
            k_slot(CLS, r, 2 * e + 1, ch1, sh);
            const half2v pair_e = {(_Float16)v[ch0], (_Float16)v[ch1]};
            w[e] = __builtin_bit_cast(uint32_t, pair_e);
        }
        Bq[r] = U4{w[0], w[1], w[2], w[3]};
    }
}

template <int HD, int G>
__device__ __forceinline__ void stage_q_split(const DecodeArgs& a, F32Smem<HD, G>& sm, int b, int kvh, int wave)
{
    const int lane = threadIdx.x & 63;
    U4 Bq[HD / 32];
    float unit, sums[2];
    if (wave >= 3) return;
    if (wave == 0) build_q_split<HD, 0, G>(a, b, kvh, Bq, unit, sums);
    else if (wave == 1) build_q_split<HD, 1, G>(a, b, kvh, Bq, unit, sums);
    else build_q_split<HD, 2, G>(a, b, kvh, Bq, unit, sums);
#pragma unroll
    for (int r = 0; r < HD / 32; r++) sm.bq[wave][r][lane] = Bq[r];
    if (wave == 0) {
        sm.qx[0][lane] = unit;
        sm.qx[1][lane] = sums[0];
        sm.qx[2][lane] = sums[1];
    }
}

// What is contracted is code - c, c the code nearest to the number zero, so that sums over many codes stay as small as those
// over the dequantized numbers themselves (with the middle of the codes, a group that one entry stretches, or one of equal
// entries, whose scale is 1, would be rounded at the size of the middle); the group's minimum goes up by c * scale.
template <int BITS>
__device__ __forceinline__ float code_of_zero(float s, float m)
{
    return __builtin_amdgcn_fmed3f(rintf(-m * __builtin_amdgcn_rcpf(fmaxf(s, 0x1p-25f))), 0.f, (float)((1 << BITS) - 1));     // (padding has scale 0)
}
// A raw operand (k_operand, v_operand: f16 subnormals code * 2^(shift - 24)) as (code - c) * 2^-9, c512 = -c * 2^-9 per slot: one
// fused multiply-add of two f16 at a time, exact
__device__ __forceinline__ half8 shifted(half8 raw, const half2v (&c512)[4], int sh0, int sh1, int sh2, int sh3)
{
    const int sh[4] = {sh0, sh1, sh2, sh3};
    const U4 u = __builtin_bit_cast(U4, raw);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const _Float16 p = (_Float16)pow2_of((float)(15 - sh[v]));
        w[v] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(half2v, w[v]), half2v{p, p}, c512[v]));
    }
    return as_half8(w[0], w[1], w[2], w[3]);
}

// Two numbers divided by 2^12, in f16; and what that leaves of them, in f16 (one instruction each: products and sums in fp32,
// rounded once)
__device__ __forceinline__ uint32_t scaled_f16(float x, float y)
{
    const half2v r = {(_Float16)fmaf(x, 1.0f / 4096.0f, 0.f), (_Float16)fmaf(y, 1.0f / 4096.0f, 0.f)};
    uint32_t u = __builtin_bit_cast(uint32_t, r);
    asm("" : "+v"(u));                             // (the second one is read where it lies, not computed again into a low half)
    return u;
}
__device__ __forceinline__ uint32_t rest_f16(float x, float y, uint32_t h)
{
    const half2v r = {(_Float16)fmaf(f16lo(h), -4096.0f, x), (_Float16)fmaf(f16hi(h), -4096.0f, y)};
    return __builtin_bit_cast(uint32_t, r);
}

template <int HD, int BITS, int G>
struct SplitFrag {
    static constexpr int KDW = (HD / 4) * BITS / 32;        // dwords of K codes per lane per 16-token tile
    static constexpr int VDW = (HD / 16) * 8 * BITS / 32;   // dwords of V codes per lane per 32-token block
    uint32_t k[2][KDW], v[VDW], km[2], vm[2];               // km, vm: metadata of token l % 16 of each tile, group j
};

// this wavefront's blocks [blk, end) of one class of one (sequence, KV head): len tokens from token slot tok_base
template <int HD, int BITS, int G, int DEPTH>
__device__ __forceinline__ void walk_class_split(const DecodeArgs& a, F32Smem<HD, G>& sm, int b, int kvh, int len, int tok_base, int blk, int end,
                                                 Tickets& tk, SplitState<HD, G>& st)
{
    static_assert(G == 1 || (G == 4 && HD == 128), "a quarter of the head lies in one group");
    constexpr int C = BITS == 2 ? 0 : (BITS == 4 ? 1 : 2), CT = HD / 16, NK = HD / 32, SETS = SplitState<HD, G>::SETS;
    using F = SplitFrag<HD, BITS, G>;
    if (blk >= end) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4, g = (lane >> 3) & 1;
    const wq_packed_kv& kv = a.kv;
    const int64_t cap = kv.cap[C];
    const uint8_t* kbase = static_cast<const uint8_t*>(kv.codes[C]) + ((int64_t)kvh * cap + tok_base) * HD * BITS / 8 + lane * (F::KDW * 4);
    const uint8_t* vbase = static_cast<const uint8_t*>(kv.codes[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * HD * BITS / 8 + lane * (F::VDW * 4);
    const uint32_t* kmeta = static_cast<const uint32_t*>(kv.meta[C]) + ((int64_t)kvh * cap + tok_base) * G + (G == 4 ? lane : lane & 15);
    const uint32_t* vmeta = static_cast<const uint32_t*>(kv.meta[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * G + (G == 4 ? lane : lane & 15);
    float* const words = sm.meta[wave][0];

    auto load = [&](int n, F& f) {
        const int64_t o = (int64_t)n * (32 * HD * BITS / 8);
        load_dwords<HD, F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o), f.k[0]);
        load_dwords<HD, F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o + 16 * HD * BITS / 8), f.k[1]);
        load_dwords<HD, F::VDW>(reinterpret_cast<const uint32_t*>(vbase + o), f.v);
#pragma unroll
        for (int t = 0; t < 2; t++) {
            f.km[t] = load_word<HD>(kmeta + (int64_t)n * (32 * G) + t * (16 * G));
            f.vm[t] = load_word<HD>(vmeta + (int64_t)n * (32 * G) + t * (16 * G));
        }
    };
    F f[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; d++)
        if (blk + d < end) load(blk + d, f[d]);
    pass_setup_barrier(b, tk);
    // B operands: column (g, h) of set s takes the channels of group 2 s + g (four groups), or of half g of the head
    half8 Bq[SETS][NK];
#pragma unroll
    for (int r = 0; r < NK; r++) {
        const U4 q = sm.bq[C][r][lane];
#pragma unroll
        for (int s = 0; s < SETS; s++) {
            const bool mine = G == 4 ? j == 2 * s + g : (j >> 1) == g;
            Bq[s][r] = as_half8(mine ? q.x : 0u, mine ? q.y : 0u, mine ? q.z : 0u, mine ? q.w : 0u);
        }
    }
    // (a finite positive number whatever the softmax scale: -inf and 0 are among the logits that it multiplies)
    const float cexp = __builtin_amdgcn_fmed3f(a.sm_scale * sm.qx[0][lane] * 512.0f, 0x1p-126f, 0x1.fffffep127f);
    float qs[SETS];
#pragma unroll
    for (int s = 0; s < SETS; s++) qs[s] = sm.qx[1 + s][lane] * (1.0f / 512.0f);

    auto compute = [&](int n, const F& f) {
        // ---- a scale beyond what the places leave room for moves them, twice as far (rarely: the first block does).  Magnitudes:
        //      a group of nearly equal fp32 values can have a negative scale ----
        uint32_t top = max(f.vm[0] & 0x7FFFu, f.vm[1] & 0x7FFFu);
        if (__builtin_amdgcn_ballot_w64(top > st.ref) != 0) {
            auto moved = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, false); };
            top = max(top, moved(top, std::integral_constant<int, 0x128>{}));
            top = max(top, moved(top, std::integral_constant<int, 0x124>{}));
            top = max(top, moved(top, std::integral_constant<int, 0x122>{}));
            top = max(top, moved(top, std::integral_constant<int, 0x121>{}));
            if (top > st.ref) st.ref = min(top + (1u << 10), 0x7BFFu);
            // weights are below 2^5.1, scales up to ref, which is below 2^(e - 14): their products below 2^15.1
            const int e = (int)(st.ref >> 10);
            st.own = st.ref == 0u ? 1.0f : pow2_of((float)(24 - e));
#pragma unroll
            for (int s = 0; s < SETS; s++) {
                float to = st.own;
                if constexpr (G == 4) {
                    const float even = lane_value(st.own, 32 * s), odd = lane_value(st.own, 32 * s + 16);
                    to = g ? odd : even;
                }
                const float by = to * (1.0f / st.place[s]);        // (powers of two)
                st.place[s] = to;
#pragma unroll
                for (int ct = s * (CT / SETS); ct < (s + 1) * (CT / SETS); ct++) {
                    st.O[ct] *= by;
                    st.P[ct] *= by;
                }
            }
        }
        // ---- scales and offsets: a lane's words in, the ones of its tokens and column out, V's scales times 2^12 of their place ----
        half2v kzero[2], vzero;
        float koff[2], voff[2];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const float kc = code_of_zero<BITS>(f16lo(f.km[t]), f16hi(f.km[t])), vc = code_of_zero<BITS>(f16lo(f.vm[t]), f16hi(f.vm[t]));
            kzero[t] = half2v{(_Float16)(kc * (-1.0f / 512.0f)), (_Float16)(kc * (-1.0f / 512.0f))};
            vzero[t] = (_Float16)(vc * (-1.0f / 512.0f));
            koff[t] = fmaf(f16lo(f.km[t]), kc, f16hi(f.km[t]));
            voff[t] = fmaf(f16lo(f.vm[t]), vc, f16hi(f.vm[t]));
        }
        if (G == 4 || lane < 16) {
#pragma unroll
            for (int t = 0; t < 2; t++) {
                float* const at = words + 16 * G * t + lane;
                at[0] = f16lo(f.km[t]);
                at[32 * G] = koff[t];
                at[64 * G] = fmaf(f16lo(f.vm[t]), st.own * 4096.0f, 0.f);
                at[96 * G] = voff[t];
            }
            sm.vzero[wave][lane] = __builtin_bit_cast(uint32_t, vzero);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        auto words_of = [&](int kind, int s, float (&w)[8]) {      // tokens 4 j + i of both tiles, the group of set s
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const float4 u = *reinterpret_cast<const float4*>(words + kind * (32 * G) + (t * G + (G == 4 ? 2 * s + g : 0)) * 16 + 4 * j);
                w[4 * t] = u.x, w[4 * t + 1] = u.y, w[4 * t + 2] = u.z, w[4 * t + 3] = u.w;
            }
        };
        // ---- logits of the two 16-token tiles ----
        float x[8], p[8], ks[SETS][8], kc[SETS][8];
#pragma unroll
        for (int s = 0; s < SETS; s++) {
            words_of(0, s, ks[s]);
            words_of(1, s, kc[s]);
        }
        floatx4 acc[2][SETS];                      // (two or four chains of products at a time)
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int s = 0; s < SETS; s++) acc[t][s] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < NK; r++) {
            int ch, sh[4];
#pragma unroll
            for (int v = 0; v < 4; v++) k_slot(C, r, 2 * v, ch, sh[v]);
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const half2v kc4[4] = {kzero[t], kzero[t], kzero[t], kzero[t]};
                const half8 codes = shifted(k_operand<BITS>(f.k[t], r), kc4, sh[0], sh[1], sh[2], sh[3]);
#pragma unroll
                for (int s = 0; s < SETS; s++) acc[t][s] = mfma(codes, Bq[s][r], acc[t][s]);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int k = 4 * t + i;
                if constexpr (G == 4) {
                    const float y = fmaf(ks[1][k], acc[t][1][i], fmaf(kc[1][k], qs[1], fmaf(ks[0][k], acc[t][0][i], kc[0][k] * qs[0])));
                    x[k] = y + ror8(y);
                } else {                           // (both halves of the head are of one group: their products first)
                    x[k] = fmaf(ks[0][k], acc[t][0][i] + ror8(acc[t][0][i]), kc[0][k] * qs[0]);
                }
            }
        const int nv = len - n * 32;               // (the class's last block of the sequence can be a partial one)
        if (nv < 32) {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (16 * (k >> 2) + 4 * j + (k & 3) >= nv) x[k] = -INFINITY;
        }
        // ---- weights, as softmax_weights ----
        float lm = max3(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5]), max3(x[6], x[7], x[7])) * cexp;      // (cexp > 0)
        if (__builtin_amdgcn_ballot_w64(lm > st.m + F32_SLACK) != 0) {
            lm = max_over_rows(lm);
            const float mn = fmaxf(st.m, lm);
            const float alpha = (mn == -INFINITY) ? 1.0f : __expf(st.m - mn);      // 0 on the first block
            st.m = mn;
            st.l *= alpha;
#pragma unroll
            for (int s = 0; s < SETS; s++) st.accM[s] *= alpha;
#pragma unroll
            for (int ct = 0; ct < CT; ct++) {
                st.O[ct] *= alpha;
                st.P[ct] *= alpha;
            }
        }
        const float ref = st.m == -INFINITY ? 0.f : st.m;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            p[k] = __expf(fmaf(x[k], cexp, -ref));
            st.l += p[k];
        }
        // ---- the weights times the scales in two f16 values each, the second 2^12 times what is left; slots (2v, 2v+1) =
        //      (tile 0, tile 1) token 4j+v ----
        half8 hi[SETS], lo[SETS];
#pragma unroll
        for (int s = 0; s < SETS; s++) {
            float vs[8], vc[8];
            words_of(2, s, vs);
            words_of(3, s, vc);
            uint32_t h[4], l[4];
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const float w0 = p[v] * vs[v], w1 = p[4 + v] * vs[4 + v];
                h[v] = scaled_f16(w0, w1);
                l[v] = rest_f16(w0, w1, h[v]);
            }
            hi[s] = as_half8(h[0], h[1], h[2], h[3]);
            lo[s] = as_half8(l[0], l[1], l[2], l[3]);
#pragma unroll
            for (int k = 0; k < 8; k++) st.accM[s] = fmaf(p[k], vc[k], st.accM[s]);
        }
        half2v vc4[G][4];
#pragma unroll
        for (int k = 0; k < G; k++) {
            const uint4 u = *reinterpret_cast<const uint4*>(sm.vzero[wave] + 16 * k + 4 * j);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int v = 0; v < 4; v++) vc4[k][v] = __builtin_bit_cast(half2v, w[v]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();           // the next block's words may overwrite the buffer after this point
        // ---- values ----
#pragma unroll
        for (int ct = 0; ct < CT; ct++) {
            constexpr int PER = CT / SETS;
            const half8 codes = shifted(v_operand<BITS>(f.v, ct), vc4[ct / (CT / G)], (int)v_slot_shift<BITS>(0), (int)v_slot_shift<BITS>(1),
                                               (int)v_slot_shift<BITS>(2), (int)v_slot_shift<BITS>(3));
            st.P[ct] = mfma(codes, lo[ct / PER], st.P[ct]);
            st.O[ct] = mfma(codes, hi[ct / PER], st.O[ct]);
        }
    };

    while (true) {
#pragma unroll
        for (int d = 0; d < DEPTH; d++) {
            compute(blk, f[d]);
            if (blk + DEPTH < end) load(blk + DEPTH, f[d]);
            if (++blk >= end) return;
        }
    }
}

// ---- the 16-bit segment: rows are plain [token][Hkv][hd], so the K side is the A operand straight from memory (a
// quarter of a token's row per lane); V rows go through LDS and are read back one channel per lane.  Rows past the end stand
// in as zeros.  new_row >= 0: row new_row (= len - 1) is not in the cache yet, it is read from k_new / v_new.
template <int HD, bool BF, int G>
__device__ __forceinline__ void walk_seg16_f32(const DecodeArgs& a, F32Smem<HD, G>& sm, int b, int kvh, int len, int first_row, int blk, int end,
                                               Tickets& tk, F32State<HD>& st, int new_row)
{
    constexpr int CT = HD / 16, KDW = HD / 8, VIT = 32 * HD * 2 / (16 * 64);       // VIT: 16-byte pieces of V per lane
    constexpr int PITCH = F32Smem<HD, G>::PITCH;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4, m = lane & 15;
    const wq_packed_kv& kv = a.kv;
    const int64_t rstride = (int64_t)kv.Hkv * HD;
    const uint16_t* k16 = static_cast<const uint16_t*>(kv.k16) + first_row * rstride + (int64_t)kvh * HD;
    const uint16_t* v16 = static_cast<const uint16_t*>(kv.v16) + first_row * rstride + (int64_t)kvh * HD;
    const uint16_t *const knew = a.k_new + ((int64_t)b * kv.Hkv + kvh) * HD, *const vnew = a.v_new + ((int64_t)b * kv.Hkv + kvh) * HD;     // (read where there is a new row)
    uint16_t* const vt = &sm.vt[wave][0][0];
    auto number = [](uint32_t u) { return BF ? wq_bf16_bits_to_float(u) : wq_f16_bits_to_float(u); };
    pass_setup_barrier(b, tk);
    for (; blk < end; blk++) {
        const int nv = len - blk * 32;
        uint32_t kd[2][KDW];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int tok = min(blk * 32 + 16 * t + m, len - 1);
            const uint16_t* src_k = tok == new_row ? knew : k16 + tok * rstride;
            load_dwords<HD, KDW>(reinterpret_cast<const uint32_t*>(src_k + j * (HD / 4)), kd[t]);
        }
        uint4 vd[VIT];
#pragma unroll
        for (int it = 0; it < VIT; it++) {
            const int chunk = it * 64 + lane, row = chunk / (HD / 8), piece = chunk % (HD / 8);
            const int tok = min(blk * 32 + row, len - 1);
            const uint16_t* src_v = tok == new_row ? vnew : v16 + tok * rstride;
            vd[it] = *reinterpret_cast<const uint4*>(src_v + piece * 8);
        }
        // ---- logits ----
        float x[8], p[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            TileAcc acc = {};
#pragma unroll
            for (int e0 = 0; e0 < HD / 8; e0 += 4) {
                float kh[2][4];
#pragma unroll
                for (int c = 0; c < 2; c++)
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const uint32_t u = kd[t][(c * (HD / 8) + e0 + e) / 2];
                        kh[c][e] = number((e & 1) ? u >> 16 : u & 0xFFFFu);
                    }
                mfma_f32_4(kh[0], st.q + e0, acc.v[0], kh[1], st.q + HD / 8 + e0, acc.v[1]);
            }
            tokens_of_group(acc, x + 4 * t);
        }
#pragma unroll
        for (int k = 0; k < 8; k++)
            if (16 * (k >> 2) + 4 * j + (k & 3) >= nv) x[k] = -INFINITY;
        softmax_weights<HD>(st, x, a.sm_scale, p);
        // ---- values ----
#pragma unroll
        for (int it = 0; it < VIT; it++) {
            const int chunk = it * 64 + lane, row = chunk / (HD / 8), piece = chunk % (HD / 8);
            const bool there = row < nv;
            uint2* const dst = reinterpret_cast<uint2*>(vt + row * PITCH + piece * 8);   // (the pitch is 8-byte aligned)
            dst[0] = there ? uint2{vd[it].x, vd[it].y} : uint2{0u, 0u};
            dst[1] = there ? uint2{vd[it].z, vd[it].w} : uint2{0u, 0u};
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int ct = 0; ct < CT; ct += 2)
#pragma unroll
            for (int t = 0; t < 2; t++) {
                float vh[2][4];
#pragma unroll
                for (int c = 0; c < 2; c++)
#pragma unroll
                    for (int i = 0; i < 4; i++) vh[c][i] = number(vt[(16 * t + 4 * j + i) * PITCH + 16 * (ct + c) + m]);
                mfma_f32_4(vh[0], p + 4 * t, st.O[ct], vh[1], p + 4 * t, st.O[ct + 1]);
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();           // the buffer is overwritten next
    }
}

// What walk_seg16_f32 leaves, as the walkers of the quantized classes carry it on: the lane groups' parts added up, and every
// lane its own channels (tokens_of_group does the same to a tile's logits)
template <int HD, int G>
__device__ __forceinline__ void carry_on(const F32State<HD>& from, SplitState<HD, G>& st)
{
    st.m = from.m;
    st.l = from.l;
#pragma unroll
    for (int ct = 0; ct < HD / 16; ct++) {
        float x[4];
        rows_of_group(from.O[ct][0], from.O[ct][1], x);
        st.O[ct] = floatx4{x[0], x[1], x[2], x[3]} * (1.0f / 512.0f) * ((G == 4 && ct >= HD / 32) ? st.place[SplitState<HD, G>::SETS - 1] : st.place[0]);
    }
}

// The wavefront's numerators, reference and weight sum to LDS for the merge
template <int HD, int G>
__device__ __forceinline__ void hand_over_split(F32Smem<HD, G>& sm, const SplitState<HD, G>& st)
{
    constexpr int CT = HD / 16, SETS = SplitState<HD, G>::SETS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4, g = (lane >> 3) & 1, h = lane & 7;
    const float l = sum_over_rows(st.l);
    float am[SETS], unit[SETS];
#pragma unroll
    for (int s = 0; s < SETS; s++) {
        am[s] = sum_over_rows(st.accM[s]);
        unit[s] = 512.0f / st.place[s];
    }
#pragma unroll
    for (int ct = 0; ct < CT; ct++) {
        const int s = ct / (CT / SETS);
        if (g == (G == 4 ? ct / (CT / 4) % 2 : 0)) {       // this column's group owns channel tile ct
            floatx4 v;
#pragma unroll
            for (int i = 0; i < 4; i++) v[i] = fmaf(fmaf(st.P[ct][i], 1.0f / 4096.0f, st.O[ct][i]), unit[s], am[s]);
            *reinterpret_cast<floatx4*>(&sm.O[wave][h][16 * ct + 4 * j]) = v;
        }
    }
    if (lane < 8) {
        sm.ml[wave][h][0] = st.m;
        sm.ml[wave][h][1] = l;
    }
}

}  // namespace
