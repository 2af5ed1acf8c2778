// a4, matrix-core path in fp32: the walkers of caches with one or four groups per head.
// (included by wq_decode_mfma.h, whose body cuts the work and merges it)
//
// These group counts keep the arithmetic of the vector kernel (k_decode_generic): a key or value is dequantized by one fp32
// fused multiply-add, fma(scale, code, minimum); queries, logits, weights and sums are fp32.  Nothing is rounded to 16 bits,
// so that neither the spread of a query nor that of the value scales costs accuracy, and v_scale_max is not read.  (Two f16
// values per weight, placed by the sequence's largest value scale, lost 2.5e-4 of a group whose scale is 2^-12 of that.)
//
// The instruction is v_mfma_f32_4x4x1_16b_f32: sixteen 4 x 4 products D += a b^T of one contraction step each, D's elements
// the fused multiply-adds that the vector unit computes (bit for bit, subnormals included).  Of its 64 A values each meets 4
// columns; with the broadcast of one A block to two neighbouring blocks (cbsz = 1, abid = 0 or 1) it meets the 8 query heads
// of a KV head, and no part of the instruction is idle (in 16 x 16 tiles half the columns would be): 115 TFLOP/s measured,
// against 146 / 2.  The storage layout (wq.h) is the A operand as it stands:
//
//   logits   lane (j, m), j = l / 16, m = l % 16, holds the codes of quarter j of token m of a 16-token tile: row m % 4 of
//            A block 4j + m / 4.  A step is one channel of every quarter.  B: lane l holds that channel of query l % 8.
//            abid a leaves in D, lane (j, m), element i: token 8 (m / 8) + 4 a + i, query l % 8, the part of quarter j.
//   values   lane (j, m) holds channel 16 ct + m of the tokens 4j .. 4j + 3 of both tiles.  A step is one token of every
//            lane group j.  B: that token's weight for query l % 8.  abid a leaves channel 16 ct + 8 (m / 8) + 4 a + i of
//            query l % 8, the part of lane group j's tokens.
//
// Between them the four quarters' parts are added up and every lane group gets its own tokens, in registers (tokens_of_group).
//
// Bound by instruction issue: a 32-token block takes 2 HD matrix instructions (9.6 cycles each) and about as much again on the
// vector unit, and neither overlaps the other to speak of, not even between the two wavefronts of a SIMD.  Codes are therefore
// converted by the dequantizing instruction itself: masked in place, a code is the f16 subnormal code * 2^(shift - 24), which
// a mixed-precision fused multiply-add takes as it is; the power of two is put into the scale (keys) or into the minimum and
// the weight (values), where it changes no rounding.  A workgroup's 32-token block takes 0.49 us with heads of 128, 0.29 with
// heads of 64 (0.60 and 0.32 in the 16-bit segment); 8 x 12795 tokens, 28 / 4 heads of 128, group 32: 917 us a call on the
// vector kernel, 34.0 here.  A wavefront's blocks are a fixed share of its workgroup's range, so that a split count fixes every bit of
// the result, as it does in the vector kernel.
#pragma once

namespace {

// cost of a 32-token block of the 2-, 4-, 8- and 16-bit class, in the unit of WQ_BLOCK_COST (the classes do the same matrix
// instructions here)
constexpr int WQ_BLOCK_COST_F32[4] = {400, 400, 420, 500};
template <int HD, int G>
constexpr int block_cost(int c)
{
    return G != 2 ? WQ_BLOCK_COST_F32[c] : HD == 64 ? WQ_BLOCK_COST_64[c] : WQ_BLOCK_COST[c];
}

template <int HD, int G>
struct F32Smem {
    static constexpr int PITCH = HD + 4;                 // 4 rows apart = 8 banks
    uint32_t meta[WQ_WAVES][32 * G];                     // per wave: V metadata words of the current block
    __attribute__((aligned(16))) uint16_t vt[WQ_WAVES][32][PITCH];     // per wave: V rows of a 16-bit block, read back one channel per lane
    // what the body uses (MfmaSmem has the same)
    float O[WQ_WAVES][WQ_MAX_REP][HD + 1];
    float ml[WQ_WAVES][WQ_MAX_REP][2];
    unsigned next_ticket;
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

// From the products of a tile (see above) to x[i] = the whole logit of token 4j + i, query l % 8, for lane (j, m)
__device__ __forceinline__ void tokens_of_group(const TileAcc& t, float* x)
{
    const floatx4 acc0 = t.v[0][0] + t.v[1][0], acc1 = t.v[0][1] + t.v[1][1];
    const int lane = threadIdx.x & 63;
    const bool own = ((lane >> 3) & 1) == (lane >> 5);   // lane (j, m) has the tokens 8 (m / 8) + ..., needs 8 (j / 2) + ...
#pragma unroll
    for (int i = 0; i < 4; i++) {
        // rows 2k and 2k + 1 of 16 lanes: the even one keeps a = 0, the odd one a = 1
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc0[i]), __float_as_uint(acc1[i]), false, false);
        const RowPair h = halves_32(__uint_as_float(r[0]) + __uint_as_float(r[1]));
        const float v = h.even + h.odd, o = ror8(v);
        x[i] = own ? v : o;
    }
}

// Weights of a block's 8 tokens per lane from their logits (-inf: not there).  A logit of -inf leaves its token out, also
// where all have been -inf so far.
template <int HD>
__device__ __forceinline__ void softmax_weights(F32State<HD>& st, float* x, float sm_scale, float* p)
{
    constexpr float SLACK = 3.5f;                  // weights stay below e^SLACK; the reference moves when a logit is farther up
#pragma unroll
    for (int k = 0; k < 8; k++) x[k] *= sm_scale;
    float lm = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    if (__builtin_amdgcn_ballot_w64(lm > st.m + SLACK) != 0) {
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

template <int HD, int BITS, int G>
struct F32Frag {
    static constexpr int KDW = (HD / 4) * BITS / 32;        // dwords of K codes per lane per 16-token tile
    static constexpr int VDW = (HD / 16) * 8 * BITS / 32;   // dwords of V codes per lane per 32-token block
    static constexpr int VM = G == 4 ? 2 : 1;               // V metadata words per lane per block
    uint32_t k[2][KDW], v[VDW], km[2], vm[VM];
};

// this wavefront's blocks [blk, end) of one class of one (sequence, KV head): len tokens from token slot tok_base
template <int HD, int BITS, int G>
__device__ __forceinline__ void walk_class_f32(const DecodeArgs& a, F32Smem<HD, G>& sm, int b, int kvh, int len, int tok_base, int blk, int end,
                                               Tickets& tk, F32State<HD>& st)
{
    static_assert(G == 1 || (G == 4 && HD == 128), "a quarter of the head lies in one group");
    constexpr int C = BITS == 2 ? 0 : (BITS == 4 ? 1 : 2), CT = HD / 16, DEPTH = 2;
    using F = F32Frag<HD, BITS, G>;
    if (blk >= end) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4;
    const wq_packed_kv& kv = a.kv;
    const int64_t cap = kv.cap[C];
    const uint8_t* kbase = static_cast<const uint8_t*>(kv.codes[C]) + ((int64_t)kvh * cap + tok_base) * HD * BITS / 8 + lane * (F::KDW * 4);
    const uint8_t* vbase = static_cast<const uint8_t*>(kv.codes[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * HD * BITS / 8 + lane * (F::VDW * 4);
    // the word of a K tile's token m and quarter j's group: the lane's own with four groups
    const uint32_t* kmeta = static_cast<const uint32_t*>(kv.meta[C]) + ((int64_t)kvh * cap + tok_base) * G + (G == 4 ? lane : lane & 15);
    const uint32_t* vmeta = static_cast<const uint32_t*>(kv.meta[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * G + (G == 4 ? lane : lane & 31);
    uint32_t* const words = sm.meta[wave];

    auto load = [&](int n, F& f) {
        const int64_t o = (int64_t)n * (32 * HD * BITS / 8);
        load_dwords<F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o), f.k[0]);
        load_dwords<F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o + 16 * HD * BITS / 8), f.k[1]);
        load_dwords<F::VDW>(reinterpret_cast<const uint32_t*>(vbase + o), f.v);
#pragma unroll
        for (int t = 0; t < 2; t++) f.km[t] = kmeta[(int64_t)n * (32 * G) + t * (16 * G)];
#pragma unroll
        for (int k = 0; k < F::VM; k++) f.vm[k] = vmeta[(int64_t)n * (32 * G) + 64 * k];
    };
    auto compute = [&](int n, const F& f) {
        // ---- value words: one or two per lane in, per group the lane group's 4 tokens x 2 tiles out ----
        if (G == 4 || lane < 32) {
#pragma unroll
            for (int k = 0; k < F::VM; k++) words[64 * k + lane] = f.vm[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // ---- logits ----
        float x[8], p[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const float s = f16lo(f.km[t]) * 16777216.0f, mn = f16hi(f.km[t]);
            TileAcc acc = {};
#pragma unroll
            for (int r = 0; r < HD / 64; r++) {
                const half8 codes[2] = {k_operand<BITS>(f.k[t], r), k_operand<BITS>(f.k[t], r + HD / 64)};
#pragma unroll
                for (int e0 = 0; e0 < 8; e0 += 4) {
                    float kh[2][4], q[2][4];
#pragma unroll
                    for (int c = 0; c < 2; c++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            int ch, sh;
                            k_slot(C, r + c * (HD / 64), e0 + e, ch, sh);
                            kh[c][e] = fmaf(s * pow2_of(-(float)sh), (float)codes[c][e0 + e], mn);
                            q[c][e] = st.q[ch];
                        }
                    mfma_f32_4(kh[0], q[0], acc.v[0], kh[1], q[1], acc.v[1]);
                }
            }
            tokens_of_group(acc, x + 4 * t);
        }
        const int nv = len - n * 32;               // (the class's last block of the sequence can be a partial one)
        if (nv < 32) {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (16 * (k >> 2) + 4 * j + (k & 3) >= nv) x[k] = -INFINITY;
        }
        softmax_weights<HD>(st, x, a.sm_scale, p);
        // ---- values: a token's codes carry 2^(shift - 24), its minimum is given the same factor, its weight the inverse ----
        float pu[8], unit[8];
#pragma unroll
        for (int tau = 0; tau < 8; tau++) {
            unit[tau] = pow2_of(v_slot_shift<BITS>(tau & 3) - 24.0f);
            pu[tau] = p[tau] * pow2_of(24.0f - v_slot_shift<BITS>(tau & 3));
        }
#pragma unroll
        for (int g = 0; g < G; g++) {
            uint32_t w[8];
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const uint4 u = *reinterpret_cast<const uint4*>(words + (t * G + g) * 16 + 4 * j);
                w[4 * t] = u.x, w[4 * t + 1] = u.y, w[4 * t + 2] = u.z, w[4 * t + 3] = u.w;
            }
            float mn[8];
#pragma unroll
            for (int tau = 0; tau < 8; tau++) mn[tau] = fmaf(f16hi(w[tau]), unit[tau], 0.f);       // (one mixed-precision instruction)
#pragma unroll
            for (int ct = g * (CT / G); ct < (g + 1) * (CT / G); ct += 2) {
                const half8 codes[2] = {v_operand<BITS>(f.v, ct), v_operand<BITS>(f.v, ct + 1)};
#pragma unroll
                for (int e0 = 0; e0 < 8; e0 += 4) {
                    float vh[2][4], pw[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int tau = 4 * (e & 1) + ((e0 + e) >> 1);
                        vh[0][e] = fmaf(f16lo(w[tau]), (float)codes[0][e0 + e], mn[tau]);
                        vh[1][e] = fmaf(f16lo(w[tau]), (float)codes[1][e0 + e], mn[tau]);
                        pw[e] = pu[tau];
                    }
                    mfma_f32_4(vh[0], pw, st.O[ct], vh[1], pw, st.O[ct + 1]);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();           // the next block's words may overwrite the buffer after this point
    };

    F f[DEPTH];                                    // one block is loaded while the other is worked on
    load(blk, f[0]);
    if (blk + 1 < end) load(blk + 1, f[1]);
    pass_setup_barrier(a, b, tk);
    while (true) {
#pragma unroll
        for (int d = 0; d < DEPTH; d++) {
            compute(blk, f[d]);
            if (blk + DEPTH < end) load(blk + DEPTH, f[d]);
            if (++blk >= end) return;
        }
    }
}

// ... and of the 16-bit segment: rows are plain [token][Hkv][hd], so the K side is the A operand straight from memory (a
// quarter of a token's row per lane); V rows go through LDS and are read back one channel per lane.  Rows past the end stand
// in as zeros.  new_row >= 0: row new_row (= len - 1) is not in the cache yet, it is read from knew / vnew.
template <int HD, bool BF, int G>
__device__ __forceinline__ void walk_seg16_f32(const DecodeArgs& a, F32Smem<HD, G>& sm, int b, int kvh, int len, int first_row, int blk, int end,
                                               Tickets& tk, F32State<HD>& st, int new_row, const uint16_t* knew, const uint16_t* vnew)
{
    constexpr int CT = HD / 16, KDW = HD / 8, VIT = 32 * HD * 2 / (16 * 64);       // VIT: 16-byte pieces of V per lane
    constexpr int PITCH = F32Smem<HD, G>::PITCH;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4, m = lane & 15;
    const wq_packed_kv& kv = a.kv;
    const int64_t rstride = (int64_t)kv.Hkv * HD;
    const uint16_t* k16 = static_cast<const uint16_t*>(kv.k16) + first_row * rstride + (int64_t)kvh * HD;
    const uint16_t* v16 = static_cast<const uint16_t*>(kv.v16) + first_row * rstride + (int64_t)kvh * HD;
    uint16_t* const vt = &sm.vt[wave][0][0];
    auto number = [](uint32_t u) { return BF ? wq_bf16_bits_to_float(u) : wq_f16_bits_to_float(u); };
    pass_setup_barrier(a, b, tk);
    for (; blk < end; blk++) {
        const int nv = len - blk * 32;
        uint32_t kd[2][KDW];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int tok = min(blk * 32 + 16 * t + m, len - 1);
            const uint16_t* src_k = tok == new_row ? knew : k16 + tok * rstride;
            load_dwords<KDW>(reinterpret_cast<const uint32_t*>(src_k + j * (HD / 4)), kd[t]);
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

// The lane groups' parts added up, the wavefront's numerators, reference exponent and weight sum to LDS for the merge
template <int HD, int G>
__device__ __forceinline__ void hand_over_f32(F32Smem<HD, G>& sm, const F32State<HD>& st)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = lane >> 4, m = lane & 15, h = lane & 7;
    const float l = sum_over_rows(st.l);
#pragma unroll
    for (int ct = 0; ct < HD / 16; ct++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            // even rows of 16 lanes keep a = 0, odd ones a = 1
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(st.O[ct][0][i]), __float_as_uint(st.O[ct][1][i]), false, false);
            const RowPair s = halves_32(__uint_as_float(r[0]) + __uint_as_float(r[1]));
            if (j < 2) sm.O[wave][h][16 * ct + 8 * (m >> 3) + 4 * j + i] = s.even + s.odd;
        }
    if (lane < 8) {
        sm.ml[wave][h][0] = st.m;
        sm.ml[wave][h][1] = l;
    }
}

}  // namespace
