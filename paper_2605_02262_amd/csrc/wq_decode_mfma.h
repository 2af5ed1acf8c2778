// a4, matrix-core path: decode attention over the packed cache (Alg. 2 decode half).
// (included by wq_decode.hip, after DecodeArgs and load_q)
//
// The walkers here and the text below are those of two groups per head (hd/group == 2).  One and four groups have walkers of
// their own, of fp32 accuracy (wq_decode_f32.h); the body at the end of this file cuts and merges the work of both.
//
// One wavefront walks 32-token blocks of a class on its own (no workgroup barrier inside the loop):
//
//   S^T = K_codes . Q^T      v_mfma_f32_16x16x32_f16, A = 16 tokens x 32 contraction slots of raw codes,
//                            B = query heads.  The 16 output columns are (group g, head h): B is block-diagonal,
//                            slots 0..15 carry group-0 channels and feed columns 0..7, slots 16..31 carry group-1
//                            channels and feed columns 8..15, so one accumulator tile holds both groups' integer
//                            dot products and every lane of the softmax has real work (7 of 8 columns per half).
//   dequant                  logit = s0*D0 + m0*sum(q over group 0) + s1*D1 + m1*sum(q over group 1): each lane
//                            applies its own group's (s, m), the two halves meet with one DPP row rotate.
//   online softmax           reference exponent per column, shared by the wavefront's four lane groups.  It starts
//                            as the first block's largest logit and moves (with a rescale of the output
//                            accumulators) only when a logit exceeds it by more than 2^8: weights stay below
//                            2^8, far inside what f32 sums and the f16 operand hold, and a new largest logit
//                            (there is one in most blocks of a short walk) costs nothing.
//   O^T += V_codes^T . P'^T  P' = p * s_v (per value group, hence the same 16 columns), raw V codes as A; the
//                            m_v part of the dequantised values is the scalar sum  p * m_v  kept per lane.
//
// Codes go into the f16 operands without arithmetic: a b-bit field masked in place inside a 16-bit half is the
// f16 subnormal  code * 2^(shift-24), which the matrix cores consume exactly; the per-slot power of two is
// folded into the other operand (q or P'), the common 2^-24 into constants applied after the contraction.
//
// The storage layout (wq.h) is exactly the per-lane operand order, so every load is one contiguous piece per
// lane, a whole tile per wavefront.  Scales and minima travel as one coalesced word per lane and block and are
// redistributed through LDS.  Each wavefront builds the query operands of the class it walks from global memory.
#pragma once

#ifdef WQ_TIMELINE   // development aid: per-workgroup phase time stamps (100 MHz clock) at the end of the workspace
#define WQ_WG ((int64_t)(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x)
#define WQ_STAMP(k) do { if (a.dbg && threadIdx.x == 0) a.dbg[WQ_WG * 64 + (k)] = wall_clock64(); } while (0)
#define WQ_WSTAMP(k, val) do { if (a.dbg && (threadIdx.x & 63) == 0) a.dbg[WQ_WG * 64 + 8 + (threadIdx.x >> 6) * 6 + (k)] = (val); } while (0)
#else
#define WQ_STAMP(k) do { } while (0)
#define WQ_WSTAMP(k, val) do { } while (0)
#endif

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct U4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ half8 as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    U4 u{a, b, c, d};
    return __builtin_bit_cast(half8, u);
}

__device__ __forceinline__ floatx4 mfma(half8 a, half8 b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float f16lo(uint32_t w) { return wq_f16_bits_to_float(w & 0xFFFFu); }
__device__ __forceinline__ float f16hi(uint32_t w) { return wq_f16_bits_to_float(w >> 16); }

// largest of three (inputs here are never signalling NaNs: results of additions)
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// (f16 in the low half of u) * p and (f16 in the low half of w) * q, each rounded to f16 (a mixed-precision fused multiply-add
// per product; left to the compiler, which keeps the distance that the matrix cores need behind a vector instruction)
__device__ __forceinline__ uint32_t mul_f16lo(uint32_t u, float p, uint32_t w, float q)
{
    const half2v r = {(_Float16)fmaf(f16lo(u), p, 0.f), (_Float16)fmaf(f16lo(w), q, 0.f)};
    return __builtin_bit_cast(uint32_t, r);
}

// rotate by 8 lanes inside each row of 16 lanes: lane (g,h) <-> lane (1-g,h)
__device__ __forceinline__ float ror8(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));
}

// ---- where contraction slot e (0..7) of k-step r finds its channel (inside the lane's quarter of hd/4
// channels) and the left shift its code keeps inside the f16 half; c = class index (0,1,2 = 2,4,8 bits) ----
__device__ __forceinline__ void k_slot(int c, int r, int e, int& ch, int& sh)
{
    const int v = e >> 1, hi = e & 1;
    if (c == 0) {               // dword d = r/2 holds 16 fields; pair p = 4*(r%2)+v is (field p, field p+8)
        const int d = r >> 1, p = 4 * (r & 1) + v;
        ch = 16 * d + p + 8 * hi;
        sh = p <= 4 ? 2 * p : 2 * (p - 5);
    } else if (c == 1) {        // dword r holds 8 fields; pair v is (field v, field v+4)
        ch = 8 * r + v + 4 * hi;
        sh = 4 * (v & 1);
    } else if (c == 2) {        // dwords 2r, 2r+1; register v = (dword v/2, bytes (v%2, v%2+2))
        const int d = 2 * r + (v >> 1);
        ch = 4 * d + (v & 1) + 2 * hi;
        sh = 0;
    } else {                    // 16-bit segment: elements in natural order
        ch = 8 * r + e;
        sh = 0;
    }
}

// unpack the K chunk of one lane (hd/4 codes of one token) into the A operand of k-step r
template <int BITS>
__device__ __forceinline__ half8 k_operand(const uint32_t* x, int r)
{
    if (BITS == 2) {
        const uint32_t w = x[r >> 1];
        if ((r & 1) == 0)
            return as_half8(w & 0x00030003u, w & 0x000C000Cu, w & 0x00300030u, w & 0x00C000C0u);
        const uint32_t y = w >> 10;
        return as_half8(w & 0x03000300u, y & 0x00030003u, y & 0x000C000Cu, y & 0x00300030u);
    } else if (BITS == 4) {
        const uint32_t w = x[r], y = w >> 8;
        return as_half8(w & 0x000F000Fu, w & 0x00F000F0u, y & 0x000F000Fu, y & 0x00F000F0u);
    } else {
        const uint32_t w0 = x[2 * r], w1 = x[2 * r + 1];
        return as_half8(w0 & 0x00FF00FFu, __builtin_amdgcn_perm(0u, w0, 0x0c030c01u), w1 & 0x00FF00FFu,
                        __builtin_amdgcn_perm(0u, w1, 0x0c030c01u));
    }
}

// power of two that P' carries in register v (slots 2v, 2v+1) so that V's in-place codes come out unscaled
template <int BITS>
__device__ __forceinline__ float v_slot_scale(int v)
{
    if (BITS == 2) return v == 0 ? 1.0f : (v == 1 ? 0.25f : (v == 2 ? 0.0625f : 0.015625f));
    if (BITS == 4) return (v & 1) ? 0.0625f : 1.0f;
    return 1.0f;
}

template <int BITS>
__device__ __forceinline__ float v_slot_shift(int v)      // -log2 of v_slot_scale
{
    if (BITS == 2) return 2.0f * (float)v;
    if (BITS == 4) return (v & 1) ? 4.0f : 0.0f;
    return 0.0f;
}

// unpack the V fragment of one lane (for channel tile ct: 8 tokens of one channel) into an A operand
template <int BITS>
__device__ __forceinline__ half8 v_operand(const uint32_t* x, int ct)
{
    if (BITS == 2) {            // dword ct/2: fields 0..7 = even tile, 8..15 = odd tile
        uint32_t y = __builtin_amdgcn_perm(0u, x[ct >> 1], 0x03010200u);   // bytes (b0,b2,b1,b3)
        if (ct & 1) y >>= 8;
        return as_half8(y & 0x00030003u, y & 0x000C000Cu, y & 0x00300030u, y & 0x00C000C0u);
    } else if (BITS == 4) {
        const uint32_t w = x[ct], y = w >> 8;
        return as_half8(w & 0x000F000Fu, w & 0x00F000F0u, y & 0x000F000Fu, y & 0x00F000F0u);
    } else {                    // dwords 2ct (tokens tau 0..3), 2ct+1 (tau 4..7)
        const uint32_t lo = x[2 * ct], hi = x[2 * ct + 1];
        return as_half8(__builtin_amdgcn_perm(hi, lo, 0x0c040c00u), __builtin_amdgcn_perm(hi, lo, 0x0c050c01u),
                        __builtin_amdgcn_perm(hi, lo, 0x0c060c02u), __builtin_amdgcn_perm(hi, lo, 0x0c070c03u));
    }
}

// The launch's arguments, read from memory once more: for what is needed late or by few.  What the whole body keeps in scalar
// registers has to fit them: one table too many, and the compiler waits for a part of the tables to set it aside before it
// sends for the next part (three round trips in front of the first block instead of one, 0.9 us a launch).
__device__ __forceinline__ const DecodeArgs& args_again()
{
    const __attribute__((address_space(4))) void* p = (const __attribute__((address_space(4))) void*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const DecodeArgs*)p;
}

// ... and a pointer among them, as what it is (arguments that the compiler did not see arrive could point anywhere)
template <class T>
__device__ __forceinline__ T* in_memory(T* p)
{
    return (T*)(__attribute__((address_space(1))) T*)p;
}

template <int HD>
struct WaveState {
    floatx4 O[HD / 16];   // O^T tiles: row = channel 16ct + 4j + i, column = (g,h)
    float m;              // reference exponent of this column (a recent largest logit), log2 domain, shared by the four lane groups
    float l;              // this lane's share of sum p
    float accM;           // this lane's share of sum p * m_v
    float up;             // log2 of the factor that the weights of the quantized classes are formed with (the same in all lanes)
};

// 32-token blocks in flight per wavefront and class: enough bytes to keep the memory system busy while a block
// is being worked on (a 2-bit block is 2.5 KB, an 8-bit block 8.5 KB)
constexpr int WQ_D2 = 4, WQ_D4 = 3, WQ_D8 = 2;
constexpr int WQ_TAPER_TICKETS = 16;   // the last blocks of a workgroup's range, two per wavefront, are walked with half the pipeline (measured: 0.45 us per call)
constexpr int WQ_FIRST_TICKETS = 4;    // blocks every wavefront starts with (the deepest pipeline's fill), in a range that has as many
constexpr int WQ_WAVES = 8;            // wavefronts per workgroup: one workgroup per compute unit, two wavefronts per SIMD
constexpr float WQ_MAX_SLACK = 5.0f;   // log2 of the largest softmax weight tolerated before the reference exponent moves
// The weights meet the value scales in fp16 (P' = p * s_v).  They are formed 2^up too large (for free, in the exponent of
// the exp2), which the sums undo exactly at the end; up is chosen per sequence from its largest value scale s_max (a table
// of the cache that the quantizer fills) so that the largest product, 2^(WQ_MAX_SLACK + up) * s_max, lies in
// [2^(WQ_P_TOP - 1), 2^WQ_P_TOP]: nothing overflows whatever the values' magnitude, and a weight has to be
// 2^-(24 + WQ_P_TOP - WQ_MAX_SLACK - 6) = 2^-29 of the largest one, in a group whose scale is the sequence's largest and
// in the slot that is shifted most, before it is lost.
constexpr int WQ_P_TOP = 15;
// up for a sequence whose largest value scale is s_max (0: no quantized token; any up will do)
__device__ __forceinline__ float weight_upscale(float s_max)
{
    const uint32_t u = __float_as_uint(s_max);
    const int ceil_log2 = (int)((u >> 23) & 0xFFu) - 127 + ((u & 0x7FFFFFu) != 0u ? 1 : 0);
    const int up = (WQ_P_TOP - (int)WQ_MAX_SLACK) - ceil_log2;
    return s_max > 0.f ? (float)min(max(up, -16), 40) : 6.0f;
}
__device__ __forceinline__ float pow2_of(float e) { return __uint_as_float((uint32_t)(127 + (int)e) << 23); }   // e an integer in [-126, 127]
constexpr int VT_PAD = 4;   // row pitch of the transposition buffer: (HD/2+4)*2 bytes, i.e. 4 rows apart = 8 banks (mod 32)

template <int HD>
struct MfmaSmem {
    struct {
        uint32_t meta[WQ_WAVES][2][64];                  // per wave: K and V metadata words of the current block
        uint16_t vt[WQ_WAVES][32][HD / 2 + VT_PAD];      // per wave: half the channels of the V rows of a 16-bit block, read back transposed
    } run;
    // per-wave numerators for the merge; rows four banks apart, written 16 bytes at a time.  A space of its own: a wavefront hands its numerators over
    // as soon as its loops end, while others still use the run-time part
    __attribute__((aligned(16))) float O[WQ_WAVES][WQ_MAX_REP][HD + 4];
    U4 bq[4][HD / 32][64];                               // query operands of the four classes (index 3 = 16-bit segment), per lane
    float qx[4][2][64];                                  // ... with the head's power of two and the group's query sum
    float ml[WQ_WAVES][WQ_MAX_REP][2];
    unsigned next_ticket;                                // the workgroup's block counter
    int expect[64], grown[64];                           // the workgroup that ends an append: per sequence, the workgroups that count themselves on it, and the new len16 (-1: unchanged)
};


// ---- a lane's value next to that of lane ^ 16 and of lane ^ 32 -------------------------------------------------
// The row-swap instructions exchange rows of 16 lanes between two registers: given the same value x twice, the first
// register comes back holding the even row of every pair of rows in both of them (the lower half of the wavefront in
// both halves, for the 32-lane form), the second one the odd row (the upper half).  No LDS, no waiting.
struct RowPair { float even, odd; };
__device__ __forceinline__ RowPair rows_16(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return RowPair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ RowPair halves_32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return RowPair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// sum / maximum over the four lanes {l, l ^ 16, l ^ 32, l ^ 48}, in every one of them
__device__ __forceinline__ float sum_over_rows(float x)
{
    const RowPair a = rows_16(x);
    const RowPair b = halves_32(a.even + a.odd);
    return b.even + b.odd;
}
__device__ __forceinline__ float max_over_rows(float x)
{
    const RowPair a = rows_16(x);
    const RowPair b = halves_32(fmaxf(a.even, a.odd));
    return fmaxf(b.even, b.odd);
}

// ---- the query operands of one class, built by the wavefront itself -------------------------------------------
// Lane (j, (g,h)) loads its quarter j of head h's query straight from global memory (hd/4 values), the head's
// largest magnitude is found with two cross-lane exchanges, the query is scaled by a power of two into [-1, 1)
// and laid out as the B operands of the k-steps: slot e of k-step r takes channel k_slot(c, r, e) of the quarter,
// times 2^-shift of that slot; lanes whose quarter is not in their column's group hold zeros (block-diagonal B).
// Returns the head's power of two (1 for the raw-bf16 operands of a bf16 16-bit segment) and the sum of the scaled
// query over the lane's group.
template <int HD, int CLS>
__device__ __forceinline__ void build_q_operands(const DecodeArgs& a, int b, int kvh, bool raw_bf16, U4* Bq, float& qexp, float& qsum)
{
    constexpr int QC = HD / 4, NK = HD / 32;
    const int lane = threadIdx.x & 63;
    const int j = lane >> 4, g = (lane & 15) >> 3, h = lane & 7;
    const bool live = h < a.rep;
    const int64_t base = ((int64_t)b * a.Hq + kvh * a.rep + (live ? h : 0)) * HD + j * QC;
    float v[QC];
    if (a.q_dtype == WQ_F32) {
        const float* p = static_cast<const float*>(a.q) + base;
#pragma unroll
        for (int k = 0; k < QC; k += 8) wq_ld8(p + k, v + k);
    } else if (a.q_dtype == WQ_BF16) {
        const __hip_bfloat16* p = static_cast<const __hip_bfloat16*>(a.q) + base;
#pragma unroll
        for (int k = 0; k < QC; k += 8) wq_ld8(p + k, v + k);
    } else {
        const __half* p = static_cast<const __half*>(a.q) + base;
#pragma unroll
        for (int k = 0; k < QC; k += 8) wq_ld8(p + k, v + k);
    }
    float mx = 0.f;
#pragma unroll
    for (int k = 0; k < QC; k++) mx = fmaxf(mx, fabsf(v[k]));   // (the columns of heads that do not exist repeat head 0: nobody reads them)
    mx = max_over_rows(mx);
    const int eb = (int)((__float_as_uint(mx) >> 23) & 0xFFu);              // biased exponent of the largest |q|
    const bool ok = eb > 0 && eb < 253;                                       // zero, denormal or non-finite: leave as is
    const float dn = ok ? __uint_as_float((uint32_t)(253 - eb) << 23) : 1.0f;     // 2^-(eb-126): max |q| lands in [0.5, 1)
    const float up = ok ? __uint_as_float((uint32_t)(eb + 1) << 23) : 1.0f;       // 2^(eb-126)
    float s = 0.f;                                 // sum of the scaled query as f16 holds it, two channels per instruction
#pragma unroll
    for (int k = 0; k < QC; k += 2) {
        const half2v pair_k = {(_Float16)(v[k] * dn), (_Float16)(v[k + 1] * dn)};
        s = __builtin_amdgcn_fdot2(pair_k, half2v{(_Float16)1.0f, (_Float16)1.0f}, s, false);
    }
    const RowPair quarters = rows_16(s);
    const float pair = quarters.even + quarters.odd;                         // both quarters of group j/2
    const RowPair groups = halves_32(pair);
    const float other = (lane & 32) ? groups.even : groups.odd;
    const bool mine = (j >> 1) == g;
    qsum = mine ? pair : other;
    qexp = raw_bf16 ? 1.0f : up;
#pragma unroll
    for (int r = 0; r < NK; r++) {
        uint32_t w[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; e2++) {
            uint32_t half[2];
#pragma unroll
            for (int t = 0; t < 2; t++) {
                int ch, sh;
                k_slot(CLS, r, 2 * e2 + t, ch, sh);
                const _Float16 f = (_Float16)(v[ch] * dn * __uint_as_float((uint32_t)(127 - sh) << 23));
                half[t] = raw_bf16 ? (__float_as_uint(v[ch]) >> 16) : (uint32_t)__builtin_bit_cast(uint16_t, f);
            }
            w[e2] = mine ? (half[0] | (half[1] << 16)) : 0u;
        }
        Bq[r] = U4{w[0], w[1], w[2], w[3]};
    }
}

// The wavefronts of a workgroup walk the same classes, so the workgroup builds the operands of all four once, one
// class per wavefront (the first four), and keeps them in LDS.
template <int HD>
__device__ __forceinline__ void stage_q_operands(const DecodeArgs& a, MfmaSmem<HD>& sm, int b, int kvh, int wave, bool bf16seg)
{
    constexpr int NK = HD / 32;
    const int lane = threadIdx.x & 63;
    U4 Bq[NK];
    float qexp, qsum;
    if (wave >= 4) return;
    if (wave == 0) build_q_operands<HD, 0>(a, b, kvh, false, Bq, qexp, qsum);
    else if (wave == 1) build_q_operands<HD, 1>(a, b, kvh, false, Bq, qexp, qsum);
    else if (wave == 2) build_q_operands<HD, 2>(a, b, kvh, false, Bq, qexp, qsum);
    else build_q_operands<HD, 3>(a, b, kvh, bf16seg, Bq, qexp, qsum);
#pragma unroll
    for (int r = 0; r < NK; r++) sm.bq[wave][r][lane] = Bq[r];
    sm.qx[wave][0][lane] = qexp;
    sm.qx[wave][1][lane] = qsum;
}

template <int HD>
__device__ __forceinline__ void fetch_q_operands(const MfmaSmem<HD>& sm, int c, U4* Bq, float& qexp, float& qsum)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < HD / 32; r++) Bq[r] = sm.bq[c][r][lane];
    qexp = sm.qx[c][0][lane];
    qsum = sm.qx[c][1][lane];
}

// ---- shares of the token axis ---------------------------------------------------------------------------------
// A workgroup owns a contiguous cost range of the stream [16-bit | 8-bit | 4-bit | 2-bit] of its (sequence, KV
// head).  Its wavefronts do not run at the same speed (of the two that share a SIMD the older one gets more issue
// slots and more of the memory system, and the classes differ), and one that is done early cannot be replaced: the
// launch is over when the slowest wavefront is.  So the 32-token blocks of the range are handed out in stream
// order through a counter in LDS (a ticket = one block): whoever is free takes the next one.  A wavefront holds a
// range of tickets (normally one) and keeps tickets that stand for blocks of a later class until it gets there.
// The ticket that replaces a spent one is drawn at the start of a block's arithmetic and read at its end; LDS
// operations have a counter of their own, so the draw never waits for the block loads that are in flight.
// With WQ_DECODE_FIXED_SHARES the range is divided among the wavefronts by cost instead: each holds its tickets from the start.
struct Tickets {
    unsigned* ctr;      // the workgroup's counter (LDS)
    unsigned held, end; // tickets held: [held, end); none left: another one is due
    bool dealt;         // the tickets held are all that this wavefront gets: there is nothing to draw
    bool synced;        // this wavefront has passed the workgroup's set-up barrier
    bool appends;       // the launch appends a token
    unsigned taper;     // from this ticket on (the workgroup's last WQ_TAPER_TICKETS) a wavefront refills only every other pipeline slot
};

// ---- a launch that appends a token (k_new != NULL) must not change len16[b] while a wavefront of a workgroup of sequence b
// may still read it (under WQ_DECODE_BY_LENGTH the split count of a sequence depends on its length).  Every workgroup of the
// sequence, also one that has nothing to do, counts itself on the sequence's counter behind a barrier that all its wavefronts
// pass with the tables in their registers: the set-up barrier, or one for this purpose where there is no work (an add that
// returns nothing: nobody waits for it).  Counted as soon as the first wavefront has the tables, a workgroup's other
// wavefronts could read the raised length where the one that raises it has nothing else to do.
// The sequence's last workgroup in dispatch order (highest KV head, highest split; every other one of the sequence was
// dispatched before it and waits for nobody before it counts itself) waits at its very end until the count is complete,
// clears the counter for the next launch and writes the new length.
__device__ __forceinline__ void count_tables_read(bool appends, int b)
{
    if (!appends) return;
    const DecodeArgs& a = args_again();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(in_memory(a.arrive) + a.B * a.kv.Hkv * a.arrive_unit + b * WQ_ARRIVE_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The set-up barrier (staged query operands, initial value of the block counter) is taken by every wavefront
// exactly once: after the first loads of the first class it walks have been issued, or, by a wavefront that has
// no blocks at all, before the final merge.
__device__ __forceinline__ void pass_setup_barrier(int b, Tickets& t)
{
    if (!t.synced) {
        __syncthreads();
        t.synced = true;
        count_tables_read(t.appends, b);
    }
}

// lane 0 draws n tickets; the first one's value is valid in lane 0 once the LDS operation has returned
__device__ __forceinline__ unsigned draw_tickets(unsigned* ctr, unsigned n)
{
    unsigned v = 0;
    if ((threadIdx.x & 63) == 0) v = __hip_atomic_fetch_add(ctr, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return v;
}

__device__ __forceinline__ unsigned ticket_value(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }

struct BlockSrc {
    int pool_first;          // first block of the class's part of the workgroup's range
    unsigned tk_lo, tk_hi;   // tickets that stand for those blocks (tk_hi = 0: there are none)
};

// Are there blocks of the class for this wavefront?  With no ticket left it draws `fill` of them and waits (at the start of a class).
__device__ __forceinline__ bool has_blocks(const BlockSrc& s, Tickets& t, unsigned fill)
{
    if (t.held == t.end) {
        t.held = t.dealt ? 0xFFFFFFFEu : ticket_value(draw_tickets(t.ctr, fill));
        t.end = t.dealt ? 0xFFFFFFFFu : t.held + fill;
    }
    return t.held < s.tk_hi;
}

// next block of the class for this wavefront, or -1 (and then -1 on every later call for the class): a ticket for a block of a
// later class is kept.  (A ticket is drawn beside the arithmetic of a block that has left none, so only a wavefront that gets no more has none here.)
__device__ __forceinline__ int next_block(const BlockSrc& s, Tickets& t)
{
    if (t.held >= min(t.end, s.tk_hi)) return -1;
    return s.pool_first + (int)(t.held++ - s.tk_lo);
}

// The first DEPTH blocks of the class (there is at least one): of the tickets held, and of those drawn where they don't reach
template <int DEPTH>
__device__ __forceinline__ void first_blocks(const BlockSrc& s, Tickets& t, int (&bi)[DEPTH])
{
    int n = (int)min(min(t.end, s.tk_hi) - t.held, (unsigned)DEPTH), at = s.pool_first + (int)(t.held - s.tk_lo);
#pragma unroll
    for (int d = 0; d < DEPTH; d++) bi[d] = d < n ? at + d : -1;
    t.held += (unsigned)n;
    if (n < DEPTH && t.held == t.end && !t.dealt) {
        const unsigned more = (unsigned)(DEPTH - n);
        t.held = ticket_value(draw_tickets(t.ctr, more));
        t.end = t.held + more;
        const unsigned in = min(max(s.tk_hi, t.held), t.end) - t.held;
        at = s.pool_first + (int)(t.held - s.tk_lo) - n;
#pragma unroll
        for (int d = 0; d < DEPTH; d++) bi[d] = d >= n && d < n + (int)in ? at + d : bi[d];
        t.held += in;
    }
}

template <int HD, int BITS>
struct Frag {
    static constexpr int KDW = (HD / 4) * BITS / 32;        // dwords of K codes per lane per 16-token tile
    static constexpr int VDW = (HD / 16) * 8 * BITS / 32;   // dwords of V codes per lane per 32-token block
    uint32_t k[2][KDW];
    uint32_t v[VDW];
    uint32_t km, vm;                                        // one metadata word per lane and plane
};

// N dwords per lane, lane after lane.  The cache is streamed once per launch, and with heads of 128 a load that takes whole lines (at most 16
// bytes per lane) says so: non-temporal.  28 layers: 8 x 12800 tokens 528 -> 507 us a step, 1 x 19735 320 -> 303; 4 x 50688 x 4 layers 102 -> 95; 32 ragged
// sequences 128 -> 120.  It costs up to 3 % where all that a program reads between two launches over a cache is less than 140 MB
// or so, which then would stay in the memory-side cache: one or two layers.  With heads of 64 that costs more (8 x 12744 tokens, 8/8 heads, three
// caches in turn: 17.4 us a call, 19.5 with non-temporal loads; 12 layers of 3336 tokens 125.5 and 118.5): plain loads.  Loads of more bytes per lane come
// in pieces that share lines, and each piece would fetch them again (all loads so: 20 % slower).  The metadata of one group per head of 128 is the exception:
// a load takes half a line, its neighbour the other half, and the two kinds are the same (22 batches, 1 to 16 sequences of 6000 to 20000 tokens, 1 to 12 layers:
// non-temporal 1.0006 times as fast on average, 0.995 to 1.014).
template <int HD, int N>
__device__ __forceinline__ void load_dwords(const uint32_t* __restrict__ p, uint32_t* dst)
{
    if constexpr (N <= 4) {
        typedef uint32_t dwords __attribute__((ext_vector_type(N)));
        const dwords* const from = reinterpret_cast<const dwords*>(p);
        const dwords u = HD == 128 ? __builtin_nontemporal_load(from) : *from;
#pragma unroll
        for (int d = 0; d < N; d++) dst[d] = u[d];
    } else {
#pragma unroll
        for (int d = 0; d < N; d += 4) {
            uint4 u = *reinterpret_cast<const uint4*>(p + d);
            dst[d] = u.x;
            dst[d + 1] = u.y;
            dst[d + 2] = u.z;
            dst[d + 3] = u.w;
        }
    }
}
template <int HD>
__device__ __forceinline__ uint32_t load_word(const uint32_t* p) { return HD == 128 ? __builtin_nontemporal_load(p) : *p; }

// One class of one (sequence, KV head): this wavefront's share of its 32-token blocks (len tokens from token slot
// tok_base of the class buffers).
template <int HD, int BITS, int DEPTH>
__device__ __forceinline__ void walk_class_mfma(const DecodeArgs& a, MfmaSmem<HD>& sm, int b, int kvh, int len, int tok_base, const BlockSrc& src,
                                                Tickets& tk, float c_log2, WaveState<HD>& st)
{
    constexpr int C = BITS == 2 ? 0 : (BITS == 4 ? 1 : 2);
    constexpr int NK = HD / 32;                    // k-steps of the logit product per 16-token tile
    constexpr int CT = HD / 16;                    // channel tiles of the value product
    using F = Frag<HD, BITS>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane >> 4, col = lane & 15, g = col >> 3;

    if (!has_blocks(src, tk, DEPTH)) return;
    const wq_packed_kv& kv = a.kv;
    const int64_t cap = kv.cap[C];
    const uint8_t* kbase = static_cast<const uint8_t*>(kv.codes[C]) + ((int64_t)kvh * cap + tok_base) * HD * BITS / 8 + lane * (F::KDW * 4);
    const uint8_t* vbase = static_cast<const uint8_t*>(kv.codes[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * HD * BITS / 8 + lane * (F::VDW * 4);
    const uint32_t* kmeta = static_cast<const uint32_t*>(kv.meta[C]) + ((int64_t)kvh * cap + tok_base) * 2 + lane;
    const uint32_t* vmeta = static_cast<const uint32_t*>(kv.meta[C]) + (((int64_t)kv.Hkv + kvh) * cap + tok_base) * 2 + lane;
    uint32_t* smeta = &sm.run.meta[wave][0][0];
    const int moff = g * 16 + 4 * j;               // (group g, tokens 4j..4j+3) inside a metadata tile of 32 words

    auto load = [&](int blk, F& f) {
        const int64_t o = (int64_t)blk * (32 * HD * BITS / 8);
        load_dwords<HD, F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o), f.k[0]);
        load_dwords<HD, F::KDW>(reinterpret_cast<const uint32_t*>(kbase + o + 16 * HD * BITS / 8), f.k[1]);
        load_dwords<HD, F::VDW>(reinterpret_cast<const uint32_t*>(vbase + o), f.v);
        f.km = load_word<HD>(kmeta + (int64_t)blk * 64);
        f.vm = load_word<HD>(vmeta + (int64_t)blk * 64);
    };

    // software pipeline: DEPTH blocks in flight per wavefront; the first loads go out before anything else
    F f[DEPTH];
    int bi[DEPTH];
    first_blocks<DEPTH>(src, tk, bi);
#pragma unroll
    for (int d = 0; d < DEPTH; d++)
        if (bi[d] >= 0) load(bi[d], f[d]);
    pass_setup_barrier(b, tk);
    U4 Bqw[NK];
    float qexp, qsum;
    fetch_q_operands<HD>(sm, C, Bqw, qexp, qsum);
    half8 Bq[NK];
#pragma unroll
    for (int r = 0; r < NK; r++) Bq[r] = __builtin_bit_cast(half8, Bqw[r]);
    // logits come out of the matrix cores as 2^-24 * sum q' code; fold 2^24, the head's power of two and
    // sm_scale*log2(e) into one constant, and pre-divide the m-term by 2^24 so both terms share it.
    const float cexp = c_log2 * qexp * 16777216.0f;
    const float qs = qsum * (1.0f / 16777216.0f);

    // added to the logits: zero, except for the tokens past the end of the sequence's last block of the class
    // (the last block this wavefront gets: shares and tickets go up the stream), which get -inf
    float pen[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // partial sums per slot register v: its weights carry 2^-shift(v) (folded into the exponent), undone after the loop
    float lv[4] = {0.f, 0.f, 0.f, 0.f}, av[4] = {0.f, 0.f, 0.f, 0.f}, ms[4];
#pragma unroll
    for (int v = 0; v < 4; v++) ms[v] = st.m + v_slot_shift<BITS>(v) - st.up;

    auto compute = [&](int blk, const F& f) {
        const bool redraw = tk.held == tk.end && !tk.dealt;
        unsigned drawn = 0;
        if (redraw) drawn = draw_tickets(tk.ctr, 1u);
        if (blk * 32 + 32 > len) {
            const int nv = len - blk * 32;         // valid tokens in this block
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) pen[4 * t + i] = (16 * t + 4 * j + i >= nv) ? -INFINITY : 0.f;
        }
        // ---- scales and minima: one word per lane in, the lane's 4 tokens x 2 tiles x {K,V} out ----
        smeta[lane] = f.km;
        smeta[64 + lane] = f.vm;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        uint32_t kw[8], vw[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const uint4 a = *reinterpret_cast<const uint4*>(smeta + t * 32 + moff);
            const uint4 c = *reinterpret_cast<const uint4*>(smeta + 64 + t * 32 + moff);
            kw[4 * t] = a.x, kw[4 * t + 1] = a.y, kw[4 * t + 2] = a.z, kw[4 * t + 3] = a.w;
            vw[4 * t] = c.x, vw[4 * t + 1] = c.y, vw[4 * t + 2] = c.z, vw[4 * t + 3] = c.w;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();   // the next block's words may overwrite the buffer after this point

        // ---- logits of the two 16-token tiles ----
        float x[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < NK; r++) acc = mfma(k_operand<BITS>(f.k[t], r), Bq[r], acc);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float y = fmaf(f16lo(kw[4 * t + i]), acc[i], fmaf(f16hi(kw[4 * t + i]), qs, pen[4 * t + i]));
                x[4 * t + i] = y + ror8(y);
            }
        }
        // ---- reference exponent: touch the other lane groups only when some logit is far above it ----
        float lm = max3(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5]), max3(x[6], x[7], x[7]));
        lm *= cexp;                                // cexp > 0
        if (__builtin_amdgcn_ballot_w64(lm > st.m + WQ_MAX_SLACK) != 0) {
            lm = max_over_rows(lm);
            const float mn = fmaxf(st.m, lm);
            const float alpha = (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(st.m - mn);   // 0 on the first block
            st.m = mn;
            st.l *= alpha;
            st.accM *= alpha;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                lv[v] *= alpha;
                av[v] *= alpha;
                ms[v] = mn + v_slot_shift<BITS>(v) - st.up;
            }
#pragma unroll
            for (int ct = 0; ct < CT; ct++) st.O[ct] *= alpha;
        }
        // ---- weights with the slot's power of two folded into the exponent, P' = p * s_v, and the m_v part ----
        float p[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            p[k] = __builtin_amdgcn_exp2f(fmaf(x[k], cexp, -ms[k & 3]));
            lv[k & 3] += p[k];
            av[k & 3] = fmaf(f16hi(vw[k]), p[k], av[k & 3]);
        }
        uint32_t bp[4];
#pragma unroll
        for (int v = 0; v < 4; v++)                // slots (2v, 2v+1) = (tile 0, tile 1) token 4j+v
            bp[v] = mul_f16lo(vw[v], p[v], vw[4 + v], p[4 + v]);
        const half8 Bp = as_half8(bp[0], bp[1], bp[2], bp[3]);
        // ---- values ----
#pragma unroll
        for (int ct = 0; ct < CT; ct++) st.O[ct] = mfma(v_operand<BITS>(f.v, ct), Bp, st.O[ct]);
        const unsigned got = ticket_value(drawn);      // read on every path: nothing is left pending at the loop edge
        if (redraw) {
            tk.held = got;
            tk.end = got + 1u;
        }
    };

    while (bi[0] >= 0) {
#pragma unroll
        for (int d = 0; d < DEPTH; d++) {
            if (bi[d] >= 0) {
                compute(bi[d], f[d]);
                // near the end of the workgroup's range the odd slots are given up: whatever is in flight when the last
                // block has been handed out is arithmetic that no load overlaps with any more
                if ((d & 1) && DEPTH > 2 && tk.held >= tk.taper) {
                    bi[d] = -1;
                    continue;
                }
                bi[d] = next_block(src, tk);
                if (bi[d] >= 0) load(bi[d], f[d]);
            }
        }
    }
    const float down = pow2_of(-st.up);            // undoes the factor that the weights were formed with
#pragma unroll
    for (int v = 0; v < 4; v++) {
        st.l = fmaf(lv[v], down * (1.0f / v_slot_scale<BITS>(v)), st.l);
        st.accM = fmaf(av[v], down * (1.0f / v_slot_scale<BITS>(v)), st.accM);
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <bool BF>
__device__ __forceinline__ floatx4 mfma16(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, const U4& b, floatx4 c)
{
    U4 a{a0, a1, a2, a3};
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// The 16-bit segment (text, generated tokens, video tail, 16-bit windows) of one (sequence, KV head): rows are
// plain [token][Hkv][hd] so the K side feeds the matrix cores straight from global memory (one token row
// quarter per lane); V rows go through LDS and are read back one channel x 8 tokens per lane.  bf16 caches use
// the bf16 instruction with the exact bf16 query and the weights split into two bf16 terms (p = hi + lo);
// fp16 caches use the f16 instruction.  Accumulators are in true units here (no 2^-24).
template <int HD, bool BF>
// new_row >= 0: row new_row (= len - 1) is not in the cache yet: it is read from k_new / v_new, the token that the launch appends.
__device__ __forceinline__ void walk_seg16_mfma(const DecodeArgs& a, MfmaSmem<HD>& sm, int b, int kvh, int len, int first_row, const BlockSrc& src,
                                                Tickets& tk, float c_log2, WaveState<HD>& st, int new_row)
{
    constexpr int NK = HD / 32, CT = HD / 16, PITCH = HD / 2 + VT_PAD, KDW = HD / 8;
    if (!has_blocks(src, tk, 1u)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane >> 4, col = lane & 15;
    const wq_packed_kv& kv = a.kv;
    const int64_t row0 = first_row;
    const int64_t rstride = (int64_t)kv.Hkv * HD;
    const uint16_t* k16 = static_cast<const uint16_t*>(kv.k16) + (int64_t)kvh * HD;
    const uint16_t* v16 = static_cast<const uint16_t*>(kv.v16) + (int64_t)kvh * HD;
    const uint16_t *const knew = a.k_new + ((int64_t)b * kv.Hkv + kvh) * HD, *const vnew = a.v_new + ((int64_t)b * kv.Hkv + kvh) * HD;     // (read where there is a new row)
    pass_setup_barrier(b, tk);
    U4 Bq[NK];
    float qexp, qsum;
    fetch_q_operands<HD>(sm, 3, Bq, qexp, qsum);
    const float cexp = c_log2 * qexp;
    uint16_t* vt = &sm.run.vt[wave][0][0];

    for (int blk = next_block(src, tk); blk >= 0; blk = next_block(src, tk)) {
        const int nv = len - blk * 32;
        const bool redraw = tk.held == tk.end && !tk.dealt;
        unsigned drawn = 0;
        if (redraw) drawn = draw_tickets(tk.ctr, 1u);
        // ---- all loads of the block up front: one memory round trip per block ----
        uint32_t kd[2][KDW];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const int tok = min(blk * 32 + 16 * t + col, len - 1);      // rows past the end re-read the last row, masked below
            const uint16_t* src_k = tok == new_row ? knew : k16 + (row0 + tok) * rstride;
            load_dwords<HD, KDW>(reinterpret_cast<const uint32_t*>(src_k + j * (HD / 4)), kd[t]);
        }
        constexpr int VIT = (32 * (HD / 2) * 2) / (16 * 64);          // 16-byte pieces per lane and channel half
        uint4 vd[2][VIT];
#pragma unroll
        for (int half = 0; half < 2; half++)
#pragma unroll
            for (int it = 0; it < VIT; it++) {
                const int chunk = it * 64 + lane;
                const int row = chunk / (HD / 16), c16 = chunk % (HD / 16);
                const int tok = min(blk * 32 + row, len - 1);
                const uint16_t* src_v = tok == new_row ? vnew : v16 + (row0 + tok) * rstride;
                vd[half][it] = *reinterpret_cast<const uint4*>(src_v + half * (HD / 2) + c16 * 8);
            }
        // ---- logits ----
        float x[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < NK; r++) acc = mfma16<BF>(kd[t][4 * r], kd[t][4 * r + 1], kd[t][4 * r + 2], kd[t][4 * r + 3], Bq[r], acc);
#pragma unroll
            for (int i = 0; i < 4; i++) x[4 * t + i] = acc[i] + ror8(acc[i]);
        }
        if (nv < 32) {
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int i = 0; i < 4; i++)
                    if (16 * t + 4 * j + i >= nv) x[4 * t + i] = -INFINITY;
        }
        float lm = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        lm *= cexp;
        if (__builtin_amdgcn_ballot_w64(lm > st.m + WQ_MAX_SLACK) != 0) {
            lm = max_over_rows(lm);
            const float mn = fmaxf(st.m, lm);
            const float alpha = (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(st.m - mn);
            st.m = mn;
            st.l *= alpha;
            st.accM *= alpha;
#pragma unroll
            for (int ct = 0; ct < CT; ct++) st.O[ct] *= alpha;
        }
        float p[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            p[k] = __builtin_amdgcn_exp2f(fmaf(x[k], cexp, -st.m));
            st.l += p[k];
        }
        // ---- weights as B operands: slots (2v, 2v+1) = (tile 0 token 4j+v, tile 1 token 4j+v) ----
        U4 Ph, Pl;
        {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int v = 0; v < 4; v++) {
                if constexpr (BF) {
                    const uint32_t u0 = __float_as_uint(p[v]), u1 = __float_as_uint(p[4 + v]);
                    const float r0 = p[v] - __uint_as_float(u0 & 0xFFFF0000u), r1 = p[4 + v] - __uint_as_float(u1 & 0xFFFF0000u);
                    hi[v] = (u0 >> 16) | (u1 & 0xFFFF0000u);
                    lo[v] = (__float_as_uint(r0) >> 16) | (__float_as_uint(r1) & 0xFFFF0000u);
                } else {
                    const _Float16 h0 = (_Float16)p[v], h1 = (_Float16)p[4 + v];
                    hi[v] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | ((uint32_t)__builtin_bit_cast(uint16_t, h1) << 16);
                    lo[v] = 0;
                }
            }
            Ph = U4{hi[0], hi[1], hi[2], hi[3]};
            Pl = U4{lo[0], lo[1], lo[2], lo[3]};
        }
        // ---- V rows -> LDS -> one channel x 8 tokens per lane, half of the channels at a time ----
#pragma unroll
        for (int half = 0; half < 2; half++) {
#pragma unroll
            for (int it = 0; it < VIT; it++) {
                const int chunk = it * 64 + lane;
                const int row = chunk / (HD / 16), c16 = chunk % (HD / 16);
                const uint4 v = vd[half][it];
                uint2* dst = reinterpret_cast<uint2*>(vt + row * PITCH + c16 * 8);   // the padded pitch is only 8-byte aligned
                dst[0] = uint2{v.x, v.y};
                dst[1] = uint2{v.z, v.w};
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int c2 = 0; c2 < CT / 2; c2++) {
                const int ct = half * (CT / 2) + c2;
                uint32_t a[4];
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const uint32_t e0 = vt[(4 * j + v) * PITCH + 16 * c2 + col];
                    const uint32_t e1 = vt[(16 + 4 * j + v) * PITCH + 16 * c2 + col];
                    a[v] = e0 | (e1 << 16);
                }
                st.O[ct] = mfma16<BF>(a[0], a[1], a[2], a[3], Ph, st.O[ct]);
                if constexpr (BF) st.O[ct] = mfma16<BF>(a[0], a[1], a[2], a[3], Pl, st.O[ct]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();          // the buffer is overwritten next
        }
        const unsigned got = ticket_value(drawn);
        if (redraw) {
            tk.held = got;
            tk.end = got + 1u;
        }
    }
}

}  // namespace

#include "wq_decode_f32.h"

namespace {

// ---- the end of an append (count_tables_read above has the protocol) ----
constexpr long long WQ_APPEND_WAIT_TICKS = 400000000ll;   // 4 s of the 100 MHz clock: far beyond any launch; a wait that long gives up

__device__ __forceinline__ void finish_append(const DecodeArgs& a, int b, int kvh, int split, int new_row)
{
    if (!a.k_new || threadIdx.x != 0 || kvh != a.kv.Hkv - 1 || split != a.splits - 1) return;
    unsigned* ctr = in_memory(a.arrive) + a.B * a.kv.Hkv * a.arrive_unit + b * WQ_ARRIVE_STRIDE;
    const unsigned all = (unsigned)a.kv.Hkv * (unsigned)a.splits;
    const long long t_start = wall_clock64();
    while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != all) {
        if (wall_clock64() - t_start > WQ_APPEND_WAIT_TICKS) {
            atomicOr(in_memory(a.status), WQ_DEV_APPEND_TIMEOUT);
            break;
        }
        __builtin_amdgcn_s_sleep(8);
    }
    __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (new_row >= 0) in_memory(a.kv.len16)[b] = new_row + 1;
}

// ---- which part of which sequence a workgroup of a launch by length gets (at most 64 sequences: one per lane) ----
// The grid is one-dimensional: sequence 0's S_0 * Hkv workgroups, then sequence 1's, ..., then those with nothing to do.
// Consecutive workgroups go to different XCDs, so every XCD gets the same share of the work whatever the lengths (with the
// workgroups of a (sequence, KV head) at a fixed distance, as launches for equal lengths have them, the long sequences'
// workgroups can all fall on the same XCDs; those without work also took compute units from the others).
// How many splits S_b a sequence gets: in a launch with a given count ceil(tokens * len_scale); in an automatic one
// ceil(cost / tau) for a cost per workgroup tau that needs no more workgroups than the launch has (slots * Hkv): three
// halvings between the mean (no rounding at all) and what is certain to fit, of which the end that fits is taken (not
// the smallest such tau, but at most an eighth of the interval above it); or even_splits each where the costs are equal to 3 %.
// Every wavefront of the launch computes the same from the same tables.
struct Place {
    int b, kvh, split, S;     // (b < 0: nothing to do)
    int len[4], off[4], end16;
    float v_scale_max;
};

template <int CTRL, int ROWS>
__device__ __forceinline__ int scan_step(int x)          // x plus the value that a data-parallel-primitive move brings (0 where none)
{
    return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, true);
}

template <int HD, int G, class Smem>
__device__ __forceinline__ Place place_by_length(const DecodeArgs& a, Smem& sm, int wg)
{
    const int lane = threadIdx.x & 63, l = min(lane, a.B - 1);
    int len[4], off[4];
#pragma unroll
    for (int c = 0; c < 3; c++) {
        len[c] = a.kv.cls_len[c][l];
        off[c] = a.kv.cls_off[c][l];
    }
    const int len16 = a.kv.len16[l], end16 = a.kv.off16[l + 1];
    off[3] = a.kv.off16[l];
    const float vmax = G == 2 ? a.kv.v_scale_max[l] : 0.f;
    const bool grows = a.k_new && off[3] + len16 < end16 && (int64_t)off[3] + len16 < a.kv.cap16;
    len[3] = len16;
    const int len16_after = len16 + (grows ? 1 : 0);     // with the token that this launch appends, as append followed by attention counts
    const bool mine = lane < a.B;
    int S;
    if (a.slots == 0) {
        const int tokens = len[0] + len[1] + len[2] + len16_after;
        S = max(1, min(a.splits, (int)ceilf((float)tokens * a.len_scale)));
    } else {
        int blocks = 1 + ((len16_after + 31) >> 5) * block_cost<HD, G>(3);
#pragma unroll
        for (int c = 0; c < 3; c++) blocks += ((len[c] + 31) >> 5) * block_cost<HD, G>(c);
        const float cost = mine ? (float)blocks : 0.f, total = wave_sum(cost), most = wave_max(cost);
        // (a sequence's share is rounded down by 0.002 first: a quotient that should be whole must not become the next whole number)
        auto splits_of = [&](float tau) { return mine ? max(1, min(a.splits, (int)ceilf(fmaf(cost, __builtin_amdgcn_rcpf(tau), -0.002f)))) : 0; };
        float lo = total / (float)a.slots;
        float hi = fmaxf(lo, a.slots > a.B ? fminf(total / (float)(a.slots - a.B), most) : most);
        const bool even = total >= 0.97f * most * (float)a.B;      // (no search then, 0.3 us)
#pragma unroll 1
        for (int k = even ? 3 : 0; k < 3; k++) {
            const float mid = 0.5f * (lo + hi);
            const bool fits = wave_sum((float)splits_of(mid)) <= (float)a.slots;
            lo = fits ? lo : mid;
            hi = fits ? mid : hi;
        }
        S = !even ? splits_of(hi) : mine ? a.even_splits : 0;
    }
    const int n = mine ? S * a.kv.Hkv : 0;
    int upto = scan_step<0x111, 0xF>(n);                 // row_shr:1, 2, 4, 8, then the rows before
    upto = scan_step<0x112, 0xF>(upto);
    upto = scan_step<0x114, 0xF>(upto);
    upto = scan_step<0x118, 0xF>(upto);
    upto = scan_step<0x142, 0xA>(upto);                  // row_bcast:15 into the odd rows
    upto = scan_step<0x143, 0xC>(upto);                  // row_bcast:31 into the upper half
    const int total = __builtin_amdgcn_readlane(upto, 63);
    if (a.k_new && wg == (int)gridDim.x - 1 && threadIdx.x < 64) {
        sm.expect[lane] = n + (lane == 0 ? (int)gridDim.x - total : 0);
        sm.grown[lane] = mine && grows ? len16_after : -1;
    }
    Place p;
    p.b = -1;
    if (wg >= total) return p;
    p.b = (int)__popcll(__builtin_amdgcn_ballot_w64(mine && upto <= wg));
    const int rem = wg - (__builtin_amdgcn_readlane(upto, p.b) - __builtin_amdgcn_readlane(n, p.b));
    p.split = __builtin_amdgcn_readfirstlane((int)(((float)rem + 0.5f) * __builtin_amdgcn_rcpf((float)a.kv.Hkv)));
    p.kvh = rem - p.split * a.kv.Hkv;
    p.S = __builtin_amdgcn_readlane(S, p.b);
#pragma unroll
    for (int c = 0; c < 4; c++) {
        p.len[c] = __builtin_amdgcn_readlane(len[c], p.b);
        p.off[c] = __builtin_amdgcn_readlane(off[c], p.b);
    }
    p.end16 = __builtin_amdgcn_readlane(end16, p.b);
    p.v_scale_max = lane_value(vmax, p.b);
    return p;
}

// ... the end of an append in such a launch: the launch's last workgroup in dispatch order (by the same reasoning as in
// finish_append) waits until every workgroup has counted itself, those with nothing to do on sequence 0's counter
template <class Smem>
__device__ __forceinline__ void finish_append_by_length(const DecodeArgs& a, Smem& sm, int wg)
{
    if (!a.k_new || threadIdx.x >= 64 || wg != (int)gridDim.x - 1) return;
    const int lane = threadIdx.x;
    const bool mine = lane < a.B;
    const unsigned expect = (unsigned)sm.expect[lane];
    unsigned* const ctr = in_memory(a.arrive) + a.B * a.kv.Hkv * a.arrive_unit + (mine ? lane : 0) * WQ_ARRIVE_STRIDE;
    const long long t_start = wall_clock64();
    while (true) {
        const bool there = !mine || __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == expect;
        if (__builtin_amdgcn_ballot_w64(!there) == 0) break;
        if (wall_clock64() - t_start > WQ_APPEND_WAIT_TICKS) {
            if (lane == 0) atomicOr(in_memory(a.status), WQ_DEV_APPEND_TIMEOUT);
            break;
        }
        __builtin_amdgcn_s_sleep(8);
    }
    if (mine) {
        __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (sm.grown[lane] >= 0) in_memory(a.kv.len16)[lane] = sm.grown[lane];
    }
}

// Shares are laid out on a cost axis in integers (a 32-token block of a class costs WQ_BLOCK_COST of it): everything
// here depends only on the sequence's tables and the workgroup's and wavefront's numbers, which are the same for all
// lanes, so the compiler keeps it in scalar registers and on the scalar unit, where it does not compete with the vector
// work of the wavefront that shares the SIMD (as float arithmetic on the vector unit it held every wavefront's first
// loads back by most of a microsecond).  Every wavefront evaluates the same expressions for the same boundary, so
// neighbouring shares meet exactly, and the mapping is monotone, which is all that the partition needs.
// first block of a class (n blocks of cost W each, starting at cost `base`) at or after cost x
template <unsigned W>
__device__ __forceinline__ int range_edge(unsigned x, unsigned base, int n)
{
    const unsigned e = x > base ? (x - base + (W - 1u)) / W : 0u;             // (division by a constant: a multiplication)
    return (int)min(e, (unsigned)n);
}

template <int HD, int G>
__device__ __forceinline__ int range_edge_of(int c, unsigned x, unsigned base, int n)
{
    return c == 0 ? range_edge<(unsigned)block_cost<HD, G>(0)>(x, base, n)
         : c == 1 ? range_edge<(unsigned)block_cost<HD, G>(1)>(x, base, n)
         : c == 2 ? range_edge<(unsigned)block_cost<HD, G>(2)>(x, base, n)
                  : range_edge<(unsigned)block_cost<HD, G>(3)>(x, base, n);
}

// ---- helpers of the two merges --------------------------------------------------------------------------------
typedef float floatx2 __attribute__((ext_vector_type(2)));

// N floats (N * 4 bytes, aligned to that) to memory with a device-scope store (one instruction)
template <int N>
__device__ __forceinline__ void store_through(float* p, const float* v)
{
    if constexpr (N == 1) {
        __hip_atomic_store(p, v[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        static_assert(N == 2, "one or two floats");
        const unsigned long long u = (unsigned long long)__float_as_uint(v[0]) | ((unsigned long long)__float_as_uint(v[1]) << 32);
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int N>
__device__ __forceinline__ void store_plain(float* p, const float* v)
{
    if constexpr (N == 1) {
        p[0] = v[0];
    } else {
        static_assert(N == 2, "one or two floats");
        *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
    }
}

// Two or four floats of a partial through a buffer descriptor, with a device-scope load (does not stop at a cache); zero
// when the offset is beyond the descriptor's range
constexpr int LD_DEVICE_SCOPE = 16;                // the sc1 bit of the instruction
__device__ __forceinline__ floatx2 ld_part2(__amdgpu_buffer_rsrc_t rsrc, unsigned byte_off)
{
    return __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)byte_off, 0, LD_DEVICE_SCOPE));
}
__device__ __forceinline__ floatx4 ld_part4(__amdgpu_buffer_rsrc_t rsrc, unsigned byte_off)
{
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, 0, LD_DEVICE_SCOPE));
}
// lane K of every row of 16 lanes, in all lanes of that row
template <int K>
__device__ __forceinline__ float row_bcast(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x150 + K, 0xF, 0xF, true));
}
template <class F, int... K>
__device__ __forceinline__ void for_each_index(const F& f, std::integer_sequence<int, K...>) { (f(std::integral_constant<int, K>{}), ...); }
// row pairs (0, 2) and (1, 3) of 16 lanes added up: a's sums in the lower half of the wavefront, b's in the upper half
__device__ __forceinline__ float fold_halves(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// ... rows 2k and 2k + 1: a's sums in the even rows, b's in the odd ones
__device__ __forceinline__ float fold_rows(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int HD, int G>
using DecodeSmem = std::conditional_t<G == 2, MfmaSmem<HD>, F32Smem<HD, G>>;

// PACKED: a launch by length whose grid place_by_length maps (an instantiation of its own: in a common one the registers it
// takes cost every other launch 0.2-0.5 us)
template <int HD, int G, bool PACKED>
__device__ void wq_decode_mfma_body(const DecodeArgs& a, void* smem_raw)
{
    constexpr bool F32 = G != 2;
    DecodeSmem<HD, G>& sm = *reinterpret_cast<DecodeSmem<HD, G>*>(smem_raw);
    // consecutive workgroups go to different (sequence, KV head) units: the units' tables and queries are then
    // read by all XCDs alike, and the workgroups of one unit do not start in a burst on neighbouring compute units
    // (the grid is (KV heads, sequences, splits): workgroups are dispatched with x fastest, and nothing here has to divide)
    int kvh = (int)blockIdx.x, b = (int)blockIdx.y, split = (int)blockIdx.z, S = a.splits;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int j = lane >> 4, col = lane & 15, g = col >> 3, h = col & 7;
    constexpr int CT = HD / 16;
    const bool bf16seg = a.kv.dtype16 == WQ_BF16;
    WQ_STAMP(0);

    // ---- the sequence's tables first ----
    int cls_len[4], cls_off[4], end16;
    float v_scale_max;
    if constexpr (PACKED) {
        const Place p = place_by_length<HD, G>(a, sm, (int)blockIdx.x);
        if (p.b < 0) {
            if (a.k_new) __syncthreads();
            count_tables_read(a.k_new != nullptr, 0);
            finish_append_by_length(a, sm, (int)blockIdx.x);
            return;
        }
        b = p.b, kvh = p.kvh, split = p.split, S = p.S;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            cls_len[c] = p.len[c];
            cls_off[c] = p.off[c];
        }
        end16 = p.end16;
        v_scale_max = p.v_scale_max;
    } else {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            cls_len[c] = a.kv.cls_len[c][b];
            cls_off[c] = a.kv.cls_off[c][b];
        }
        cls_len[3] = a.kv.len16[b];
        cls_off[3] = a.kv.off16[b];
        end16 = a.kv.off16[b + 1];
        v_scale_max = F32 ? 0.f : a.kv.v_scale_max[b];
    }
    // The arguments' line with the classes' pointers comes with the tables: first touched where a class begins, it was a round trip of its own in
    // front of the first block loads (28 launches: 8 x 12800 tokens 508 -> 502 us, 1 x 19735 302 -> 297; place_by_length touches it anyway)
    if constexpr (!PACKED) asm volatile("" :: "s"(a.kv.group));
    const int unit = b * a.kv.Hkv + kvh;
    // a token appended by this launch becomes the last row of the 16-bit segment: read from k_new / v_new by whoever
    // walks its block, copied into the cache by the first split's workgroup (at its end: the copy is a round trip to memory that
    // stood in front of that workgroup's first loads), counted in len16 once every workgroup of the sequence has read len16 (finish_append)
    int new_row = -1;
    if (a.k_new) {
        const uint32_t row = (uint32_t)cls_off[3] + (uint32_t)cls_len[3];
        const bool room = row < (uint32_t)end16 && ((uint64_t)a.kv.cap16 >> 32 != 0 || row < (uint32_t)a.kv.cap16);
        new_row = room ? cls_len[3] : -1;
        cls_len[3] += room ? 1 : 0;
        if (!room && split == 0 && kvh == 0 && tid == 0) atomicOr(in_memory(args_again().status), WQ_DEV_SEG16_OVERFLOW);      // the segment is full: nothing is appended
    }
    WQ_WSTAMP(5, wall_clock64() + (long long)((cls_len[0] + cls_len[1] + cls_len[2] + cls_len[3] + cls_off[0] + cls_off[1] + cls_off[2] + cls_off[3]) & 0));   // the tables have arrived
    if (!PACKED && a.len_scale > 0.f) {     // (more than 64 sequences: the sequence's share of the launch's splits, the other workgroups have nothing to do)
        const int tokens = cls_len[0] + cls_len[1] + cls_len[2] + cls_len[3];
        S = max(1, min(a.splits, (int)ceilf((float)tokens * a.len_scale)));
        if (split >= S) {
            if (a.k_new) __syncthreads();
            count_tables_read(a.k_new != nullptr, b);
            finish_append(a, b, kvh, split, new_row);
            return;
        }
    }
    // ---- the query operands of all classes, one class per wavefront ----
    if constexpr (F32) stage_q_split<HD, G>(a, sm, b, kvh, wave);
    else stage_q_operands<HD>(a, sm, b, kvh, wave, bf16seg);

    // ---- the workgroup's range of the stream [16-bit | 8-bit | 4-bit | 2-bit] of (b, kvh), and what of it this wavefront has from the
    //      start: a few tickets, all of them where the launch asks for fixed shares, or (one and four groups) blocks own[c] up to own_end[c] ----
    Tickets tk;
    tk.synced = false;
    tk.appends = a.k_new != nullptr;
    BlockSrc src[4];
    int own[4], own_end[4];
    {
        int nb[4];
#pragma unroll
        for (int c = 0; c < 3; c++) nb[c] = (cls_len[c] + 31) >> 5;
        nb[3] = a.mfma16 ? (cls_len[3] + 31) >> 5 : 0;
        unsigned total = 0u;
#pragma unroll
        for (int c = 0; c < 4; c++) total += (unsigned)nb[c] * (unsigned)block_cost<HD, G>(c);
        // cost at which split x starts: floor(total * x / S) up to rounding (one reciprocal, the same bits in every wavefront of
        // the launch; even lanes find this split's, odd ones the next one's); split 0 starts at cost 0, the last one ends behind everything
        const unsigned start = min(total, (unsigned)((float)total * ((float)(split + (lane & 1)) * __builtin_amdgcn_rcpf((float)S))));
        const unsigned G0 = (unsigned)__builtin_amdgcn_readlane((int)start, 0), next = (unsigned)__builtin_amdgcn_readlane((int)start, 1);
        const unsigned G1 = split == S - 1 ? total : next;
        // ... and the wavefront's share of the cost, where it has one: 5 parts for the older of the two that share a SIMD, 3 for the
        // younger, whose instructions wait for the older one's (with equal shares the older four were done at 13.1 us, the others
        // at 17.5).  8 x 12795 tokens, 28/4 heads of 128, group 32: 21.6 -> 21.0 us a call, all of 8 bits 26.0 -> 24.5; 6 x 19700, 8/8 heads of 64,
        // group 64: 25.1 -> 23.8; one sequence of 3271: 9.8 either way.  (9 : 7 gains 1 %, 19 : 13 2 %, this 3 % over 14 shapes.)  Equal
        // shares up to a block each, where 5 parts would be two for some: 3 sequences of up to 2592 tokens, 32/8 heads of 128, 64.7 us a step of 4
        // layers, so 58.5.
        static_assert(WQ_WAVES == 8, "the shares");
        const unsigned cost = G1 - G0;
        const bool few = cost < 9u * (unsigned)block_cost<HD, G>(1);
        unsigned t = 0u;
        if constexpr (F32) {
            // A share is whole blocks, and those of the 16-bit class cost as much as three others: which wavefronts get one more, and
            // which SIMD two wavefronts with some, decides a short range.  So both ways of sharing are laid out, 5 : 3 in lanes 0 to 8 and equal ones in
            // lanes 16 to 24 (lane w: where wavefront w begins), and the one whose slowest SIMD is done first is taken: after the older
            // one's cost, or the younger one's and two fifths of the older one's (it gets 3 instructions in while the older one issues 5).  Ranges of up to 16
            // 16-bit blocks; above, rounding to blocks matters less than the 5 : 3.  8 x 4000 tokens, 500 of them in 16 bits, 28/4 heads of 128, group
            // 128: equal shares 12.6 us a call, 5 : 3 13.8, so 12.7; 13 x 2600, 100 in 16 bits, 14/2 heads of 64: 8.3, 7.5 and 7.6; 16 x 1040, 60 in 16 bits, 32/8
            // heads of 128: 11.7, 12.7 and 11.6; over 300 shapes 1.012 times as fast as by the count of blocks alone (all edges by lanes, instead of two per
            // class one after the other on the scalar unit, is 0.1 us of it), 0.93 at least.
            const unsigned w = min((unsigned)lane & 15u, (unsigned)WQ_WAVES), parts = (lane & 16) ? 4u * w : min(5u * w, 3u * w + 8u);
            const unsigned x = G0 + (cost >> 5) * parts + (((cost & 31u) * parts) >> 5);
            int at[4], mine = 0;
            unsigned base = 0u;
#pragma unroll
            for (int c = 3; c >= 0; c--) {
                at[c] = range_edge_of<HD, G>(c, x, base, nb[c]);
                const int n = __builtin_amdgcn_update_dpp(0, at[c], 0x101, 0xF, 0xF, true) - at[c];         // (row_shl:1: the next lane's)
                mine += __mul24(n, block_cost<HD, G>(c));
                base += (unsigned)nb[c] * (unsigned)block_cost<HD, G>(c);
            }
            const int younger = __builtin_amdgcn_update_dpp(0, mine, 0x104, 0xF, 0xF, true);                // (row_shl:4)
            int done = 2 * mine + max(3 * mine, 5 * younger);                                               // (fifths)
            done = max(done, __builtin_amdgcn_update_dpp(0, done, 0xB1, 0xF, 0xF, true));                   // (quad_perm: of the four SIMDs, lanes 0 to 3 of a row)
            done = max(done, __builtin_amdgcn_update_dpp(0, done, 0x4E, 0xF, 0xF, true));
            const int uneven = __builtin_amdgcn_readlane(done, 0), equal = __builtin_amdgcn_readlane(done, 16);
            const int l = wave + (cost <= 16u * (unsigned)block_cost<HD, G>(3) && (equal < uneven || (equal == uneven && few)) ? 16 : 0);
#pragma unroll
            for (int c = 3; c >= 0; c--) {
                own[c] = __builtin_amdgcn_readlane(at[c], l);
                own_end[c] = __builtin_amdgcn_readlane(at[c], l + 1);
            }
        } else {
            auto parts_before = [&](int w) { return (unsigned)(few ? 4 * w : min(5 * w, 3 * w + 8)); };
            const unsigned long long span = cost;
            const unsigned x0 = G0 + (unsigned)((span * parts_before(wave)) >> 5), x1 = G0 + (unsigned)((span * parts_before(wave + 1)) >> 5);
            unsigned base = 0u;
            unsigned bases[4];
#pragma unroll
            for (int c = 3; c >= 0; c--) {
                bases[c] = base;
                const int e0 = range_edge_of<HD, G>(c, G0, base, nb[c]);
                const int e1 = range_edge_of<HD, G>(c, G1, base, nb[c]);
                src[c].pool_first = e0;
                src[c].tk_lo = t;
                t += (unsigned)(e1 - e0);
                src[c].tk_hi = e1 > e0 ? t : 0u;
                base += (unsigned)nb[c] * (unsigned)block_cost<HD, G>(c);
            }
            // The first tickets are fixed, so that the first loads can go out before the workgroup's set-up barrier; the counter
            // starts behind them.  WQ_FIRST_TICKETS consecutive blocks per wavefront, or, in a range of fewer blocks, what
            // spreads them over all eight: a block's arithmetic is half a microsecond, and with four blocks each the first
            // wavefronts of a short range walked it one block after the other beside idle ones (5 blocks, heads of 64: 9.0 -> 6.6 us
            // a call; 13 blocks, heads of 128: 15.8 -> 13.3)
            const unsigned first = min((unsigned)WQ_FIRST_TICKETS, (t + (unsigned)WQ_WAVES - 1u) / (unsigned)WQ_WAVES);
            tk.held = (unsigned)wave * first;
            tk.end = tk.held + first;
            tk.dealt = first * (unsigned)WQ_WAVES >= t;
            tk.taper = t > (unsigned)WQ_TAPER_TICKETS ? t - (unsigned)WQ_TAPER_TICKETS : 0xFFFFFFFFu;
            tk.ctr = &sm.next_ticket;
            if (tid == 0) sm.next_ticket = first * (unsigned)WQ_WAVES;
            if (a.fixed_shares) {
                tk.held = tk.end = 0u;
#pragma unroll
                for (int c = 3; c >= 0; c--) {
                    tk.held += (unsigned)(range_edge_of<HD, G>(c, x0, bases[c], nb[c]) - src[c].pool_first);
                    tk.end += (unsigned)(range_edge_of<HD, G>(c, x1, bases[c], nb[c]) - src[c].pool_first);
                }
                tk.dealt = true;
                tk.taper = 0xFFFFFFFFu;
            }
        }
    }

    WQ_STAMP(1);
#ifdef WQ_TIMELINE
    if (a.dbg && threadIdx.x == 0) {
        a.dbg[WQ_WG * 64 + 6] = __builtin_amdgcn_s_getreg((31 << 11) | 4);    // HW_ID
        a.dbg[WQ_WG * 64 + 7] = -(long long)__builtin_readcyclecounter();
    }
#endif

    if constexpr (F32) {
        SplitState<HD, G> st;
#pragma unroll
        for (int ct = 0; ct < CT; ct++) st.O[ct] = st.P[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
        st.m = -INFINITY;
        st.l = 0.f;
        st.ref = 0u;
        st.own = 1.0f;
#pragma unroll
        for (int s = 0; s < SplitState<HD, G>::SETS; s++) {
            st.accM[s] = 0.f;
            st.place[s] = 1.0f;
        }
        if (own[3] < own_end[3]) {
            F32State<HD> st16;
#pragma unroll
            for (int ct = 0; ct < CT; ct++) st16.O[ct][0] = st16.O[ct][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            st16.m = -INFINITY;
            st16.l = 0.f;
            load_q_quarter<HD>(a, b, kvh, st16.q);
            if (bf16seg)
                walk_seg16_f32<HD, true, G>(a, sm, b, kvh, cls_len[3], cls_off[3], own[3], own_end[3], tk, st16, new_row);
            else
                walk_seg16_f32<HD, false, G>(a, sm, b, kvh, cls_len[3], cls_off[3], own[3], own_end[3], tk, st16, new_row);
            carry_on<HD, G>(st16, st);
        }
        walk_class_split<HD, 8, G, G == 4 ? 1 : 2>(a, sm, b, kvh, cls_len[2], cls_off[2], own[2], own_end[2], tk, st);
        walk_class_split<HD, 4, G, 2>(a, sm, b, kvh, cls_len[1], cls_off[1], own[1], own_end[1], tk, st);
        walk_class_split<HD, 2, G, 2>(a, sm, b, kvh, cls_len[0], cls_off[0], own[0], own_end[0], tk, st);
        hand_over_split<HD, G>(sm, st);
    } else {
        const float c_log2 = a.sm_scale * 1.4426950408889634f;
        WaveState<HD> st;
#pragma unroll
        for (int ct = 0; ct < CT; ct++) st.O[ct] = floatx4{0.f, 0.f, 0.f, 0.f};
        st.m = -INFINITY;
        st.l = 0.f;
        st.accM = 0.f;
        st.up = weight_upscale(v_scale_max);
        const float o_unit = pow2_of(24.0f - st.up);   // what an accumulator of the value product counts in units of
        WQ_WSTAMP(0, wall_clock64());
        if (has_blocks(src[3], tk, 1u)) {              // (most wavefronts have no block of the 16-bit segment and go straight on)
            if (bf16seg)
                walk_seg16_mfma<HD, true>(a, sm, b, kvh, cls_len[3], cls_off[3], src[3], tk, c_log2, st, new_row);
            else
                walk_seg16_mfma<HD, false>(a, sm, b, kvh, cls_len[3], cls_off[3], src[3], tk, c_log2, st, new_row);
            // the quantized classes accumulate 2^(up-24) * (p s_v code); bring the 16-bit part to the same unit (exact)
            const float to_unit = pow2_of(st.up - 24.0f);
#pragma unroll
            for (int ct = 0; ct < CT; ct++) st.O[ct] *= to_unit;
        }
        WQ_WSTAMP(1, wall_clock64());
        walk_class_mfma<HD, 8, WQ_D8>(a, sm, b, kvh, cls_len[2], cls_off[2], src[2], tk, c_log2, st);
        WQ_WSTAMP(2, wall_clock64());
        walk_class_mfma<HD, 4, WQ_D4>(a, sm, b, kvh, cls_len[1], cls_off[1], src[1], tk, c_log2, st);
        WQ_WSTAMP(3, wall_clock64());
        walk_class_mfma<HD, 2, WQ_D2>(a, sm, b, kvh, cls_len[0], cls_off[0], src[0], tk, c_log2, st);
        WQ_WSTAMP(4, wall_clock64());

        WQ_STAMP(4);
#ifdef WQ_TIMELINE
        if (a.dbg && threadIdx.x == 0) a.dbg[WQ_WG * 64 + 7] += (long long)__builtin_readcyclecounter();
#endif
        // ---- reduce the lane groups' shares, hand the wave's numerators to LDS ----
        float l = st.l, am = st.accM;
        l = sum_over_rows(l);
        am = sum_over_rows(am);
#pragma unroll
        for (int ct = 0; ct < CT / 2; ct++) {          // this column's group owns the channel tiles g CT / 2 ...
            floatx4 v;
#pragma unroll
            for (int i = 0; i < 4; i++) v[i] = fmaf(g ? st.O[CT / 2 + ct][i] : st.O[ct][i], o_unit, am);
            *reinterpret_cast<floatx4*>(&sm.O[wave][h][g * (HD / 2) + 16 * ct + 4 * j]) = v;
        }
        if (j == 0 && g == 0) {
            sm.ml[wave][h][0] = st.m;
            sm.ml[wave][h][1] = l;
        }
    }
    pass_setup_barrier(b, tk);
    // what the end needs of the arguments: there when the other wavefronts are
    const DecodeArgs& e = F32 ? a : args_again();         // (with the walkers of one and four groups they fit the scalar registers)
    int rep = e.rep, nparts = e.nparts, Hq = e.Hq, fused = e.fused, arrive_unit = e.arrive_unit;
    unsigned* arrive = e.arrive;
    float *part = e.part, *part_ml = e.part_ml, *out = e.out, *lse = e.lse;
    if constexpr (!F32)
        asm volatile("" : "+s"(rep), "+s"(nparts), "+s"(Hq), "+s"(fused), "+s"(arrive_unit), "+s"(arrive), "+s"(part), "+s"(part_ml), "+s"(out), "+s"(lse));
    if (new_row >= 0 && split == 0 && wave == WQ_WAVES - 1 && lane < 2 * (HD / 8)) {
        const int plane = lane / (HD / 8), piece = lane % (HD / 8);
        uint16_t* const dst = in_memory(static_cast<uint16_t*>(plane ? e.kv.v16 : e.kv.k16)) + (((int64_t)cls_off[3] + new_row) * e.kv.Hkv + kvh) * HD + piece * 8;
        *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(in_memory(plane ? e.v_new : e.k_new) + (int64_t)unit * HD + piece * 8);
    }
    __syncthreads();
    // ---- merge the wavefronts, write the partial (m in natural-log units): wavefront r takes head r, a lane CPL
    //      neighbouring channels, so the eight scales of a head are computed once per lane ----
    constexpr int CPL = HD / 64;                   // channels per lane
    static_assert(WQ_WAVES >= WQ_MAX_REP, "one wavefront per head");
    const int64_t part_row = (int64_t)unit * nparts * rep;          // the unit's first row (split 0, head 0)
    if (wave < rep) {
        const int64_t row = part_row + split * rep + wave;
        float mw[WQ_WAVES];
#pragma unroll
        for (int w = 0; w < WQ_WAVES; w++) mw[w] = sm.ml[w][wave][0];
        float M = mw[0];
#pragma unroll
        for (int w = 1; w < WQ_WAVES; w++) M = fmaxf(M, mw[w]);
        float num[CPL], L = 0.f;
#pragma unroll
        for (int c = 0; c < CPL; c++) num[c] = 0.f;
#pragma unroll
        for (int w = 0; w < WQ_WAVES; w++) {
            const float sc = (mw[w] == -INFINITY) ? 0.f : F32 ? __expf(mw[w] - M) : __builtin_amdgcn_exp2f(mw[w] - M);
#pragma unroll
            for (int c = 0; c < CPL; c++) num[c] = fmaf(sm.O[w][wave][CPL * lane + c], sc, num[c]);
            L = fmaf(sm.ml[w][wave][1], sc, L);
        }
        // device-scope stores go through to memory (every XCD has an L2 of its own), so that no cache write-back
        // is needed to hand the partial to the workgroup that merges the splits
        store_through<CPL>(in_memory(part) + row * HD + CPL * lane, num);
        if (lane == 0) {
            const float ml2[2] = {F32 ? M : M * 0.6931471805599453f, L};       // (the walkers of one and four groups keep the reference in natural units)
            store_through<2>(in_memory(part_ml) + row * 2, ml2);
        }
    }
    WQ_STAMP(5);
    if (!fused) return;

    // ---- the last workgroup of (b, kvh) to get here merges the partials of all splits, in the order of merge_weights_lanes; head by head:
    //      head r's partial was written by wavefront r alone, so wavefront r reports in for it on a counter of its own
    //      and, if it is the last to do so, merges head r, without a word to the other wavefronts ----
    // The partial was stored with device-scope stores, which go through to memory.  The wavefront waits until the
    // memory system has acknowledged its stores (vmcnt(0): what a fence of narrower scope does not make the compiler
    // emit) and only then counts itself, so the wavefront that finds itself last reads partials that have arrived, with
    // device-scope loads that do not stop at a cache.  This costs one memory round trip; a device-scope release fence
    // would add a write-back of the whole L2 (measured: 19 us per call).
    bool last = false;
    if (wave < rep) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        WQ_STAMP(56);
        unsigned* const counter = in_memory(arrive) + unit * arrive_unit + wave * (arrive_unit / WQ_MAX_REP);
        static_assert(WQ_ARRIVE_STRIDE >= WQ_MAX_REP, "one counter per head inside a unit's piece");
        unsigned old = 0u;
        if (lane == 0) old = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = (unsigned)__builtin_amdgcn_readfirstlane((int)old) == (unsigned)S - 1u;
        WQ_STAMP(57);
        if (last && lane == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    }
    // What follows runs once per (b, kvh, head) while the rest of the chip waits, and an instruction of a lone wavefront takes
    // about 2 ns: every instruction counts.  Lane l holds (m, l) of split split_of_lane(l) (the launch takes this path with at most 64
    // splits), the weights come from reductions inside the wavefront.  The four rows of 16 lanes take every fourth split each,
    // 16 bytes of it per lane and load, all of them in flight together; a split's weight is lane k of its row
    // (row_bcast), and the rows' sums are folded into each other, two of them at a time and half the channels
    // each.  No LDS, no barrier.  The partials are read through buffer descriptors, whose range check returns zero beyond the last split.
    // Against a split per load, 8 bytes per lane, the weight read back as a scalar, and numerators handed over 4 bytes at a time: a step of
    // 28 launches with 32 splits 360 -> 331 us, with 8 splits 552 -> 537; 4 calls with 16 splits 100.6 -> 99.0.
    if (last) {
        const int np = S;                          // (the splits are all the partials there are in a launch that merges them itself)
        const int r = lane >> 4, k16 = lane & 15;
        constexpr int PIECES = HD / 64;            // 16-byte pieces of a split's channels per lane
        const unsigned rows = (unsigned)(np * rep);
        const int first_row = __builtin_amdgcn_readfirstlane((int)part_row);         // (few units, few splits: merges_itself)
        const __amdgpu_buffer_rsrc_t mls = __builtin_amdgcn_make_buffer_rsrc(part_ml + (int64_t)first_row * 2, 0, (int)(rows * 8u), 0x00020000);
        const __amdgpu_buffer_rsrc_t nums = __builtin_amdgcn_make_buffer_rsrc(part + (int64_t)first_row * HD, 0, (int)(rows * (HD * 4u)), 0x00020000);
        const int s_l = split_of_lane(lane);
        const floatx2 ml = ld_part2(mls, (unsigned)(s_l * rep + wave) * 8u);
        const unsigned chan = (unsigned)(r * rep + wave) * (HD * 4u) + (unsigned)k16 * 16u, step = (unsigned)rep * (MERGE_CHAINS * HD * 4u);
        float w_s = 0.f, M = -INFINITY, L = 0.f;
        floatx4 acc[PIECES];
#pragma unroll
        for (int p = 0; p < PIECES; p++) acc[p] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto gather = [&](auto N) {                // N splits per row
            constexpr int NS = decltype(N)::value;
            floatx4 pre[NS][PIECES];
#pragma unroll
            for (int k = 0; k < NS; k++)
#pragma unroll
                for (int p = 0; p < PIECES; p++) pre[k][p] = ld_part4(nums, chan + (unsigned)k * step + p * 256u);
            merge_weights_lanes(s_l < np ? ml[0] : -INFINITY, ml[1], w_s, M, L);
            auto add = [&](auto K) {               // (a split beyond the last one: zeros times zero)
                constexpr int k = decltype(K)::value;
                const float wk = row_bcast<k>(w_s);
#pragma unroll
                for (int p = 0; p < PIECES; p++)
#pragma unroll
                    for (int c = 0; c < 4; c++) acc[p][c] = fmaf(wk, pre[k][p][c], acc[p][c]);
            };
            for_each_index(add, std::make_integer_sequence<int, NS>{});
        };
        if (np <= 16) gather(std::integral_constant<int, 4>{});
        else if (np <= 32) gather(std::integral_constant<int, 8>{});
        else gather(std::integral_constant<int, 16>{});
        WQ_STAMP(58);
        const int hq = kvh * rep + wave;
        float o[CPL];
        int ch;                                    // the first of the lane's channels
        if constexpr (PIECES == 2) {
            float h[4];
#pragma unroll
            for (int c = 0; c < 4; c++) h[c] = fold_halves(acc[0][c], acc[1][c]);
#pragma unroll
            for (int c = 0; c < 2; c++) o[c] = fold_rows(h[c], h[c + 2]);
            ch = 64 * (r >> 1) + 4 * k16 + 2 * (r & 1);
        } else {
            o[0] = fold_rows(fold_halves(acc[0][0], acc[0][2]), fold_halves(acc[0][1], acc[0][3]));
            ch = 4 * k16 + 2 * (r >> 1) + (r & 1);
        }
#pragma unroll
        for (int c = 0; c < CPL; c++) o[c] = L > 0.f ? o[c] / L : 0.f;
        store_plain<CPL>(in_memory(out) + ((int64_t)b * Hq + hq) * HD + ch, o);
        if (lse && lane == 0) in_memory(lse)[(int64_t)b * Hq + hq] = L > 0.f ? M + logf(L) : -INFINITY;
    }
    WQ_STAMP(59);
    if constexpr (PACKED)
        finish_append_by_length(e, sm, (int)blockIdx.x);
    else
        finish_append(e, b, kvh, split, new_row);
}

}  // namespace
