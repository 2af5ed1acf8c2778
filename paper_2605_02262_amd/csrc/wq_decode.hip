// a4: decode attention over the packed mixed-precision cache (Alg. 2 decode half; Sec. 3.3.2 shows that the
// block order does not matter without a mask, which is also what makes the split over tokens legal).
//
// One workgroup per (split, KV head, sequence) walks its share of the 2-, 4-, 8- and 16-bit segments with an
// online softmax (running max m, running sum l, unnormalised accumulator), writes one partial (m, l, acc) per
// query head; k_combine, or the matrix-core kernel itself, merges the partials of all splits by log-sum-exp: splits s, s + 4, ... one after the
// other for s = 0..3, then (0 + 2) + (1 + 3).  No float atomics: with fixed shares, which one and four groups per head always have, and in the
// vector kernel a split count fixes every bit.
//
// k_decode_generic: plain vector-ALU kernel that reads codes field by field from the storage layout.  It
// handles every supported (hd, group) and query type and is the reference implementation inside the library; the
// matrix-core body in wq_decode_mfma.h is the fast path (use_matrix_cores below says where it is taken).
#include <stddef.h>
#include <stdlib.h>

#include <initializer_list>
#include <type_traits>
#include <utility>

#include "wq_internal.h"

namespace {

struct DecodeArgs {         // (what the matrix-core kernel reads of it comes first)
    int q_dtype;
    int B, Hq, rep, splits;
    float sm_scale;
    float len_scale;        // > 0: a (sequence, KV head) with n tokens uses ceil(n * len_scale) of the launch's splits (at least one)
    int nparts;             // partials per (b, KV head): splits + splits16
    int mfma16;             // the matrix-core kernel also walks the 16-bit segment
    int fused;              // the matrix-core kernel merges the splits itself (last workgroup per (b, KV head))
    int fixed_shares;       // every wavefront of the matrix-core kernel gets a fixed share of its workgroup's range
    int arrive_unit;
    unsigned* arrive;       // [B*Hkv] pieces of arrive_unit words (WQ_MAX_REP arrival counters each), then [B] append counters, zero between launches
    wq_packed_kv kv;
    const void* q;
    // appending one generated token per sequence in the same launch (matrix-core kernel, merged splits only):
    const uint16_t* k_new;  // [B][Hkv][hd] in the cache's 16-bit type, or NULL
    const uint16_t* v_new;
    uint32_t* status;       // device status word (a full 16-bit segment is reported there)
    float* part;            // numerators of the partials [B][Hkv][nparts][rep][hd]
    float* part_ml;         // ... their references and weight sums [B][Hkv][nparts][rep][2]
    float* out;
    float* lse;
    int slots;              // splits by length, workgroups with work numbered without gaps (place_by_length); > 0: automatic, at most this many splits of all sequences together
    int even_splits;        // ... and what a sequence gets where the kernel finds all of them equally long
    int packed_grid;
    int splits16;           // workgroups of the vector kernel on the 16-bit segment
    int use_mfma;
#ifdef WQ_TIMELINE
    long long* dbg;
#endif
};
static_assert(offsetof(DecodeArgs, slots) <= 5 * 64, "the matrix-core kernel touches five lines of arguments, all of them with its first loads (by length one more, behind its tables): a sixth is a round trip of 0.3 us");

// ---- the weights of the splits -----------------------------------------------------------------------------
// Reductions over the 64 lanes of a wavefront in a fixed order: four rotations inside the rows of 16 lanes (one
// data-parallel-primitive instruction each, no LDS), then the four rows' results as scalars.
template <int CTRL>
__device__ __forceinline__ float lanes_moved(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_value(float x, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ __forceinline__ float wave_max(float x)
{
    x = fmaxf(x, lanes_moved<0x128>(x));           // row_ror:8, 4, 2, 1
    x = fmaxf(x, lanes_moved<0x124>(x));
    x = fmaxf(x, lanes_moved<0x122>(x));
    x = fmaxf(x, lanes_moved<0x121>(x));
    return fmaxf(fmaxf(lane_value(x, 0), lane_value(x, 16)), fmaxf(lane_value(x, 32), lane_value(x, 48)));
}
__device__ __forceinline__ float wave_sum(float x)
{
    x += lanes_moved<0x128>(x);
    x += lanes_moved<0x124>(x);
    x += lanes_moved<0x122>(x);
    x += lanes_moved<0x121>(x);
    return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// Up to 64 splits, one per lane: lane l holds m_s (-inf beyond the last split) and l_s of split s = split_of_lane(l); it gets
// the weight w_s = e^{m_s - M}, and every lane M = max m_s and L = sum l_s w_s.  Both merges (the one inside the matrix-core
// kernel and k_combine) go through this function when there are at most 64 splits and then sum the numerators in the
// same order (splits s, s + 4, ... one after the other for s = 0..3, then (0 + 2) + (1 + 3)), which is why their results agree bit for bit.
constexpr int MERGE_CHAINS = 4;                    // one per row of 16 lanes
__device__ __forceinline__ int split_of_lane(int lane) { return MERGE_CHAINS * (lane & 15) + (lane >> 4); }
__device__ __forceinline__ void merge_weights_lanes(float m, float l, float& w, float& M, float& L)
{
    M = wave_max(m);
    w = (m == -INFINITY) ? 0.f : __expf(m - M);
    L = wave_sum(l * w);
}

// More than 64 splits (k_combine only): one wavefront turns the m_s of n splits (in w) into the weights in place and
// returns M and L.  Lane i takes the splits i, i + 64, ..., then the lanes are reduced as above.
__device__ __forceinline__ void merge_weights(float* w, const float* l, int n, float& M, float& L)
{
    const int lane = threadIdx.x & 63;
    float mx = -INFINITY;
    for (int s = lane; s < n; s += 64) mx = fmaxf(mx, w[s]);
    mx = wave_max(mx);
    float sum = 0.f;
    for (int s = lane; s < n; s += 64) {
        const float ms = w[s];
        const float e = (ms == -INFINITY) ? 0.f : __expf(ms - mx);
        w[s] = e;
        sum = fmaf(l[s], e, sum);
    }
    M = mx;
    L = wave_sum(sum);
}

__device__ __forceinline__ float load_q(const void* q, int dtype, int64_t i)
{
    if (dtype == WQ_F32) return static_cast<const float*>(q)[i];
    if (dtype == WQ_BF16) return wq_bf16_bits_to_float(static_cast<const uint16_t*>(q)[i]);
    return wq_f16_bits_to_float(static_cast<const uint16_t*>(q)[i]);
}

}  // namespace

#include "wq_decode_mfma.h"

namespace {

// field n (BITS wide) of a little-endian packed byte image
template <int BITS>
__device__ __forceinline__ int field(const uint8_t* base, int64_t n)
{
    int64_t bit = n * BITS;
    return (base[bit >> 3] >> (bit & 7)) & ((1 << BITS) - 1);
}

template <int HD>
struct Smem {
    float q[WQ_MAX_REP][HD];
    float logit[WQ_MAX_REP][32];
    float p[WQ_MAX_REP][32];
    float red[256 / HD][WQ_MAX_REP][HD];
    float m[WQ_MAX_REP], l[WQ_MAX_REP], scale[WQ_MAX_REP];
};

// One 32-token step: logits are in sm.logit (-inf for invalid tokens).  Thread (r = tid/32, u = tid%32) owns one
// (head, token) pair: block max and sum by wavefront shuffles inside its 32 lanes, running (m, l) in LDS; leaves the
// weights in sm.p and rescales every thread's accumulators.
template <int HD>
__device__ __forceinline__ void softmax_step(Smem<HD>& sm, int rep, float* acc)
{
    const int tid = threadIdx.x;
    const int r = tid >> 5, u = tid & 31;
    const float lg = r < rep ? sm.logit[r][u] : -INFINITY;
    float bm = lg;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) bm = fmaxf(bm, __shfl_xor(bm, o, 64));
    const float mo = sm.m[r];
    const float mn = fmaxf(mo, bm);
    const float p = (mn == -INFINITY) ? 0.f : __expf(lg - mn);
    float ps = p;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) ps += __shfl_xor(ps, o, 64);
    sm.p[r][u] = p;
    __syncthreads();                      // every lane has read the old m before it changes
    if (u == 0) {
        const float sc = (mn == -INFINITY) ? 1.0f : __expf(mo - mn);
        sm.scale[r] = sc;
        sm.m[r] = mn;
        sm.l[r] = sm.l[r] * sc + ps;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < WQ_MAX_REP; k++) acc[k] *= sm.scale[k];
}

template <int HD, int BITS>
__device__ void walk_class(const DecodeArgs& a, Smem<HD>& sm, int b, int kvh, int share, int nshare, float* acc)
{
    constexpr int C = BITS == 2 ? 0 : (BITS == 4 ? 1 : 2);
    constexpr int Q = HD / 4, CT = HD / 16, PARTS = 256 / HD;
    const wq_packed_kv& kv = a.kv;
    const int tid = threadIdx.x;
    const int G = HD / kv.group;
    const int len = kv.cls_len[C][b];
    const int nblk = (len + 31) / 32;
    const int blk_lo = (int)((int64_t)share * nblk / nshare), blk_hi = (int)((int64_t)(share + 1) * nblk / nshare);
    const int64_t tok_base = kv.cls_off[C][b];
    const int64_t cap = kv.cap[C];
    const uint8_t* kcodes = static_cast<const uint8_t*>(kv.codes[C]) + (int64_t)kvh * cap * HD * BITS / 8;
    const uint8_t* vcodes = static_cast<const uint8_t*>(kv.codes[C]) + ((int64_t)kv.Hkv + kvh) * cap * HD * BITS / 8;
    const uint32_t* kmeta = static_cast<const uint32_t*>(kv.meta[C]) + (int64_t)kvh * cap * G;
    const uint32_t* vmeta = static_cast<const uint32_t*>(kv.meta[C]) + ((int64_t)kv.Hkv + kvh) * cap * G;

    for (int blk = blk_lo; blk < blk_hi; blk++) {
        const int64_t t0 = tok_base + (int64_t)blk * 32;       // absolute token slot of the block
        // ---- logits: thread = (token u, eighth p of the channels) ----
        {
            const int u = tid >> 3, p = tid & 7;
            const int64_t t = t0 + u;
            const int64_t tile = t >> 4;
            const int mrow = (int)(t & 15);
            const uint8_t* tb = kcodes + tile * (16 * HD * BITS / 8);
            float part[WQ_MAX_REP];
#pragma unroll
            for (int r = 0; r < WQ_MAX_REP; r++) part[r] = 0.f;
            for (int i = 0; i < HD / 8; i++) {
                int ch = p * (HD / 8) + i;
                int j = ch / Q, e = ch % Q;
                int code = field<BITS>(tb, (int64_t)(j * 16 + mrow) * Q + e);
                uint32_t w = kmeta[(tile * G + ch / kv.group) * 16 + mrow];
                float kh = fmaf(wq_f16_bits_to_float(w & 0xFFFF), (float)code, wq_f16_bits_to_float(w >> 16));
#pragma unroll
                for (int r = 0; r < WQ_MAX_REP; r++)
                    if (r < a.rep) part[r] = fmaf(sm.q[r][ch], kh, part[r]);
            }
#pragma unroll
            for (int r = 0; r < WQ_MAX_REP; r++) {
                float v = part[r];
                v += __shfl_xor(v, 1, 64);
                v += __shfl_xor(v, 2, 64);
                v += __shfl_xor(v, 4, 64);
                if (p == 0 && r < a.rep) sm.logit[r][u] = (blk * 32 + u < len) ? v * a.sm_scale : -INFINITY;
            }
        }
        __syncthreads();
        softmax_step<HD>(sm, a.rep, acc);
        // ---- values: thread = (channel c, token part tp) ----
        {
            const int c = tid % HD, tp = tid / HD;
            const int ct = c / 16, mm = c % 16;
            const uint8_t* vb = vcodes + (t0 >> 5) * (32 * HD * BITS / 8);
            for (int u = tp * (32 / PARTS); u < (tp + 1) * (32 / PARTS); u++) {
                int jj = (u % 16) / 4, tau = 4 * (u / 16) + u % 4;
                int code = field<BITS>(vb, ((int64_t)(jj * 16 + mm) * CT + ct) * 8 + tau);
                const int64_t t = t0 + u;
                uint32_t w = vmeta[((t >> 4) * G + c / kv.group) * 16 + (t & 15)];
                float vh = fmaf(wq_f16_bits_to_float(w & 0xFFFF), (float)code, wq_f16_bits_to_float(w >> 16));
#pragma unroll
                for (int r = 0; r < WQ_MAX_REP; r++)
                    if (r < a.rep) acc[r] = fmaf(sm.p[r][u], vh, acc[r]);
            }
        }
        __syncthreads();
    }
}

template <int HD>
__device__ void walk_seg16(const DecodeArgs& a, Smem<HD>& sm, int b, int kvh, int share, int nshare, float* acc)
{
    constexpr int PARTS = 256 / HD;
    const wq_packed_kv& kv = a.kv;
    const int tid = threadIdx.x;
    const int len = kv.len16[b];
    const int nblk = (len + 31) / 32;
    const int blk_lo = (int)((int64_t)share * nblk / nshare), blk_hi = (int)((int64_t)(share + 1) * nblk / nshare);
    const uint16_t* k16 = static_cast<const uint16_t*>(kv.k16);
    const uint16_t* v16 = static_cast<const uint16_t*>(kv.v16);
    const bool bf = kv.dtype16 == WQ_BF16;
    for (int blk = blk_lo; blk < blk_hi; blk++) {
        {
            const int u = tid >> 3, p = tid & 7;
            const int i = blk * 32 + u;
            const bool valid = i < len;
            const int64_t row = ((int64_t)kv.off16[b] + (valid ? i : 0)) * kv.Hkv + kvh;
            float part[WQ_MAX_REP];
#pragma unroll
            for (int r = 0; r < WQ_MAX_REP; r++) part[r] = 0.f;
            for (int k = 0; k < HD / 8; k++) {
                int ch = p * (HD / 8) + k;
                uint32_t h = valid ? k16[row * HD + ch] : 0;
                float kh = bf ? wq_bf16_bits_to_float(h) : wq_f16_bits_to_float(h);
#pragma unroll
                for (int r = 0; r < WQ_MAX_REP; r++)
                    if (r < a.rep) part[r] = fmaf(sm.q[r][ch], kh, part[r]);
            }
#pragma unroll
            for (int r = 0; r < WQ_MAX_REP; r++) {
                float v = part[r];
                v += __shfl_xor(v, 1, 64);
                v += __shfl_xor(v, 2, 64);
                v += __shfl_xor(v, 4, 64);
                if (p == 0 && r < a.rep) sm.logit[r][u] = valid ? v * a.sm_scale : -INFINITY;
            }
        }
        __syncthreads();
        softmax_step<HD>(sm, a.rep, acc);
        {
            const int c = tid % HD, tp = tid / HD;
            for (int u = tp * (32 / PARTS); u < (tp + 1) * (32 / PARTS); u++) {
                const int i = blk * 32 + u;
                if (i >= len) break;
                const int64_t row = ((int64_t)kv.off16[b] + i) * kv.Hkv + kvh;
                uint32_t h = v16[row * HD + c];
                float vh = bf ? wq_bf16_bits_to_float(h) : wq_f16_bits_to_float(h);
#pragma unroll
                for (int r = 0; r < WQ_MAX_REP; r++)
                    if (r < a.rep) acc[r] = fmaf(sm.p[r][u], vh, acc[r]);
            }
        }
        __syncthreads();
    }
}

template <int HD>
__device__ void decode_generic_body(const DecodeArgs& a, void* smem_raw, bool quantized, int share, int nshare, int part_idx)
{
    Smem<HD>& sm = *reinterpret_cast<Smem<HD>*>(smem_raw);
    const int kvh = blockIdx.y, b = blockIdx.z;
    const int tid = threadIdx.x;
    for (int i = tid; i < a.rep * HD; i += 256) {
        int r = i / HD, ch = i % HD;
        sm.q[r][ch] = load_q(a.q, a.q_dtype, ((int64_t)b * a.Hq + kvh * a.rep + r) * HD + ch);
    }
    __syncthreads();
    if (tid < WQ_MAX_REP) {
        sm.m[tid] = -INFINITY;
        sm.l[tid] = 0.f;
        sm.scale[tid] = 1.f;
    }
    __syncthreads();
    float acc[WQ_MAX_REP];
#pragma unroll
    for (int r = 0; r < WQ_MAX_REP; r++) acc[r] = 0.f;
    if (quantized) {
        walk_class<HD, 2>(a, sm, b, kvh, share, nshare, acc);
        walk_class<HD, 4>(a, sm, b, kvh, share, nshare, acc);
        walk_class<HD, 8>(a, sm, b, kvh, share, nshare, acc);
    }
    walk_seg16<HD>(a, sm, b, kvh, share, nshare, acc);

    // reduce the token parts, write the partial
    constexpr int PARTS = 256 / HD;
    const int c = tid % HD, tp = tid / HD;
#pragma unroll
    for (int r = 0; r < WQ_MAX_REP; r++)
        if (r < a.rep) sm.red[tp][r][c] = acc[r];
    __syncthreads();
    const int64_t row0 = (((int64_t)b * a.kv.Hkv + kvh) * a.nparts + part_idx) * a.rep;
    if (tp == 0) {
        for (int r = 0; r < a.rep; r++) {
            float s = 0.f;
            for (int k = 0; k < PARTS; k++) s += sm.red[k][r][c];
            a.part[(row0 + r) * HD + c] = s;
        }
    }
    if (tid < a.rep) {
        a.part_ml[(row0 + tid) * 2] = sm.m[tid];
        a.part_ml[(row0 + tid) * 2 + 1] = sm.l[tid];
    }
}

// Generic kernel: every segment (use_mfma == 0), or only the 16-bit segment next to a matrix-core launch, in
// which case its partials follow the matrix-core ones (slot splits + x).
template <int HD>
__global__ __launch_bounds__(256) void k_decode_generic(DecodeArgs a)
{
    __shared__ __align__(16) unsigned char smem[sizeof(Smem<HD>)];
    const int x = blockIdx.x;
    if (!a.use_mfma)
        decode_generic_body<HD>(a, smem, true, x, a.splits, x);
    else
        decode_generic_body<HD>(a, smem, false, x, a.splits16, a.splits + x);
}

// Matrix-core kernel: the quantized classes of one (split, KV head, sequence).
template <int HD, int G, bool PACKED>
__global__ __launch_bounds__(64 * WQ_WAVES) void k_decode_mfma(DecodeArgs a)
{
    __shared__ __align__(16) unsigned char smem[sizeof(DecodeSmem<HD, G>)];
    wq_decode_mfma_body<HD, G, PACKED>(a, smem);
}

// out[b,h,:] = sum_s acc_s e^{m_s - M} / sum_s l_s e^{m_s - M},  M = max_s m_s;  lse = M + log(sum).
// One workgroup per (b, h); the weights come from merge_weights (first wavefront), the numerators are summed with all loads
// of a thread independent of each other (no data-dependent control flow around them): the same arithmetic in the same order as
// the merge inside the matrix-core kernel.
__global__ __launch_bounds__(128) void k_combine(const float* __restrict__ part, const float* __restrict__ part_ml, int Hq, int rep, int nparts,
                                                 int hd, float* __restrict__ out, float* __restrict__ lse)
{
    __shared__ float s_w[1024 + 32];
    __shared__ float s_l[1024 + 32];
    __shared__ float s_red[2];
    const int h = blockIdx.x, b = blockIdx.y;
    const int kvh = h / rep, r = h % rep;
    const int Hkv = Hq / rep;
    const int tid = threadIdx.x;
    const int64_t row0 = (((int64_t)b * Hkv + kvh) * nparts) * rep + r, stride = (int64_t)rep * hd;
    const float* base = part + row0 * hd;
    const float* ml = part_ml + row0 * 2;
    constexpr int CHUNK = 32;
    float pre[CHUNK];                      // this channel's numerators of the first CHUNK splits: in flight while the weights are found
#pragma unroll
    for (int k = 0; k < CHUNK; k++) pre[k] = (k < nparts && tid < hd) ? base[(int64_t)k * stride + tid] : 0.f;
    for (int s = tid; s < nparts; s += 128) {
        s_w[s] = ml[(int64_t)s * rep * 2];
        s_l[s] = ml[(int64_t)s * rep * 2 + 1];
    }
    __syncthreads();
    if (tid < 64) {
        float M, L;
        if (nparts <= 64) {
            const int s = split_of_lane(tid);
            float w;
            merge_weights_lanes(s < nparts ? s_w[s] : -INFINITY, s < nparts ? s_l[s] : 0.f, w, M, L);
            if (s < nparts) s_w[s] = w;
        } else {
            merge_weights(s_w, s_l, nparts, M, L);
        }
        if (tid == 0) {
            s_red[0] = M;
            s_red[1] = L;
        }
    }
    __syncthreads();
    const float M = s_red[0], L = s_red[1];
    float acc[MERGE_CHAINS] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < CHUNK; k++) acc[k % MERGE_CHAINS] = fmaf(pre[k], k < nparts ? s_w[k] : 0.f, acc[k % MERGE_CHAINS]);
    if (tid < hd) {
        for (int s0 = CHUNK; s0 < nparts; s0 += CHUNK) {
            float v[CHUNK];
#pragma unroll
            for (int k = 0; k < CHUNK; k++) v[k] = (s0 + k < nparts) ? base[(int64_t)(s0 + k) * stride + tid] : 0.f;
#pragma unroll
            for (int k = 0; k < CHUNK; k++) acc[k % MERGE_CHAINS] = fmaf(v[k], (s0 + k < nparts) ? s_w[s0 + k] : 0.f, acc[k % MERGE_CHAINS]);
        }
        const float sum = (acc[0] + acc[2]) + (acc[1] + acc[3]);
        out[((int64_t)b * Hq + h) * hd + tid] = L > 0.f ? sum / L : 0.f;
    }
    if (lse && tid == 0) lse[(int64_t)b * Hq + h] = L > 0.f ? M + logf(L) : -INFINITY;
}

}  // namespace

// workgroups per (sequence, KV head) given to the 16-bit segment by the matrix-core launch: about one per
// 32 rows of the average sequence's capacity, between 1 and 32
static int wq_decode_splits16(int B, int64_t cap16)
{
    int64_t per = B > 0 ? cap16 / B : 0;
    int64_t n = (per + 31) / 32;
    return (int)(n < 1 ? 1 : (n > 32 ? 32 : n));
}

size_t wq_decode_ws_bytes(int B, int Hq, int hd, int splits)
{
    if (B <= 0 || Hq <= 0 || hd <= 0 || splits <= 0) return 0;
    return wq_align256(sizeof(float) * (size_t)B * Hq * (splits + 32) * (hd + 2));
}

// The matrix-core kernel's work is cut on a 32-bit cost axis (at most 500 per 32-token block).
static bool fits_cost_axis(const wq_packed_kv* kv)
{
    return (int64_t)kv->cap[0] + kv->cap[1] + kv->cap[2] + kv->cap16 <= (int64_t)1 << 27;
}

static bool aligned_16(std::initializer_list<const void*> pointers)
{
    uintptr_t bits = 0;
    for (const void* p : pointers) bits |= reinterpret_cast<uintptr_t>(p);
    return bits % 16 == 0;
}

// Which kernel walks the quantized classes.  Two groups per head: the matrix-core kernel, with the weights in one f16 value.
// One and four groups: the matrix-core kernel with its walkers of fp32 accuracy for 16-bit queries (measured, 8 x 12795 tokens,
// 28 / 4 heads of 128, group 32: 917 us a call on the vector kernel, 21.0 on them); fp32 queries and caches beyond the cost axis stay with the
// vector kernel, which also takes what does not lie on 16-byte boundaries (a query cut out of a larger tensor): it reads
// element by element.
static bool use_matrix_cores(const void* q, int q_dtype, const wq_packed_kv* kv, int balgo)
{
    if (balgo != WQ_DECODE_AUTO) return balgo == WQ_DECODE_MFMA;
    return kv->hd / kv->group == 2 ||
           (q_dtype != WQ_F32 && fits_cost_axis(kv) && aligned_16({q, kv->k16, kv->v16, kv->codes[0], kv->codes[1], kv->codes[2]}));
}

// Does a launch with these arguments merge the splits itself (all but their number looked at)?
static bool merges_itself(const void* q, int q_dtype, int B, const wq_packed_kv* kv, int algo)
{
    return !(algo & (WQ_DECODE_PARTIALS_ONLY | WQ_DECODE_SEPARATE_MERGE)) && use_matrix_cores(q, q_dtype, kv, algo & ~WQ_DECODE_FLAGS) &&
           !(kv->dtype16 == WQ_BF16 && q_dtype != WQ_BF16) && (int64_t)B * kv->Hkv <= WQ_MAX_ARRIVE;
}

// Splits of an automatic launch that merges them itself (0: this one does not), for sequences of up to max_seq_tokens.  The
// kernel's registers leave room for one workgroup per compute unit, so the launch runs in rounds of 256 workgroups: what
// counts is (rounds) x (fixed cost of a workgroup + its blocks).  A round begun for a few workgroups costs as much as a full
// one (9 sequences x 4 KV heads of 12800 tokens: 7 splits 20.8 us, 8 splits 30.4 us; 5 sequences: 12 splits 15.3, 13 splits
// 22.9), and several full rounds can beat one with idle compute units (20 x 8 of 12800: 1 split 68.8, 3 splits 63.3).  Up
// to 16 splits are merged with 4 loads in flight per row of lanes, up to 32 with 8, up to 64 with 16: 0.3 and 1.4 us in the sum (28/4 heads of
// 128, 1600 tokens, batch 1: 16 splits 7.5 us, 20 splits 7.9, 40 splits 8.9, 64 splits 9.7).
// Within that, the finer the better down to a few blocks per workgroup (28/4 heads of 128, 12800 tokens, batch 1: 16
// splits 10.5 us, 32 splits 9.7, 64 splits 9.9; 39200 tokens: 17.8, 13.3, 12.8; 14/2 heads of 64, 12800 tokens: 16 splits 8.1, 32 splits 7.4; group 64, 39200 tokens: 32 splits 12.3, 64 splits 9.7).
static int splits_for_rounds(int B, const wq_packed_kv* kv, int64_t max_seq_tokens, int most)
{
    const int64_t units = (int64_t)B * kv->Hkv, blocks = (max_seq_tokens + 31) / 32;
    const bool two = kv->hd / kv->group == 2, large = kv->hd == 128;
    // a block's cost, averaged over the cache's slots
    const double slots = (double)kv->cap[0] + (double)kv->cap[1] + (double)kv->cap[2] + (double)kv->cap16;
    const int* const unit = !two ? WQ_BLOCK_COST_F32 : large ? WQ_BLOCK_COST : WQ_BLOCK_COST_64;
    const double cost = slots > 0 ? ((double)kv->cap[0] * unit[0] + (double)kv->cap[1] * unit[1] +
                                     (double)kv->cap[2] * unit[2] + (double)kv->cap16 * unit[3]) / slots : unit[0];
    // a compute unit's time for it, with little traffic besides (what memory takes when the whole chip is at it depends little on the splits)
    const double block_us = cost * (two ? (large ? 0.85e-3 : 0.55e-3) : (large ? 1.45e-3 : 0.95e-3)), fixed_us = large ? 8.0 : 6.5;
    int best = 1;
    double best_us = 0;
    for (int s = 1; s <= most && s <= (blocks > 1 ? blocks : 1); s++) {
        const double us = (double)((units * s + 255) / 256) * (fixed_us + block_us * (double)blocks / s) + (s > 32 ? 1.4 : s > 16 ? 0.3 : 0.0);
        if (s == 1 || us < best_us) { best_us = us; best = s; }
    }
    return best;
}

// Under WQ_DECODE_BY_LENGTH with a given count: are the workgroups with work numbered by the kernel (place_by_length)?  That
// takes 0.9 us of the launch (8 even sequences: 17.7 us, numbered 18.6), which uneven ones repay (20 that fill 0.49 of the
// longest one's length, 8 splits: 37.6 -> 36.1).  Room in the cache for less than 3/4 of B longest sequences proves that they
// differ; room for more than B of them (and their last blocks' padding) says nothing, the caller's flag is believed.
static bool packs_by_length(int B, const wq_packed_kv* kv, int64_t max_seq_tokens)
{
    const double slots = (double)kv->cap[0] + (double)kv->cap[1] + (double)kv->cap[2] + (double)kv->cap16;
    return B <= 64 && (slots < 0.75 * (double)B * (double)max_seq_tokens || slots > (double)B * ((double)max_seq_tokens + 128.0));
}

// Splits of an automatic call (0: the launch would not merge them itself, the caller decides).  Under WQ_DECODE_BY_LENGTH the
// kernel finds every sequence's count (place_by_length) and this is the most that one can get.  The caller's flag alone
// decides that: the capacities say what the classes have room for, not what they hold (where thresholds decide, every class
// has room for all tokens; a cache in use has room to grow).  Even sequences lose 1 to 2 us by it (8 x 12800: 17.0 us, 18.7
// with the flag), uneven ones gain far more (20 that fill 0.49 of the longest one's length: 40.2 us with even counts, 29.5 so;
// 32 that fill 0.52: 78.6 and 57.4); one sequence has nothing to differ from.  Up to 900 blocks in the longest sequence 32 splits at
// most: beyond, the merge has 16 loads in flight per row of lanes instead of 8, and short sequences are cut into more workgroups than they have work for
// (2 sequences of up to 3300 tokens, 28/4 heads of 128, group 64: 8.9 us a call, 9.9 with up to 48 or 64; up to 12900: 9.3 and 10.3).  Over 300 batches of 2 to 8
// sequences of up to 100 to 1100 blocks 48 and 64 are 0.995 times as fast: 0.98 with two groups per head, 1.00 with four, 1.02 with one and heads of 64
// (2 of up to 12900 tokens, 14/2 heads: 9.3 us, with 48 8.6), 1.005 above 1000 blocks.
int wq_decode_pick_splits(const void* q, int q_dtype, int B, const wq_packed_kv* kv, int64_t max_seq_tokens, int plain_splits, int algo)
{
    // the same count where the caller has the merge done by a second kernel or left out (there are no counts by length then):
    // the two merges give the same bits, and a launch without its merge does the same work
    constexpr int NO_MERGE = WQ_DECODE_SEPARATE_MERGE | WQ_DECODE_PARTIALS_ONLY;
    const bool by_length = (algo & WQ_DECODE_BY_LENGTH) != 0 && !(algo & NO_MERGE) && B > 1;
    if (!merges_itself(q, q_dtype, B, kv, algo & ~NO_MERGE) || max_seq_tokens <= 0 || (by_length && B > 64)) return 0;
    // what a workspace for plain_splits has room for (wq_decode_ws_bytes), and no more where there is more: the same call then
    // cuts its work alike, and gives the same bits, whatever the workspace
    const int most = plain_splits + 32 < WQ_MAX_FUSED_SPLITS ? plain_splits + 32 : WQ_MAX_FUSED_SPLITS;
    if (by_length) return most > 32 && max_seq_tokens <= 900 * 32 ? 32 : most;
    return splits_for_rounds(B, kv, max_seq_tokens, most);
}

// Can wq_launch_decode append k_new, v_new (element type new_dtype) itself with these arguments?  Only the matrix-core
// kernel that walks every segment and merges its splits does: it needs the new rows in the cache's own 16-bit type and on
// 16-byte boundaries, and one more counter per sequence in the workspace header.
bool wq_decode_can_append(const void* q, int q_dtype, int B, int Hq, const wq_packed_kv* kv, int num_splits, int algo, const void* k_new,
                          const void* v_new, int new_dtype)
{
    return merges_itself(q, q_dtype, B, kv, algo) && new_dtype == kv->dtype16 && aligned_16({k_new, v_new}) && (int64_t)B * kv->Hkv + B <= WQ_MAX_ARRIVE &&
           num_splits <= WQ_MAX_FUSED_SPLITS && Hq / kv->Hkv <= WQ_MAX_REP;
}

template <bool PACKED>
static auto mfma_kernel(int hd, int groups) -> void (*)(DecodeArgs)
{
    if (hd == 128) return groups == 2 ? k_decode_mfma<128, 2, PACKED> : groups == 1 ? k_decode_mfma<128, 1, PACKED> : k_decode_mfma<128, 4, PACKED>;
    return groups == 2 ? k_decode_mfma<64, 2, PACKED> : k_decode_mfma<64, 1, PACKED>;
}

int wq_launch_decode(wq_ctx* ctx, const void* q, int q_dtype, int B, int Hq, const wq_packed_kv* kv, float sm_scale,
                     int num_splits, int algo, float* out, float* lse, const void* k_new, const void* v_new,
                     int64_t longest_tokens)
{
    const bool partials_only = (algo & WQ_DECODE_PARTIALS_ONLY) != 0;
    const bool fixed_shares = (algo & WQ_DECODE_FIXED_SHARES) != 0;
    const bool fused = merges_itself(q, q_dtype, B, kv, algo);
    algo &= ~WQ_DECODE_FLAGS;
    DecodeArgs a;
    a.q = q;
    a.q_dtype = q_dtype;
    a.B = B;
    a.Hq = Hq;
    a.rep = Hq / kv->Hkv;
    a.splits = num_splits;
    a.sm_scale = sm_scale;
    a.use_mfma = use_matrix_cores(q, q_dtype, kv, algo);
    // a bf16 cache needs the exact bf16 query for the bf16 instruction; other query types send the 16-bit
    // segment to the generic kernel
    a.mfma16 = a.use_mfma && !(kv->dtype16 == WQ_BF16 && q_dtype != WQ_BF16);
    a.splits16 = (a.use_mfma && !a.mfma16) ? wq_decode_splits16(B, kv->cap16) : 0;
    a.nparts = a.splits + a.splits16;
    a.kv = *kv;
    a.fixed_shares = fixed_shares;
    a.arrive = reinterpret_cast<unsigned*>(ctx->ws + 256);
    // A device-scope atomic takes 12-16 ns of the cache line it is for, and a unit's splits times its heads report in within
    // a microsecond or two: with a unit's counters in one line, the last of 32 splits x 7 heads was counted 3 us after its
    // partial had landed.  So a unit gets as many lines as the workspace header has room for, up to one per head.
    a.arrive_unit = WQ_ARRIVE_STRIDE;
    while (a.arrive_unit < WQ_ARRIVE_STRIDE * WQ_MAX_REP && (2 * (int64_t)(a.arrive_unit / WQ_ARRIVE_STRIDE) * kv->Hkv + 1) * B <= WQ_MAX_ARRIVE)
        a.arrive_unit *= 2;
    // one launch does it all when the matrix-core kernel walks every segment, the counters fit the workspace
    // header and a wavefront's lanes hold the splits' weights
    a.fused = fused && a.nparts <= WQ_MAX_FUSED_SPLITS;
    if (a.use_mfma && !fits_cost_axis(kv))
        return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "the matrix-core decode kernel takes caches of up to 2^27 token slots");
    a.part = reinterpret_cast<float*>(ctx->ws + WQ_WS_HEADER);
    a.part_ml = a.part + (int64_t)B * Hq * a.nparts * kv->hd;
    a.out = out;
    a.k_new = static_cast<const uint16_t*>(k_new);
    a.v_new = static_cast<const uint16_t*>(v_new);
    a.status = wq_status_ptr(ctx);
    if (k_new && !a.fused) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "this decode launch cannot append");
    // splits by length: only where the kernel merges the splits itself (the separate merge kernel reads every partial)
    a.len_scale = (a.fused && longest_tokens > 0) ? (float)a.splits / (float)longest_tokens : 0.f;
    a.packed_grid = a.fused && (longest_tokens < 0 || (longest_tokens > 0 && packs_by_length(B, kv, longest_tokens)));
    // Automatic splits by length: 256 workgroups, one per compute unit, if that is at least two per (sequence, KV head), so
    // that rounding to whole splits leaves few of them with little to do; else 512
    const int auto_wgs = (int64_t)B * kv->Hkv <= 128 ? 256 : 512;
    a.slots = a.packed_grid && longest_tokens < 0 ? auto_wgs / kv->Hkv : 0;
    // (sequences that turn out to be even get the count of a call without the flag: 40 x 3200 tokens, 4 KV heads, are 480
    // workgroups with the whole quotient 3, 28.8 us, and 160 so, 23.7 us; 22.4 without the flag)
    a.even_splits = a.slots > 0 ? splits_for_rounds(B, kv, -longest_tokens, a.splits < a.slots / B ? a.splits : a.slots / B) : 0;
#ifdef WQ_TIMELINE
    a.dbg = getenv("WQ_TIMELINE") ? reinterpret_cast<long long*>(ctx->ws + ctx->ws_bytes - (8 << 20)) : nullptr;
#endif
    a.lse = lse;
    const dim3 blk(256);
    const dim3 grid_q(a.splits, kv->Hkv, B), grid_16(a.splits16 > 0 ? a.splits16 : 1, kv->Hkv, B);
    // the matrix-core kernel maps workgroups (of WQ_WAVES wavefronts) to units itself
    const dim3 blk_m(64 * WQ_WAVES), grid_m = a.packed_grid ? dim3((unsigned)(a.slots > 0 ? a.slots * kv->Hkv : a.splits * kv->Hkv * B))
                                                            : dim3((unsigned)kv->Hkv, (unsigned)B, (unsigned)a.splits);
    const int tslot = (int)(ctx->ev_calls % WQ_TIMING_RING);
    if (ctx->timing) (void)hipEventRecord(ctx->ev[2 * tslot], ctx->stream);
    const int groups = kv->hd / kv->group;
    if (a.use_mfma) {
        void (*const kernel)(DecodeArgs) = a.packed_grid ? mfma_kernel<true>(kv->hd, groups) : mfma_kernel<false>(kv->hd, groups);
        hipLaunchKernelGGL(kernel, grid_m, blk_m, 0, ctx->stream, a);
    } else {
        hipLaunchKernelGGL(kv->hd == 128 ? k_decode_generic<128> : k_decode_generic<64>, grid_q, blk, 0, ctx->stream, a);
    }
    if (ctx->timing) (void)hipEventRecord(ctx->ev[2 * tslot + 1], ctx->stream);
    if (a.splits16 > 0) hipLaunchKernelGGL(kv->hd == 128 ? k_decode_generic<128> : k_decode_generic<64>, grid_16, blk, 0, ctx->stream, a);
    if (!partials_only && !a.fused)
        hipLaunchKernelGGL(k_combine, dim3(Hq, B), dim3(128), 0, ctx->stream, a.part, a.part_ml, Hq, a.rep, a.nparts, kv->hd, out, lse);
    if (ctx->timing) ctx->ev_calls++;
    WQ_HIP_CHECK(ctx, hipGetLastError());
    return WQ_OK;
}
