// a3: reorder + asymmetric round-to-nearest quantization + packing (Sec. 3.3.1, Sec. 3.3.3, Alg. 2 prefill half).
//
//   k_plan      one workgroup: per-class padded offsets / lengths of every sequence, 16-bit row counts,
//               capacity checks (device status word)
//   k_quantize_small  the whole call in one launch, for a few hundred workgroups
//   k_quantize_all  one launch for the three classes and the 16-bit rows.  A class workgroup takes one
//               (32-token destination block, KV head): gathers the source rows through
//               perm (the window reorder is fused into the load), finds each group's min/max with
//               wavefront shuffles, computes codes with the exact fp32 sequence of the format definition,
//               stages them in LDS and writes the K tile / V block / metadata images with coalesced stores
//               The remaining workgroups copy eight rows each of the 16-bit windows, video tail and text -> k16/v16
// HBM-bound: reads 2 x 2 bytes per (K,V) element pair once, writes b/8 + 4/group bytes per element.
// This file is compiled with floating-point contraction off: the code sequence must round exactly as stated.
#include <type_traits>

#include "wq_internal.h"

#pragma clang fp contract(off)

namespace {

__device__ __forceinline__ int pad32(int n) { return (n + 31) & ~31; }

// A store of the quantizer for rows of type T: non-temporal for the 16-bit types (k_quantize_all).  Behind fp32 rows an fp32 query
// comes, which the vector kernel takes with one and four groups per head: it reads the cache in small pieces, one round trip after the other, and
// pays for a cache that is not near (a layer's prefill and decode, 4 x 4804 tokens, 28/4 heads of 128, group 32: 631 us, 655 with non-temporal stores).
template <typename T, typename V>
__device__ __forceinline__ void put(void* p, V v)
{
    if constexpr (sizeof(T) == 2) wq_store_once(p, v);
    else *static_cast<V*>(p) = v;
}

// Class c's place for every sequence: off[B + 1], len[B]; n_of(b): its tokens.  True where something did not fit.
template <typename Tokens>
__device__ __forceinline__ bool plan_class(int B, int64_t cap, Tokens n_of, int32_t* off, int32_t* len)
{
    int64_t run = 0;
    bool over = false;
    off[0] = 0;
    for (int b = 0; b < B; b++) {
        int n = n_of(b);
        int64_t nxt = run + pad32(n);
        if (nxt > cap) {                // does not fit: drop the sequence's share of this class
            over = true;
            n = 0;
            nxt = run;
        }
        len[b] = n;
        run = nxt;
        off[b + 1] = (int32_t)run;
    }
    return over;
}
// n 16-bit rows between `at` and the next sequence's first one
__device__ __forceinline__ bool rows_fit(int at, int next, int n, int64_t cap16) { return n <= next - at && (int64_t)at + n <= cap16 && at >= 0; }
// ... and of the 16-bit rows: len[B], and their running count pre[B + 1]; begins(b): where sequence b's begin
template <typename Tokens, typename Begins>
__device__ __forceinline__ bool plan_rows(int B, int64_t cap16, Tokens n_of, Begins begins, int32_t* pre, int32_t* len)
{
    int64_t run = 0;
    bool over = false;
    pre[0] = 0;
    for (int b = 0; b < B; b++) {
        int n = n_of(b);
        if (!rows_fit(begins(b), begins(b + 1), n, cap16)) {
            over = true;
            n = 0;
        }
        len[b] = n;
        run += n;
        pre[b + 1] = (int32_t)run;
    }
    return over;
}

// Sum over the lanes up to and including this one
__device__ __forceinline__ int64_t lanes_upto(int64_t x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o *= 2) {
        const int64_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

// A wavefront per class and one for the 16-bit rows, a lane per sequence, 64 sequences at a time: bound by the round trip to the
// tables (one sequence after the other it took 5.7 us for 8 sequences and 8.7 for 16).  Only where a class does not hold
// everything does what a sequence gets depend on the ones before it: then plan_class does the class over.
__global__ __launch_bounds__(256) void k_plan(int B, const int32_t* __restrict__ kv_off, const int32_t* __restrict__ win_size,
                                              const int32_t* __restrict__ win_off, const int32_t* __restrict__ seg_windows,
                                              wq_packed_kv pk, int32_t* __restrict__ pre16, uint32_t* __restrict__ status)
{
    const int tid = threadIdx.x, lane = tid & 63, c = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int b = tid; b < B; b += 256) pk.v_scale_max[b] = 0.f;               // k_v_scale_max raises it
    int64_t run = 0;                                      // of the sequences before the 64
    bool over = false;
    if (c < 3) {
        int32_t *off = pk.cls_off[c], *len = pk.cls_len[c];
        const int64_t cap = pk.cap[c];
        auto tokens = [&](int b) { return seg_windows[4 * b + c] * win_size[b]; };
        if (lane == 0) off[0] = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            const int b = b0 + lane, n = b < B ? tokens(b) : 0;
            const int64_t upto = run + lanes_upto(pad32(n));
            over = over || upto > cap;
            if (b < B) {
                len[b] = n;
                off[b + 1] = (int32_t)upto;
            }
            run = __shfl(upto, 63, 64);
        }
        if (__builtin_amdgcn_ballot_w64(over) != 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");                // (what is written above is written over)
            if (lane == 0 && plan_class(B, cap, tokens, off, len)) atomicOr(status, WQ_DEV_CLASS_OVERFLOW);
        }
    } else {
        if (lane == 0) pre16[0] = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            const int b = b0 + lane;
            int n = 0;
            if (b < B) {
                const int size = win_size[b];
                n = seg_windows[4 * b + 3] * size + (kv_off[b + 1] - kv_off[b] - (win_off[b + 1] - win_off[b]) * size);
                if (!rows_fit(pk.off16[b], pk.off16[b + 1], n, pk.cap16)) {
                    over = true;
                    n = 0;
                }
            }
            const int64_t upto = run + lanes_upto(n);
            if (b < B) {
                pk.len16[b] = n;
                pre16[b + 1] = (int32_t)upto;
            }
            run = __shfl(upto, 63, 64);
        }
        if (over) atomicOr(status, WQ_DEV_SEG16_OVERFLOW);
    }
}

// maximum of an unsigned value over the 64 lanes of a wavefront: four rotations inside the rows of 16 lanes (one
// data-parallel-primitive instruction each, no LDS), then the four rows' results as scalars
template <int CTRL>
__device__ __forceinline__ uint32_t lanes_moved(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t lanes_max(uint32_t x)
{
    x = max(x, lanes_moved<0x128>(x));             // row_ror:8, 4, 2, 1
    x = max(x, lanes_moved<0x124>(x));
    x = max(x, lanes_moved<0x122>(x));
    x = max(x, lanes_moved<0x121>(x));
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)x, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)x, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    return max(max(a, b), max(c, d));
}

// v_scale_max holds [B] results, then one float per (32-token block, KV head) of the three classes (class c's blocks
// behind those of the classes before it, by capacity)
__device__ __forceinline__ int64_t v_scale_slot(const wq_packed_kv& pk, int B, int c, int64_t blk, int kvh)
{
    int64_t base = 0;
    for (int k = 0; k < c; k++) base += pk.cap[k] / 32;
    return (int64_t)B + (base + blk) * pk.Hkv + kvh;
}

// per sequence: the largest of its blocks' largest value scales (0 if it has no quantized token).  WQ_VS_PARTS workgroups
// per sequence take a slice of the blocks each and raise the sequence's entry, which k_plan has set to zero (positive
// floats order like their bit patterns)
constexpr int WQ_VS_PARTS = 16;
__global__ __launch_bounds__(256) void k_v_scale_max(int B, wq_packed_kv pk)
{
    __shared__ uint32_t s_top[4];
    const int b = blockIdx.x / WQ_VS_PARTS, part = blockIdx.x % WQ_VS_PARTS, tid = threadIdx.x;
    const float* src[3];
    int64_t count[3], longest = 0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int64_t t0 = pk.cls_off[c][b] / 32, t1 = pk.cls_off[c][b + 1] / 32;
        const int64_t n = (t1 - t0) * pk.Hkv, per = (n + WQ_VS_PARTS - 1) / WQ_VS_PARTS, lo = part * per;
        src[c] = pk.v_scale_max + v_scale_slot(pk, B, c, t0, 0) + lo;
        count[c] = min(n, lo + per) - lo;
        longest = max(longest, count[c]);
    }
    float mx = 0.f;
#pragma unroll 2
    for (int64_t i = tid; i < longest; i += 256) { // (the three classes' loads in flight together)
        float x[3];
#pragma unroll
        for (int c = 0; c < 3; c++) x[c] = i < count[c] ? src[c][i] : 0.f;
        mx = fmaxf(fmaxf(mx, x[0]), fmaxf(x[1], x[2]));
    }
    const uint32_t top = lanes_max(__float_as_uint(mx));
    if ((tid & 63) == 0) s_top[tid >> 6] = top;
    __syncthreads();
    if (tid == 0) {
        const uint32_t most = max(max(s_top[0], s_top[1]), max(s_top[2], s_top[3]));
        if (most != 0u) atomicMax(reinterpret_cast<unsigned*>(pk.v_scale_max + b), most);
    }
}

// bits -> class index
__host__ __device__ constexpr int cls_index(int bits) { return bits == 2 ? 0 : (bits == 4 ? 1 : 2); }

// V codes of a 32-token block on their way into operand order, one byte each: the 8 tokens x HD/16 channel tiles of a
// lane of the decode kernel's matrix operand (lane = 16 jj + mm holds channels 16 ct + mm of tokens 16 (tau >> 2) +
// 4 jj + (tau & 3)) lie together, [ct][tau], at lane x VT_PITCH; the 16 bytes of padding keep the readers' 16-byte
// reads in different banks
template <int HD>
struct QuantSmem {
    static constexpr int VT_PITCH = (HD / 16) * 8 + 16;
    __attribute__((aligned(16))) uint8_t vt[64 * VT_PITCH];
    uint32_t meta[2][4][32];                    // [plane][group][token]
};

template <int CTRL>
__device__ __forceinline__ float lanes_moved_f(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// 16 codes of BITS bits, one per byte of x[0..3], as consecutive fields: 2 BITS bytes in y
template <int BITS>
__device__ __forceinline__ void pack16(const uint32_t (&x)[4], uint32_t (&y)[4])
{
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 4; i++) y[i] = x[i];
    } else if constexpr (BITS == 4) {
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const uint32_t a = x[2 * i] | (x[2 * i] >> 4), b = x[2 * i + 1] | (x[2 * i + 1] >> 4);     // bytes 0 and 2 hold two codes each
            y[i] = __builtin_amdgcn_perm(b, a, 0x06040200u);                                          // a.b0 a.b2 b.b0 b.b2
        }
    } else {
        uint32_t z[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t a = x[i] | (x[i] >> 6);          // bytes 0 and 2 hold two codes each
            z[i] = a | (a >> 12);                           // byte 0 holds all four
        }
        y[0] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(z[3], z[2], 0x0C0C0400u), __builtin_amdgcn_perm(z[1], z[0], 0x0C0C0400u), 0x05040100u);
    }
}

// one (32-token destination block `blk` of class BITS, KV head `kvh`); off, lens: the class's tables (cls_off, cls_len).
// SMALL: in a launch of few workgroups, where latency counts: the values are sent for with the keys, and the block's largest
// value scale goes through to memory, for another workgroup of the launch
template <typename T, int HD, int BITS, bool SMALL = false>
__device__ __forceinline__ void quantize_block(QuantSmem<HD>& sm, int blk, int kvh, const int32_t* off, const int32_t* lens,
                                               const T* __restrict__ K, const T* __restrict__ V,
                                               int B, int group, const int32_t* __restrict__ kv_off,
                                               const int32_t* __restrict__ win_size, const int32_t* __restrict__ win_off,
                                               const int32_t* __restrict__ perm, const int32_t* __restrict__ seg_windows,
                                               const wq_packed_kv& pk)
{
    constexpr int C = cls_index(BITS);
    constexpr int QMAX = (1 << BITS) - 1;
    constexpr int CPT = HD / 8;                 // channels per thread: 8 threads share one token row
    auto& s_meta = sm.meta;
    const int tid = threadIdx.x;
    const int Hkv = pk.Hkv;
    const int G = HD / group;
    const int64_t tok0 = (int64_t)blk * 32;
    if (tok0 >= off[B]) return;                 // unused capacity
    const int b = wq_find_seq(off, B, tok0);
    const int d0 = (int)(tok0 - off[b]);        // first destination token of the block inside the segment
    const int len = lens[b];
    const int S = win_size[b];
    int pos0 = 0;                               // windows of lower classes come first in perm
    for (int c = 0; c < C; c++) pos0 += seg_windows[4 * b + c];

    // ---- gather + quantize: thread = (token u, part p) -------------------------------------------------
    const int u = tid >> 3, p = tid & 7;
    const int d = d0 + u;
    const bool valid = d < len;
    int64_t src = 0;
    if (valid) {
        int r = d / S, o = d - r * S;
        int win = perm[win_off[b] + pos0 + r];
        src = (int64_t)kv_off[b] + (int64_t)win * S + o;
    }
    const int tpg = group / CPT;                // threads per group (2, 4 or 8; 16 when group=128, hd=64 is excluded)
    const int64_t base = (src * Hkv + kvh) * HD + p * CPT;
    float later[CPT];
    if (SMALL && valid) {
#pragma unroll
        for (int i = 0; i < CPT; i += 8) wq_ld8(V + base + i, later + i);
    }
#pragma unroll
    for (int plane = 0; plane < 2; plane++) {
        const T* X = plane == 0 ? K : V;
        float x[CPT];
        float lo = INFINITY, hi = -INFINITY;
        if (valid) {
            if (SMALL && plane == 1) {
#pragma unroll
                for (int i = 0; i < CPT; i++) x[i] = later[i];
            } else {
#pragma unroll
                for (int i = 0; i < CPT; i += 8) wq_ld8(X + base + i, x + i);     // 16-byte pieces (rows are 16-byte aligned)
            }
#pragma unroll
            for (int i = 0; i < CPT; i++) {
                lo = fminf(lo, x[i]);
                hi = fmaxf(hi, x[i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < CPT; i++) x[i] = 0.f;
            lo = hi = 0.f;
        }
        // lanes p..p+tpg-1 of a token are adjacent lanes of one wavefront: partners p ^ 1, p ^ 2, p ^ 7 (lane moves
        // inside quads and half rows, no LDS)
        lo = fminf(lo, lanes_moved_f<0xB1>(lo));
        hi = fmaxf(hi, lanes_moved_f<0xB1>(hi));
        if (tpg >= 4) {
            lo = fminf(lo, lanes_moved_f<0x4E>(lo));
            hi = fmaxf(hi, lanes_moved_f<0x4E>(hi));
        }
        if (tpg >= 8) {
            lo = fminf(lo, lanes_moved_f<0x141>(lo));
            hi = fmaxf(hi, lanes_moved_f<0x141>(hi));
        }
        if (lo == 0.0f) lo = 0.0f;               // a zero minimum is stored as +0
        const __half mh = __float2half_rn(lo);
        const float m = __half2float(mh);
        const float r = hi - m;
        const float s0 = r / (float)QMAX;       // correctly rounded fp32 divide
        __half sh = __float2half_rn(s0);
        float s = __half2float(sh);
        if (s == 0.0f) {
            s = 1.0f;
            sh = __float2half_rn(1.0f);
        }
        const float inv = 1.0f / s;
        // This thread's codes: the K plane takes them as consecutive BITS-wide fields of its token's row quarter
        // (pw, stored below); the V plane goes through LDS, a byte per code, to where the operand order wants it.
        // A token past the end has x = 0 everywhere, which gives m = 0, s = 1 and codes 0.
        constexpr int NB = CPT * BITS / 8;      // bytes of the K fields: 2..16
        uint32_t pw[(NB + 3) / 4];
#pragma unroll
        for (int i = 0; i < (NB + 3) / 4; i++) pw[i] = 0;
        uint8_t* const vt = sm.vt + ((u >> 2) & 3) * (16 * QuantSmem<HD>::VT_PITCH) + (u & 3) + 4 * (u >> 4);    // lane 16 jj (+ mm), byte tau (+ 8 ct)
#pragma unroll
        for (int i = 0; i < CPT; i++) {
            float t = (x[i] - m) * inv;         // contraction is off: subtract, round, multiply, round
            float q = rintf(t);
            q = __builtin_amdgcn_fmed3f(q, 0.0f, (float)QMAX);      // (the clamp: no NaN comes here)
            const uint32_t code = (uint32_t)(int)q;
            if (plane == 0) {
                pw[(i * BITS) >> 5] |= code << ((i * BITS) & 31);
            } else {
                const int ch = p * CPT + i;     // (ch & 15, ch >> 4 are fixed per i once p is known: CPT divides 16)
                vt[(ch & 15) * QuantSmem<HD>::VT_PITCH + (ch >> 4) * 8] = (uint8_t)code;
            }
        }
        if (plane == 0) {
            constexpr int Q = HD / 4;
            const int j = (p * CPT) / Q, e0 = (p * CPT) % Q;
            uint8_t* out = static_cast<uint8_t*>(pk.codes[C]) + ((int64_t)kvh * pk.cap[C] + tok0) * HD * BITS / 8 +
                           (u >> 4) * (16 * HD * BITS / 8) + ((j * 16 + (u & 15)) * Q + e0) * BITS / 8;
            if constexpr (NB == 2) {
                put<T>(out, (uint16_t)pw[0]);
            } else if constexpr (NB == 4) {
                put<T>(out, pw[0]);
            } else if constexpr (NB == 8) {
                put<T>(out, uint2{pw[0], pw[1]});
            } else {
                put<T>(out, uint4{pw[0], pw[1], pw[2], pw[3]});
            }
        }
        if ((p * CPT) % group == 0) {
            uint32_t word = valid ? ((uint32_t)__half_as_ushort(sh) | ((uint32_t)__half_as_ushort(mh) << 16)) : 0u;
            s_meta[plane][(p * CPT) / group][u] = word;
        }
    }
    __syncthreads();

    // ---- the block's largest value scale (the decode kernel places its fp16 weights by the sequence's largest one): the
    //      scales are the low halves of the V metadata words, zero for tokens past the end; their magnitudes (a group of
    //      nearly equal fp32 values can have a negative scale) order like their bit patterns.  One plain store per workgroup into the table's scratch part; k_v_scale_max collects them ----
    if (tid < 64) {
        uint32_t top = 0;
        for (int i = tid; i < 32 * G; i += 64) top = max(top, s_meta[1][i >> 5][i & 31] & 0x7FFFu);
        top = lanes_max(top);
        if (tid == 0) {
            float* const slot = pk.v_scale_max + v_scale_slot(pk, B, C, blk, kvh);
            if constexpr (SMALL) __hip_atomic_store(slot, wq_f16_bits_to_float(top), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else *slot = wq_f16_bits_to_float(top);
        }
    }

    // ---- V plane: block of 32 tokens, field n = ((jj*16 + mm)*(HD/16) + ct)*8 + tau: LDS holds the codes in this
    //      order, a byte each; a thread packs 16 of them (two channel tiles of a lane) into 2 BITS bytes ----------
    {
        constexpr int CT = HD / 16;
        uint8_t* out = static_cast<uint8_t*>(pk.codes[C]) + (((int64_t)Hkv + kvh) * pk.cap[C] + tok0) * HD * BITS / 8;
        for (int r = tid; r < 64 * CT / 2; r += 256) {
            const uint4 c = *reinterpret_cast<const uint4*>(sm.vt + (r / (CT / 2)) * QuantSmem<HD>::VT_PITCH + (r % (CT / 2)) * 16);
            const uint32_t x[4] = {c.x, c.y, c.z, c.w};
            uint32_t y[4];
            pack16<BITS>(x, y);
            if constexpr (BITS == 8)
                put<T>(out + r * 16, uint4{y[0], y[1], y[2], y[3]});
            else if constexpr (BITS == 4)
                put<T>(out + r * 8, uint2{y[0], y[1]});
            else
                put<T>(out + r * 4, y[0]);
        }
    }
    // ---- metadata: [tile of 16][group][16 tokens] ---------------------------------------------------------
    {
        const int lg = G >> 1;                  // log2 of G = 1, 2 or 4: at most 256 words, one per thread
        if (tid < (64 << lg)) {
            const int plane = tid >> (5 + lg), r = tid & ((32 << lg) - 1);
            const int tile = r >> (4 + lg), gi = (r >> 4) & (G - 1), mrow = r & 15;
            uint32_t* out = static_cast<uint32_t*>(pk.meta[C]) + (((int64_t)plane * Hkv + kvh) * pk.cap[C] + tok0) * G;
            put<T>(out + r, s_meta[plane][gi][tile * 16 + mrow]);
        }
    }
}

// rows r0 .. r0 + ROWS16 - 1 of all 16-bit rows of the batch, 8 elements (one store of 16 bytes) per thread at a time.  A
// workgroup per row, an element per thread, took 150 us where the whole cache stays in 16 bits (8 x 12800 tokens, 4 KV heads
// of 128, bf16), this way 84.
constexpr int ROWS16 = 8;
template <typename T>
__device__ __forceinline__ void copy16_rows(int64_t r0, const T* __restrict__ K, const T* __restrict__ V, int B, int pieces,
                                            const int32_t* __restrict__ kv_off, const int32_t* __restrict__ win_size,
                                            const int32_t* __restrict__ win_off, const int32_t* __restrict__ perm,
                                            const int32_t* __restrict__ seg_windows, const int32_t* pre16,
                                            const wq_packed_kv& pk)
{
    __shared__ int64_t s_src[ROWS16], s_dst[ROWS16];
    if (r0 >= pre16[B]) return;
    const int rows = (int)min((int64_t)ROWS16, pre16[B] - r0);
    if (threadIdx.x < rows) {
        const int64_t r = r0 + threadIdx.x;
        const int b = wq_find_seq(pre16, B, r);
        const int i = (int)(r - pre16[b]);
        const int S = win_size[b];
        const int W = win_off[b + 1] - win_off[b];
        const int n16w = seg_windows[4 * b + 3] * S;
        int64_t src;
        if (i < n16w) {
            int pos0 = seg_windows[4 * b] + seg_windows[4 * b + 1] + seg_windows[4 * b + 2];
            int rr = i / S, o = i - rr * S;
            src = (int64_t)kv_off[b] + (int64_t)perm[win_off[b] + pos0 + rr] * S + o;
        } else {
            src = (int64_t)kv_off[b] + (int64_t)W * S + (i - n16w);
        }
        s_src[threadIdx.x] = src * pieces;
        s_dst[threadIdx.x] = ((int64_t)pk.off16[b] + i) * pieces;
    }
    __syncthreads();
    // (a test of every store's address, in the loop, kept a piece's two loads from being sent together: 83.5 us -> 87.8)
    auto copy = [&](auto aligned) {
        for (int e = threadIdx.x; e < rows * pieces; e += 256) {
            const int row = e / pieces, piece = e - row * pieces;
            const int64_t from = s_src[row] + piece, to = s_dst[row] + piece;
#pragma unroll
            for (int plane = 0; plane < 2; plane++) {
                const T* const src = (plane ? V : K) + from * 8;
                uint16_t* const dst = static_cast<uint16_t*>(plane ? pk.v16 : pk.k16) + to * 8;
                uint4 x;
                if constexpr (std::is_same_v<T, float>) {      // fp32 -> fp16 (nearest even)
                    float f[8];
                    wq_ld8(src, f);
                    uint32_t o[4];
#pragma unroll
                    for (int k = 0; k < 4; k++)
                        o[k] = (uint32_t)__half_as_ushort(__float2half_rn(f[2 * k])) | (uint32_t)__half_as_ushort(__float2half_rn(f[2 * k + 1])) << 16;
                    x = make_uint4(o[0], o[1], o[2], o[3]);
                } else {
                    x = wq_load_once(src);
                }
                if constexpr (decltype(aligned)::value) {
                    put<T>(dst, x);
                } else {
                    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                    for (int k = 0; k < 8; k++) dst[k] = (uint16_t)(w[k >> 1] >> (16 * (k & 1)));
                }
            }
        }
    };
    if ((reinterpret_cast<uintptr_t>(pk.k16) | reinterpret_cast<uintptr_t>(pk.v16)) % 16 == 0) copy(std::true_type{});
    else copy(std::false_type{});                              // (a segment that does not begin on a 16-byte boundary)
}

// The whole call after k_plan in one launch.  The blocks of the classes first (consecutive workgroups = the KV heads of one
// token block: together they read whole source rows), the 2-bit ones, then 4-bit, then 8-bit; then ROWS16 16-bit rows each.
// The blocks are numbered by the capacities (n0 workgroups for the 2-bit class, n1 for the 4-bit one) or, with n0 =
// WQ_BY_USE, without gaps by what k_plan has found to be in use.  The latter where the capacities hold more than all rows
// together fill: where thresholds decide, every class has room for all tokens, and a call for 16 ragged sequences (198 500
// tokens, fp16) took 144 us with workgroups for the unused room, 136 without.  Else the former: reading the tables first
// costs 2.5 of 61 us (8 x 12800 tokens).
// Everything the launch writes is written once, for 16-bit rows with non-temporal stores, which leave the memory to the reads: 4 x 50688 tokens, 4 KV heads of 128,
// 352 -> 348 us for a layer's prefill (377 -> 364 before the scoring read its rows so), 4 x 12644, 8 KV heads of 64, 75.7 -> 67.8; a decode call behind it
// takes what it took.  Small calls pay where what they write would have stayed near: the same caches written again and again, 8 x 2369 tokens, 4 KV heads of 128,
// 18.1 -> 19.3 us (17 x 1148: 20.9 -> 22.7), and 17 x 1148 into one of 33 caches with a decode call behind it 35.0 -> 37.0; they gain where K and V have just been written and the
// cache has not, as in a model's prefill (two copies and the call: 32.5 -> 30.5, 35.9 -> 34.4; 12 shapes of up to 70 MB 0.99 to 1.09).  (The rows of K and V so: 1 to 10 % slower, a wavefront reads them in pieces; the 16-bit rows' copies take whole lines: 209.6 ->
// 202.7 us where all of 8 x 12644 tokens stay in 16 bits.)
// n: workgroups for the blocks, a bound on their number.
constexpr unsigned WQ_BY_USE = 0xFFFFFFFFu;
template <typename T, int HD>
__global__ __launch_bounds__(256) void k_quantize_all(const T* __restrict__ K, const T* __restrict__ V, int B, int group,
                                                      const int32_t* __restrict__ kv_off, const int32_t* __restrict__ win_size,
                                                      const int32_t* __restrict__ win_off, const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ seg_windows, const int32_t* __restrict__ pre16,
                                                      wq_packed_kv pk, unsigned n, unsigned n0, unsigned n1)
{
    __shared__ QuantSmem<HD> sm;
    unsigned w = blockIdx.y * gridDim.x + blockIdx.x;
    const unsigned Hkv = (unsigned)pk.Hkv;
    if (w >= n) {
        copy16_rows<T>((int64_t)(w - n) * ROWS16, K, V, B, pk.Hkv * HD / 8, kv_off, win_size, win_off, perm, seg_windows, pre16, pk);
        return;
    }
    if (n0 == WQ_BY_USE) {
        n0 = (unsigned)pk.cls_off[0][B] / 32u * Hkv;
        n1 = (unsigned)pk.cls_off[1][B] / 32u * Hkv;
    }
    if (w < n0) {
        quantize_block<T, HD, 2>(sm, (int)(w / Hkv), (int)(w % Hkv), pk.cls_off[0], pk.cls_len[0], K, V, B, group, kv_off, win_size, win_off, perm, seg_windows, pk);
        return;
    }
    w -= n0;
    if (w < n1) {
        quantize_block<T, HD, 4>(sm, (int)(w / Hkv), (int)(w % Hkv), pk.cls_off[1], pk.cls_len[1], K, V, B, group, kv_off, win_size, win_off, perm, seg_windows, pk);
        return;
    }
    w -= n1;
    quantize_block<T, HD, 8>(sm, (int)(w / Hkv), (int)(w % Hkv), pk.cls_off[2], pk.cls_len[2], K, V, B, group, kv_off, win_size, win_off, perm, seg_windows, pk);
}

// The whole call in one launch, where it is a few hundred workgroups and launches are most of what it costs (8 windows of 16
// tokens, 2 KV heads of 64: three launches 8.6 us, this one 6.2): every workgroup works the plan out for itself, in LDS (two
// round trips to memory and a loop over the sequences), the first one writes it out, and the last one to finish collects the
// sequences' largest value scales.  Workgroups report in on counters of the workspace header, zero between launches: on one up to
// SMALL_LINE of them (12-16 ns each, as device-scope atomics on one address take), above on SMALL_LINES, whose last ones report in on
// the one (a round trip more: 100 workgroups 8.4 us on one counter, 8.7 so; 200 9.7 and 9.0, 250 10.2 and 8.9).  Against three launches, 1 to 15 sequences,
// 2 to 8 KV heads of 64 and 128: 400 workgroups 11.0 -> 9.5 us, 700 11.6 -> 10.5, 1000 12.9 -> 11.8; from 1200 to 1500 on equal, 1990 16.5 and 16.8.
// n: workgroups for the blocks (numbered by use), a bound on their number; the rest take ROWS16 16-bit rows each.
constexpr int SMALL_SEQS = 16, SMALL_WGS = 1024, SMALL_LINE = 150, SMALL_LINES = 16;
template <typename T, int HD>
__global__ __launch_bounds__(256) void k_quantize_small(const T* __restrict__ K, const T* __restrict__ V, int B, int group,
                                                        const int32_t* __restrict__ kv_off, const int32_t* __restrict__ win_size,
                                                        const int32_t* __restrict__ win_off, const int32_t* __restrict__ perm,
                                                        const int32_t* __restrict__ seg_windows, wq_packed_kv pk, unsigned n,
                                                        uint32_t* __restrict__ status, unsigned* __restrict__ arrive, unsigned* __restrict__ arrive_lines)
{
    __shared__ QuantSmem<HD> sm;
    // the tables' own values, and the plan
    __shared__ int32_t s_kv[SMALL_SEQS + 1], s_win[SMALL_SEQS + 1], s_size[SMALL_SEQS], s_seg[4 * SMALL_SEQS], s_begin[SMALL_SEQS + 1];
    __shared__ int32_t s_off[3][SMALL_SEQS + 1], s_len[4][SMALL_SEQS], s_pre16[SMALL_SEQS + 1];
    __shared__ unsigned s_top[SMALL_SEQS], s_last;
    const int tid = threadIdx.x;
    if (tid <= B) {
        s_kv[tid] = kv_off[tid];
        s_win[tid] = win_off[tid];
    }
    if (tid < B) s_size[tid] = win_size[tid];
    if (tid < 4 * B) s_seg[tid] = seg_windows[tid];
    if (tid <= B) s_begin[tid] = pk.off16[tid];
    if (tid < SMALL_SEQS) s_top[tid] = 0u;
    __syncthreads();
    if (tid < 3) {
        if (plan_class(B, pk.cap[tid], [&](int b) { return s_seg[4 * b + tid] * s_size[b]; }, s_off[tid], s_len[tid]) && blockIdx.x == 0)
            atomicOr(status, WQ_DEV_CLASS_OVERFLOW);
    } else if (tid == 3) {
        auto rows = [&](int b) { return s_seg[4 * b + 3] * s_size[b] + (s_kv[b + 1] - s_kv[b] - (s_win[b + 1] - s_win[b]) * s_size[b]); };
        if (plan_rows(B, pk.cap16, rows, [&](int b) { return s_begin[b]; }, s_pre16, s_len[3]) && blockIdx.x == 0)
            atomicOr(status, WQ_DEV_SEG16_OVERFLOW);
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid <= B) {
#pragma unroll
        for (int c = 0; c < 3; c++) {
            pk.cls_off[c][tid] = s_off[c][tid];
            if (tid < B) pk.cls_len[c][tid] = s_len[c][tid];
        }
        if (tid < B) pk.len16[tid] = s_len[3][tid];
    }
    const unsigned Hkv = (unsigned)pk.Hkv, n0 = (unsigned)s_off[0][B] / 32u * Hkv, n1 = (unsigned)s_off[1][B] / 32u * Hkv;
    unsigned w = blockIdx.x;
    if (w >= n) {
        copy16_rows<T>((int64_t)(w - n) * ROWS16, K, V, B, pk.Hkv * HD / 8, s_kv, s_size, s_win, perm, s_seg, s_pre16, pk);
    } else if (w < n0) {
        quantize_block<T, HD, 2, true>(sm, (int)(w / Hkv), (int)(w % Hkv), s_off[0], s_len[0], K, V, B, group, s_kv, s_size, s_win, perm, s_seg, pk);
    } else if ((w -= n0) < n1) {
        quantize_block<T, HD, 4, true>(sm, (int)(w / Hkv), (int)(w % Hkv), s_off[1], s_len[1], K, V, B, group, s_kv, s_size, s_win, perm, s_seg, pk);
    } else {
        w -= n1;
        quantize_block<T, HD, 8, true>(sm, (int)(w / Hkv), (int)(w % Hkv), s_off[2], s_len[2], K, V, B, group, s_kv, s_size, s_win, perm, s_seg, pk);
    }
    // The thread that has stored the block's value scale (device scope: past the XCD's L2) waits for the store to be
    // acknowledged before it counts the workgroup, so whoever finds itself last reads scales that have arrived.
    if (tid == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        auto last_of = [](unsigned* counter, unsigned all) { return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == all - 1u; };
        if (gridDim.x <= SMALL_LINE) {
            s_last = last_of(arrive, gridDim.x) ? 1u : 0u;
        } else {
            const unsigned line = blockIdx.x % SMALL_LINES;
            unsigned* const counter = arrive_lines + line * WQ_ARRIVE_STRIDE;
            s_last = 0u;
            if (last_of(counter, (gridDim.x - line + SMALL_LINES - 1u) / SMALL_LINES)) {
                __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_last = last_of(arrive, SMALL_LINES) ? 1u : 0u;
            }
        }
    }
    __syncthreads();
    if (s_last == 0u) return;
    if (tid == 0) __hip_atomic_store(arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // for the next launch
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int slots = s_off[c][B] / 32 * (int)Hkv;
        const float* const src = pk.v_scale_max + v_scale_slot(pk, B, c, 0, 0);
        for (int i = tid; i < slots; i += 256) {
            const float top = fmaxf(__hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), 0.f);
            atomicMax(&s_top[wq_find_seq(s_off[c], B, (int64_t)(i / (int)Hkv) * 32)], __float_as_uint(top));
        }
    }
    __syncthreads();
    if (tid < B) pk.v_scale_max[tid] = __uint_as_float(s_top[tid]);
}

// one generated token per sequence -> the end of its 16-bit segment
template <typename T>
__global__ __launch_bounds__(256) void k_append16(const T* __restrict__ k_new, const T* __restrict__ v_new, int row_elems,
                                                  wq_packed_kv pk, uint32_t* __restrict__ status)
{
    const int b = blockIdx.x;
    const int64_t row = (int64_t)pk.off16[b] + pk.len16[b];
    const bool full = row >= pk.off16[b + 1] || row >= pk.cap16;
    __syncthreads();                       // every lane has read len16[b] before it changes
    if (full) {
        if (threadIdx.x == 0) atomicOr(status, WQ_DEV_SEG16_OVERFLOW);
        return;
    }
    uint16_t* k16 = static_cast<uint16_t*>(pk.k16) + row * row_elems;
    uint16_t* v16 = static_cast<uint16_t*>(pk.v16) + row * row_elems;
    for (int e = threadIdx.x; e < row_elems; e += 256) {
        const float kx = wq_ld(k_new, (int64_t)b * row_elems + e), vx = wq_ld(v_new, (int64_t)b * row_elems + e);
        if constexpr (std::is_same_v<T, __hip_bfloat16>) {
            k16[e] = (uint16_t)(__float_as_uint(kx) >> 16);
            v16[e] = (uint16_t)(__float_as_uint(vx) >> 16);
        } else {
            k16[e] = __half_as_ushort(__float2half_rn(kx));
            v16[e] = __half_as_ushort(__float2half_rn(vx));
        }
    }
    if (threadIdx.x == 0) pk.len16[b] += 1;
}

// ---- the unfused variant of the operator-fusion ablation (Sec. 3.3.3, Sec. 4.4): packed classes back to 16-bit rows -------------
// dst's 16-bit segment receives, per sequence, the dequantized tokens of src's 2-, 4- and 8-bit classes (in this order,
// the order of the cache) and then src's 16-bit rows; dst's classes are empty.  Decode attention over dst is then the
// plain 16-bit attention that a dequantize-to-memory implementation would run.
// One launch: a workgroup per (32-token block of a class, KV head), value = fma(code, s, m) in fp32, rounded to nearest even
// into the 16-bit type; a workgroup per DENSE_ROWS rows of src's 16-bit segment; and one for dst's tables.
// Bound by the 16-bit rows that it writes, if the vector unit keeps up: a lane instruction per element costs the whole call
// 3 us at 8 x 12800 tokens, 4 KV heads of 128.  So a thread turns 8 consecutive channels of a token (16 bytes of a row, a
// row's pieces by consecutive lanes) from codes that lie one per byte (a conversion instruction takes any byte of a
// register), two values at a time; and the V codes, whose operand order has 8 tokens of one channel together, are
// transposed as bytes, 8 lanes x 8 tokens at a time, in three exchanges between lanes (11 instructions per 8 codes).
// Field by field from LDS, in a launch per class, the call took 93 us (275 MB read and written: 2.9 TB/s); this way 59 us (4.7
// TB/s; a plain copy of 1 GiB runs at 5.0), and with non-temporal stores of the rows 42 us (6.5 TB/s).  Whoever reads the rows next finds less of
// them in the memory-side cache: with a plain read of all of them behind it the call takes 87 us either way (12.1 and 12.2 with 1568 tokens, 32.0 and 32.8
// with 4 x 9408).  1 x 12644 tokens 8.2 -> 6.5 us, 16 x 15780 144 -> 134.  (The metadata's loads so too: 56 us.  The 16-bit rows' loads: no gain.)
constexpr int DENSE_ROWS = 8;

__device__ __forceinline__ int dense_total(const wq_packed_kv& src, int b)
{
    return src.cls_len[0][b] + src.cls_len[1][b] + src.cls_len[2][b] + src.len16[b];
}
__device__ __forceinline__ bool dense_fits(const wq_packed_kv& src, const wq_packed_kv& dst, int b)
{
    const int n = dense_total(src, b);
    return dst.off16[b] >= 0 && n <= dst.off16[b + 1] - dst.off16[b] && (int64_t)dst.off16[b] + n <= dst.cap16;
}

__device__ __forceinline__ void dense_plan(int B, const wq_packed_kv& src, const wq_packed_kv& dst, uint32_t* __restrict__ status)
{
    for (int b = threadIdx.x; b < B; b += 256) {
        const bool ok = dense_fits(src, dst, b);
        dst.len16[b] = ok ? dense_total(src, b) : 0;
        if (!ok) atomicOr(status, WQ_DEV_SEG16_OVERFLOW);
#pragma unroll
        for (int c = 0; c < 3; c++) dst.cls_len[c][b] = 0;
        dst.v_scale_max[b] = 0.f;
    }
    for (int b = threadIdx.x; b <= B; b += 256)
#pragma unroll
        for (int c = 0; c < 3; c++) dst.cls_off[c][b] = 0;
}

typedef float float2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// two values rounded to nearest even into the 16-bit type
template <bool BF>
__device__ __forceinline__ uint32_t pair_16bit(float x, float y)
{
    const float2v v = {x, y};
    if constexpr (BF) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, half2v));
}

__device__ __forceinline__ float byte_of(uint32_t x, int k) { return (float)((x >> (8 * k)) & 0xFFu); }

template <int NB>
__device__ __forceinline__ void load_bytes(const uint8_t* p, uint32_t* x)      // NB bytes, aligned to NB
{
    if constexpr (NB == 2) {
        x[0] = *reinterpret_cast<const uint16_t*>(p);
    } else if constexpr (NB == 4) {
        x[0] = *reinterpret_cast<const uint32_t*>(p);
    } else if constexpr (NB == 8) {
        const uint2 t = *reinterpret_cast<const uint2*>(p);
        x[0] = t.x, x[1] = t.y;
    } else {
        const uint4 t = *reinterpret_cast<const uint4*>(p);
        x[0] = t.x, x[1] = t.y, x[2] = t.z, x[3] = t.w;
    }
}

// 8 consecutive fields of BITS bits as numbers
template <int BITS>
__device__ __forceinline__ void codes_of(const uint32_t* w, float (&c)[8])
{
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 8; i++) c[i] = byte_of(w[i >> 2], i & 3);
    } else if constexpr (BITS == 4) {
        const uint32_t even = w[0] & 0x0F0F0F0Fu, odd = (w[0] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
        for (int i = 0; i < 8; i++) c[i] = byte_of((i & 1) ? odd : even, i >> 1);
    } else {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t x = (w[0] >> (2 * k)) & 0x0303u;       // fields k and k + 4
            c[k] = byte_of(x, 0);
            c[k + 4] = byte_of(x, 1);
        }
    }
}

// 8 values m + s * code of a token -> 16 bytes of its row
template <bool BF>
__device__ __forceinline__ uint4 dense_piece(const float (&c)[8], uint32_t word)
{
    const float s = __half2float(__ushort_as_half((uint16_t)(word & 0xFFFFu))), m = __half2float(__ushort_as_half((uint16_t)(word >> 16)));
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] = pair_16bit<BF>(fmaf(c[2 * i], s, m), fmaf(c[2 * i + 1], s, m));
    return make_uint4(o[0], o[1], o[2], o[3]);
}

__device__ __forceinline__ uint32_t byte_perm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// The V codes of a lane of the operand order for one channel tile: 8 tokens of one channel, as bytes in d0, d1 in the order
// v_tau below.  Eight lanes (channels) x 8 tokens are transposed: lane l = mm & 7 is left with token v_tau(l) and the
// channels 0..7 of the eight, in order.  Each exchange (partners l ^ 7, l ^ 2, l ^ 1) halves the tokens and doubles the
// channels; byte i of (hi, lo) is then the channel l ^ x with i = index(x), index linear over xor: 1 -> 4, 2 -> 2, 4 -> 7.
__device__ __forceinline__ uint2 transpose_codes(uint32_t d0, uint32_t d1, int l)
{
    const bool b0 = l & 1, b1 = l & 2, b2 = l & 4;
    const uint32_t a = b2 ? d1 : d0, b = lanes_moved<0x141>(b2 ? d0 : d1);
    const uint32_t k = byte_perm(b, a, b1 ? 0x07060302u : 0x05040100u), r = lanes_moved<0x4E>(byte_perm(b, a, b1 ? 0x05040100u : 0x07060302u));
    const uint32_t lo = byte_perm(r, k, b0 ? 0x07050301u : 0x06040200u), hi = lanes_moved<0xB1>(byte_perm(r, k, b0 ? 0x06040200u : 0x07050301u));
    const uint32_t own = ((b0 ? 4u : 0u) ^ (b1 ? 2u : 0u) ^ (b2 ? 7u : 0u)) * 0x01010101u;
    return make_uint2(byte_perm(hi, lo, 0x06020400u ^ own), byte_perm(hi, lo, 0x01050307u ^ own));
}
template <int BITS>
__device__ __forceinline__ int v_tau(int l)      // the token (tau) that byte l & 3 of d[l >> 2] belongs to
{
    constexpr uint32_t order = BITS == 8 ? 0x76543210u : BITS == 4 ? 0x75316420u : 0x73625140u;
    return (int)((order >> (4 * l)) & 7u);
}

template <int HD>
struct DenseSmem {
    static constexpr int PITCH = HD + 8;
    __attribute__((aligned(16))) uint8_t v[32 * PITCH];      // V codes, a byte each, [token][channel]
};

template <int HD, int BITS, bool BF>
__device__ __forceinline__ void dequantize_block(DenseSmem<HD>& sm, int blk, int kvh, int B, const wq_packed_kv& src, const wq_packed_kv& dst)
{
    constexpr int C = cls_index(BITS);
    constexpr int Q = HD / 4, CT = HD / 16, CTW = CT / 4;       // CTW: channel tiles that a wavefront transposes
    constexpr int ITEMS = HD / 64;                              // pieces of 8 channels per thread and plane
    const int tid = threadIdx.x, Hkv = src.Hkv, G = HD / src.group;
    const int32_t* off = src.cls_off[C];
    const int64_t tok0 = (int64_t)blk * 32;
    const uint8_t* kc = static_cast<const uint8_t*>(src.codes[C]) + ((int64_t)kvh * src.cap[C] + tok0) * HD * BITS / 8;
    const uint8_t* vc = static_cast<const uint8_t*>(src.codes[C]) + (((int64_t)Hkv + kvh) * src.cap[C] + tok0) * HD * BITS / 8;
    const uint32_t* km = static_cast<const uint32_t*>(src.meta[C]) + ((int64_t)kvh * src.cap[C] + tok0) * G;
    const uint32_t* vm = static_cast<const uint32_t*>(src.meta[C]) + (((int64_t)Hkv + kvh) * src.cap[C] + tok0) * G;
    // every load of the block first: this lane's V codes of the wavefront's channel tiles, its K pieces, the words of both
    const int lane = tid & 63, wave = tid >> 6, jj = lane >> 4, mm = lane & 15;
    constexpr int VB = CTW * BITS, KB = BITS;                   // bytes
    uint32_t vw[(VB + 3) / 4], kw[ITEMS][(KB + 3) / 4], kword[ITEMS], vword[ITEMS];
    load_bytes<VB>(vc + lane * (CT * BITS) + wave * VB, vw);
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        const int item = i * 256 + tid, u = item / (HD / 8), ch = (item % (HD / 8)) * 8, tile = u >> 4, m = u & 15;
        const int word = (tile * G + ch / src.group) * 16 + m;
        load_bytes<KB>(kc + tile * (16 * HD * BITS / 8) + ((ch / Q * 16 + m) * Q + ch % Q) * BITS / 8, kw[i]);
        kword[i] = km[word];
        vword[i] = vm[word];
    }
    const int b = wq_find_seq(off, B, tok0);
    if (!dense_fits(src, dst, b)) return;                       // (the same for the whole workgroup)
    const int d0 = (int)(tok0 - off[b]), len = src.cls_len[C][b];
    int before = 0;                                             // tokens of the lower classes come first
    for (int c = 0; c < C; c++) before += src.cls_len[c][b];

    const int l = mm & 7, tau = v_tau<BITS>(l);
    uint8_t* const vt = sm.v + (16 * (tau >> 2) + 4 * jj + (tau & 3)) * DenseSmem<HD>::PITCH + 8 * (mm >> 3);
#pragma unroll
    for (int k = 0; k < CTW; k++) {
        uint32_t c0, c1;
        if constexpr (BITS == 8) {
            c0 = vw[2 * k], c1 = vw[2 * k + 1];
        } else if constexpr (BITS == 4) {
            c0 = vw[k] & 0x0F0F0F0Fu, c1 = (vw[k] >> 4) & 0x0F0F0F0Fu;
        } else {
            const uint32_t x = k == 0 ? vw[0] & 0xFFFFu : vw[0] >> 16, y = (x << 14) | x;
            c0 = y & 0x03030303u, c1 = (y >> 4) & 0x03030303u;
        }
        *reinterpret_cast<uint2*>(vt + 16 * (wave * CTW + k)) = transpose_codes(c0, c1, l);
    }
    __syncthreads();
    const int64_t row0 = (int64_t)dst.off16[b] + before + d0;
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
        const int item = i * 256 + tid, u = item / (HD / 8), ch = (item % (HD / 8)) * 8;
        if (d0 + u >= len) continue;
        const int64_t o = ((row0 + u) * Hkv + kvh) * HD + ch;
        float c[8];
        codes_of<BITS>(kw[i], c);
        wq_store_once(static_cast<uint16_t*>(dst.k16) + o, dense_piece<BF>(c, kword[i]));
        const uint2 v = *reinterpret_cast<const uint2*>(sm.v + u * DenseSmem<HD>::PITCH + ch);
#pragma unroll
        for (int k = 0; k < 8; k++) c[k] = byte_of(k < 4 ? v.x : v.y, k & 3);
        wq_store_once(static_cast<uint16_t*>(dst.v16) + o, dense_piece<BF>(c, vword[i]));
    }
}

__device__ __forceinline__ void dense_copy(int64_t r0, int B, int pieces, const wq_packed_kv& src, const wq_packed_kv& dst)
{
    for (int e = threadIdx.x; e < DENSE_ROWS * pieces; e += 256) {
        const int64_t r = r0 + e / pieces;      // a row of src's 16-bit segment
        if (r < src.off16[0] || r >= src.off16[B] || r >= src.cap16) continue;
        const int b = wq_find_seq(src.off16, B, r);
        const int i = (int)(r - src.off16[b]);
        if (i >= src.len16[b] || !dense_fits(src, dst, b)) continue;
        const int64_t d = (int64_t)dst.off16[b] + src.cls_len[0][b] + src.cls_len[1][b] + src.cls_len[2][b] + i;
        const int64_t from = r * pieces + e % pieces, to = d * pieces + e % pieces;
        const uint4 k = static_cast<const uint4*>(src.k16)[from], v = static_cast<const uint4*>(src.v16)[from];
        wq_store_once(static_cast<uint4*>(dst.k16) + to, k);
        wq_store_once(static_cast<uint4*>(dst.v16) + to, v);
    }
}

// workgroup 0: the tables; then the 16-bit rows (rows16 workgroups), then the blocks of the classes that are in use, numbered
// without gaps (the capacities can be far larger: every class then has room for all tokens), but never more of them than the
// class has room for, whatever its table says
template <int HD, bool BF>
__global__ __launch_bounds__(256) void k_dequantize(int B, wq_packed_kv src, wq_packed_kv dst, unsigned rows16, uint32_t* __restrict__ status)
{
    __shared__ DenseSmem<HD> sm;
    unsigned w = blockIdx.y * gridDim.x + blockIdx.x;
    if (w == 0) {
        dense_plan(B, src, dst, status);
        return;
    }
    w -= 1;
    if (w < rows16) {
        dense_copy((int64_t)w * DENSE_ROWS, B, src.Hkv * HD / 8, src, dst);
        return;
    }
    w -= rows16;
    const unsigned Hkv = (unsigned)src.Hkv;
    auto blocks = [&](int c) { return (unsigned)(max((int64_t)0, min((int64_t)src.cls_off[c][B], src.cap[c])) / 32) * Hkv; };
    const unsigned n0 = blocks(0), n1 = blocks(1), n2 = blocks(2);
    if (w < n0)
        dequantize_block<HD, 2, BF>(sm, (int)(w / Hkv), (int)(w % Hkv), B, src, dst);
    else if (w - n0 < n1)
        dequantize_block<HD, 4, BF>(sm, (int)((w - n0) / Hkv), (int)((w - n0) % Hkv), B, src, dst);
    else if (w - n0 - n1 < n2)
        dequantize_block<HD, 8, BF>(sm, (int)((w - n0 - n1) / Hkv), (int)((w - n0 - n1) % Hkv), B, src, dst);
}

// Workgroups numbered row by row.  A dimension of a launch ends at 2^32 threads without an error (2^24 workgroups: one each for
// the blocks of 2^29 tokens times KV heads), so more than 2^22 of them go into two.
dim3 grid_of(int64_t wgs)
{
    constexpr int64_t MAX_X = 1 << 22;
    return dim3((unsigned)(wgs < MAX_X ? wgs : MAX_X), (unsigned)((wgs + MAX_X - 1) / MAX_X));
}

template <int HD>
int run_dequantize(wq_ctx* ctx, int B, const wq_packed_kv* src, const wq_packed_kv* dst)
{
    const int64_t rows16 = (src->cap16 + DENSE_ROWS - 1) / DENSE_ROWS;
    const int64_t blocks = (src->cap[0] + src->cap[1] + src->cap[2]) / 32;
    const int64_t wgs = 1 + rows16 + blocks * src->Hkv;
    if (wgs > 0x7FFFFFFF) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "too many blocks for one launch");
    hipLaunchKernelGGL((dst->dtype16 == WQ_BF16 ? k_dequantize<HD, true> : k_dequantize<HD, false>), grid_of(wgs), dim3(256), 0, ctx->stream, B,
                       *src, *dst, (unsigned)rows16, wq_status_ptr(ctx));
    WQ_HIP_CHECK(ctx, hipGetLastError());
    return WQ_OK;
}

template <typename T, int HD>
int run(wq_ctx* ctx, const void* K_, const void* V_, int B, const int32_t* kv_off, const int32_t* win_size,
        const int32_t* win_off, const int32_t* perm, const int32_t* seg_windows, int64_t total_rows, const wq_packed_kv* pk)
{
    const T* K = static_cast<const T*>(K_);
    const T* V = static_cast<const T*>(V_);
    hipStream_t st = ctx->stream;
    // blocks in use: no more than the capacities hold, nor than the rows fill if every sequence's last block of every class is
    // a partial one
    const int64_t held = (pk->cap[0] + pk->cap[1] + pk->cap[2]) / 32, filled = total_rows / 32 + 3 * (int64_t)B;
    const int64_t n = (held < filled ? held : filled) * pk->Hkv;
    const unsigned n0 = held <= filled ? (unsigned)(pk->cap[0] / 32 * pk->Hkv) : WQ_BY_USE, n1 = (unsigned)(pk->cap[1] / 32 * pk->Hkv);
    const int64_t rows16 = pk->cap16 > 0 ? (total_rows < pk->cap16 ? total_rows : pk->cap16) : 0;
    const int64_t wgs16 = (rows16 + ROWS16 - 1) / ROWS16;
    if (n + wgs16 > 0x7FFFFFFF) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "too many blocks for one launch");
    if (B <= SMALL_SEQS && n + wgs16 <= SMALL_WGS) {
        hipLaunchKernelGGL((k_quantize_small<T, HD>), dim3((unsigned)(n + wgs16 > 0 ? n + wgs16 : 1)), dim3(256), 0, st, K, V, B, pk->group, kv_off,
                           win_size, win_off, perm, seg_windows, *pk, (unsigned)n, wq_status_ptr(ctx), wq_small_arrive_ptr(ctx), wq_arrive_lines_ptr(ctx));
        WQ_HIP_CHECK(ctx, hipGetLastError());
        return WQ_OK;
    }
    int32_t* pre16 = reinterpret_cast<int32_t*>(ctx->ws + WQ_WS_HEADER);
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(256), 0, st, B, kv_off, win_size, win_off, seg_windows, *pk, pre16,
                       wq_status_ptr(ctx));
    if (n + wgs16 > 0)
        hipLaunchKernelGGL((k_quantize_all<T, HD>), grid_of(n + wgs16), dim3(256), 0, st, K, V, B, pk->group, kv_off, win_size,
                           win_off, perm, seg_windows, pre16, *pk, (unsigned)n, n0, n1);
    if (B > 0) hipLaunchKernelGGL(k_v_scale_max, dim3((unsigned)B * WQ_VS_PARTS), dim3(256), 0, st, B, *pk);
    WQ_HIP_CHECK(ctx, hipGetLastError());
    return WQ_OK;
}

}  // namespace

int wq_launch_append(wq_ctx* ctx, const void* k_new, const void* v_new, int dtype, int B, const wq_packed_kv* kv)
{
    const int row_elems = kv->Hkv * kv->hd;
    hipStream_t st = ctx->stream;
    switch (dtype) {
        case WQ_F32:
            hipLaunchKernelGGL(k_append16<float>, dim3(B), dim3(256), 0, st, static_cast<const float*>(k_new),
                               static_cast<const float*>(v_new), row_elems, *kv, wq_status_ptr(ctx));
            break;
        case WQ_BF16:
            hipLaunchKernelGGL(k_append16<__hip_bfloat16>, dim3(B), dim3(256), 0, st, static_cast<const __hip_bfloat16*>(k_new),
                               static_cast<const __hip_bfloat16*>(v_new), row_elems, *kv, wq_status_ptr(ctx));
            break;
        default:
            hipLaunchKernelGGL(k_append16<__half>, dim3(B), dim3(256), 0, st, static_cast<const __half*>(k_new),
                               static_cast<const __half*>(v_new), row_elems, *kv, wq_status_ptr(ctx));
    }
    WQ_HIP_CHECK(ctx, hipGetLastError());
    return WQ_OK;
}

int wq_launch_dequantize(wq_ctx* ctx, int B, const wq_packed_kv* src, const wq_packed_kv* dst)
{
    if (src->hd == 64 && src->group == 128) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "group larger than hd");
    return src->hd == 128 ? run_dequantize<128>(ctx, B, src, dst) : run_dequantize<64>(ctx, B, src, dst);
}

int wq_launch_quantize(wq_ctx* ctx, const void* K, const void* V, int dtype, int B, const int32_t* kv_off,
                       const int32_t* win_size, const int32_t* win_off, const int32_t* perm,
                       const int32_t* seg_windows, int64_t total_rows, const wq_packed_kv* out)
{
    if (out->hd == 64 && out->group == 128) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "group larger than hd");
#define WQ_RUN(T)                                                                                                   \
    (out->hd == 128 ? run<T, 128>(ctx, K, V, B, kv_off, win_size, win_off, perm, seg_windows, total_rows, out)      \
                    : run<T, 64>(ctx, K, V, B, kv_off, win_size, win_off, perm, seg_windows, total_rows, out))
    switch (dtype) {
        case WQ_F32: return WQ_RUN(float);
        case WQ_BF16: return WQ_RUN(__hip_bfloat16);
        default: return WQ_RUN(__half);
    }
#undef WQ_RUN
}
