// a1: window/text similarity (Sec. 3.2.1, similarity equation).
//
// Pooled path: by linearity the mean of all pairwise cosines of a window equals
//     (mean_j t_j/|t_j|) . (mean_k w_k/|w_k|),
// so every embedding row is read exactly once: the kernels are bound by HBM bandwidth.
//   k_text_norm   one wavefront per text token  -> 1/|t_j|                       (0 for a zero row)
//   k_text_mean   thread per channel            -> tbar[b][d] = 1/N sum_j t_j[d]/|t_j|
//   k_token_score one wavefront per visual row  -> c_k = (w_k . tbar) / |w_k|    (0 for a zero row)
//   k_window_mean one wavefront per window      -> score = 1/S sum_k c_k, fixed order (part of k_token_score up to FOLD_ROWS, FOLD_BYTES where the counters fit)
//   k_scores_small  all of it for a short text and few rows, a workgroup per window
// All accumulation is fp32 and every reduction has a fixed order (no atomics): results are deterministic.
#include "wq_internal.h"

#include <type_traits>

namespace {

constexpr int WAVE = 64;
// k_token_score: visual rows per wavefront, and how far the loop over a row's elements is unrolled (measured on 4 x 50176 rows of
// 3584 bf16: 2 rows, unrolled twice: 257 us for the whole call; 4 rows: 277; 1 row: 269; 8 rows: 390)
constexpr int WQ_TS_ROWS = 2;
#define WQ_TS_UNROLL 2

// x of the lane that a data-parallel-primitive control pairs this lane with (rows of 16 lanes)
template <int CTRL>
__device__ __forceinline__ float lanes_moved(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// Sum over the wavefront, in every lane: lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1 in turn, by moves between registers (exchanging
// through LDS takes six round trips).  Once lanes that differ in the bits above are equal, a rotation by 8, 4, 2, 1 inside a
// row of 16 lanes brings the value of lane ^ 8, ^ 4, ^ 2, ^ 1.
__device__ __forceinline__ float wave_sum(float v)
{
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v += lanes_moved<0x128>(v);
    v += lanes_moved<0x124>(v);
    v += lanes_moved<0x122>(v);
    v += lanes_moved<0x121>(v);
    return v;
}

// VEC: rows are read 8 elements per lane (needs D % 8 == 0), WQ_TEXT_FLIGHT pieces in flight; otherwise element by element.  The two
// kernels of the text read a few MB and are bound by the latency of their loads: one piece after the other 4 x 512 tokens of 3584 bf16 take
// 5.9 and 8.0 us, so 4.7 and 4.8; 512 of them 4.5 and 8.2, so 4.0 and 4.5.  Pieces past the row's or the text's end are loaded all the same: with eight in
// flight short texts lose by it (a call for 2000 rows of 512: 14 tokens 9.1 us with one, 8.6 with four, 9.1 with eight; 600 tokens 14.6, 10.7, 11.2;
// 100 sizes, 5 to 600 tokens of 512 to 4096: four 1.146 times as fast as one on average, 0.991 at least; eight 1.111 and 0.982, two 1.119 and 0.996).
constexpr int WQ_TEXT_FLIGHT = 4;
// What k_token_score needs to make the windows' means itself (FOLD).  folded windows: k_text_norm clears their counters, a line each
constexpr int FOLD_STRIDE = 16;
struct WindowFold {
    const int32_t *win_size, *win_off, *txt_off;
    unsigned* rows_done;
    float* scores;
};
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_text_norm(const T* __restrict__ txt, int D, int64_t total_txt,
                                                   float* __restrict__ inv_norm, WindowFold fold, int64_t folded)
{
    for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < folded; w += (int64_t)gridDim.x * 256) {
        fold.rows_done[w * FOLD_STRIDE] = 0u;
        fold.scores[w] = 0.f;                             // (what a window without rows has)
    }
    int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= total_txt) return;
    int lane = threadIdx.x & 63;
    const T* p = txt + row * D;
    float ss = 0.f;
    if (VEC) {
        for (int d0 = lane * 8; d0 < D; d0 += WAVE * 8 * WQ_TEXT_FLIGHT) {
            float x[WQ_TEXT_FLIGHT][8];
#pragma unroll
            for (int i = 0; i < WQ_TEXT_FLIGHT; i++) wq_ld8(p + min(d0 + i * WAVE * 8, D - 8), x[i]);
#pragma unroll
            for (int i = 0; i < WQ_TEXT_FLIGHT; i++)
#pragma unroll
                for (int k = 0; k < 8; k++) ss = d0 + i * WAVE * 8 < D ? fmaf(x[i][k], x[i][k], ss) : ss;
        }
    } else {
        for (int d = lane; d < D; d += WAVE) {
            float x = wq_ld(p, d);
            ss = fmaf(x, x, ss);
        }
    }
    ss = wave_sum(ss);
    if (lane == 0) inv_norm[row] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
}

// tbar[b][d] = 1/N sum_j t_j[d]/|t_j|.  VEC: a workgroup takes 64 columns, thread = (8 columns, one of 32 token slices),
// slices merged in LDS in slice order (many small workgroups: the kernel is bound by the latency of its row loads);
// otherwise one thread per column.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_text_mean(const T* __restrict__ txt, const float* __restrict__ inv_norm, int D,
                                                   const int32_t* __restrict__ txt_off, float* __restrict__ tbar)
{
    const int b = blockIdx.y;
    const int j0 = txt_off[b], j1 = txt_off[b + 1];
    if (VEC) {
        __shared__ float s_acc[32][8][9];
        const int cc = threadIdx.x & 7, ts = threadIdx.x >> 3;
        const int d0 = (blockIdx.x * 8 + cc) * 8;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (d0 < D)
            for (int j = j0 + ts; j < j1; j += 32 * WQ_TEXT_FLIGHT) {
                float x[WQ_TEXT_FLIGHT][8], w[WQ_TEXT_FLIGHT];
#pragma unroll
                for (int i = 0; i < WQ_TEXT_FLIGHT; i++) {
                    const int row = min(j + 32 * i, j1 - 1);
                    wq_ld8(txt + (int64_t)row * D + d0, x[i]);
                    w[i] = inv_norm[row];
                }
#pragma unroll
                for (int i = 0; i < WQ_TEXT_FLIGHT; i++)
#pragma unroll
                    for (int k = 0; k < 8; k++) acc[k] = j + 32 * i < j1 ? fmaf(x[i][k], w[i], acc[k]) : acc[k];
            }
#pragma unroll
        for (int k = 0; k < 8; k++) s_acc[ts][cc][k] = acc[k];
        __syncthreads();
        const int c2 = threadIdx.x >> 3, k2 = threadIdx.x & 7;      // 8 chunks x 8 columns
        const int d = (blockIdx.x * 8 + c2) * 8 + k2;
        if (threadIdx.x < 64 && d < D) {
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < 32; t++) s += s_acc[t][c2][k2];
            tbar[(int64_t)b * D + d] = j1 > j0 ? s / (float)(j1 - j0) : 0.f;
        }
    } else {
        int d = blockIdx.x * 256 + threadIdx.x;
        if (d >= D) return;
        float acc = 0.f;
        for (int j = j0; j < j1; j++) acc = fmaf(wq_ld(txt, (int64_t)j * D + d), inv_norm[j], acc);
        tbar[(int64_t)b * D + d] = j1 > j0 ? acc / (float)(j1 - j0) : 0.f;
    }
}

// c_k = (w_k . tbar) / |w_k|.  VEC: one wavefront takes WQ_TS_ROWS consecutive rows so that each 32-byte piece of the pooled
// text vector is loaded once per WQ_TS_ROWS rows; 16 bytes of every row per lane and iteration.  Bound by HBM.  With ONCE the
// rows' loads say that they are read once (non-temporal): 4 x 50176 rows of 3584 bf16 246 -> 229 us a call (6.0 -> 6.5 TB/s in this kernel), 50176 of 896
// 35.8 -> 31.6, 64.3 -> 61.4 with a copy that has just written the 12544 of 3584 in front of it.  Below ONCE_FROM bytes plain loads, which the memory-side
// cache serves where a few such inputs are scored in turn (three of 30000 rows of 896: 22.7 us with non-temporal loads, 21.0 so; three of 10000 of 3584: 21.8 and 20.8; four
// launches, 8624 rows of 896 and a text of 14 tokens: 12.1 and 11.6; behind a matrix product that writes them the two are the same to 1 %).  fp32 rows keep plain loads (10 % faster: wq_ld8_once).
// FOLD (VEC only): the workgroup that finishes a window's last row makes the window's mean, as k_window_mean does.
template <typename T, bool VEC, bool FOLD, bool ONCE>
__global__ __launch_bounds__(256) void k_token_score(const T* __restrict__ vis, const float* __restrict__ tbar, int D, int B,
                                                     const int32_t* __restrict__ vis_off, int64_t total_vis,
                                                     float* __restrict__ tok_score, WindowFold fold)
{
    const int lane = threadIdx.x & 63;
    if (VEC) {
        constexpr int R = WQ_TS_ROWS, ROWS = 4 * R;
        const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * R;
        if (!FOLD && row0 >= total_vis) return;
        __shared__ float s_score[FOLD ? ROWS : 1];
        int bs[R];
        const T* p[R];
        int first = 0, size = 0, window = 0, windows_end = 0, text = 0;      // FOLD: of the sequence of the workgroup's row number `lane`
        if constexpr (FOLD) {
            const int b = wq_find_seq(vis_off, B, min((int64_t)blockIdx.x * ROWS + lane % ROWS, total_vis - 1));
            first = vis_off[b];
            size = fold.win_size[b];
            window = fold.win_off[b];
            windows_end = fold.win_off[b + 1];
            text = fold.txt_off[b + 1] - fold.txt_off[b];
            const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
            for (int r = 0; r < R; r++) bs[r] = __builtin_amdgcn_readlane(b, wave * R + r);
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t row = row0 + r < total_vis ? row0 + r : total_vis - 1;
            if constexpr (!FOLD) bs[r] = wq_find_seq(vis_off, B, row);
            p[r] = vis + row * D;
        }
        const bool same = bs[0] == bs[R - 1];      // rows are ordered by sequence: all of them share one text vector
        float ss[R], dt[R];
#pragma unroll
        for (int r = 0; r < R; r++) ss[r] = dt[r] = 0.f;
#pragma unroll WQ_TS_UNROLL
        for (int d = lane * 8; d < D; d += WAVE * 8) {
            float t[8];
            wq_ld8(tbar + (int64_t)bs[0] * D + d, t);
#pragma unroll
            for (int r = 0; r < R; r++) {
                float x[8], tr[8];
                if constexpr (ONCE) wq_ld8_once(p[r] + d, x);
                else wq_ld8(p[r] + d, x);
                if (!same && bs[r] != bs[0]) wq_ld8(tbar + (int64_t)bs[r] * D + d, tr);
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const float tk = (!same && bs[r] != bs[0]) ? tr[k] : t[k];
                    ss[r] = fmaf(x[k], x[k], ss[r]);
                    dt[r] = fmaf(x[k], tk, dt[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; r++) {
            const float s = wave_sum(ss[r]), d2 = wave_sum(dt[r]);
            const float c = s > 0.f ? d2 / sqrtf(s) : 0.f;
            if constexpr (FOLD) {
                if (lane == 0) s_score[(int)(threadIdx.x >> 6) * R + r] = c;
            } else {
                if (lane == 0 && row0 + r < total_vis) tok_score[row0 + r] = c;
            }
        }
        if constexpr (FOLD) {
            __syncthreads();
            if (threadIdx.x >= WAVE) return;
            // A lane per row.  The scores are stored past the XCD's L2 and acknowledged before the rows are counted, so whoever completes a window
            // reads scores that have arrived.  (At most FOLD_ROWS rows: 32 bits hold everything.)
            const int base = (int)blockIdx.x * ROWS, row = base + lane, end = min(base + ROWS, (int)total_vis);
            // (rows may lie in front of the first sequence's, whose windows are counted back from it as k_window_mean does; the ones that
            // would come before the first window or begin before the first row are none)
            const int ahead = row - first, nth = size <= 0 ? 0 : ahead >= 0 ? ahead / size : ~(~ahead / size), begin = first + nth * size;
            window += nth;
            const bool counted = row < end && size > 0 && window >= 0 && window < windows_end && begin >= 0;
            if (row < end) __hip_atomic_store(tok_score + row, s_score[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            bool done = false;
            if (counted && row == max(base, begin)) {     // the workgroup's first row of the window
                const unsigned n = (unsigned)(min(end, begin + size) - row);
                done = __hip_atomic_fetch_add(fold.rows_done + (int64_t)window * FOLD_STRIDE, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + n == (unsigned)size;
            }
            for (uint64_t left = __builtin_amdgcn_ballot_w64(done); left != 0; left &= left - 1) {
                const int l = __builtin_ctzll(left), S = __builtin_amdgcn_readlane(size, l), r0 = __builtin_amdgcn_readlane(begin, l);
                const int tokens = __builtin_amdgcn_readlane(text, l), w = __builtin_amdgcn_readlane(window, l);
                float acc = 0.f;
#pragma unroll 4
                for (int k = lane; k < S; k += WAVE) acc += __hip_atomic_load(tok_score + r0 + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                acc = wave_sum(acc);
                if (lane == 0) fold.scores[w] = tokens > 0 ? acc / (float)S : 0.f;
            }
        }
    } else {
        int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
        if (row >= total_vis) return;
        int b = wq_find_seq(vis_off, B, row);
        const T* p = vis + row * D;
        const float* t = tbar + (int64_t)b * D;
        float ss = 0.f, dt = 0.f;
        for (int d = lane; d < D; d += WAVE) {
            float x = wq_ld(p, d);
            ss = fmaf(x, x, ss);
            dt = fmaf(x, t[d], dt);
        }
        ss = wave_sum(ss);
        dt = wave_sum(dt);
        if (lane == 0) tok_score[row] = ss > 0.f ? dt / sqrtf(ss) : 0.f;
    }
}

__global__ __launch_bounds__(256) void k_window_mean(const float* __restrict__ tok_score, int B,
                                                     const int32_t* __restrict__ vis_off, const int32_t* __restrict__ txt_off,
                                                     const int32_t* __restrict__ win_size, const int32_t* __restrict__ win_off,
                                                     int64_t total_win, float* __restrict__ scores)
{
    int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (w >= total_win) return;
    int lane = threadIdx.x & 63;
    // Bound by round trips to memory: up to 64 sequences a lane has a sequence's tables, all of them in one (searched by halves and then read,
    // four for 4 sequences, six for 16).  One sequence needs no search, and scalar loads (0.1 us less)
    int S, tokens;
    int64_t r0;
    if (B > 1 && B <= WAVE) {
        const int l = min(lane, B - 1), size = win_size[l], first = win_off[l], after = win_off[l + 1], row = vis_off[l], text = txt_off[l + 1] - txt_off[l];
        const int b = min(B - 1, (int)__popcll(__builtin_amdgcn_ballot_w64(lane < B && (int64_t)after <= w)));
        S = __builtin_amdgcn_readlane(size, b);
        tokens = __builtin_amdgcn_readlane(text, b);
        r0 = (int64_t)__builtin_amdgcn_readlane(row, b) + (w - __builtin_amdgcn_readlane(first, b)) * S;
    } else {
        const int b = wq_find_seq(win_off, B, w);
        S = win_size[b];
        tokens = txt_off[b + 1] - txt_off[b];
        r0 = (int64_t)vis_off[b] + (w - win_off[b]) * S;
    }
    float acc = 0.f;
#pragma unroll 4
    for (int k = lane; k < S; k += WAVE) acc += tok_score[r0 + k];
    acc = wave_sum(acc);
    if (lane == 0) scores[w] = (S > 0 && tokens > 0) ? acc / (float)S : 0.f;
}

// A call of a few windows in one launch: a workgroup per window finds the norms and the mean of its sequence's text for itself
// (in LDS), then its rows' scores and their mean, in the order of the four kernels above, so that the bits are theirs.
// Launches and round trips to memory are all that such a call costs, so the text is read once, into LDS, and a wavefront's
// first row is on its way meanwhile: 8 windows of 16 rows, 16 text tokens, 896 floats: four launches, 16 us; this one 6.
// A workgroup goes through its sequence's tokens and its window's rows in a chain of 0.07 to 0.1 us each, the four launches over
// all of them at once: 9 to 12 us whatever the sizes (11 to 17 where a call waits for its launches to be submitted).  So the tokens of a sequence and the
// rows of a window together are no more than SMALL_CHAIN, on average (the host knows the totals only), with a text of up to 64 KB a sequence (two: 96 KB), and
// SMALL_CHAIN_LONG with more (all must fit LDS).  Inside these lines, over 1700 combinations (1 to 64 tokens and rows, D 128 to 4096, bf16 and fp32), 0.38 to
// 1.02 of the four launches' time in a replayed graph, 0.36 to 0.82 of it otherwise; beyond: 96 tokens 9 to 11 us against 9, 256 tokens 20 against 10, 64 tokens and
// rows of 64 11 to 13 against 9, 32 tokens of 2048 bf16 and rows of 32 11.3 against 9.8.
constexpr int SMALL_THREADS = 1024, SMALL_TOKENS = 256, SMALL_TEXT = 128 << 10, SMALL_ROWS = 1024, SMALL_WINDOWS = 256, SMALL_DIM = 4096;
constexpr int64_t SMALL_BYTES = 1 << 20, SMALL_SEQ_TEXT = 32 << 10, SMALL_CHAIN = 72, SMALL_CHAIN_LONG = 32;
template <typename T>
__global__ __launch_bounds__(SMALL_THREADS) void k_scores_small(const T* __restrict__ vis, const T* __restrict__ txt, int D, int B,
                                                                const int32_t* __restrict__ vis_off, const int32_t* __restrict__ txt_off,
                                                                const int32_t* __restrict__ win_size, const int32_t* __restrict__ win_off,
                                                                float* __restrict__ scores)
{
    __shared__ float s_inv[SMALL_TOKENS], s_tok[SMALL_ROWS];
    __shared__ __align__(16) float s_tbar[SMALL_DIM];
    __shared__ __align__(16) T s_txt[SMALL_TEXT / sizeof(T)];
    constexpr int WAVES = SMALL_THREADS / WAVE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, w = (int)blockIdx.x;
    const int b = wq_find_seq(win_off, B, w);
    const int n0 = txt_off[b], N = txt_off[b + 1] - n0, S = win_size[b];
    const int64_t r0 = (int64_t)vis_off[b] + (int64_t)(w - win_off[b]) * S;
    constexpr int FIRST = 2;                              // pieces per lane of the first row that are sent for at once
    float first[FIRST][8];
#pragma unroll
    for (int i = 0; i < FIRST; i++)
        if (wave < S && lane * 8 + i * WAVE * 8 < D) wq_ld8(vis + (r0 + wave) * D + lane * 8 + i * WAVE * 8, first[i]);
    for (int j = wave; j < N; j += WAVES) {               // (k_text_norm)
        const T* p = txt + (int64_t)(n0 + j) * D;
        float ss = 0.f;
        for (int d = lane * 8; d < D; d += WAVE * 8) {
            constexpr int W = sizeof(T) / 2;              // 16-byte words of 8 elements
            uint4 u[W];
#pragma unroll
            for (int i = 0; i < W; i++) u[i] = reinterpret_cast<const uint4*>(p + d)[i];
#pragma unroll
            for (int i = 0; i < W; i++) reinterpret_cast<uint4*>(s_txt + j * D + d)[i] = u[i];
            float x[8];
            wq_ld8(reinterpret_cast<const T*>(u), x);
#pragma unroll
            for (int k = 0; k < 8; k++) ss = fmaf(x[k], x[k], ss);
        }
        ss = wave_sum(ss);
        if (lane == 0) s_inv[j] = ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
    }
    __syncthreads();
    for (int d = tid; d < D; d += SMALL_THREADS) {        // (k_text_mean: 32 slices of the tokens, then their sums)
        float s = 0.f;
#pragma unroll 1
        for (int t0 = 0; t0 < min(N, 32); t0 += 8) {
            float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int j = t0; j < N; j += 32) {
                float x[8], v[8];
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const int i = min(j + k, N - 1);
                    x[k] = wq_ld(s_txt, i * D + d);
                    v[k] = s_inv[i];
                }
#pragma unroll
                for (int k = 0; k < 8; k++) acc[k] = j + k < N ? fmaf(x[k], v[k], acc[k]) : acc[k];
            }
#pragma unroll
            for (int k = 0; k < 8; k++) s += acc[k];
        }
        s_tbar[d] = N > 0 ? s / (float)N : 0.f;
    }
    __syncthreads();
    for (int r = wave; r < S; r += WAVES) {               // (k_token_score)
        const T* p = vis + (r0 + r) * D;
        float ss = 0.f, dt = 0.f;
        auto piece = [&](const float (&x)[8], int d) {
            float t[8];
            wq_ld8(s_tbar + d, t);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                ss = fmaf(x[k], x[k], ss);
                dt = fmaf(x[k], t[k], dt);
            }
        };
        int d = lane * 8;
        if (r == wave) {
#pragma unroll
            for (int i = 0; i < FIRST; i++, d += WAVE * 8)
                if (d < D) piece(first[i], d);
        }
        for (; d < D; d += WAVE * 8) {
            float x[8];
            wq_ld8(p + d, x);
            piece(x, d);
        }
        ss = wave_sum(ss);
        dt = wave_sum(dt);
        if (lane == 0) s_tok[r] = ss > 0.f ? dt / sqrtf(ss) : 0.f;
    }
    __syncthreads();
    if (wave == 0) {                                      // (k_window_mean)
        float acc = 0.f;
        for (int k = lane; k < S; k += WAVE) acc += s_tok[k];
        acc = wave_sum(acc);
        if (lane == 0) scores[w] = (S > 0 && N > 0) ? acc / (float)S : 0.f;
    }
}

// ---- pairwise path on the matrix cores --------------------------------------------------------------------------
// The similarity equation taken literally: C = E_v E_t^T (every window token against every text token), then
// c_k = 1/(N |w_k|) sum_j C[k,j] / |t_j|.  A tile is up to 256 visual rows of one sequence (128 where it has more than 256
// text tokens); its text tokens are walked in passes of up to 256 (512) columns, so that the visual rows are read from memory
// once when the sequence has at most 512 text tokens.  One workgroup of eight wavefronts per compute unit takes a contiguous
// share of the launch's rows.  Over D it goes in steps of KS elements (64, or 128 with 128-row tiles: 32 KB of rows each):
//   visual rows   memory -> LDS directly (buffer loads with the LDS bit, two or three steps ahead, three or four buffers, one
//                 barrier per step) -> A operands of all wavefronts, read two product groups ahead of their use;
//   text rows     each wavefront owns 16 CT columns of the pass (CT = 4, or 2 with up to 256 columns), so its B operands are
//                 private to it.  An operand is 16 rows x 16 bytes per lane group: read from the row-major text that is 64
//                 scattered pieces per load, which the memory pipeline takes one lane at a time.  k_pack_text therefore
//                 rewrites the text once (a few MB) into operand order, [tile of 16 rows][32 elements of D][lane][8 elements],
//                 so that a wavefront's operand is one contiguous KB; it goes from there (L2) straight into registers, 64 of
//                 them whatever CT, 16 / CT instructions deep ahead.
// A wavefront multiplies a [16 RT] x [16 CT] tile per step with v_mfma_f32_16x16x32 bf16/f16 (up to 128 accumulator registers,
// two wavefronts per SIMD).  At the end of a pass the products are multiplied by 1/|t_j| and summed over the columns, so C
// never leaves the registers.  |w_k|^2 comes from the A operands of one or two row tiles per wavefront during the first pass.
// Reductions have a fixed order: results are deterministic.
// What bounds it: above 256 columns the matrix cores, which sustain about three quarters of their nominal rate with operands
// that change from product to product (wq_probe_mfma measures it: the clock drops under the load) and are kept busy three
// quarters of the kernel's cycles.  Up to 256 columns what passes the compute unit's memory pipeline: a wavefront's loads
// complete in order, so the text operands wait for the rows sent for before them, and have to be sent for about as far ahead;
// and LDS, 72 % of whose cycles are reads of operands that feed two products each and the rows' writes.
// 8 x 12544 rows of 3584 bf16, us per call (a read of the rows alone: 117), tiles of 128 rows x 64 columns of a wavefront ->
// tiles of up to 256 rows x 32: 256 text tokens 264 -> 192, 128: 230 -> 159, 20: 219 -> 128; 32 x 3136 rows of 4096, 256 text
// tokens: 430 -> 234; one sequence of 19600 rows, 200 text tokens: 63 -> 57.  (64 columns and two row groups of 128 rows: 206 at
// 256 text tokens; every text operand is then loaded twice, and only half as far ahead.)
// Variants measured and dropped because they were not faster: text operands sent for one by one, three quarters of a step
// ahead; the 32x32x16 form of the instruction; each XCD or each workgroup beginning elsewhere in D.
typedef float floatx4s __attribute__((ext_vector_type(4)));
typedef _Float16 half8s __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8s __attribute__((ext_vector_type(8)));

template <bool BF>
__device__ __forceinline__ floatx4s mfma_s(const uint4& a, const uint4& b, floatx4s c)
{
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8s, a), __builtin_bit_cast(bf16x8s, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8s, a), __builtin_bit_cast(half8s, b), c, 0, 0, 0);
}

typedef __bf16 bf16x2s __attribute__((ext_vector_type(2)));
typedef _Float16 half2s __attribute__((ext_vector_type(2)));

// sum of the squares of eight 16-bit elements (v_dot2_f32: both products and the sum in fp32)
template <bool BF>
__device__ __forceinline__ float sumsq8(const uint4& u)
{
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        if constexpr (BF) {
            const bf16x2s p = __builtin_bit_cast(bf16x2s, w[k]);
            s = __builtin_amdgcn_fdot2_f32_bf16(p, p, s, false);
        } else {
            const half2s p = __builtin_bit_cast(half2s, w[k]);
            s = __builtin_amdgcn_fdot2(p, p, s, false);
        }
    }
    return s;
}

constexpr int PA_THREADS = 512, PA_WAVES = 8;
constexpr int PA_BUF = 16384;            // elements of one LDS buffer: 128 rows of 128 elements, or 256 rows of 64
constexpr int PA_DMA = PA_BUF / 8 / (64 * PA_WAVES);   // loads to LDS per wavefront and step (64 16-byte pieces each)
constexpr int PA_ROW_POLICY = 2;         // cache policy of the visual rows' loads: non-temporal (read once; measured 1 % fewer cycles)

// Tiles of 16 text rows in operand order.  Sequence b's tiles start at tile txt_off[b] / 16 + b: room for
// ceil(N_b / 16) tiles each, whatever the lengths.  Rows past N_b are zero.
__device__ __forceinline__ int pair_tile_base(const int32_t* txt_off, int b) { return (txt_off[b] >> 4) + b; }

// A workgroup takes a tile: its wavefronts the chunks of 32 elements in turn, PT_FLIGHT of them in flight, and 1/|t_j| of its rows
// on the way (0 for a zero row).  Bound by the latency of its loads.  (Chunk by chunk over four times the wavefronts, behind
// a kernel of its own for the norms: 14 us of a call for 8 x 256 rows of 3584 between them, this one 8.)
constexpr int PT_THREADS = 1024, PT_FLIGHT = 4;
template <bool BF>
__global__ __launch_bounds__(PT_THREADS) void k_pack_text(const uint16_t* __restrict__ txt, int D, int B, const int32_t* __restrict__ txt_off,
                                                          uint4* __restrict__ packed, float* __restrict__ inv_norm)
{
    constexpr int WAVES = PT_THREADS / 64;
    __shared__ float s_sum[WAVES][16];
    const int chunks = D / 32, tile = (int)blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lm = lane & 15, lj = lane >> 4;
    // the sequence that owns this tile: the last b with pair_tile_base(b) <= tile
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pair_tile_base(txt_off, mid) <= tile) lo = mid; else hi = mid - 1;
    }
    const int n0 = txt_off[lo], N = txt_off[lo + 1] - n0;
    const int row = (tile - pair_tile_base(txt_off, lo)) * 16 + lm;
    const uint16_t* const src = txt + ((int64_t)n0 + row) * D + lj * 8;
    uint4* const dst = packed + (int64_t)tile * chunks * 64 + lane;
    float ss = 0.f;
    for (int c0 = wave; c0 < chunks; c0 += WAVES * PT_FLIGHT) {
        uint4 v[PT_FLIGHT];
#pragma unroll
        for (int k = 0; k < PT_FLIGHT; k++) {
            const int c = c0 + k * WAVES;
            v[k] = (row < N && c < chunks) ? *reinterpret_cast<const uint4*>(src + c * 32) : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < PT_FLIGHT; k++) {
            const int c = c0 + k * WAVES;
            if (c < chunks) dst[c * 64] = v[k];
            const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float x = BF ? wq_bf16_bits_to_float(w[e] & 0xFFFFu) : wq_f16_bits_to_float(w[e] & 0xFFFFu);
                const float y = BF ? wq_bf16_bits_to_float(w[e] >> 16) : wq_f16_bits_to_float(w[e] >> 16);
                ss = fmaf(y, y, fmaf(x, x, ss));
            }
        }
    }
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (lane < 16) s_sum[wave][lane] = ss;
    __syncthreads();
    if (threadIdx.x < 16 && row < N) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; w++) t += s_sum[w][lane];
        inv_norm[n0 + row] = t > 0.f ? 1.0f / sqrtf(t) : 0.f;
    }
}

// The buffers of visual rows are separate arrays on purpose: the compiler then knows that a read of one cannot
// see a load in flight to another, and makes a wavefront wait for exactly the loads it reads behind.
__shared__ __attribute__((aligned(16))) uint16_t pair_a0[PA_BUF];
__shared__ __attribute__((aligned(16))) uint16_t pair_a1[PA_BUF];
__shared__ __attribute__((aligned(16))) uint16_t pair_a2[PA_BUF];
__shared__ __attribute__((aligned(16))) uint16_t pair_a3[PA_BUF];
template <int P>
__device__ __forceinline__ uint16_t* pair_buf()
{
    static_assert(P >= 0 && P < 4, "four buffers");
    return P == 0 ? pair_a0 : (P == 1 ? pair_a1 : (P == 2 ? pair_a2 : pair_a3));
}
// Where 16-byte piece c of row r lies in its row of a buffer.  A wavefront's 16-byte reads go to LDS sixteen lanes at a time,
// eight of one lane group (rows 0-3, 12-15 or 4-11 of a tile) and eight of the next (the other rows, the next piece): so
// placed, the sixteen touch every bank once, without padding (with rows 288 bytes apart a sixth of the loads filled it).
template <int KS>
__device__ __forceinline__ int pair_place(int r, int c)
{
    return KS == 128 ? c ^ (r & 15) : c ^ ((r >> 1) & 7);
}

// One stage of a sum over the 16 lanes of a row, for NV values per lane at once: the lane and its partner (which
// differ in `upper`) split the values between them, each adding the other's half of the pair's sums to its own, so
// the lane is left with NV / 2 values, v[0 .. NV/2): the lower half of the indices if !upper, else the upper half.
// With a single value left both keep the sum.
template <int CTRL, int NV>
__device__ __forceinline__ void pair_halve(float (&v)[32], bool upper)
{
    if constexpr (NV >= 2) {
#pragma unroll
        for (int j = 0; j < NV / 2; j++) {
            const float give = upper ? v[j] : v[j + NV / 2];
            const float keep = upper ? v[j + NV / 2] : v[j];
            v[j] = keep + lanes_moved<CTRL>(give);
        }
    } else {
        v[0] += lanes_moved<CTRL>(v[0]);
    }
}

constexpr int PA_WCAP = 1024;            // text columns whose 1/|t_j| stay in LDS for a whole run
struct PairSmem {
    float W[PA_WCAP];                    // 1/|t_j| (0 past the end): of all passes if they fit, else of the current one
    float R[2048];                       // row sums, one array per column block
    float N2[256];                       // |w_k|^2
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
template <int P> struct PairBuf { static constexpr int value = P; };
struct PairUnit { int tile, pass; };     // a row tile of the sequence x a pass of columns
struct PairCursor { PairUnit u; int s; }; // a step of a unit

// A run: rows [row0, row_end) of one sequence in `ntiles` tiles of `rows` rows (a multiple of 16; the last tile may have
// fewer), each walked in ceil(N / PASS) passes of PASS
// text columns; a (tile, pass) is a unit of D / KS steps.  All units of a run form one pipeline: visual rows are sent
// for AL steps ahead and text operands BL steps ahead, across the ends of units, so the matrix cores do not wait for
// memory at the start of a tile, and what a unit leaves behind (scaling by 1/|t_j|, the sum over its columns, at a
// tile's end the scores) happens while those loads are in flight.
// The eight wavefronts are NCB column blocks of 16 CT text columns x RG = 8 / NCB row groups of RT row tiles of 16.
// A wavefront whose column block's number is c also
// sums |w_k|^2 of the row tiles c, c + NCB of its row group (read from LDS once more, a quarter at a time).
template <bool BF, int RT, int CT, int NCB, int KS>
__device__ __forceinline__ void pair_run(PairSmem& sm, const uint16_t* __restrict__ va, const char* __restrict__ tbb,
                                         const float* __restrict__ inv_tn, int D, int N, int row0, int row_end, int ntiles, int rows,
                                         float* __restrict__ out)
{
    constexpr int WCOLS = CT * 16, PASS = NCB * WCOLS;    // columns per wavefront, per pass
    constexpr int RG = PA_WAVES / NCB, OWN = (RT + NCB - 1) / NCB, CAP = RT * RG * 16;   // row groups, |w_k|^2 tiles per wavefront, most rows of a tile
    constexpr int AHEAD = 16 / CT;                        // quarters (32 elements of D, one matrix instruction deep) that text operands are sent for ahead: 64 registers
    constexpr int Q = KS / 32, NB = AHEAD == Q ? 3 : 4, AL = NB - 1, BL = AHEAD / Q;     // quarters per step, buffers, lead of rows and text in steps
    constexpr int PCS = KS / 8, DMA = (CAP * PCS + 64 * PA_WAVES - 1) / (64 * PA_WAVES); // 16-byte pieces of a row, loads to LDS per wavefront and step
    static_assert(DMA <= PA_DMA && NCB * CAP <= 2048 && CAP <= 256 && CAP * KS <= PA_BUF, "LDS arrays too small");
    static_assert(NB % BL == 0 || BL == 1, "a step's text registers are fixed by its buffer");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane >> 4, lm = lane & 15;
    const int cb = wave % NCB, rb = (wave / NCB) * RT;
    const int steps = D / KS, ntile = (N + 15) >> 4, npass = (N + PASS - 1) / PASS;

    // visual rows: memory -> LDS without passing registers.  A load instruction fills 64 consecutive 16-byte pieces
    // of the buffer, one per lane; the lane fetches the piece that belongs there.  The descriptor covers the tile's
    // rows only: rows past its end lie outside it and read as zero.
    auto rows_of = [&](PairUnit u) {
        const int r0 = row0 + u.tile * rows;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(va + (int64_t)r0 * D), 0, min(rows, row_end - r0) * D * 2, 0x00020000);
    };
    constexpr int RSTEP = 64 * PA_WAVES / PCS;            // rows from one load of a wavefront to its next (a multiple of 16: the same places)
    static_assert(RSTEP % 16 == 0, "pair_place repeats");
    const int pr = (wave * 64 + lane) / PCS, voff = (pr * D + pair_place<KS>(pr, lane % PCS) * 8) * 2;
    auto send_rows = [&](auto P, __amdgpu_buffer_rsrc_t tile_rows, int byte0) {     // 2 KS bytes of every row, from byte0 -> buffer P
        uint16_t* const dst = pair_buf<decltype(P)::value>();
        int v = voff;
        asm volatile("" : "+v"(v));                       // (the other loads' offsets: computed here, not kept)
#pragma unroll
        for (int t = 0; t < DMA; t++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(tile_rows, (lds_ptr_t)(dst + (wave + PA_WAVES * t) * 512), 16, v + t * (RSTEP * D * 2), byte0, 0,
                                                     PA_ROW_POLICY);
    };
    // byte offset of this lane's operand piece: of the wavefront's first tile (the tiles follow each other by 16 rows),
    // first quarter; a quarter further its place changes by an exclusive or (pair_place)
    constexpr int TILE_BYTES = 16 * KS * 2;
    const int ro = (rb * 16 + lm) * KS * 2 + pair_place<KS>(lm, lj) * 16;
    // A read from the buffer that this wavefront has sent loads for: the compiler puts the wait for those loads in
    // front of it (loads land in the order sent), whatever else it has moved around them.
    auto peek = [&](auto P) {
        const char* const src = reinterpret_cast<const char*>(pair_buf<decltype(P)::value>());
        return *reinterpret_cast<const uint32_t*>(src + ro);
    };
    auto use = [&](uint32_t x) { asm volatile("" ::"v"(x)); };
    // the wavefront's column tiles of a pass in the packed text (tiles past the end re-read the last one: their
    // weights are zero); a lane's 16 bytes of operand c of a tile sit at 1024 c + 16 lane
    auto text_of = [&](PairUnit u, const char* (&t)[CT]) {
#pragma unroll
        for (int k = 0; k < CT; k++)
            t[k] = tbb + (int64_t)min((u.pass * PASS + cb * WCOLS) / 16 + k, ntile - 1) * (D / 32) * 1024;
    };
    auto load_b = [&](const char* const (&t)[CT], int c, uint4 (&gb)[CT]) {      // elements 32 c .. 32 c + 31 of D
        const uint32_t off = (uint32_t)(c * 1024) + (uint32_t)lane * 16u;
#pragma unroll
        for (int k = 0; k < CT; k++) gb[k] = *reinterpret_cast<const uint4*>(t[k] + off);
    };
    auto after = [&](PairUnit u) {                        // the unit after u; the run's last unit is followed by itself
        if (++u.pass == npass) { u.pass = 0; ++u.tile; }
        if (u.tile == ntiles) { u.tile = ntiles - 1; u.pass = npass - 1; }
        return u;
    };
    // 1/|t_j| in LDS: all passes' at once if they fit, else pass by pass (the slow way: behind a barrier at a unit's end)
    const bool w_all = npass * PASS <= PA_WCAP;
    auto stage_weights = [&](int col0, int n) {
        for (int k = threadIdx.x; k < n; k += PA_THREADS) sm.W[k] = col0 + k < N ? inv_tn[col0 + k] : 0.f;
    };

    // Three cursors walk the run's steps: (uc, s) the step whose products are being summed; cb_, BL steps ahead, the
    // step whose text operands are sent for (tc: its unit's text); ca, AL steps ahead, the step whose visual rows are
    // sent for (dc: its tile's rows).  Past the run's end they stay in its last unit.
    auto advance = [&](PairCursor& c) {                   // true when it has entered another unit
        if (++c.s < steps) return false;
        c.s = 0;
        c.u = after(c.u);
        return true;
    };
    PairUnit uc{0, 0};
    PairCursor cb_{uc, 0}, ca{uc, 0};
    __amdgpu_buffer_rsrc_t dc = rows_of(uc);
    const char* tc[CT];
    text_of(uc, tc);
    floatx4s acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
        for (int k = 0; k < CT; k++) acc[i][k] = floatx4s{0.f, 0.f, 0.f, 0.f};
    float nsq[OWN];
#pragma unroll
    for (int o = 0; o < OWN; o++) nsq[o] = 0.f;
    int s = 0;

    __syncthreads();                                      // whoever used the buffers before is done with them
    stage_weights(0, w_all ? npass * PASS : PASS);
    __syncthreads();
    // gq: B operands of AHEAD quarters
    uint4 gq[AHEAD][CT];
    // the first loads in the order of the steps: otherwise the waits of the loop's first steps are those of the way into it
    auto load_step = [&](auto slot) {                     // the text operands of the step at cb_
#pragma unroll
        for (int q = 0; q < Q; q++) load_b(tc, Q * cb_.s + q, gq[decltype(slot)::value * Q + q]);
        if (advance(cb_)) text_of(cb_.u, tc);
    };
    auto before = [&](auto V) {                           // what step V - LEAD would send for
        constexpr int LEAD = AL > BL ? AL : BL, r = decltype(V)::value - LEAD + AL, t = decltype(V)::value - LEAD + BL;
        if constexpr (r >= 0 && r < AL) {
            send_rows(PairBuf<(r < NB ? r : 0)>{}, dc, ca.s * (KS * 2));
            if (advance(ca)) dc = rows_of(ca.u);
        }
        if constexpr (t >= 0 && t < BL) load_step(PairBuf<t>{});
    };
    before(PairBuf<0>{});
    before(PairBuf<1>{});
    before(PairBuf<2>{});
    before(PairBuf<3>{});
    use(peek(PairBuf<0>{}));

    // What a unit leaves behind.  The lane holds, of its i-th row tile, rows 4 lj + e at column lm of column tile k.
    // Scale by 1/|t_j| and sum over the wavefront's columns: over k in the lane, over lm across the 16 lanes of a
    // row in four stages of pairwise exchanges, each of which halves the number of values a lane carries (the
    // partners are lm ^ 8, lm ^ 7, lm ^ 2, lm ^ 1; the stages split on bits 3, 2, 1, 0 of lm).
    // (Both work from a copy of the thread's number that the compiler cannot trace: what they derive from it is then
    // computed here, once per unit, rather than kept in registers throughout the steps.)
    auto unit_done = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        const int lm = t & 15, lj = (t >> 4) & 3;
        float wk[CT];
#pragma unroll
        for (int k = 0; k < CT; k++) wk[k] = sm.W[(w_all ? uc.pass * PASS : 0) + cb * WCOLS + k * 16 + lm];
#pragma unroll
        for (int i0 = 0; i0 < RT; i0 += 8) {              // eight row tiles at a time
            constexpr int MOST = RT < 8 ? RT : 8;
            float v[32];
#pragma unroll
            for (int i = 0; i < MOST; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    float x = 0.f;
#pragma unroll
                    for (int k = 0; k < CT; k++) x = i0 + i < RT ? fmaf(acc[i0 + i < RT ? i0 + i : 0][k][e], wk[k], x) : 0.f;
                    v[i * 4 + e] = x;
                }
            constexpr int NV = MOST > 4 ? 32 : MOST > 2 ? 16 : MOST * 4;      // a power of two
#pragma unroll
            for (int j = MOST * 4; j < NV; j++) v[j] = 0.f;
            pair_halve<0x128, NV>(v, (lm & 8) != 0);                    // row_ror:8
            pair_halve<0x141, NV / 2>(v, (lm & 4) != 0);                // row_half_mirror
            pair_halve<0x4E, (NV >= 4 ? NV / 4 : 1)>(v, (lm & 2) != 0); // quad_perm [2,3,0,1]
            pair_halve<0xB1, (NV >= 8 ? NV / 8 : 1)>(v, (lm & 1) != 0); // quad_perm [1,0,3,2]
            // what is left: values j0 .. j0 + KEEP - 1 of the NV (j = 4 i + e), j0 made of the bits of lm that split a
            // stage; a stage that did not split left the sum in both lanes, the lower one writes
            constexpr int KEEP = NV >= 16 ? NV / 16 : 1;
            int j0 = 0;
            bool writer = true;
            if constexpr (NV >= 2) j0 += (lm & 8) ? NV / 2 : 0;
            if constexpr (NV >= 4) j0 += (lm & 4) ? NV / 4 : 0;
            if constexpr (NV >= 8) j0 += (lm & 2) ? NV / 8 : 0; else writer = writer && !(lm & 2);
            if constexpr (NV >= 16) j0 += (lm & 1) ? NV / 16 : 0; else writer = writer && !(lm & 1);
            if (writer) {
#pragma unroll
                for (int r = 0; r < KEEP; r++) {
                    const int j = j0 + r, i = i0 + (j >> 2);
                    if (i < RT) sm.R[cb * CAP + (rb + i) * 16 + 4 * lj + (j & 3)] += v[r];    // one writer per (column block, row)
                }
            }
        }
#pragma unroll
        for (int i = 0; i < RT; i++)
#pragma unroll
            for (int k = 0; k < CT; k++) acc[i][k] = floatx4s{0.f, 0.f, 0.f, 0.f};
    };
    // A tile's last unit is done: its scores.  |w_k|^2: lane (lm, lj) of a wavefront holds, for each of its own row tiles,
    // the sum over the pieces lj, lj + 4, ... of row lm.
    auto tile_done = [&](int tile) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
#pragma unroll
        for (int o = 0; o < OWN; o++) {
            nsq[o] += __shfl_xor(nsq[o], 16, 64);
            nsq[o] += __shfl_xor(nsq[o], 32, 64);
            if (lane < 16 && cb + NCB * o < RT) sm.N2[(rb + cb + NCB * o) * 16 + lane] = nsq[o];
            nsq[o] = 0.f;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (no fence: loads for the next unit are in flight)
        const int row = row0 + tile * rows + tid;
        if (tid < CAP) {
            float r = 0.f;
#pragma unroll
            for (int c = 0; c < NCB; c++) {
                r += sm.R[c * CAP + tid];
                sm.R[c * CAP + tid] = 0.f;                // for the next tile; the barriers of its steps come before its sums
            }
            const float nn = sm.N2[tid];
            if (tid < rows && row < row_end) out[row] = nn > 0.f ? r / (sqrtf(nn) * (float)N) : 0.f;
        }
    };

    // A step: LDS buffer P x the B operands, a quarter (32 elements of D) at a time.  The products' part has no
    // branches: it stays one block, which keeps the wait counts of the loads in flight exact.
    auto step = [&](auto P) {
        using Cur = decltype(P);
        using Nxt = PairBuf<(Cur::value + 1) % NB>;
        using Far = PairBuf<(Cur::value + AL) % NB>;
        constexpr int G0 = (Cur::value % BL) * Q;         // the step's first quarter in gq
        // every wavefront's rows of this step have landed (each waited for its own before it came here), and all are
        // done reading the buffer of the step before, which takes the rows AL steps ahead.  No fence: a fence would
        // wait for the B operands in flight.
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        send_rows(Far{}, dc, ca.s * (KS * 2));
        const float count = uc.pass == 0 ? 1.f : 0.f;     // |w_k|^2 is summed during the first pass (a factor, not a branch)
        const char* const sa = reinterpret_cast<const char*>(pair_buf<Cur::value>());
        int r1 = ro;
        asm volatile("" : "+v"(r1));                      // (the quarters' and buffers' addresses: computed here, not kept)
        auto place = [&](int q) { return r1 ^ (q * 64); };
        // Q RT groups of CT products: row tile i, quarter q; the A operand is read from LDS two groups
        // ahead.  A quarter's B operands are replaced as soon as their last product has issued.
        auto read_a = [&](int g) { return *reinterpret_cast<const uint4*>(sa + place(g / RT) + (g % RT) * TILE_BYTES); };
        uint4 f[3], own[OWN];
        uint32_t landed = 0u;
        f[0] = read_a(0);
        f[1] = read_a(1);
#pragma unroll
        for (int g = 0; g < Q * RT; g++) {
            const int i = g % RT, q = g / RT;
            if (g + 2 < Q * RT) f[(g + 2) % 3] = read_a(g + 2);
            if (i == 0) {
#pragma unroll
                for (int o = 0; o < OWN; o++)             // (a wavefront without such a tile reads its first one: nothing is made of it)
                    own[o] = *reinterpret_cast<const uint4*>(sa + place(q) + (cb + NCB * o < RT ? cb + NCB * o : 0) * TILE_BYTES);
            }
            if (g == Q * RT - 2) landed = peek(Nxt{});                // waits for the next step's rows, as late as it can
            if (i == RT - 1) {
#pragma unroll
                for (int o = 0; o < OWN; o++) nsq[o] = fmaf(sumsq8<BF>(own[o]), count, nsq[o]);
            }
#pragma unroll
            for (int k = 0; k < CT; k++) acc[i][k] = mfma_s<BF>(f[g % 3], gq[G0 + q][k], acc[i][k]);
            if (i == RT - 1) load_b(tc, Q * cb_.s + q, gq[G0 + q]);
            __builtin_amdgcn_sched_barrier(0);            // issue order as written: one LDS read, then the group's products
        }
        use(landed);
        if (s == steps - 1) {
            const PairUnit un = after(uc);
            unit_done();
            if (uc.pass == npass - 1) tile_done(uc.tile);
            if (!w_all) {
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // all have read this unit's weights
                stage_weights(un.pass * PASS, PASS);
            }
            s = 0;
            uc = un;
        } else {
            ++s;
        }
        if (advance(cb_)) text_of(cb_.u, tc);
        if (advance(ca)) dc = rows_of(ca.u);
    };
    const int total = ntiles * npass * steps;
    int gs = 0;
    for (; gs + NB <= total; gs += NB) {
        step(PairBuf<0>{});
        step(PairBuf<1>{});
        step(PairBuf<2>{});
        if constexpr (NB == 4) step(PairBuf<3>{});
    }
    if (gs < total) step(PairBuf<0>{});
    if (gs + 1 < total) step(PairBuf<1>{});
    if constexpr (NB == 4) {
        if (gs + 2 < total) step(PairBuf<2>{});
        use(peek(PairBuf<3>{}));
    }
    use(peek(PairBuf<0>{}));                              // nothing of this run is in flight to LDS any more
    use(peek(PairBuf<1>{}));
    use(peek(PairBuf<2>{}));
}

// What 16 rows of a sequence with N text tokens cost: reading them, up to 256 columns (the products take no longer), or the
// products of 512 columns and more.  (Not above 32: the rows that a card's memory holds then fit 32 bits.)
__device__ __forceinline__ uint32_t pair_cost(int N)
{
    return N <= 256 ? 1u : min(32u, 2u * ((uint32_t)(N + 511) / 512u));
}

// Whole numbers of workgroups per sequence, so that none has the end of one sequence and the beginning of the next: a run
// costs about PAIR_SLACK sixteens of rows however short it is (5 x 4704 rows of 3584, 64 text tokens, 5.7 sixteens a
// workgroup: 95 us a call with equal shares of all rows, 62 so; 7 x 12544 at most, 200 tokens: 138 and 122).  The smallest share
// from an equal one on that needs no more workgroups than there are, if one below PAIR_SLACK more does; a larger one costs more than the
// runs it saves (50 short sequences: 67 us with up to 6, 79 with 3).  With more than 256 text tokens, whose products bind a
// tile, a sequence gets no more workgroups than give them PAIR_LEAST sixteens, the smallest form's height: each reads all the text (4 x 3920 rows of
// 3584, 300 tokens: 77 us, so 73).  A lane looks at four sequences, and there are no more workgroups than 256 (65 x 500 rows, 200 tokens:
// 150 us cut evenly, 131 so; 100 x 128, 20 tokens: 120 and 81).  b: this workgroup's sequence, -1 if it has nothing to do.
constexpr uint32_t PAIR_SLACK = 6, PAIR_LEAST = 6;
struct PairWhole { bool fits; int b, part, parts; };
__device__ __forceinline__ PairWhole pair_whole(int B, const int32_t* vis_off, const int32_t* txt_off, uint32_t total)
{
    PairWhole p{false, -1, 0, 1};
    constexpr int PER = 4;                                // sequences per lane
    if (B > 64 * PER) return p;
    const int lane = threadIdx.x & 63;
    uint32_t cost[PER], most[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) {
        cost[i] = most[i] = 0u;
        if (i * 64 >= B) continue;
        const int b = i * 64 + lane, l = min(b, B - 1), N = txt_off[l + 1] - txt_off[l];
        const uint32_t T = b < B ? (uint32_t)(vis_off[l + 1] - vis_off[l] + 15) >> 4 : 0u;
        cost[i] = T * pair_cost(N);
        most[i] = N > 256 ? (T + PAIR_LEAST - 1) / PAIR_LEAST : T;
    }
    const uint32_t equal = (total + gridDim.x - 1) / gridDim.x;
    int n[PER] = {}, used = 0;
#pragma unroll 1
    for (uint32_t share = max(equal, 1u); share < equal + PAIR_SLACK && !p.fits; share++) {
        float sum = 0.f;                                  // (at most gridDim.x + B of them together: exact)
#pragma unroll
        for (int i = 0; i < PER; i++) {
            if (i * 64 < B) n[i] = (int)min(most[i], (cost[i] + share - 1) / share);
            sum += (float)n[i];
        }
        used = __builtin_amdgcn_readfirstlane((int)wave_sum(sum));
        p.fits = used <= (int)gridDim.x;
    }
    // (as many of the used ones on every XCD)
    const int xcd = (int)blockIdx.x % 8, wg = gridDim.x % 8 == 0 ? xcd * used / 8 + (int)blockIdx.x / 8 : (int)blockIdx.x;
    if (gridDim.x % 8 == 0 && wg >= (xcd + 1) * used / 8) return p;
    int upto = 0;
#pragma unroll
    for (int i = 0; i < PER; i++)
        for (int b = i * 64; p.fits && p.b < 0 && b < min(B, i * 64 + 64); b++) {
            const int m = __builtin_amdgcn_readlane(n[i], b - i * 64);
            if (wg < upto + m) p.b = b, p.part = wg - upto, p.parts = m;
            upto += m;
        }
    return p;
}

// The launch's rows, sixteen at a time, are laid out sequence after sequence on an axis of their cost; a workgroup takes an
// equal share of it, or of a sequence (pair_whole), and walks it as runs of rows of one sequence, a run in tiles of equal height (as few as there can be).
// Forms: what is left of 256 columns without text halves the column blocks and doubles the row groups.  Up to 8 sixteens of
// rows steps of 128 elements (half the barriers, and only half the LDS buffers' rows are there).  Every height that more than 8
// sixteens in tiles of at most 16 can come to has a form of its own (with those of even height and 13 only, shares of 18, 22 and 30 sixteens, tiles of
// 9, 11 and 15, took 148, 170 and 214 us a call instead of 145, 164 and 208: 8 sequences, 200 text tokens, D 3584).  Lower
// shares go to the next of 4 and 8 (6, 7 and 8 with more than 256 text tokens): the same sequences in shares of 1 to 8 sixteens
// take 47, 48, 51, 55, 64, 69, 74 and 79 us.  The forms stand in order of their columns and heights, the smallest first: a form pays for the
// branches and the registers held over them in front of it (the other way round 32 sequences of 1000 to 2550 rows, 30 tokens, took 99.8 us a call
// instead of 93.4, 16 x 3136, 100 tokens, 99.4 instead of 95.1, the larger ones the same).
template <bool BF>
__global__ __launch_bounds__(PA_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_pair_mfma(const uint16_t* __restrict__ vis, const uint4* __restrict__ packed_txt,
                                                          const float* __restrict__ inv_tnorm, int D, int B,
                                                          const int32_t* __restrict__ vis_off, const int32_t* __restrict__ txt_off,
                                                          float* __restrict__ tok_score)
{
    __shared__ PairSmem sm;
    const int tid = threadIdx.x;
    auto tiles_of = [&](int b) { return (uint32_t)(vis_off[b + 1] - vis_off[b] + 15) >> 4; };
    uint32_t total = 0;
    for (int b = 0; b < B; b++) total += tiles_of(b) * pair_cost(txt_off[b + 1] - txt_off[b]);
    // neighbouring shares on one XCD (workgroups go to the eight in turn): each then reads one or two sequences' text through its L2
    const uint32_t wg = gridDim.x % 8 == 0 ? blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8 : blockIdx.x;
    const uint32_t lo = (uint32_t)((uint64_t)total * wg / gridDim.x), hi = (uint32_t)((uint64_t)total * (wg + 1) / gridDim.x);
    for (int k = tid; k < 2048; k += PA_THREADS) sm.R[k] = 0.f;     // (a run starts with a barrier)
    const PairWhole whole = pair_whole(B, vis_off, txt_off, total);
    if (whole.fits && whole.b < 0) return;
    uint32_t at = 0;                                      // cost of the sequences before b
    const int last = whole.fits ? whole.b : B - 1;
    for (int b = whole.fits ? whole.b : 0; b <= last && (whole.fits || at < hi); b++) {
        const int n0 = txt_off[b], N = txt_off[b + 1] - n0;
        const uint32_t T = tiles_of(b), cost = pair_cost(N), begin = at;
        at += T * cost;
        if (at <= lo && !whole.fits) continue;
        auto edge = [&](uint32_t x) {                     // (a sequence that costs no more than a run is not cut: 400 x 64 rows, 20 tokens, 252 -> 219 us)
            if (x <= begin) return 0;
            if (T * cost <= PAIR_SLACK) return 2 * (x - begin) > T * cost ? (int)T : 0;
            return (int)min(T, (x - begin + cost - 1) / cost);
        };
        const int t0 = whole.fits ? (int)((uint64_t)T * whole.part / whole.parts) : edge(lo);
        const int t1 = whole.fits ? (int)((uint64_t)T * (whole.part + 1) / whole.parts) : edge(hi);
        if (t0 >= t1) continue;
        const int m0 = vis_off[b], M = vis_off[b + 1] - m0, row0 = t0 * 16, row_end = min(M, t1 * 16);
        const uint16_t* va = vis + (int64_t)m0 * D;
        const char* tb = reinterpret_cast<const char*>(packed_txt) + (int64_t)pair_tile_base(txt_off, b) * (D / 32) * 1024;
        float* out = tok_score + m0;
        const int most = N > 256 ? 8 : 16, n = (t1 - t0 + most - 1) / most, h = (t1 - t0 + n - 1) / n, rows = h * 16;     // tiles, their height
#define WQ_PAIR(RT, CT, NCB, KS) pair_run<BF, RT, CT, NCB, KS>(sm, va, tb, inv_tnorm + n0, D, N, row0, row_end, n, rows, out)
        if (N <= 0) {
            for (int r = row0 + tid; r < row_end; r += PA_THREADS) out[r] = 0.f;
        } else if (N <= 32) {
            WQ_PAIR(2, 2, 1, 64);
        } else if (N <= 64) {
            WQ_PAIR(4, 2, 2, 64);
        } else if (N <= 128) {
            WQ_PAIR(8, 2, 4, 64);
        } else if (N > 256) {
            if (h == 8) WQ_PAIR(8, 4, 8, 128);
            else if (h == 7) WQ_PAIR(7, 4, 8, 128);
            else WQ_PAIR(6, 4, 8, 128);
        } else {
            if (h <= 4) WQ_PAIR(4, 2, 8, 128);
            else if (h <= 8) WQ_PAIR(8, 2, 8, 128);
            else if (h == 9) WQ_PAIR(9, 2, 8, 64);
            else if (h == 10) WQ_PAIR(10, 2, 8, 64);
            else if (h == 11) WQ_PAIR(11, 2, 8, 64);
            else if (h == 12) WQ_PAIR(12, 2, 8, 64);
            else if (h == 13) WQ_PAIR(13, 2, 8, 64);
            else if (h == 14) WQ_PAIR(14, 2, 8, 64);
            else if (h == 15) WQ_PAIR(15, 2, 8, 64);
            else WQ_PAIR(16, 2, 8, 64);
        }
#undef WQ_PAIR
    }
}

// tiles of 16 text rows that the packed text of B sequences with total_txt rows can take (see pair_tile_base)
int64_t pair_total_tiles(int B, int64_t total_txt) { return total_txt / 16 + B; }

// Up to here k_token_score makes the windows' means itself: a launch saved against a wait at the end of every workgroup, which costs more where
// the rows keep the chip busy for long.  Four launches -> three, bf16: 6272 rows of 3584 18.2 -> 17.6 us, 25088 39.8 -> 39.0, 50176 69.1 -> 68.9, 75264
// (539 MB) 93.1 -> 95.2; 8192 rows of 512 12.3 -> 11.3, 65536 31.0 -> 27.8, 100352 of 896 (180 MB) 57.8 -> 54.3; 32768 of 4096 (268 MB) 54.4 -> 53.9.
// The counters must fit where the pairwise form has its packed text, D / 2 windows per 16 text tokens and per sequence: more windows over a short text, or no text at
// all, keep the fourth launch.
constexpr int64_t FOLD_ROWS = 1 << 17, FOLD_BYTES = 320 << 20;
// 16-bit rows from here on have non-temporal loads, whoever makes the means (k_token_score)
constexpr int64_t ONCE_FROM = 80 << 20;
template <typename T, bool VEC>
int run_pooled(wq_ctx* ctx, const void* vis_, const void* txt_, int B, int D, const int32_t* vis_off, const int32_t* txt_off,
               const int32_t* win_size, const int32_t* win_off, int64_t total_vis, int64_t total_txt, int64_t total_win,
               float* scores)
{
    const T* vis = static_cast<const T*>(vis_);
    const T* txt = static_cast<const T*>(txt_);
    char* ws = ctx->ws + WQ_WS_HEADER;
    float* inv_norm = reinterpret_cast<float*>(ws);
    ws += wq_align256(sizeof(float) * (size_t)(total_txt > 0 ? total_txt : 1));
    float* tbar = reinterpret_cast<float*>(ws);
    ws += wq_align256(sizeof(float) * (size_t)B * D);
    float* tok_score = reinterpret_cast<float*>(ws);
    hipStream_t st = ctx->stream;
    const int64_t text_bytes = total_txt * D * (int64_t)sizeof(T), chain = total_txt * total_win + total_vis * B, per = (int64_t)B * total_win;
    if (VEC && total_txt <= SMALL_TOKENS && total_vis <= SMALL_ROWS && total_win <= SMALL_WINDOWS && D <= SMALL_DIM && text_bytes <= SMALL_TEXT &&
        total_vis * D * (int64_t)sizeof(T) <= SMALL_BYTES &&
        chain <= (text_bytes <= SMALL_SEQ_TEXT * (B + 1) ? SMALL_CHAIN : SMALL_CHAIN_LONG) * per) {
        hipLaunchKernelGGL(k_scores_small<T>, dim3((unsigned)total_win), dim3(SMALL_THREADS), 0, st, vis, txt, D, B, vis_off, txt_off, win_size,
                           win_off, scores);
        WQ_HIP_CHECK(ctx, hipGetLastError());
        return WQ_OK;
    }
    // the windows' counters lie where the pairwise form has its packed text
    float* const counters = tok_score + wq_align256(sizeof(float) * (size_t)(total_vis > 0 ? total_vis : 1)) / sizeof(float);
    const WindowFold fold{win_size, win_off, txt_off, reinterpret_cast<unsigned*>(counters), scores};
    const int64_t row_bytes = total_vis * D * (int64_t)sizeof(T);
    const bool folds = VEC && total_vis > 0 && total_vis <= FOLD_ROWS && row_bytes <= FOLD_BYTES && total_txt > 0 &&
                       total_win * FOLD_STRIDE * (int64_t)sizeof(unsigned) <= pair_total_tiles(B, total_txt) * 16 * D * 2;
    if (total_txt > 0)
        hipLaunchKernelGGL((k_text_norm<T, VEC>), dim3((unsigned)((total_txt + 3) / 4)), dim3(256), 0, st, txt, D, total_txt, inv_norm, fold,
                           folds ? total_win : 0);
    hipLaunchKernelGGL((k_text_mean<T, VEC>), dim3(VEC ? (D + 63) / 64 : (D + 255) / 256, B), dim3(256), 0, st, txt, inv_norm, D, txt_off, tbar);
    if (total_vis > 0) {
        const int64_t rows_per_block = VEC ? 4 * WQ_TS_ROWS : 4;
        constexpr bool CAN = VEC && sizeof(T) == 2;       // (other rows have one kind of loads)
        const bool once = CAN && row_bytes >= ONCE_FROM;
        hipLaunchKernelGGL((folds ? once ? k_token_score<T, VEC, VEC, CAN> : k_token_score<T, VEC, VEC, false>
                                  : once ? k_token_score<T, VEC, false, CAN> : k_token_score<T, VEC, false, false>),
                           dim3((unsigned)((total_vis + rows_per_block - 1) / rows_per_block)), dim3(256), 0, st, vis, tbar, D, B, vis_off, total_vis,
                           tok_score, fold);
    }
    if (!folds) hipLaunchKernelGGL(k_window_mean, dim3((unsigned)((total_win + 3) / 4)), dim3(256), 0, st, tok_score, B, vis_off, txt_off,
                       win_size, win_off, total_win, scores);
    WQ_HIP_CHECK(ctx, hipGetLastError());
    return WQ_OK;
}

}  // namespace


size_t wq_scores_ws_bytes(int B, int64_t total_vis, int64_t total_txt, int D)
{
    if (B <= 0 || D <= 0) return 0;
    return wq_align256(sizeof(float) * (size_t)(total_txt > 0 ? total_txt : 1)) + wq_align256(sizeof(float) * (size_t)B * D) +
           wq_align256(sizeof(float) * (size_t)(total_vis > 0 ? total_vis : 1)) +
           wq_align256((size_t)pair_total_tiles(B, total_txt) * 16 * (size_t)D * 2);      // text in operand order (pairwise path)
}

int wq_launch_scores(wq_ctx* ctx, const void* vis, const void* txt, int dtype, int B, int D, const int32_t* vis_off,
                     const int32_t* txt_off, const int32_t* win_size, const int32_t* win_off, int64_t total_vis,
                     int64_t total_txt, int64_t total_win, int algo, float* scores)
{
    if (algo == WQ_SCORE_PAIRWISE_MFMA) {
        if (D % 128 != 0) return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "the matrix-core scoring path needs D %% 128 == 0");
        if ((reinterpret_cast<uintptr_t>(vis) | reinterpret_cast<uintptr_t>(txt)) % 16 != 0)
            return wq_fail(ctx, WQ_ERR_ARG, "embeddings must be 16-byte aligned");
        const int64_t tiles = pair_total_tiles(B, total_txt);
        if (tiles * 16 * (int64_t)D * 2 > (int64_t)UINT32_MAX)
            return wq_fail(ctx, WQ_ERR_UNSUPPORTED, "the matrix-core scoring path takes at most 4 GiB of text embeddings");
        char* ws = ctx->ws + WQ_WS_HEADER;
        float* inv_norm = reinterpret_cast<float*>(ws);
        ws += wq_align256(sizeof(float) * (size_t)(total_txt > 0 ? total_txt : 1));
        ws += wq_align256(sizeof(float) * (size_t)B * D);
        float* tok_score = reinterpret_cast<float*>(ws);
        ws += wq_align256(sizeof(float) * (size_t)(total_vis > 0 ? total_vis : 1));
        uint4* packed = reinterpret_cast<uint4*>(ws);
        hipStream_t st = ctx->stream;
        const uint16_t* v16 = static_cast<const uint16_t*>(vis);
        const uint16_t* t16 = static_cast<const uint16_t*>(txt);
        if (total_vis > 0) {
            hipLaunchKernelGGL((dtype == WQ_BF16 ? k_pack_text<true> : k_pack_text<false>), dim3((unsigned)tiles), dim3(PT_THREADS), 0, st, t16, D, B,
                               txt_off, packed, inv_norm);
            static int cus = 0;
            if (cus <= 0) {
                int dev = 0;
                if (hipGetDevice(&dev) != hipSuccess ||
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
                    cus = 256;
            }
            // one workgroup per compute unit, or fewer if there are fewer tiles of 16 rows (a sequence has at most one partial one)
            const int64_t tiles_most = (total_vis + 15) / 16 + B;
            const dim3 grid((unsigned)(tiles_most < cus ? tiles_most : cus));
            if (dtype == WQ_BF16)
                hipLaunchKernelGGL(k_pair_mfma<true>, grid, dim3(PA_THREADS), 0, st, v16, packed, inv_norm, D, B, vis_off, txt_off, tok_score);
            else
                hipLaunchKernelGGL(k_pair_mfma<false>, grid, dim3(PA_THREADS), 0, st, v16, packed, inv_norm, D, B, vis_off, txt_off, tok_score);
        }
        hipLaunchKernelGGL(k_window_mean, dim3((unsigned)((total_win + 3) / 4)), dim3(256), 0, st, tok_score, B, vis_off, txt_off,
                           win_size, win_off, total_win, scores);
        WQ_HIP_CHECK(ctx, hipGetLastError());
        return WQ_OK;
    }
    // 16-byte row pieces need D % 8 == 0 and 16-byte aligned bases (rows then stay aligned for every element type)
    const bool vec = D % 8 == 0 && (reinterpret_cast<uintptr_t>(vis) | reinterpret_cast<uintptr_t>(txt)) % 16 == 0;
#define WQ_RUN(T)                                                                                                         \
    (vec ? run_pooled<T, true>(ctx, vis, txt, B, D, vis_off, txt_off, win_size, win_off, total_vis, total_txt, total_win, scores) \
         : run_pooled<T, false>(ctx, vis, txt, B, D, vis_off, txt_off, win_size, win_off, total_vis, total_txt, total_win, scores))
    switch (dtype) {
        case WQ_F32: return WQ_RUN(float);
        case WQ_BF16: return WQ_RUN(__hip_bfloat16);
        default: return WQ_RUN(__half);
    }
#undef WQ_RUN
}
