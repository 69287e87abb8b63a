// Fused log-softmax + cumulative score + top-k beam selection.
//
// At level t the search keeps the b_t best of the n_t*V_t candidates
// score(i,v) = c_i + log_softmax(z_i)[v] of a request (section 3.2 beam search,
// section 4.2 Dynamic Beam Width).  The selection is two-stage, as TopK Pre-Cut
// (appendix A.2) describes: every beam row first keeps its own min(b_t, V_t)
// best tokens, then the request keeps the b_t best of those.  Both stages are
// exact selections, so the result equals a full sort of all candidates.
// The per-row cut is tightened by a bound per request: b_t candidates that are known
// to exist put a floor under the survivors.  The first R rows hold the best beams, and
// their ceil(b_t / R) best candidates each are b_t candidates, so nothing below the worst
// of those can survive; the tightest of R = 1, 2, 4, ... is used (one row where the beams'
// scores fall off steeply, many where they are level).  All rows write only what
// reaches that bound (at most their own cut), compacted per request.
//
// Candidates travel between the stages as unique 64-bit keys
//     (order-preserving bits of the fp32 score) << 32 | (0xFFFFFFFF - flat index)
// so "larger key" means "higher score, then lower flat index i*V + v": equal
// scores resolve deterministically and the final order is a plain key sort.
#include <stdlib.h>

#include <type_traits>

#include "common.h"

// The running candidate count of a request sits on a cache line of its own where there is room (select_plan): the rows of all requests
// count at once, and atomics on one line are served one after the other, about 20 ns each.  Measured: 64 requests of 256 rows of 4096
// half-precision logits, 157 us with the counts side by side, 40 us apart.
#define COUNT_PITCH_MAX 32
#define BOUND_ROWS_MAX 32  // rows per request that go into its bound

__device__ __forceinline__ uint32_t score_key(float f) {
    f += 0.0f;  // -0 -> +0 so equal scores have equal keys
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t k) {
    uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}
#define LAST_KEY 0x003FFFFFu  // score_key of the NaN that ranks below all numbers

// inclusive scan over a 256-thread block (4 wavefronts)
__device__ __forceinline__ int block_scan_256(int v, int *wave_tot /*[4] LDS*/) {
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    if (lane == 63) wave_tot[wv] = v;
    __syncthreads();
    int add = 0;
    for (int w = 0; w < wv; w++) add += wave_tot[w];
    __syncthreads();
    return v + add;
}

// ---------------------------------------------------------------------------
// stage A: one workgroup per beam row
// ---------------------------------------------------------------------------
// The row (V logits) is read once and stays in registers: ITEMS values per thread,
// token v = j*256 + tid.  After the log-sum-exp, the row's min(b_t, V_t) best scores
// are cut out with about two dozen vector operations per logit, so the kernel stays
// bound by the HBM read of the logits:
//   1. a histogram of the scores over ROW_BINS equal-width bins between the row's
//      minimum and maximum (LDS atomics, spread over the bins by the values themselves),
//   2. a scan from the top bin finds the bin T that holds the m-th best score,
//   3. everything above bin T is a candidate; the few scores inside bin T are ranked
//      exactly against each other (64-bit keys, so ties go to the lowest token).
// If bin T is crowded (degenerate rows, e.g. all logits equal) the row falls back to an
// exact radix selection on the score keys that walks two bits at a time and only counts.
#define ROW_BINS 1024
#define ROW_LIST 1024

struct RowShared {
    float f[3][4];
    uint32_t u[2][4][2];
    int wave_tot[4];
    int scan_base, out_gt, out_eq, sel_bin, sel_krem, sel_cnt, list_n;
    int hist[ROW_BINS + 64];  // (past the bins: one place per lane for what is not counted)
    unsigned long long list[ROW_LIST];
};

__device__ __forceinline__ float block_max_256(float v, RowShared &sh, int slot) {
    v = wave_max(v);
    if (threadIdx.x % 64 == 0) sh.f[slot][threadIdx.x / 64] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh.f[slot][0], sh.f[slot][1]), fmaxf(sh.f[slot][2], sh.f[slot][3]));
}
__device__ __forceinline__ float block_sum_256(float v, RowShared &sh, int slot) {
    v = wave_sum(v);
    if (threadIdx.x % 64 == 0) sh.f[slot][threadIdx.x / 64] = v;
    __syncthreads();
    return (sh.f[slot][0] + sh.f[slot][1]) + (sh.f[slot][2] + sh.f[slot][3]);
}

// Every score of the row is a number.  False: a NaN or +inf logit or nothing but -inf (the log-sum-exp is no number then), or a cumulative
// score of NaN or +inf.  NaN passes no comparison, so such a row takes no part in the bounded pass; see select_rows_wave.
__device__ __forceinline__ bool row_is_numbers(float c, float lse) { return fabsf(lse) < INFINITY && c < INFINITY; }

// The sum whose NaN is a's where both are NaN.  Candidates rank by the bits of their scores, a NaN above or below all numbers by its sign, and a row's cumulative score and its
// log-softmax may be NaN of either sign: kernels that promise each other the same bits cannot leave the order to the compiler.
__device__ __forceinline__ float sum_a_first(float a, float b) {
    float r;
    asm("v_add_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// Score of a token in the wavefront kernels: NaN of the log-softmax first for rows of up to 2048 tokens, of the cumulative score for longer ones
template <bool SHORT> __device__ __forceinline__ float wave_score(float c, float log_p) { return SHORT ? sum_a_first(log_p, c) : sum_a_first(c, log_p); }

__device__ __forceinline__ unsigned long long pack_candidate(float score, uint32_t flat) {
    return ((unsigned long long)score_key(score) << 32) | (0xFFFFFFFFu - flat);
}

// Exact fallback: radix selection on the order-preserving keys of the scores held in
// sc[] (padding slots hold -inf and are skipped by the v < V test).
template <int ITEMS>
__device__ __noinline__ void select_row_radix(const float (&sc)[ITEMS], int V, int m, uint32_t flat0, unsigned long long *dst,
                                              RowShared &sh) {
    const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
    uint32_t k_and = 0xFFFFFFFFu, k_or = 0u;
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        if (j * 256 + tid < V) { const uint32_t k = score_key(sc[j]); k_and &= k; k_or |= k; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        k_and &= __shfl_xor(k_and, o, 64);
        k_or |= __shfl_xor(k_or, o, 64);
    }
    __syncthreads();
    if (lane == 0) { sh.u[0][wv][0] = k_and; sh.u[0][wv][1] = k_or; }
    if (tid == 0) { sh.out_gt = 0; sh.out_eq = 0; }
    __syncthreads();
    k_and = sh.u[0][0][0] & sh.u[0][1][0] & sh.u[0][2][0] & sh.u[0][3][0];
    k_or = sh.u[0][0][1] | sh.u[0][1][1] | sh.u[0][2][1] | sh.u[0][3][1];
    // decided: bits already fixed in `prefix`; a key is still active while (key & decided) == prefix
    const uint32_t diff = k_and ^ k_or;
    uint32_t decided = 0xFFFFFFFFu, prefix = k_and;
    int krem = m, active = V;
    if (diff != 0) {
        const int top = 31 - __clz(diff);
        decided = ~((2u << top) - 1u);  // top == 31 gives 0
        prefix = k_and & decided;
        int slot = 1;
        for (int shb = top & ~1; shb >= 0; shb -= 2) {
            uint32_t c12 = 0, c3 = 0;  // active keys with digit >= 1 (low half), >= 2 (high half), >= 3
#pragma unroll
            for (int j = 0; j < ITEMS; j++) {
                const uint32_t k = score_key(sc[j]);
                const uint32_t d = (k >> shb) & 3u;
                const uint32_t act = (((k ^ prefix) & decided) == 0u && (j * 256 + tid) < V) ? 1u : 0u;
                c12 += (d >= 1u ? act : 0u) + (d >= 2u ? (act << 16) : 0u);
                c3 += d >= 3u ? act : 0u;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                c12 += __shfl_xor(c12, o, 64);
                c3 += __shfl_xor(c3, o, 64);
            }
            if (lane == 0) { sh.u[slot][wv][0] = c12; sh.u[slot][wv][1] = c3; }
            __syncthreads();
            c12 = sh.u[slot][0][0] + sh.u[slot][1][0] + sh.u[slot][2][0] + sh.u[slot][3][0];
            c3 = sh.u[slot][0][1] + sh.u[slot][1][1] + sh.u[slot][2][1] + sh.u[slot][3][1];
            slot ^= 1;  // the next step writes the other slot, so one barrier per step is enough
            const int C1 = (int)(c12 & 0xFFFFu), C2 = (int)(c12 >> 16), C3 = (int)c3;
            uint32_t dsel;
            if (C3 >= krem) { dsel = 3; active = C3; }
            else if (C2 >= krem) { dsel = 2; krem -= C3; active = C2 - C3; }
            else if (C1 >= krem) { dsel = 1; krem -= C2; active = C1 - C2; }
            else { dsel = 0; krem -= C1; active = active - C1; }
            prefix |= dsel << shb;
            decided |= 3u << shb;
            if (active == krem) break;  // every key still active is taken
        }
    }
    // (key & decided) > prefix: above the threshold; == prefix: `active` keys tie at it, krem of them are taken
    const int n_gt = m - krem;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    if (active == krem) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            const int v = j * 256 + tid;
            const uint32_t kk = score_key(sc[j]) & decided;
            const bool gt = v < V && kk > prefix, eq = v < V && kk == prefix;
            const unsigned long long mg = __ballot(gt), me = __ballot(eq);
            int bg = 0, be = 0;
            if (lane == 0) {
                if (mg) bg = atomicAdd(&sh.out_gt, __popcll(mg));
                if (me) be = atomicAdd(&sh.out_eq, __popcll(me));
            }
            bg = __shfl(bg, 0, 64);
            be = __shfl(be, 0, 64);
            if (gt) dst[bg + __popcll(mg & lt_mask)] = pack_candidate(sc[j], flat0 + (uint32_t)v);
            if (eq) dst[n_gt + be + __popcll(me & lt_mask)] = pack_candidate(sc[j], flat0 + (uint32_t)v);
        }
    } else {
        // more keys tie at the threshold than are needed: take the lowest tokens, in token order
        int base = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            const int v = j * 256 + tid;
            const uint32_t kk = score_key(sc[j]) & decided;
            const bool gt = v < V && kk > prefix;
            const int flag = (v < V && kk == prefix) ? 1 : 0;
            const int incl = block_scan_256(flag, sh.wave_tot);
            if (gt) dst[atomicAdd(&sh.out_gt, 1)] = pack_candidate(sc[j], flat0 + (uint32_t)v);
            const int rank = base + incl - flag;
            if (flag && rank < krem) dst[n_gt + rank] = pack_candidate(sc[j], flat0 + (uint32_t)v);
            if (tid == 255) sh.scan_base = base + incl;
            __syncthreads();
            base = sh.scan_base;
            __syncthreads();
        }
    }
}

template <int ITEMS>
__global__ __launch_bounds__(256) void select_rows(const float *__restrict__ logits, const float *__restrict__ cum, int n, int V, int m,
                                                   unsigned long long *__restrict__ cand) {
    __shared__ RowShared sh;
    extern __shared__ unsigned long long out_stage[];  // m candidates, gathered here and written out in one coalesced sweep
    const int tid = threadIdx.x;
    const int64_t row = blockIdx.x;
    const float *z = logits + row * (int64_t)V;
    const float c = cum ? cum[row] : 0.0f;
    for (int i = tid; i < ROW_BINS; i += 256) sh.hist[i] = 0;
    if (tid == 0) { sh.out_gt = 0; sh.list_n = 0; }

    float x[ITEMS];
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int v = j * 256 + tid;
        x[j] = v < V ? z[v] : -INFINITY;
        mx = fmaxf(mx, x[j]);
        if (v < V) mn = fminf(mn, x[j]);
    }
    mx = block_max_256(mx, sh, 0);
    mn = -block_max_256(-mn, sh, 1);
    float sum = 0.0f;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) sum += __expf(x[j] - mx);  // exp(-inf) = 0 for the padding
    const float lse = mx + __logf(block_sum_256(sum, sh, 2));
#pragma unroll
    for (int j = 0; j < ITEMS; j++) x[j] = sum_a_first(c, x[j] - lse);  // scores from here on (padding stays -inf)

    unsigned long long *dst = cand + row * (int64_t)m;
    const uint32_t flat0 = (uint32_t)((row % n) * (int64_t)V);
    if (m >= V) {  // nothing to cut: every token is a candidate
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            const int v = j * 256 + tid;
            if (v < V) dst[v] = pack_candidate(x[j], flat0 + (uint32_t)v);
        }
        return;
    }
    // 1. histogram over equal-width bins of [lo, hi]; the bin index is monotone in the score
    const float lo = c + (mn - lse), hi = c + (mx - lse);
    const float inv_w = (hi > lo) ? (float)ROW_BINS / (hi - lo) : 0.0f;
    int bin[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        int bi = (int)((x[j] - lo) * inv_w);
        bi = bi < 0 ? 0 : (bi > ROW_BINS - 1 ? ROW_BINS - 1 : bi);
        bin[j] = bi;
        if (j * 256 + tid < V) atomicAdd(&sh.hist[bi], 1);
    }
    __syncthreads();
    // 2. thread t owns bins 1023-4t .. 1020-4t; inclusive scan from the top bin down
    {
        const int b0 = ROW_BINS - 1 - 4 * tid;
        const int h0 = sh.hist[b0], h1 = sh.hist[b0 - 1], h2 = sh.hist[b0 - 2], h3 = sh.hist[b0 - 3];
        const int incl = block_scan_256(h0 + h1 + h2 + h3, sh.wave_tot);
        int above = incl - (h0 + h1 + h2 + h3);  // scores in bins above this thread's four
        if (above < m && incl >= m) {
            int bsel = b0, cnt = h0;
            if (above + h0 < m) { above += h0; bsel = b0 - 1; cnt = h1;
                if (above + h1 < m) { above += h1; bsel = b0 - 2; cnt = h2;
                    if (above + h2 < m) { above += h2; bsel = b0 - 3; cnt = h3; } } }
            sh.sel_bin = bsel;
            sh.sel_krem = m - above;
            sh.sel_cnt = cnt;
        }
    }
    __syncthreads();
    const int T = sh.sel_bin, krem = sh.sel_krem, cntT = sh.sel_cnt;
    if (cntT > ROW_LIST) {  // crowded threshold bin: exact radix selection over the whole row
        float sc[ITEMS];  // a copy, so that only this branch keeps the scores in addressable memory
#pragma unroll
        for (int j = 0; j < ITEMS; j++) sc[j] = x[j];
        select_row_radix<ITEMS>(sc, V, m, flat0, dst, sh);
        return;
    }
    // 3. bins above T are candidates; bin T goes to the list for exact ranking.  One scan of the
    //    per-thread counts (low half: above T, high half: inside T) gives every thread its slots.
    const int n_gt = m - krem;
    int mine = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const bool ok = j * 256 + tid < V;
        mine += (ok && bin[j] > T ? 1 : 0) + (ok && bin[j] == T ? (1 << 16) : 0);
    }
    const int incl = block_scan_256(mine, sh.wave_tot);
    int pos_gt = (incl - mine) & 0xFFFF, pos_eq = (incl - mine) >> 16;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) {
        const int v = j * 256 + tid;
        if (v < V && bin[j] > T) out_stage[pos_gt++] = pack_candidate(x[j], flat0 + (uint32_t)v);
        if (v < V && bin[j] == T) sh.list[pos_eq++] = pack_candidate(x[j], flat0 + (uint32_t)v);
    }
    __syncthreads();
    // rank every listed candidate among the cntT listed ones; the krem best go out
    for (int i = tid; i < cntT; i += 256) {
        const unsigned long long mine = sh.list[i];
        int rank = 0;
        for (int q = 0; q < cntT; q++) rank += sh.list[q] > mine ? 1 : 0;
        if (rank < krem) out_stage[n_gt + rank] = mine;
    }
    __syncthreads();
    for (int i = tid; i < m; i += 256) dst[i] = out_stage[i];
}

template <typename LT> struct LogitPiece;  // one 16-byte piece of a row of logits as floats
template <> struct LogitPiece<float> {
    static constexpr int E = 4;
    static __device__ __forceinline__ void unpack(const uint4 &r, float *o) {
        o[0] = __uint_as_float(r.x); o[1] = __uint_as_float(r.y); o[2] = __uint_as_float(r.z); o[3] = __uint_as_float(r.w);
    }
};
template <> struct LogitPiece<_Float16> {
    static constexpr int E = 8;
    static __device__ __forceinline__ void unpack(const uint4 &r, float *o) {
        const halfx8 v = __builtin_bit_cast(halfx8, r);
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = (float)v[e];
    }
};

// ---------------------------------------------------------------------------
// request bounds
// ---------------------------------------------------------------------------
// One workgroup per row r < R of a request (R a power of two): the scores below which the row has its ceil(m / Q) best candidates, for every
// power of two Q in (r, R], go to rb[b * 2R + Q + r].  A bound may lie below the exact value (that only lets a few more candidates
// through), so a histogram of the logits is enough: the lower edge of the bin that holds the ranked value, a margin above the error of
// bin and log-sum-exp (the sweep computes its own).  Q = 1 is ranked exactly inside its bin and its logit kept too (slot 0 of the
// request): the first row takes the threshold from that, since the margin would let it over its m slots now and then.
// Masked tokens must not cost the request its bound: -inf stays out of the histogram (a row with fewer numbers than a rank has no bound
// there), and where finite masks (-1e4, -65504) press the others into the top bins, the histogram is taken again over those bins alone, at
// most twice (masks of two magnitudes).  64 requests of 128 float32 rows of 4096 of which 1024 are not masked, level scores, k = 512: 55 us
// masked with -inf and 60 with -1e4, as against 560 and 350 with bounds lost to the masks; 55 without a mask.
template <int ITEMS, typename LT>
__global__ __launch_bounds__(256) void row_bounds(const LT *__restrict__ logits, const float *__restrict__ cum, int n, int V, int m, int R,
                                                  float *__restrict__ rb, int *__restrict__ req_count, int count_pitch, int *__restrict__ todo_count) {
    __shared__ RowShared sh;
    const int tid = threadIdx.x, r = blockIdx.x % R;
    const int64_t b = blockIdx.x / R, row = b * n + r;
    if (blockIdx.x == 0 && tid == 0) *todo_count = 0;
    if (r == 0 && tid == 0) req_count[b * count_pitch] = 0;
    for (int i = tid; i < ROW_BINS; i += 256) sh.hist[i] = 0;
    if (tid == 0) sh.list_n = 0;
    const uint4 *z = (const uint4 *)(logits + row * (int64_t)V);
    constexpr int E = LogitPiece<LT>::E, G = ITEMS / E;
    float x[ITEMS];
    float mx = -INFINITY, lo = INFINITY;
#pragma unroll
    for (int g = 0; g < G; g++) {
        const bool ok = (g * 256 + tid) * E < V;  // V % E == 0
        if (ok) LogitPiece<LT>::unpack(z[g * 256 + tid], &x[g * E]);
#pragma unroll
        for (int e = 0; e < E; e++) {
            if (!ok) x[g * E + e] = -INFINITY;
            mx = fmaxf(mx, x[g * E + e]);
            if (x[g * E + e] > -INFINITY) lo = fminf(lo, x[g * E + e]);
        }
    }
    mx = block_max_256(mx, sh, 0);
    lo = -block_max_256(-lo, sh, 1);
    float sum = 0.0f;
#pragma unroll
    for (int j = 0; j < ITEMS; j++) sum += __expf(x[j] - mx);
    const float lse = mx + __logf(block_sum_256(sum, sh, 2));
    const float c = cum ? cum[row] : 0.0f;
    if (!row_is_numbers(c, lse)) {  // bounds nothing
        if (tid == 0) {
            for (int Q = 1; Q <= R; Q <<= 1)
                if (Q > r) rb[b * (2 * R) + Q + r] = -INFINITY;
            if (r == 0) rb[b * (2 * R)] = -INFINITY;
        }
        return;
    }
    // (from here on the logits are numbers or -inf, and some are numbers)
    auto rank_of = [&](int q) { return (m + (1 << q) - 1) >> q; };  // ceil(m / Q), Q = 1 << q
    const int q0 = 32 - __clz(r), rank_max = rank_of(q0);           // the smallest Q above r: the row's lowest rank
    const int b0 = ROW_BINS - 1 - 4 * tid;  // thread t owns bins 1023-4t .. 1020-4t
    float inv_w;
    int h[4], incl, excl;
    // (-1 a bin or more below lo; bin 0 reaches a bin below lo, which is of no harm to ranks at or above lo)
    auto bin_of = [&](float v) { return (int)__builtin_amdgcn_fmed3f((v - lo) * inv_w, -1.0f, (float)(ROW_BINS - 1)); };
    auto find = [&](int rank, int &above, int &cnt) {  // the bin of a rank in (excl, incl], how many values lie above it and in it
        int at = 0;
        above = excl;
        cnt = h[0];
#pragma unroll
        for (int i = 0; i < 3; i++)
            if (at == i && above + h[i] < rank) { above += h[i]; cnt = h[i + 1]; at = i + 1; }
        return b0 - at;
    };
    for (int pass = 0;; pass++) {
        inv_w = mx > lo && mx - lo < INFINITY ? (float)ROW_BINS / (mx - lo) : 0.0f;
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            const int bin = bin_of(x[j]);
            atomicAdd(&sh.hist[bin >= 0 ? bin : ROW_BINS + tid % 64], 1);
        }
        if (tid == 0) sh.sel_bin = -1;
        __syncthreads();
        // inclusive scan from the top bin down
#pragma unroll
        for (int i = 0; i < 4; i++) h[i] = sh.hist[b0 - i];
        incl = block_scan_256(h[0] + h[1] + h[2] + h[3], sh.wave_tot);
        excl = incl - (h[0] + h[1] + h[2] + h[3]);
        if (excl < rank_max && incl >= rank_max) {
            int above, cnt;
            sh.sel_bin = find(rank_max, above, cnt);
            sh.sel_krem = rank_max - above;
            sh.sel_cnt = cnt;
        }
        __syncthreads();
        const int T = sh.sel_bin, cnt = sh.sel_cnt;
        // (a rank in the top 16 of 1024 bins: they say little about the ranked values)
        if (pass == 2 || T < 0 || !(inv_w > 0.0f) || !(cnt > ROW_LIST || (cnt > 8 && T >= ROW_BINS - 16))) break;
        float from = INFINITY;
#pragma unroll
        for (int j = 0; j < ITEMS; j++)
            if (bin_of(x[j]) >= T) from = fminf(from, x[j]);
        from = -block_max_256(-from, sh, 1);
        if (from == lo) break;
        lo = from;
        for (int i = tid; i < ROW_BINS; i += 256) sh.hist[i] = 0;
        __syncthreads();
    }
    auto put = [&](int Q, float v) {
        const float sc = c + (v - lse), low = sc - (1e-5f + 4e-7f * (fabsf(c) + fabsf(v) + fabsf(lse)));
        rb[b * (2 * R) + Q + r] = low == low ? low : -INFINITY;
    };
    // the value at the lower edge of a bin
    auto edge = [&](int bin) { return inv_w > 0.0f ? lo + ((float)bin - 0.01f) / inv_w : lo; };
    for (int q = q0; (1 << q) <= R; q++) {
        const int rank = rank_of(q);
        int above, cnt;
        if (q > 0 && excl < rank && incl >= rank) put(1 << q, edge(find(rank, above, cnt)));
        if (tid == 255 && incl < rank) put(1 << q, -INFINITY);  // fewer numbers than that
    }
    if (r != 0) return;
    const int T = sh.sel_bin, krem = sh.sel_krem, cnt = sh.sel_cnt;
    if (T < 0 || cnt > ROW_LIST || !(inv_w > 0.0f)) {  // no such rank, or a crowded bin (degenerate rows): its edge will do
        if (tid == 0) {
            if (T >= 0) put(1, edge(T));
            rb[b * (2 * R)] = -INFINITY;
        }
        return;
    }
    float *list = (float *)sh.list;
#pragma unroll
    for (int j = 0; j < ITEMS; j++)
        if (bin_of(x[j]) == T) list[atomicAdd(&sh.list_n, 1)] = x[j];
    __syncthreads();
    for (int i = tid; i < cnt; i += 256) {
        const float v = list[i];
        int gt = 0, ge = 0;
        for (int q = 0; q < cnt; q++) { gt += list[q] > v ? 1 : 0; ge += list[q] >= v ? 1 : 0; }
        if (gt < krem && ge >= krem) {  // (equal values write the same)
            put(1, v);
            rb[b * (2 * R)] = v;
        }
    }
}

// The request's bound by one wavefront, v: slot `lane` of the request's scores (anything past them).  Slots [Q, 2Q) hold the rows of
// Q, an aligned group of lanes: the minimum of every group, then the best group.
__device__ __forceinline__ float request_bound(float v, int R, int lane) {
#pragma unroll
    for (int s = 1; s < BOUND_ROWS_MAX; s <<= 1) {
        const float o = __shfl_xor(v, s, 64);
        if (lane >= 2 * s) v = fminf(v, o);
    }
    return wave_max_dpp(lane >= 1 && lane < 2 * R ? v : -INFINITY);
}
// the same for the request's first row, whose own m-th best logit x0 (slot 0) is known
__device__ __forceinline__ float first_row_bound(float x0, float bound, float c, float lse) { return fmaxf(bound, c + (x0 - lse)); }

// ---------------------------------------------------------------------------
// stage A, wavefront form: one wavefront per beam row (V <= 8192)
// ---------------------------------------------------------------------------
// Same cut as select_rows, but a row never leaves one wavefront: no workgroup barrier anywhere, the V logits sit in VEC*4
// registers per lane, read as 16-byte pieces of E = 4 float32 or E = 8 half-precision values (lane l, piece g holds tokens
// (g*64 + l)*E .. +E-1; V % E == 0), every reduction is a wave reduction, and the histogram, the threshold-bin list and the
// staged output live in a private LDS region per wavefront.  The kernel is bound by vector instructions per logit, so the
// common case, select_rows_sweep, is kept to a maximum, one exp2 and one comparison per logit: with a request-level bound in
// force the row is swept in the logit domain against a threshold a hair below the exact one, and only the few logits that pass it
// are turned into scores and tested exactly.  Rows that need their own cut (select_rows_wave: more than m candidates at the bound,
// or no bound) turn all logits into scores, histogram them and rank the threshold bin exactly; score bits are staged raw and
// turned into sortable keys only for the survivors on the way out.
#define WROW_BINS 1024
#define WROW_LIST 512  // threshold-bin candidates ranked exactly; the list reuses the histogram's 4 KB
#define WROW_SLOTS 544  // 8-byte slots of a wavefront's histogram with the 64 places in front (list), before the staged output
#define WROW_FEW 64    // up to here at once (each lane reads the whole list: 230 candidates took 50 us)

// (pointers that say they are into LDS: functions of their own would take generic ones, whose offsets the compiler may fold so that the address in the registers lies below the
// memory's window, where the hardware finds the window by that address alone)
typedef __attribute__((address_space(3))) unsigned long long LdsKey;
typedef __attribute__((address_space(3))) int LdsInt;
typedef __attribute__((address_space(3))) intx4 LdsInt4;

__device__ __forceinline__ unsigned long long staged_to_key(unsigned long long st) {
    return ((unsigned long long)score_key(__uint_as_float((uint32_t)(st >> 32))) << 32) | (st & 0xFFFFFFFFull);
}

// token held in register i of a lane: piece i / E of the lane, element i % E of the piece
template <int E> __device__ __forceinline__ int wave_tok(int i, int lane) { return ((i / E) * 64 + lane) * E + (i % E); }
// whether it is one of the row's: V % E == 0, so a piece is in or out as a whole.  (One mask to a piece: a mask to a token, kept over the rows, filled the scalar registers and was put away in
// vector registers before the first row, and a wavefront often has only one: 36 to 206 of them, now 16 to 72.)
template <int E> __device__ __forceinline__ bool wave_has(int i, int lane, int V) { return ((i / E) * 64 + lane) * E < V; }

// exact fallback on the registers of one wavefront: radix selection on the score keys, two bits per step (ALONE: a function for each kernel that calls
// it, or all of them get the registers of the one with the most)
template <int VEC, int E, bool ALONE>
__device__ __noinline__ void select_row_radix_wave(const float (&sc)[VEC * 4], int V, int m, uint32_t flat0, LdsKey *stage, bool tied, uint32_t tie,
                                                   int tie_krem) {
    const int lane = threadIdx.x % 64;
    uint32_t k_and = 0xFFFFFFFFu, k_or = 0u;
#pragma unroll
    for (int i = 0; i < VEC * 4; i++)
        if (wave_has<E>(i, lane, V)) { const uint32_t k = score_key(sc[i]); k_and &= k; k_or |= k; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { k_and &= __shfl_xor(k_and, o, 64); k_or |= __shfl_xor(k_or, o, 64); }
    const uint32_t diff = k_and ^ k_or;
    uint32_t decided = 0xFFFFFFFFu, prefix = k_and;
    int krem = m, active = V;
    if (tied) {  // the threshold is known: tie_krem of the scores equal to `tie` are taken, all above them
        prefix = tie;
        krem = tie_krem;
    } else if (diff != 0) {
        const int top = 31 - __clz(diff);
        decided = ~((2u << top) - 1u);  // top == 31 gives 0
        prefix = k_and & decided;
        for (int shb = top & ~1; shb >= 0; shb -= 2) {
            uint32_t c12 = 0, c3 = 0;  // active keys with digit >= 1 (low half), >= 2 (high half), >= 3
#pragma unroll
            for (int i = 0; i < VEC * 4; i++) {
                const uint32_t k = score_key(sc[i]);
                const uint32_t d = (k >> shb) & 3u;
                const uint32_t act = (((k ^ prefix) & decided) == 0u && wave_has<E>(i, lane, V)) ? 1u : 0u;
                c12 += (d >= 1u ? act : 0u) + (d >= 2u ? (act << 16) : 0u);
                c3 += d >= 3u ? act : 0u;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) { c12 += __shfl_xor(c12, o, 64); c3 += __shfl_xor(c3, o, 64); }
            const int C1 = (int)(c12 & 0xFFFFu), C2 = (int)(c12 >> 16), C3 = (int)c3;
            uint32_t dsel;
            if (C3 >= krem) { dsel = 3; active = C3; }
            else if (C2 >= krem) { dsel = 2; krem -= C3; active = C2 - C3; }
            else if (C1 >= krem) { dsel = 1; krem -= C2; active = C1 - C2; }
            else { dsel = 0; krem -= C1; active = active - C1; }
            prefix |= dsel << shb;
            decided |= 3u << shb;
            if (active == krem) break;  // every key still active is taken
        }
    }
    // (key & decided) > prefix: above the threshold; == prefix: `active` keys tie there and the krem lowest tokens are taken.
    // Tokens ascend with (piece, lane, element), so a tie's rank is the count of ties in earlier pieces, in lower lanes of
    // this piece, and in lower elements.
    const int n_gt = m - krem;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    int base_gt = 0, base_eq = 0;
#pragma unroll
    for (int g = 0; g < VEC * 4 / E; g++) {
        int my_eq = 0;
        bool gt[E], eq[E];
#pragma unroll
        for (int e = 0; e < E; e++) {
            const bool ok = (g * 64 + lane) * E < V;
            const uint32_t kk = score_key(sc[g * E + e]) & decided;
            gt[e] = ok && kk > prefix;
            eq[e] = ok && kk == prefix;
            my_eq += eq[e] ? 1 : 0;
        }
        int incl = my_eq;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (lane >= o) incl += t; }
        int rank = base_eq + incl - my_eq;
        base_eq += __shfl(incl, 63, 64);
#pragma unroll
        for (int e = 0; e < E; e++) {
            const unsigned long long mg = __ballot(gt[e]);
            const uint32_t flat = flat0 + (uint32_t)((g * 64 + lane) * E + e);
            const unsigned long long st = ((unsigned long long)__float_as_uint(sc[g * E + e] + 0.0f) << 32) | (0xFFFFFFFFu - flat);
            if (gt[e]) stage[base_gt + __popcll(mg & lt_mask)] = st;
            base_gt += __popcll(mg);
            if (eq[e]) { if (rank < krem) stage[n_gt + rank] = st; rank++; }
        }
    }
}

// The scores' bins, monotone in the score: WROW_LOW and up to WROW_BINS - 1 more; what lies below them all is in bin WROW_LOW - 1.
#define WROW_LOW 64
__device__ __forceinline__ uint32_t mid_u(uint32_t v, uint32_t lo, uint32_t hi) { return min(max(v, lo), hi); }
__device__ __forceinline__ int score_bin(float x, float inv_w, float k0) {
    return (int)mid_u((uint32_t)__builtin_fmaf(x, inv_w, k0), WROW_LOW - 1, WROW_LOW + WROW_BINS - 1);  // negative and NaN convert to 0
}
// The bin T of the m-th best score, by one wavefront: krem of its cnt scores are among the m best.  Scores below the bins are counted in a place per lane in front of them and are what
// the bins leave of the row's V (masked tokens in one bin would be served one after the other: 64 x 64 rows of 1024 half-precision logits, 70 % of them masked, 25.2 us a selection, now 17.6).
struct RowCut { int T, krem, cnt; };
template <int VEC, bool FULL, int E>
__device__ __forceinline__ RowCut find_cut(const float (&x)[VEC * 4], float inv_w, float k0, int V, int m, LdsInt *hist, int lane) {
#pragma unroll
    for (int i = 0; i < WROW_BINS / 256; i++) ((LdsInt4 *)(hist + WROW_LOW))[i * 64 + lane] = (intx4){0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < VEC * 4; i++) {
        const uint32_t at = mid_u((uint32_t)__builtin_fmaf(x[i], inv_w, k0), (uint32_t)lane, WROW_LOW + WROW_BINS - 1);
        if (FULL || wave_has<E>(i, lane, V)) __hip_atomic_fetch_add(&hist[at], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // lane l owns the bins 1023-16l .. 1008-16l; inclusive scan from the top bin down
    const LdsInt *own = hist + WROW_LOW + WROW_BINS - 16 - 16 * lane;
    int h[16];
#pragma unroll
    for (int i = 0; i < 4; i++) { const intx4 t = ((const LdsInt4 *)own)[i]; h[4 * i] = t[0]; h[4 * i + 1] = t[1]; h[4 * i + 2] = t[2]; h[4 * i + 3] = t[3]; }
    int mine = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) mine += h[i];
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (lane >= o) incl += t; }
    int above = incl - mine, selT = WROW_LOW - 1, selK = m - incl, selC = 0;
    const bool owner = above < m && incl >= m;
    if (owner) {
#pragma unroll
        for (int i = 15; i >= 0; i--) {  // h[15] is this lane's top bin
            if (selC == 0 && above + h[i] >= m) { selT = WROW_LOW + WROW_BINS - 16 - 16 * lane + i; selK = m - above; selC = h[i]; }
            if (selC == 0) above += h[i];
        }
    } else {
        selC = V - incl;
    }
    const unsigned long long owners = __ballot(owner);
    const int src_lane = owners ? __ffsll((long long)owners) - 1 : 63;  // (nobody's: below the bins, as lane 63 has it)
    return {__shfl(selT, src_lane, 64), __shfl(selK, src_lane, 64), __shfl(selC, src_lane, 64)};
}
// bins above the cut's go straight to the staged output, its bin to the list (over the dead histogram) for exact ranking
template <int VEC, bool FULL, int E>
__device__ __forceinline__ void stage_cut(const float (&x)[VEC * 4], const RowCut &cut, float inv_w, float k0, uint32_t nflat, int V, int m, LdsKey *list,
                                          LdsKey *stage, int lane) {
    const int n_gt = m - cut.krem;
    int base_gt = 0, base_eq = 0;
    // The bins are recomputed, not kept: opaque copies of the two constants stop the compiler from holding
    // all bin indices of the histogram pass in registers until here.
    float inv_w2 = inv_w, k02 = k0;
    asm volatile("" : "+v"(inv_w2), "+v"(k02));
#pragma unroll
    for (int i = 0; i < VEC * 4; i++) {
        const int bi = score_bin(x[i], inv_w2, k02);
        const bool ok = FULL || wave_has<E>(i, lane, V);
        const bool gt = ok && bi > cut.T, eq = ok && bi == cut.T;
        const unsigned long long mg = __ballot(gt), me = __ballot(eq);
        const unsigned long long st = ((unsigned long long)__float_as_uint(x[i] + 0.0f) << 32) | (nflat - (uint32_t)((i / E) * 64 * E + (i % E)));
        if (gt) stage[base_gt + __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0))] = st;
        base_gt += __popcll(mg);
        if (me != 0) {
            if (eq) list[base_eq + __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0))] = st;
            base_eq += __popcll(me);
        }
    }
    // rank every listed candidate among the listed ones; the krem best go out
    for (int i = lane; i < cut.cnt; i += 64) {
        const unsigned long long st = list[i], key = staged_to_key(st);
        int rank = 0;
        for (int q = 0; q < cut.cnt; q++) rank += staged_to_key(list[q]) > key ? 1 : 0;
        if (rank < cut.krem) stage[n_gt + rank] = st;
    }
}

// A crowded bin: equal scores go by their tokens, others take another histogram over the span of this bin's alone, then an exact ranking.  numbers: the row's best score is below +inf, so all
// are numbers or -inf.  Otherwise - a NaN logit or log-sum-exp, a cumulative score of +inf over masked tokens - some may be NaN, which minima and maxima pass over, and equal extremes would
// not mean equal scores: the ranking at once.  In a function of its own
// on scores in memory: in line it cost the other rows registers (172 for up to 2048 tokens, two wavefronts to a SIMD, now 157 and three).  Whole selections in us, in line with a mask to a
// token / now: 326 requests of 329 rows of 8 tokens, k = 10 74.2 / 69.6; 138 of 606 rows of 56 76.1 / 68.9; 546 of 15 rows of 1760, half of them without a number 130.6 / 121.9.
template <int VEC, int E>
__device__ __noinline__ void select_row_crowded(const float (&sc)[VEC * 4], RowCut cut, float inv_w, float k0, bool numbers, uint32_t flat0, int V, int m,
                                                LdsKey *list, LdsKey *stage) {
    const int lane = threadIdx.x % 64;
    bool tied = false;
    float tie = 0.0f;
    for (int zoom = 0; zoom < 3 && numbers && cut.cnt > WROW_FEW; zoom++) {
        float lo_t = INFINITY, hi_t = -INFINITY, least = INFINITY;  // least: that is not -inf
#pragma unroll
        for (int i = 0; i < VEC * 4; i++) {
            if (score_bin(sc[i], inv_w, k0) == cut.T && wave_has<E>(i, lane, V)) {
                lo_t = fminf(lo_t, sc[i]);
                hi_t = fmaxf(hi_t, sc[i]);
                least = fminf(least, sc[i] > -INFINITY ? sc[i] : INFINITY);
            }
        }
        lo_t = -wave_max(-lo_t);
        hi_t = wave_max(hi_t);
        least = -wave_max(-least);
        tied = lo_t == hi_t;
        tie = hi_t;
        if (tied || !(hi_t >= least)) break;
        const float finer = hi_t > least ? (float)(WROW_BINS - 3) / (hi_t - least) : 1.0f;
        if (!(finer < INFINITY)) break;  // (the cut stands for the bins of inv_w and k0)
        inv_w = finer;
        k0 = (float)WROW_LOW + 0.5f - least * inv_w;  // (-inf below the bins)
        cut = find_cut<VEC, false, E>(sc, inv_w, k0, V, m, (LdsInt *)list, lane);
    }
    if (tied || cut.cnt > WROW_LIST) select_row_radix_wave<VEC, E, false>(sc, V, m, flat0, stage, tied, score_key(tie), cut.krem);
    else stage_cut<VEC, false, E>(sc, cut, inv_w, k0, 0xFFFFFFFFu - flat0 - (uint32_t)lane * (uint32_t)E, V, m, list, stage, lane);
}

// The row's own top-m cut.  x[i]: the logit of token wave_tok<E>(i, lane), padding -inf; mx, lse: the row's maximum and
// log-sum-exp; the m best (score, token) pairs go to dst.
template <int VEC, bool FULL, int E, bool ALONE>
__device__ __forceinline__ void select_row_own_cut(float (&x)[VEC * 4], float c, float mx, float lse, unsigned long long *__restrict__ dst,
                                                   uint32_t flat0, uint32_t nflat, int V, int m, LdsKey *list, int lane) {
    constexpr int NX = VEC * 4;
    // Rows of more than 2048 tokens have no registers left for another histogram (77 x 338 listed rows of 7016 tokens that are all masked 1048 us without, 1535 with)
    constexpr bool AGAIN = VEC <= 8;
    LdsInt *hist = (LdsInt *)list;
    LdsKey *stage = list + WROW_SLOTS;
    // scores from here on (padding stays -inf)
    float mn = INFINITY;
#pragma unroll
    for (int i = 0; i < NX; i++) {
        x[i] = wave_score<AGAIN>(c, x[i] - lse);
        mn = fminf(mn, ((FULL || wave_has<E>(i, lane, V)) && (!AGAIN || x[i] > -INFINITY)) ? x[i] : INFINITY);
    }
    if (m >= V) {  // nothing to cut: every token is a candidate
#pragma unroll
        for (int i = 0; i < NX; i++) {
            const int v = wave_tok<E>(i, lane);
            if (FULL || wave_has<E>(i, lane, V)) dst[v] = pack_candidate(x[i], flat0 + (uint32_t)v);
        }
        return;
    }
    // A histogram of the scores over equal-width bins of [lo, hi] finds the bin of the m-th best; the bin index is monotone in the score.  (AGAIN: lo is the least that is not -inf, which a
    // masked token has, and at most 64 below the best: a low finite mask would press the other scores into a few bins: 16 requests of 128 rows of 2048, k = 32 35.5 us, now 16.5)
    float lo = -wave_max(-mn), hi = c + (mx - lse);
    if (AGAIN) lo = fmaxf(lo, hi - 64.0f);
    const float inv_w = (hi > lo) ? ((float)WROW_BINS - 0.01f) / (hi - lo) : 0.0f;
    const float k0 = (float)WROW_LOW - lo * inv_w;
    const RowCut cut = find_cut<VEC, FULL, E>(x, inv_w, k0, V, m, hist, lane);
    if (cut.cnt > (AGAIN ? WROW_FEW : WROW_LIST)) {  // crowded (e.g. all logits equal)
        float sc[NX];  // a copy, so that only this branch keeps the scores in addressable memory
#pragma unroll
        for (int i = 0; i < NX; i++) sc[i] = x[i];
        if constexpr (AGAIN) select_row_crowded<VEC, E>(sc, cut, inv_w, k0, hi < INFINITY, flat0, V, m, list, stage);
        else select_row_radix_wave<VEC, E, ALONE>(sc, V, m, flat0, stage, false, 0u, 0);
    } else {
        stage_cut<VEC, FULL, E>(x, cut, inv_w, k0, nflat, V, m, list, stage, lane);
    }
    for (int i = lane; i < m; i += 64) dst[i] = staged_to_key(stage[i]);
}

// FULL: V == VEC*256, every register holds a token (the validity tests fold away).
// todo / todo_count (both or neither): the launch visits only the listed rows {row, slot}; each gets its
// own cut, written at slot `slot` of its request's segment.  Wavefronts walk their rows with the launch's stride.
// The row and the cut's state need 119 (VEC 4) to 511 registers (VEC 32): with the 168 of three wavefronts per SIMD most of a row of 4096 and
// 8192 tokens lived in scratch.  ALONE: one wavefront per SIMD, the shortest time of a row of 8192 tokens (m = 256: a few listed rows 17.7 us, 21.8 with two wavefronts
// per SIMD, 22.2 with three).  Otherwise two: what a long list takes (32768 rows all listed 318 us with one, 206 with two, 226 with three).
template <int VEC, bool FULL, bool ALONE, typename LT>
__global__ __launch_bounds__(256, ALONE ? 1 : 2) void select_rows_wave(const LT *__restrict__ logits, const float *__restrict__ cum, int64_t rows, int n, int V,
                                                          int m, unsigned long long *__restrict__ cand, const int2 *__restrict__ todo,
                                                          const int *__restrict__ todo_count, bool numbers_first) {
    constexpr int E = LogitPiece<LT>::E, NX = VEC * 4, G = NX / E;
    extern __shared__ unsigned long long wave_lds[];  // per wavefront: WROW_SLOTS of histogram / list, then m slots of staged output
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
    const int64_t nwaves = (int64_t)gridDim.x * 4;
    const int64_t count = todo ? (int64_t)*todo_count : rows;
    LdsKey *list = (LdsKey *)wave_lds + (size_t)wv * ((WROW_SLOTS + m + 1) & ~1);  // even number of 8-byte slots: 16-byte accesses stay aligned
    // whole wavefronts leave the loop; nothing below synchronises across wavefronts
    for (int64_t at = (int64_t)blockIdx.x * 4 + wv; at < count; at += nwaves) {
        int64_t vrow = at, dst_at = -1;
        if (todo) {
            const int2 t = todo[at];
            vrow = t.x;
            dst_at = (vrow / n) * ((int64_t)n * m) + t.y;
        }
        const uint4 *z = (const uint4 *)(logits + vrow * (int64_t)V);
        float x[NX];
#pragma unroll
        for (int g = 0; g < G; g++) {
            if (FULL || (g * 64 + lane) * E < V) {
                LogitPiece<LT>::unpack(z[g * 64 + lane], &x[g * E]);
            } else {
#pragma unroll
                for (int e = 0; e < E; e++) x[g * E + e] = -INFINITY;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < NX; i++) mx = fmaxf(mx, x[i]);
        mx = wave_max_dpp(mx);
        const float mxl = mx * 1.4426950408889634f;
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < NX; i++) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], 1.4426950408889634f, -mxl));  // padding gives 0
        const float lse = mx + __logf(wave_sum_dpp(sum));
        const uint32_t flat0 = (uint32_t)((vrow % n) * (int64_t)V);
        // low word of a staged candidate: 0xFFFFFFFF - (flat0 + token)
        const uint32_t nflat = 0xFFFFFFFFu - flat0 - (uint32_t)lane * (uint32_t)E;
        const float c = cum ? cum[vrow] : 0.0f;
        unsigned long long *dst = cand + (dst_at >= 0 ? dst_at : vrow * (int64_t)m);
        if (numbers_first && (lse != lse || c != c)) {
            // No score of the row is a number (a beam whose tokens are all masked, say).  Its tokens rank below every number, -inf too, so they
            // survive only where the request has fewer than k numbers.  (m <= V)
            for (int i = lane; i < m; i += 64) dst[i] = (unsigned long long)LAST_KEY << 32 | (0xFFFFFFFFu - (flat0 + (uint32_t)i));
            continue;
        }
        select_row_own_cut<VEC, FULL, E, ALONE>(x, c, mx, lse, dst, flat0, nflat, V, m, list, lane);
    }
}

// The bounded pass.  A row stays in registers as it was read (raw[g]: tokens (g*64 + lane)*E .. +E-1; pieces past V hold -inf): maximum,
// log-sum-exp and the sweep for candidates at or above the request's bound read it in place.  Bound by the memory's latency: a wavefront's row is loaded at once
// and worked on when it is there, so what keeps the memory busy is the other wavefronts of the SIMD.  (A half-precision row used to be requested while the one before it was
// worked on, in as many registers again: 95 instead of 71 for rows of 4096 tokens, 168 instead of 109 for 8192, five and three wavefronts instead of seven and
// four, and the last row of each wavefront was requested twice.  65536 rows of 4096 tokens 157 us, 140 without; 32768 of 8192 150 and 127; 262144 of 8192 912 and 856; a million
// 3.51 and 3.34 ms, whole selections.  AHEAD keeps that for other rows and candidates than these: see rows_walked.  Those are selections one after the other.  One waited for, a row ahead and
// without, on logits that no cache holds: 64 x 256 rows of 4096 62.1 us and 61.6, of 8192 96.3 and 90.5; right behind 600 MB of writes elsewhere, whose lines the caches still have to give back:
// 78.9 and 82.2, 132.7 and 136.0, 128 x 256 of 4096 136.1 and 132.4.)  Wavefronts walk the rows with the launch's
// stride (neighbouring rows in flight together; consecutive rows per wavefront, with one reservation for several rows'
// candidates, were 15 % slower).  A row with more than m candidates at the bound reserves m slots and is
// put on the list for select_rows_wave, which gives it its own cut; this kernel carries none of that code or its registers.
template <int VEC, bool FULL, bool AHEAD, typename LT>
__global__ __launch_bounds__(256, VEC >= 32 ? 2 : (VEC >= 16 ? 3 : 4)) void select_rows_sweep(
    const LT *__restrict__ logits, const float *__restrict__ cum, int64_t rows, int n, int V, int m, unsigned long long *__restrict__ cand,
    const float *__restrict__ rb, int R, int *__restrict__ req_count, int count_pitch, int2 *__restrict__ todo, int *__restrict__ todo_count) {
    constexpr bool HALF = sizeof(LT) == 2;
    constexpr int NX = VEC * 4, E = LogitPiece<LT>::E, G = NX / E;
    extern __shared__ unsigned long long wave_lds[];  // per wavefront: m slots of staged output
    // The row index is made a scalar of the wavefront (rows < 2^31, checked by the host): its cumulative score and bound then
    // come through scalar loads, which do not queue behind the vector loads of a row.
    const int lane = threadIdx.x % 64, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const uint32_t nwaves = gridDim.x * 4u;
    uint32_t row = blockIdx.x * 4u + (uint32_t)wv;
    if (row >= (uint64_t)rows) return;  // whole wavefronts leave; nothing below synchronises across wavefronts
    unsigned long long *stage = wave_lds + (size_t)wv * m;
    auto request_row = [&](uint32_t r, uint4 (&raw)[G]) {
        const uint4 *z = (const uint4 *)(logits + (int64_t)r * V);
#pragma unroll
        for (int g = 0; g < G; g++) {
            if (FULL || (g * 64 + lane) * E < V) raw[g] = z[g * 64 + lane];
            else raw[g] = HALF ? make_uint4(0xFC00FC00u, 0xFC00FC00u, 0xFC00FC00u, 0xFC00FC00u)  // -inf
                               : make_uint4(0xFF800000u, 0xFF800000u, 0xFF800000u, 0xFF800000u);
        }
    };
    // per row: request, beam, cumulative score and this lane's slot of the request's bound, fetched one row ahead
    // (the slot by a vector load, so before the row's: loads return in order)
    auto row_scalars = [&](uint32_t r, uint32_t &req, uint32_t &beam, float &c, float &rbv) {
        req = r / (uint32_t)n;
        beam = r % (uint32_t)n;
        c = cum ? cum[r] : 0.0f;
        rbv = rb[(int64_t)req * (2 * R) + (lane < 2 * R ? lane : 0)];
    };
    auto pk_max = [](halfx2 a, halfx2 b) {  // (the plain instruction: the generic maximum first quiets both operands)
        halfx2 r;
        asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
        return r;
    };
    uint4 raw[G];
    uint32_t req, beam;
    float c, rbv;
    row_scalars(row, req, beam, c, rbv);
    request_row(row, raw);
    for (;;) {
        const uint64_t next = (uint64_t)row + nwaves;
        const bool more = next < (uint64_t)rows;
        const uint32_t ahead = more ? (uint32_t)next : row;
        uint4 nxt[AHEAD ? G : 1];
        uint32_t req_n, beam_n;
        float c_n, rbv_n;
        row_scalars(ahead, req_n, beam_n, c_n, rbv_n);
        // (unconditional - the last row is asked for twice: a branch here would make the compiler wait for these loads at the first use of the current
        // row, as if they had been skipped)
        if constexpr (AHEAD) request_row(ahead, nxt);
        __builtin_amdgcn_sched_barrier(0);  // the loads go out here, not where the instruction scheduler finds the registers cheapest

        typename std::conditional<HALF, halfx2, float>::type pmax[G];  // per piece: the maximum (half precision: of its even and of its odd tokens)
        float lane_mx;
        auto piece_max = [&](int g) {
            if constexpr (HALF) return fmaxf((float)pmax[g][0], (float)pmax[g][1]);
            else return pmax[g];
        };
        if constexpr (HALF) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                const halfx8 v = __builtin_bit_cast(halfx8, raw[g]);
                const halfx2 p0 = {v[0], v[1]}, p1 = {v[2], v[3]}, p2 = {v[4], v[5]}, p3 = {v[6], v[7]};
                pmax[g] = pk_max(pk_max(p0, p1), pk_max(p2, p3));
            }
            halfx2 rm = pmax[0];
#pragma unroll
            for (int g = 1; g < G; g++) rm = pk_max(rm, pmax[g]);
            lane_mx = fmaxf((float)rm[0], (float)rm[1]);
        } else {
            lane_mx = -INFINITY;
#pragma unroll
            for (int g = 0; g < G; g++) {
                float v[E];
                LogitPiece<LT>::unpack(raw[g], v);
                pmax[g] = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
                lane_mx = fmaxf(lane_mx, pmax[g]);
            }
        }
        const float mx = wave_max_dpp(lane_mx);
        const float mxl = mx * 1.4426950408889634f;
        float sum = 0.0f;
#pragma unroll
        for (int g = 0; g < G; g++) {
            float v[E];
            LogitPiece<LT>::unpack(raw[g], v);
#pragma unroll
            for (int e = 0; e < E; e++) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(v[e], 1.4426950408889634f, -mxl));  // padding gives 0
        }
        const float lse = mx + __logf(wave_sum_dpp(sum));
        float sstar = request_bound(rbv, R, lane);
        if (beam == 0) sstar = first_row_bound(__shfl(rbv, 0, 64), sstar, c, lse);
        // (opaque to the compiler: otherwise it keeps the NX widened logits of the sum above in registers for the sweep below)
#pragma unroll
        for (int g = 0; g < G; g++) asm volatile("" : "+v"(raw[g].x), "+v"(raw[g].y), "+v"(raw[g].z), "+v"(raw[g].w));

        // score(x) = c + (x - lse) >= sstar is tested exactly, but only inside the pieces whose maximum passes a threshold in the
        // logit domain placed a few roundings below the exact one (every candidate at or above the bound passes it); most
        // rows of a request's weaker beams have no such piece at all
        uint32_t nflat = 0xFFFFFFFFu - beam * (uint32_t)V - (uint32_t)lane * (uint32_t)E;
        asm volatile("" : "+v"(nflat));  // (opaque: keeps the compiler from carrying NX row-independent parts of the token words across rows)
        const float t0 = (sstar - c) + lse;
        // (no bound: everything passes, also where the scores are -inf and t0 is NaN)
        const float thr = sstar > -INFINITY ? t0 - 1e-6f * (fabsf(sstar) + fabsf(c) + fabsf(lse) + fabsf(t0)) : -INFINITY;
        int cnt = row_is_numbers(c, lse) ? 0 : m + 1;  // (to the list, whatever the sweep finds)
        if (__ballot(lane_mx >= thr) != 0) {
#pragma unroll
            for (int g = 0; g < G; g++) {
                const unsigned long long any = __ballot(piece_max(g) >= thr);
                if (any != 0) {
                    float v[E];
                    LogitPiece<LT>::unpack(raw[g], v);
#pragma unroll
                    for (int e = 0; e < E; e++) {
                        const float sc = c + (v[e] - lse);
                        const bool hit = sc >= sstar;
                        const unsigned long long mk = __ballot(hit);
                        const unsigned long long st = ((unsigned long long)__float_as_uint(sc + 0.0f) << 32) | (nflat - (uint32_t)(g * 64 * E + e));
                        const int at = cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0));
                        if (hit && at < m) stage[at] = st;
                        cnt += __popcll(mk);
                    }
                }
            }
        }
        if (cnt > 0) {  // (wavefront-uniform)
            const int take = cnt <= m ? cnt : m;
            int base = 0;
            if (lane == 0) {
                base = atomicAdd(&req_count[(int64_t)req * count_pitch], take);
                if (cnt > m) todo[atomicAdd(todo_count, 1)] = make_int2((int)row, base);  // its m slots are filled by the listed pass
            }
            base = __shfl(base, 0, 64);
            if (cnt <= m) {
                unsigned long long *dst = cand + (int64_t)req * ((int64_t)n * m) + base;
                for (int i = lane; i < cnt; i += 64) dst[i] = staged_to_key(stage[i]);
            }
        }
        if (!more) break;
        row = (uint32_t)next;
        if constexpr (AHEAD) {
#pragma unroll
            for (int g = 0; g < G; g++) raw[g] = nxt[g];
        } else {
            request_row(row, raw);
        }
        req = req_n; beam = beam_n; c = c_n; rbv = rbv_n;
    }
}

// ---------------------------------------------------------------------------
// stage B: one workgroup per request
// ---------------------------------------------------------------------------
#define SELB_THREADS 1024
#define SELB_SORT_MAX 4096

// the key of lane ^ X for X = 1, 2, 4, 8 (inside a row of 16 lanes)
template <int X> __device__ __forceinline__ unsigned lane_xor_u(unsigned v) {
    if constexpr (X == 1) return dpp_move_u<0xB1, 0xF>(v, v);
    else if constexpr (X == 2) return dpp_move_u<0x4E, 0xF>(v, v);
    else if constexpr (X == 4) { const unsigned r = dpp_move_u<0x141, 0xF>(v, v); return dpp_move_u<0x1B, 0xF>(r, r); }  // ^ 7, then ^ 3
    else return dpp_move_u<0x128, 0xF>(v, v);
}
// one exchange of the sort with lane ^ X: the greater key stays where take_max holds
template <int X> __device__ __forceinline__ unsigned long long sort_exchange(unsigned long long v, bool take_max) {
    const unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    unsigned long long a, b;  // the pair, in the same order for both lanes or not: the greater and the smaller one are what counts
    if constexpr (X >= 16) {
        uintx2 l, h;
        if constexpr (X == 16) { l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false); h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false); }
        else { l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false); h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false); }
        a = (unsigned long long)h[0] << 32 | l[0];
        b = (unsigned long long)h[1] << 32 | l[1];
    } else {
        a = (unsigned long long)lane_xor_u<X>(hi) << 32 | lane_xor_u<X>(lo);
        b = v;
    }
    return (a > b) == take_max ? a : b;
}

// Bitonic sort, descending, of np keys (a power of two, np <= E * SELB_THREADS; the registers past np hold nothing).  Element
// i = tid * E + e sits in v[e]: exchanges over less than 64 * E elements stay inside a lane or a wavefront (DPP and permlane moves: an LDS
// permute of 8 bytes per step and wavefront held up all of them), the ten or so longer ones go through LDS, in two halves by
// turns where both fit (one barrier per step).  Wavefronts past np only keep the barriers.
template <int E>
__device__ __forceinline__ void sort_desc(unsigned long long (&v)[E], int np, unsigned long long *lds) {
    const int tid = threadIdx.x;
    const bool busy = __builtin_amdgcn_readfirstlane(tid) * E < np;
    constexpr bool TURNS = 2 * E * SELB_THREADS <= SELB_SORT_MAX;
    int turn = 1;  // (the first half may still be read)
    for (int k = 2; k <= np; k <<= 1) {
        for (int x = k / E >> 1; x >= 64; x >>= 1) {
            unsigned long long *buf = lds + (TURNS ? turn * E * SELB_THREADS : 0);
            if (!TURNS) __syncthreads();
            if (busy) {
#pragma unroll
                for (int e = 0; e < E; e++) buf[e * SELB_THREADS + tid] = v[e];
            }
            __syncthreads();
            if (busy) {
                const bool low = (tid & x) == 0;
#pragma unroll
                for (int e = 0; e < E; e++) {
                    const unsigned long long o = buf[e * SELB_THREADS + (tid ^ x)];
                    const bool desc = ((tid * E + e) & k) == 0;
                    v[e] = (o > v[e]) == (desc == low) ? o : v[e];
                }
            }
            turn ^= 1;
        }
        if (!busy) continue;
#define LANES_(X) \
        if (k > X * E) { \
            const bool low = (tid & X) == 0; \
            _Pragma("unroll") for (int e = 0; e < E; e++) v[e] = sort_exchange<X>(v[e], (((tid * E + e) & k) == 0) == low); \
        }
        LANES_(32) LANES_(16) LANES_(8) LANES_(4) LANES_(2) LANES_(1)
#undef LANES_
#pragma unroll
        for (int q = E / 2; q > 0; q >>= 1)
            if (k > q) {
#pragma unroll
                for (int e = 0; e < E; e++)
                    if (!(e & q)) {
                        const bool desc = ((tid * E + e) & k) == 0;
                        const unsigned long long a = v[e], b = v[e | q];
                        if (desc ? a < b : a > b) { v[e] = b; v[e | q] = a; }
                    }
            }
    }
}

// sorts the first np keys of lds (np <= SELB_SORT_MAX, a power of two) in place
template <int E>
__device__ __forceinline__ void sort_keys_lds(unsigned long long *lds, int np) {
    const int tid = threadIdx.x;
    unsigned long long v[E];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; e++) v[e] = tid * E + e < np ? lds[tid * E + e] : 0ull;
    sort_desc<E>(v, np, lds);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; e++)
        if (tid * E + e < np) lds[tid * E + e] = v[e];
    __syncthreads();
}
__device__ __forceinline__ void bitonic_sort_desc(unsigned long long *lds, int np) {
    if (np <= SELB_THREADS) sort_keys_lds<1>(lds, np);
    else if (np <= 2 * SELB_THREADS) sort_keys_lds<2>(lds, np);
    else sort_keys_lds<4>(lds, np);
}

// every key of a request's candidate list, 16 bytes per lane and four loads in flight (the list is streamed several times)
template <typename F>
__device__ __forceinline__ void for_each_key(const unsigned long long *__restrict__ src, int64_t ncand, F f) {
    const int tid = threadIdx.x;
    if ((((uintptr_t)src) & 15) == 0) {
        const ulonglong2 *src2 = (const ulonglong2 *)src;
        const int64_t pairs = ncand / 2;
        int64_t i = tid;
        for (; i + 3 * SELB_THREADS < pairs; i += 4 * SELB_THREADS) {
            const ulonglong2 a = src2[i], b = src2[i + SELB_THREADS], c = src2[i + 2 * SELB_THREADS], d = src2[i + 3 * SELB_THREADS];
            f(a.x); f(a.y); f(b.x); f(b.y); f(c.x); f(c.y); f(d.x); f(d.y);
        }
        for (; i < pairs; i += SELB_THREADS) { const ulonglong2 a = src2[i]; f(a.x); f(a.y); }
        if ((ncand & 1) && tid == 0) f(src[ncand - 1]);
    } else {
        for (int64_t i = tid; i < ncand; i += SELB_THREADS) f(src[i]);
    }
}

// Usual path of stage B: the candidates are read once into registers, SELB_HELD per thread (twice from memory where there are more), and
// swept twice.  A sample of one key per thread gives the span of the score bits; the first sweep counts the keys in 2048 equal bins of that
// span (keys outside it fall into the end bins; the bin index is monotone in the key, and the counts spread over the bins, unlike the leading
// radix digit, which most keys of a request share), the second collects every key from the threshold bin up into LDS: those above it, then its
// own, of which a few comparisons keep the ones still needed, so that a sort of k keys (not of the next power of two) finishes the job.
// Bound by latency, one workgroup per request.  256 requests of 128 and 256 rows of 4096 tokens, k = 256 and 512: 16.4 and 21.1 us with two reads,
// a sort of twice as many keys through LDS permutes and the tables gathered level by level, now 12.9 and 15.4; one request (k = 128 and 256)
// 12.6 and 15.9, now 10.2 and 12.0.
// Returns false, having selected nothing, when more than SELB_SORT_MAX keys lie from the threshold bin up (the exact radix selection then runs).
#define SELB_HELD 8
#define SELB_SORT_ALL 256  // up to here all keys are sorted
#define SELB_TIES 256  // keys of the threshold bin that are ranked against each other
struct SelbShared {  // (one request's)
    unsigned long long skeys[SELB_SORT_MAX];
    int hist[2048];
    int wave_tot[16];
    uint32_t span_hi[SELB_THREADS / 64], span_lo[SELB_THREADS / 64];
    int sel_digit, sel_krem, sel_cnt, out_cnt, gathered;
};
// x: the keys of this thread (0: none), all of them (held) or not yet; each(f): every key that is not held; smp_hi, smp_lo: this thread's part of the sampled span
template <int H, typename EACH>
__device__ __forceinline__ bool select_binned(unsigned long long (&x)[H], bool held, EACH each, uint32_t smp_hi, uint32_t smp_lo, int k, SelbShared &sh) {
    const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
    for (int i = tid; i < 2048; i += SELB_THREADS) sh.hist[i] = 0;
    if (tid == 0) sh.out_cnt = sh.gathered = 0;
    uint32_t smax = wave_max_u(smp_hi), smin = ~wave_max_u(~smp_lo);
    if (lane == 0) { sh.span_hi[wv] = smax; sh.span_lo[wv] = smin; }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SELB_THREADS / 64; q++) { smax = max(smax, sh.span_hi[q]); smin = min(smin, sh.span_lo[q]); }
    const uint32_t span = smax - smin;
    int nsh = span < 2048u ? 0 : 21 - __clz((int)span);
    if ((span >> nsh) >= 2040u) nsh++;
    auto digit = [&](unsigned long long key) {  // 4 .. 2043 inside the span, 0 below it, up to 2047 above (the addition cannot wrap)
        const uint32_t s = (uint32_t)(key >> 32);
        return s < smin ? 0 : (int)(min((s - smin) >> nsh, 2043u) + 4u);
    };
    if (held) {
#pragma unroll
        for (int j = 0; j < H; j++)
            if (x[j]) atomicAdd(&sh.hist[digit(x[j])], 1);
    } else {
        each([&](unsigned long long key) { atomicAdd(&sh.hist[digit(key)], 1); });
    }
    __syncthreads();
    // thread t owns digits 2047-2t (hi) and 2046-2t (lo); scan from the top digit down
    const int hi = sh.hist[2047 - 2 * tid], lo = sh.hist[2046 - 2 * tid];
    const int v = wave_scan(hi + lo);
    if (lane == 63) sh.wave_tot[wv] = v;
    __syncthreads();
    int add = 0;
#pragma unroll
    for (int q = 0; q < SELB_THREADS / 64; q++) add += q < wv ? sh.wave_tot[q] : 0;
    const int incl = v + add, excl = incl - hi - lo;
    if (excl < k && incl >= k) {
        if (excl + hi >= k) { sh.sel_digit = 2047 - 2 * tid; sh.sel_krem = k - excl; sh.sel_cnt = hi; }
        else { sh.sel_digit = 2046 - 2 * tid; sh.sel_krem = k - excl - hi; sh.sel_cnt = lo; }
    }
    __syncthreads();
    const int T = sh.sel_digit, krem = sh.sel_krem, cnt = sh.sel_cnt, n_gt = k - krem, total = n_gt + cnt;
    if (total > SELB_SORT_MAX) return false;  // uniform: every thread read the same shared values
    const bool rank_ties = cnt > krem && cnt <= SELB_TIES;
    const int want = rank_ties ? k : total;
    int np = 1;
    while (np < want) np <<= 1;
    unsigned long long *skeys = sh.skeys;
    for (int i = total + tid; i < np; i += SELB_THREADS) skeys[i] = 0ull;
    if (!held) {  // the keys from bin T up, at most SELB_SORT_MAX (a counter for either end in this sweep cost 20 to 60 us of a million keys)
        each([&](unsigned long long key) {
            if (digit(key) >= T) skeys[atomicAdd(&sh.gathered, 1)] = key;
        });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < H; j++) x[j] = j < SELB_SORT_MAX / SELB_THREADS && j * SELB_THREADS + tid < total ? skeys[j * SELB_THREADS + tid] : 0ull;
        __syncthreads();
    }
    // keys above bin T go to [0, n_gt), those of bin T behind them; out_cnt counts both, 16 bits each (at most SELB_SORT_MAX of either); one reservation
    // per wavefront
    unsigned long long mg[H], me[H];
    int c = 0;
#pragma unroll
    for (int j = 0; j < H; j++) {
        const int d = x[j] ? digit(x[j]) : -1;
        mg[j] = __ballot(d > T);
        me[j] = __ballot(d == T);
        c += __popcll(mg[j]) + (__popcll(me[j]) << 16);
    }
    if (c) {
        int at = lane == 0 ? atomicAdd(&sh.out_cnt, c) : 0;
        at = __builtin_amdgcn_readfirstlane(at);
        int ag = at & 0xFFFF, ae = n_gt + (int)((unsigned)at >> 16);
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int j = 0; j < H; j++) {
            if (mg[j] >> lane & 1) skeys[ag + __popcll(mg[j] & below)] = x[j];
            if (me[j] >> lane & 1) skeys[ae + __popcll(me[j] & below)] = x[j];
            ag += __popcll(mg[j]);
            ae += __popcll(me[j]);
        }
    }
    if (rank_ties) {
        __syncthreads();
        const unsigned long long key = tid < cnt ? skeys[n_gt + tid] : 0ull;
        int rank = 0;
        if (__builtin_amdgcn_readfirstlane(tid) < cnt)
            for (int q = 0; q < cnt; q++) rank += skeys[n_gt + q] > key ? 1 : 0;
        __syncthreads();
        if (tid < cnt && rank < krem) skeys[n_gt + rank] = key;
        for (int i = k + tid; i < np; i += SELB_THREADS) skeys[i] = 0ull;
    }
    bitonic_sort_desc(skeys, np);
    return true;
}

// Exact whatever the keys: radix selection on the unique 64-bit keys, 11-bit digits from the top; stops as soon as the chosen bin holds exactly the number of
// keys still needed.  each(f): every key.
template <typename EACH> __device__ __forceinline__ void select_radix(EACH each, int k, int kp, SelbShared &sh) {
    const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
    unsigned long long prefix = 0;  // value of key >> shift
    int krem = k, shift = 64;
    const int widths[6] = {11, 11, 11, 11, 11, 9};
    for (int pass = 0; pass < 6; pass++) {
        const int w = widths[pass];
        const int nshift = shift - w;
        for (int i = tid; i < 2048; i += SELB_THREADS) sh.hist[i] = 0;
        __syncthreads();
        each([&](unsigned long long key) {
            if (pass == 0 || (key >> shift) == prefix) atomicAdd(&sh.hist[(int)((key >> nshift) & ((1u << w) - 1))], 1);
        });
        __syncthreads();
        // thread t owns digits 2047-2t (hi) and 2046-2t (lo); scan from the top digit down
        const int hi = sh.hist[2047 - 2 * tid], lo = sh.hist[2046 - 2 * tid];
        const int v = wave_scan(hi + lo);
        if (lane == 63) sh.wave_tot[wv] = v;
        __syncthreads();
        int add = 0;
        for (int q = 0; q < wv; q++) add += sh.wave_tot[q];
        const int incl = v + add, excl = incl - hi - lo;
        if (excl < krem && incl >= krem) {
            if (excl + hi >= krem) { sh.sel_digit = 2047 - 2 * tid; sh.sel_krem = krem - excl; sh.sel_cnt = hi; }
            else { sh.sel_digit = 2046 - 2 * tid; sh.sel_krem = krem - excl - hi; sh.sel_cnt = lo; }
        }
        __syncthreads();
        prefix = (prefix << w) | (unsigned long long)sh.sel_digit;
        krem = sh.sel_krem;
        shift = nshift;
        const int cnt = sh.sel_cnt;
        __syncthreads();
        if (cnt == krem || shift == 0) break;  // uniform: all threads read the same shared values
    }
    if (tid == 0) sh.out_cnt = 0;
    for (int i = tid; i < kp; i += SELB_THREADS) sh.skeys[i] = 0ull;
    __syncthreads();
    each([&](unsigned long long key) {
        if ((key >> shift) >= prefix) {
            int p = atomicAdd(&sh.out_cnt, 1);
            if (p < kp) sh.skeys[p] = key;
        }
    });
    __syncthreads();
    bitonic_sort_desc(sh.skeys, kp);
}

// What a selection returns
struct Survivors {
    int32_t *parent, *tok;
    float *score;
    const int32_t *sid_old;
    int32_t *sid_new;
    const int32_t *anc_old;
    int32_t *anc_new;
    int T, level;
};
__device__ __forceinline__ void write_survivors(const Survivors &o, const unsigned long long *skeys, int64_t b, int n, int V, int k) {
    for (int j = threadIdx.x; j < k; j += SELB_THREADS) {
        const unsigned long long key = skeys[j];
        const uint32_t flat = 0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull);
        // (a request lists at least k candidates; the clamp keeps what is read through the parent inside the batch whatever the keys hold)
        const int par = min((int)(flat / (uint32_t)V), n - 1), tk = (int)(flat % (uint32_t)V);
        o.parent[b * k + j] = par;
        o.tok[b * k + j] = tk;
        o.score[b * k + j] = key_score((uint32_t)(key >> 32));
        // sids, and the row (over the whole batch) of the survivor's ancestor at every level so far: the reorder is this index table
        // (every load ahead of the stores)
        const int64_t from = (b * n + par) * o.T, to = (b * k + j) * o.T;
        int32_t sid[GR4AD_MAX_LEVELS], anc[GR4AD_MAX_LEVELS];
#pragma unroll
        for (int t = 0; t < GR4AD_MAX_LEVELS; t++) {
            sid[t] = o.sid_new && t < o.level ? o.sid_old[from + t] : (t == o.level ? tk : 0);
            anc[t] = o.anc_new && t < o.level ? o.anc_old[from + t] : (int32_t)(b * n + par);
        }
#pragma unroll
        for (int t = 0; t < GR4AD_MAX_LEVELS; t++) {
            if (o.sid_new && t < o.T) o.sid_new[to + t] = sid[t];
            if (o.anc_new && t <= o.level) o.anc_new[to + t] = anc[t];
        }
    }
}

__global__ __launch_bounds__(SELB_THREADS) void select_request(const unsigned long long *__restrict__ cand, int64_t req_stride, const int *__restrict__ req_count,
                                                               int count_pitch, int V, int k, int n, Survivors out) {
    __shared__ SelbShared sh;
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const unsigned long long *src = cand + b * req_stride;  // the request's candidates: the first keys of its segment, all of them without a count
    const int64_t ncand = req_count ? req_count[b * count_pitch] : req_stride;
    int kp = 1;
    while (kp < k) kp <<= 1;
    auto each = [&](auto f) { for_each_key(src, ncand, f); };

    // few enough to sort them all (a cut down to k keys costs two sweeps; worth it from 1024 keys on, and from 257 where three quarters of them go)
    if (ncand <= SELB_SORT_ALL || ncand <= kp || (ncand <= SELB_THREADS && ncand < 4 * k)) {
        int np = 1;
        while (np < ncand) np <<= 1;
        for (int i = tid; i < (np > kp ? np : kp); i += SELB_THREADS) sh.skeys[i] = i < ncand ? src[i] : 0ull;
        __syncthreads();
        bitonic_sort_desc(sh.skeys, np);
    } else {
        const bool held = ncand <= SELB_HELD * SELB_THREADS;
        unsigned long long x[SELB_HELD];  // 0: none
        if (held) {
            const bool pairs = (((uintptr_t)src) & 15) == 0;
#pragma unroll
            for (int j = 0; j < SELB_HELD; j += 2) {
                const int i = j * SELB_THREADS + (pairs ? 2 * tid : tid), i2 = pairs ? i + 1 : i + SELB_THREADS;
                x[j] = x[j + 1] = 0ull;
                if (pairs && i2 < ncand) {
                    const ulonglong2 a = *(const ulonglong2 *)(src + i);
                    x[j] = a.x;
                    x[j + 1] = a.y;
                } else {
                    if (i < ncand) x[j] = src[i];
                    if (i2 < ncand) x[j + 1] = src[i2];
                }
            }
        }
        const uint32_t smp = (uint32_t)(src[(int64_t)tid * ncand / SELB_THREADS] >> 32);
        if (!select_binned<SELB_HELD>(x, held, each, smp, smp, k, sh)) select_radix(each, k, kp, sh);
    }
    write_survivors(out, sh.skeys, b, n, V, k);
}

// ---------------------------------------------------------------------------
// A request of one row - the first level of every decode - in one launch
// ---------------------------------------------------------------------------
// The row's cut and the request's sort were two launches, the first of a single wavefront (or of 256 threads) per request.  Here 1024 threads hold the row, PER logits each:
// maximum, exponentials and keys are formed side by side, and only the sum of the exponentials, whose order decides the last bit of every score, is
// added up as the row kernels add it (ORDER_WAVE: select_rows_wave, a lane walks its pieces; else select_rows, a thread walks every 256th token), from LDS.
// LOG_P_FIRST: the operand order of wave_score<true>
template <int PER, bool ORDER_WAVE, bool LOG_P_FIRST, typename LT>
__global__ __launch_bounds__(SELB_THREADS) void select_single(const LT *__restrict__ logits, const float *__restrict__ cum, int V, int k, Survivors out) {
    constexpr int E = ORDER_WAVE ? LogitPiece<LT>::E : 1, J = PER / E;  // tokens of a load; loads of a thread
    __shared__ SelbShared sh;
    __shared__ float red[SELB_THREADS / 64], lse_s;
    extern __shared__ __attribute__((aligned(16))) float expo[];  // [V]
    const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
    const int64_t b = blockIdx.x;
    const LT *z = logits + b * V;
    const float c = cum ? cum[b] : 0.0f;
    float x[PER];
    auto token = [&](int i) { return ((i / E) * SELB_THREADS + tid) * E + i % E; };
#pragma unroll
    for (int j = 0; j < J; j++) {
        const int at = token(j * E);
        if constexpr (ORDER_WAVE) {
            if (at < V) {  // (V is a multiple of a piece)
                LogitPiece<LT>::unpack(((const uint4 *)z)[at / E], &x[j * E]);
            } else {
#pragma unroll
                for (int e = 0; e < E; e++) x[j * E + e] = -INFINITY;
            }
        } else {
            x[j] = at < V ? (float)z[at] : -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; i++) mx = fmaxf(mx, x[i]);
    mx = wave_max_dpp(mx);
    if (lane == 0) red[wv] = mx;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SELB_THREADS / 64; q++) mx = fmaxf(mx, red[q]);
    const float mxl = mx * 1.4426950408889634f;
#pragma unroll
    for (int i = 0; i < PER; i++)
        if (token(i) < V) expo[token(i)] = ORDER_WAVE ? __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], 1.4426950408889634f, -mxl)) : __expf(x[i] - mx);
    __syncthreads();
    if constexpr (ORDER_WAVE) {
        if (wv == 0) {
            float sum = 0.0f;
#pragma unroll 4
            for (int at = lane * E; at < V; at += 64 * E) {
#pragma unroll
                for (int e = 0; e < E; e += 4) {
                    const floatx4 p = *(const floatx4 *)(expo + at + e);
                    sum += p[0];
                    sum += p[1];
                    sum += p[2];
                    sum += p[3];
                }
            }
            const float lse = mx + __logf(wave_sum_dpp(sum));
            if (lane == 0) lse_s = lse;
        }
    } else {
        if (wv < 4) {
            float sum = 0.0f;
#pragma unroll 8
            for (int at = tid; at < V; at += 256) sum += expo[at];
            sum = wave_sum(sum);
            if (lane == 0) red[wv] = sum;
        }
        __syncthreads();
        if (tid == 0) lse_s = mx + __logf((red[0] + red[1]) + (red[2] + red[3]));
    }
    __syncthreads();
    const float lse = lse_s;
    unsigned long long key[PER];
    uint32_t hi = 0u, lo = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        key[i] = token(i) < V ? pack_candidate(wave_score<LOG_P_FIRST>(c, x[i] - lse), (uint32_t)token(i)) : 0ull;
        if (i == 0 && key[i]) hi = lo = (uint32_t)(key[i] >> 32);
    }
    int kp = 1;
    while (kp < k) kp <<= 1;
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < PER; i++)
            if (key[i]) f(key[i]);
    };
    if (V <= SELB_SORT_ALL) {
        int np = 1;
        while (np < V) np <<= 1;
        for (int i = V + tid; i < np; i += SELB_THREADS) sh.skeys[i] = 0ull;
#pragma unroll
        for (int i = 0; i < PER; i++)
            if (key[i]) sh.skeys[token(i)] = key[i];
        __syncthreads();
        bitonic_sort_desc(sh.skeys, np);
    } else if (!select_binned<PER>(key, true, each, hi, lo, k, sh)) {
        // (a row without a number, or of one score: its first tokens.  Counted digit by digit, one after the other, 341 requests of 7560 such tokens took 102.9 us, now 25.1)
        hi = 0u, lo = 0xFFFFFFFFu;
        each([&](unsigned long long ky) {
            hi = max(hi, (uint32_t)(ky >> 32));
            lo = min(lo, (uint32_t)(ky >> 32));
        });
        hi = wave_max_u(hi);
        lo = ~wave_max_u(~lo);
        if (lane == 0) { sh.span_hi[wv] = hi; sh.span_lo[wv] = lo; }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < SELB_THREADS / 64; q++) { hi = max(hi, sh.span_hi[q]); lo = min(lo, sh.span_lo[q]); }
        if (hi == lo) {
            for (int i = tid; i < k; i += SELB_THREADS) sh.skeys[i] = (unsigned long long)hi << 32 | (0xFFFFFFFFu - (uint32_t)i);
            __syncthreads();
        } else {
            select_radix(each, k, kp, sh);
        }
    }
    write_survivors(out, sh.skeys, b, 1, V, k);
}

template <int PER, bool ORDER_WAVE, bool LOG_P_FIRST, typename LT>
static int launch_select_single(const void *logits, const float *cum, int B, int V, int k, const Survivors &out, hipStream_t st) {
    auto kern = select_single<PER, ORDER_WAVE, LOG_P_FIRST, LT>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, PER * SELB_THREADS * (int)sizeof(float)) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    ProfScope ps(KC_SELECT_REQUEST, st, 0.0, (double)B * V * sizeof(LT) + (double)B * k * 12);
    hipLaunchKernelGGL(kern, dim3((unsigned)B), dim3(SELB_THREADS), (size_t)V * sizeof(float), st, (const LT *)logits, cum, V, k, out);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// what the row kernels of one selection share
struct RowsLaunch {
    hipStream_t st;
    const void *logits;
    int logits_f16;
    const float *cum;
    int n, V, m;
    unsigned long long *cand;
    float *rb;  // scores behind the request bounds, R rows per request
    int R;
    int *req_count;
    int count_pitch;
    int2 *todo;
    int *todo_count;
    bool numbers_first;  // rows whose scores are no numbers rank below all numbers (requests that a bound could serve)
};
static int compute_units() {
    static int n_cu = 0;
    if (!n_cu) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
        n_cu = prop.multiProcessorCount;
    }
    return n_cu;
}
// mode 0: every row its own cut; mode 1: the listed rows' own cuts
template <int VEC, bool FULL, bool ALONE, typename LT>
static int launch_rows_wave_as(const RowsLaunch &a, int64_t rows, int mode) {
    auto kern = select_rows_wave<VEC, FULL, ALONE, LT>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (WROW_SLOTS + GR4AD_MAX_BEAM + 2) * 8) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const size_t lds = 4 * (size_t)((WROW_SLOTS + a.m + 1) & ~1) * sizeof(unsigned long long);  // <= 4 * (4.25 KB + 32 KB)
    int64_t grid = ceil_div64(rows, 4);  // one wavefront per row, four rows per workgroup
    if (mode == 1) {  // the list is short as a rule: a few workgroups per compute unit walk it
        const int n_cu = compute_units();
        if (!n_cu) return GR4AD_EHIP;
        if (grid > (int64_t)n_cu * 4) grid = (int64_t)n_cu * 4;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, a.st, (const LT *)a.logits, a.cum, rows, a.n, a.V, a.m, a.cand,
                       mode == 1 ? (const int2 *)a.todo : nullptr, mode == 1 ? (const int *)a.todo_count : nullptr, a.numbers_first);
    return GR4AD_OK;
}
// (The length of a list is known on the device only, and it is short as a rule: beside a sweep of more than 8192 rows the four microseconds of a short one do not
// show, while a long one takes half as long again on wavefronts of their own.  Selections whose rows are all listed, shared and alone: 6400 rows of 8192 tokens 138 us and 136, of
// 8000 tokens 253 and 199; 16384 rows of 8192 tokens 324 and 366, of 8000 522 and 541; 32768 rows of 8000 tokens 854 and 934.)
template <int VEC, bool FULL, typename LT>
static int launch_rows_wave_kind(const RowsLaunch &a, int64_t rows, int mode) {
    if constexpr (VEC >= 32)
        if (rows <= 8192) return launch_rows_wave_as<VEC, FULL, true, LT>(a, rows, mode);
    return launch_rows_wave_as<VEC, FULL, false, LT>(a, rows, mode);
}
// mode 2: the bounded pass, which lists the rows that need their own cut
template <int VEC, bool FULL, bool AHEAD, typename LT>
static int launch_rows_sweep_as(const RowsLaunch &a, int64_t rows, int64_t rows_per) {
    auto kern = select_rows_sweep<VEC, FULL, AHEAD, LT>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * GR4AD_MAX_BEAM * 8) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const size_t lds = 4 * (size_t)a.m * sizeof(unsigned long long);
    const int64_t grid = ceil_div64(ceil_div64(rows, rows_per), 4);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, a.st, (const LT *)a.logits, a.cum, rows,
                       a.n, a.V, a.m, a.cand, (const float *)a.rb, a.R, a.req_count, a.count_pitch, a.todo, a.todo_count);
    return GR4AD_OK;
}
// Float32: up to eight rows per wavefront, but 64 wavefronts per compute unit come first.  Half precision: one row per wavefront, or as many as float32 with the next one requested while one
// is worked on.  Whole selections, time of one row over that of several (rows_per: how many), the popular tokens of a decode and normal logits, 256, 512 and 847 rows per request:
//   2048, 4096 and 8192 tokens   0.83 to 1.03, k = 1 to 512 (65536 rows of 4096 tokens, k = 512 128 us and 150; 262144 of 8192, k = 32 761 and 800): never
//   1024 tokens                  rows_per 2 0.97 to 1.04, 3 0.96 to 1.10, 4 0.95 to 1.09, 7 and 8 0.95 to 1.20 (128000 rows, k = 128 93 us and 88)
//   up to 1016 and up to 2040    rows_per 2 0.97 to 1.17, 3 to 5 0.97 to 1.17, 6 to 8 0.97 to 1.32 (128000 rows of 776, k = 32 88 us and 79; 160000 of 1584, k = 128 187 and 145)
//   2056 to 4088                 rows_per 2 and 3 0.90 to 1.20, 4 to 8 0.94 to 1.23 (k = 512 on popular tokens 0.94 to 1.05; 65536 rows of 3096, k = 8 114 us and 100, k = 512 139 and 145)
//   4104 to 8184                 rows_per 2 to 5 0.75 to 1.04, 7 and 8 0.95 to 1.22 for k <= 32, 0.84 to 1.22 above (160000 rows of 8000, k = 8 565 us and 495, k = 512 765 and 772)
// (rows of so many tokens that every lane has all its pieces gain from the registers alone: see the kernel; what the others pay for each row they have a wavefront to themselves for is
// not known).  And where the LDS of m staged candidates to a wavefront leaves no more wavefronts than the registers of a row ahead do, some five to a SIMD up to 4096 tokens and three above: k = 1024
// 1.00 to 1.33 up to 4088 tokens, 0.95 to 1.04 for 4096, where k = 1400 gives 0.99 to 1.11; k = 2048 1.02 to 1.57, and above 4096 tokens 0.99 to 1.54, where k = 1400 gives 0.88 to 1.17
// (160000 rows of 4096, k = 4096 1061 us and 829; 128000 of 8000, k = 2048 981 and 637).
template <int VEC, bool FULL> static bool rows_walked(int64_t rows_per, int m) {
    if (rows_per < 2) return false;
    if (160 * 1024 / (4 * 8 * m) <= (VEC > 16 ? 2 : VEC == 16 && FULL ? 4 : 5)) return true;
    if (FULL) return VEC == 4 && rows_per >= 3;
    if (VEC <= 8) return true;
    return VEC == 16 ? rows_per >= 4 && m <= 256 : rows_per >= 7 && m <= 64;
}
template <int VEC, bool FULL, typename LT>
static int launch_rows_sweep_kind(const RowsLaunch &a, int64_t rows) {
    const int n_cu = compute_units();
    if (!n_cu) return GR4AD_EHIP;
    int64_t rows_per = rows / ((int64_t)n_cu * 64);
    rows_per = rows_per < 1 ? 1 : (rows_per > 8 ? 8 : rows_per);
    if constexpr (sizeof(LT) == 2) {
        if (rows_walked<VEC, FULL>(rows_per, a.m)) return launch_rows_sweep_as<VEC, FULL, true, LT>(a, rows, rows_per);
        rows_per = 1;
    }
    return launch_rows_sweep_as<VEC, FULL, false, LT>(a, rows, rows_per);
}
// the request bounds: R rows of every request
template <int ITEMS>
static int launch_row_bounds(const RowsLaunch &a, int B) {
    const dim3 grid((unsigned)((int64_t)B * a.R));
    if (a.logits_f16)
        hipLaunchKernelGGL((row_bounds<ITEMS, _Float16>), grid, dim3(256), 0, a.st, (const _Float16 *)a.logits, a.cum, a.n, a.V, a.m, a.R, a.rb,
                           a.req_count, a.count_pitch, a.todo_count);
    else
        hipLaunchKernelGGL((row_bounds<ITEMS, float>), grid, dim3(256), 0, a.st, (const float *)a.logits, a.cum, a.n, a.V, a.m, a.R, a.rb, a.req_count,
                           a.count_pitch, a.todo_count);
    return GR4AD_OK;
}
template <int VEC>
static int launch_rows_vec(const RowsLaunch &a, int64_t rows, int mode) {
    const bool full = a.V == VEC * 256;
    if (mode == 3) return launch_row_bounds<(VEC < 8 ? 8 : VEC)>(a, (int)rows);
    if (mode == 2) {
        if (a.logits_f16) return full ? launch_rows_sweep_kind<VEC, true, _Float16>(a, rows) : launch_rows_sweep_kind<VEC, false, _Float16>(a, rows);
        return full ? launch_rows_sweep_kind<VEC, true, float>(a, rows) : launch_rows_sweep_kind<VEC, false, float>(a, rows);
    }
    if (a.logits_f16) return full ? launch_rows_wave_kind<VEC, true, _Float16>(a, rows, mode) : launch_rows_wave_kind<VEC, false, _Float16>(a, rows, mode);
    return full ? launch_rows_wave_kind<VEC, true, float>(a, rows, mode) : launch_rows_wave_kind<VEC, false, float>(a, rows, mode);
}
// mode 3: the request bounds (rows = requests)
static int launch_rows(const RowsLaunch &a, int64_t rows, int mode) {
    if (a.V <= 1024) return launch_rows_vec<4>(a, rows, mode);
    if (a.V <= 2048) return launch_rows_vec<8>(a, rows, mode);
    if (a.V <= 4096) return launch_rows_vec<16>(a, rows, mode);
    return launch_rows_vec<32>(a, rows, mode);
}

// Half-precision logits are taken by the wavefront kernel only: 16-byte pieces of 8 values.
bool select_takes_f16(int V) { return V >= 8 && V <= 8192 && V % 8 == 0; }

// Workspace: candidates [B][n*m] keys, the request counts, the scores behind the bounds [B][2R], the count of listed rows (one int in 256
// bytes) and the list {row, slot} [B*n].  The size callers are told, r() rounding up to 256 bytes, is
// r(8 B n m) + r(8 B m) + r(8 B) + r(4 B) + 256 + r(8 B n): the parts never need more (counts: at most 4 m bytes per request; scores: 8, or at
// most 2 m where R > 1), so how counts and scores are spread changes neither it nor what the static scratch accepts.
struct SelectPlan {
    int R, count_pitch;
    size_t counts, scores, todo_count, todo, total;
};
static SelectPlan select_plan(int B, int n, int V, int k) {
    SelectPlan p;
    const int m = k < V ? k : V;
    p.R = 1;
    while (p.R < BOUND_ROWS_MAX && p.R * 64 <= n && p.R * 4 <= m) p.R <<= 1;  // at most one row in 32 is read for the bound
    p.count_pitch = m < COUNT_PITCH_MAX ? m : COUNT_PITCH_MAX;
    p.counts = align256((size_t)B * n * m * sizeof(unsigned long long));
    p.scores = p.counts + align256((size_t)B * p.count_pitch * sizeof(int));
    p.todo_count = p.scores + align256((size_t)B * 2 * p.R * sizeof(float));
    p.todo = p.todo_count + 256;
    p.total = p.counts + align256((size_t)B * m * 8) + align256((size_t)B * 8) + align256((size_t)B * 4) + 256 + align256((size_t)B * n * sizeof(int2));
    return p;
}
size_t select_workspace_bytes(int B, int n, int V, int k) { return select_plan(B, n, V, k).total; }

// Few short rows are faster cut one by one (one launch of wavefronts that each take a row, then the request's sort over all n * m keys, which it holds up to 8192) than
// bounded, swept and listed in three launches.  Whole selections in us, bounded / row by row: 4 requests of 16 rows of 256 tokens, k = 16 16.8 / 11.6; 64 of 64 rows of 1024,
// k = 64 (4096 rows) 21.2 / 16.9, 64 of 128 rows, k = 32 (8192 rows) 21.7 / 21.3; of 2048 tokens 16 of 128 rows, k = 32 (2048 rows) 18.8 / 16.0, 64 of 64 rows, k = 64 24.4 / 23.9.
// Requests of 2 to 7 rows would gain as much (256 of 2 rows of 1024, k = 64 21.2 / 11.1; 16 of 5 rows of 256, k = 128 22.3 / 15.1; 256 of 7 rows of 2048, k = 256 29.5 / 20.0): they stay
// bounded so that the workspace shows how many candidates a masked request lists (test_gpu_select_masked.py reads it, 5 rows of 264), not because a measurement says so.
static bool rows_cut_alone(int64_t rows, int n, int V, int m) {
    return n >= 8 && (int64_t)n * m <= SELB_HELD * SELB_THREADS && V <= 2048 && rows <= (V <= 1024 ? 4096 : 2048);
}
int launch_select(const void *logits_any, int logits_f16, const float *cum, int B, int n, int V, int k, void *ws, size_t ws_bytes, int32_t *parent,
                  int32_t *tok, float *score, const int32_t *sid_old, int32_t *sid_new, const int32_t *anc_old, int32_t *anc_new, int T, int level,
                  hipStream_t st) {
    if (B <= 0 || n <= 0 || V <= 0 || k <= 0 || (int64_t)k > (int64_t)n * V) return GR4AD_EINVAL;
    if (logits_f16 && (!select_takes_f16(V) || ((uintptr_t)logits_any % 16))) return GR4AD_EUNSUPPORTED;
    const float *logits = (const float *)logits_any;  // (float32 unless logits_f16: only the wavefront kernel then reads them)
    if (k > GR4AD_MAX_BEAM || V > GR4AD_MAX_CODEBOOK || (int64_t)n * V >= 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    if (ws_bytes < select_workspace_bytes(B, n, V, k) || ((uintptr_t)ws % 8)) return GR4AD_EWORKSPACE;
    const int m = k < V ? k : V;
    const int64_t rows = (int64_t)B * n;
    if (rows > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    const SelectPlan p = select_plan(B, n, V, k);
    unsigned long long *cand = (unsigned long long *)ws;
    int *req_count = (int *)((char *)ws + p.counts), *todo_count = (int *)((char *)ws + p.todo_count);
    const bool wave_path = V <= 8192 && V % 4 == 0 && ((uintptr_t)logits % 16) == 0;
    const Survivors out = {parent, tok, score, sid_old, sid_new, anc_old, anc_new, T, level};
    // (in one round of workgroups, of which two share a compute unit up to 8192 tokens; us, two launches / one: 64 requests of 256 tokens, k = 16 10.4 / 7.7; of 4096, k = 128
    // 15.8 / 9.0; of 8192, k = 256 23.4 / 11.5; of 16384, k = 128 21.1 / 13.8; but 1024 requests of 256 tokens 15.8 / 20.0, of 8192 36.8 / 41.2)
    if (n == 1 && B <= (wave_path ? 512 : 256)) {
        if (wave_path && V <= 2048)
            return logits_f16 ? launch_select_single<8, true, true, _Float16>(logits_any, cum, B, V, k, out, st) : launch_select_single<4, true, true, float>(logits_any, cum, B, V, k, out, st);
        if (wave_path && logits_f16) return launch_select_single<8, true, false, _Float16>(logits_any, cum, B, V, k, out, st);
        if (wave_path && V <= 4096) return launch_select_single<4, true, false, float>(logits_any, cum, B, V, k, out, st);
        if (wave_path) return launch_select_single<8, true, false, float>(logits_any, cum, B, V, k, out, st);
        if (V <= 4096) return launch_select_single<4, false, false, float>(logits_any, cum, B, V, k, out, st);
        return launch_select_single<16, false, false, float>(logits_any, cum, B, V, k, out, st);
    }
    // Request-level bound (several rows per request, a cut smaller than the row): see row_bounds.  One row per request is its own cut: a bound would only
    // read the row twice.
    const bool bounded = wave_path && n > 1 && k <= V && !rows_cut_alone(rows, n, V, m);
    {
        // algorithmic bytes: every logit once; the candidates written depend on the data (between k per request and m per row):
        // the lower bound is counted when the request-level bound is in use
        ProfScope ps(KC_SELECT_ROWS, st, 0.0, (double)rows * V * (logits_f16 ? 2 : 4) + (bounded ? (double)B * k : (double)rows * m) * 8);
        if (wave_path) {
            const RowsLaunch a = {st, logits_any, logits_f16, cum, n, V, m, cand, (float *)((char *)ws + p.scores), p.R, req_count, p.count_pitch,
                            (int2 *)((char *)ws + p.todo), todo_count, n > 1 && k <= V};
            int s;
            if (bounded) {
                if ((s = launch_rows(a, B, 3))) return s;
                GR4AD_LAUNCH_CHECK();
                if ((s = launch_rows(a, rows, 2))) return s;
                GR4AD_LAUNCH_CHECK();
                if ((s = launch_rows(a, rows, 1))) return s;
            } else if ((s = launch_rows(a, rows, 0))) {
                return s;
            }
        } else {
            const size_t stage_bytes = (size_t)m * sizeof(unsigned long long);  // <= 32 KB (GR4AD_MAX_BEAM)
            if (V <= 1024)
                hipLaunchKernelGGL(select_rows<4>, dim3((unsigned)rows), dim3(256), stage_bytes, st, logits, cum, n, V, m, cand);
            else if (V <= 4096)
                hipLaunchKernelGGL(select_rows<16>, dim3((unsigned)rows), dim3(256), stage_bytes, st, logits, cum, n, V, m, cand);
            else if (V <= 8192)
                hipLaunchKernelGGL(select_rows<32>, dim3((unsigned)rows), dim3(256), stage_bytes, st, logits, cum, n, V, m, cand);
            else
                hipLaunchKernelGGL(select_rows<64>, dim3((unsigned)rows), dim3(256), stage_bytes, st, logits, cum, n, V, m, cand);
        }
        GR4AD_LAUNCH_CHECK();
    }
    ProfScope ps(KC_SELECT_REQUEST, st, 0.0, (bounded ? (double)B * k : (double)rows * m) * 8 + (double)B * k * 12);  // (same convention)
    hipLaunchKernelGGL(select_request, dim3((unsigned)B), dim3(SELB_THREADS), 0, st, (const unsigned long long *)ws, (int64_t)n * m, bounded ? req_count : nullptr, p.count_pitch, V, k, n, out);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// ---------------------------------------------------------------------------
// The same selection for callers that cannot allocate device memory (code under HIP graph capture, tight serving loops,
// harnesses that forbid hipMalloc): the candidate lists, the scores behind the request bounds and the counts live in a fixed device
// array of this library instead of a caller workspace.  Host code never uses the array's name as an address: the device
// address is looked up once per device and kept.  Every call on a GPU shares that GPU's array (overlapping calls race);
// nothing in it has to start at zero - the counts are written by a kernel of every call before they are read.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[GR4AD_SELECT_STATIC_BYTES];

namespace {
const int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device (NULL: not looked up yet)
}  // namespace

extern "C" int gr4ad_op_select_static(const float *logits, const float *cum, int32_t B, int32_t n, int32_t V, int32_t k, int32_t *parent,
                                      int32_t *tok, float *score, void *hip_stream) {
    if (!logits || !parent || !tok || !score) return gr4ad_set_thread_error(GR4AD_EINVAL, "gr4ad_op_select_static: a required pointer is NULL");
    if (B < 1 || n < 1 || V < 1 || k < 1 || (int64_t)k > (int64_t)n * V)
        return gr4ad_set_thread_error(GR4AD_EINVAL, "gr4ad_op_select_static: need B, n, V >= 1 and 1 <= k <= n*V");
    if (k > GR4AD_MAX_BEAM || V > GR4AD_MAX_CODEBOOK)
        return gr4ad_set_thread_error(GR4AD_EUNSUPPORTED, "gr4ad_op_select_static: k > %d or V > %d", GR4AD_MAX_BEAM, GR4AD_MAX_CODEBOOK);
    const int m = k < V ? k : V;
    // (computed in 64 bits before select_workspace_bytes multiplies the sizes)
    if ((double)B * n * m * 8.0 > (double)GR4AD_SELECT_STATIC_BYTES || select_workspace_bytes(B, n, V, k) > (size_t)GR4AD_SELECT_STATIC_BYTES)
        return gr4ad_set_thread_error(GR4AD_EWORKSPACE, "gr4ad_op_select_static: B=%d n=%d V=%d k=%d needs more than the %u bytes of static scratch", B, n,
                                      V, k, (unsigned)GR4AD_SELECT_STATIC_BYTES);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return gr4ad_set_thread_error(GR4AD_EHIP, "gr4ad_op_select_static: hipGetDevice failed");
    if (dev < 0 || dev >= kMaxDevices) return gr4ad_set_thread_error(GR4AD_EUNSUPPORTED, "gr4ad_op_select_static: device index %d", dev);
    if (!g_scratch_ptr[dev]) {  // once per device, with that device current: each GPU holds its own copy of the array
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return gr4ad_set_thread_error(GR4AD_EHIP, "gr4ad_op_select_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    const int s = launch_select(logits, 0, cum, B, n, V, k, g_scratch_ptr[dev], (size_t)GR4AD_SELECT_STATIC_BYTES, parent, tok, score, nullptr, nullptr,
                                nullptr, nullptr, 0, 0, (hipStream_t)hip_stream);
    return s == GR4AD_OK ? s : gr4ad_set_thread_error(s, "gr4ad_op_select_static: selection failed: %s", gr4ad_strerror(s));
}
