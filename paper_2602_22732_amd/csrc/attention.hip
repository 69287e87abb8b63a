// Attention kernels of the decoder layer (section 3.2: cross-attention between
// decoder states and the context X, self-attention over decoder states).
//
//  * cross_attn_flash_bf16  beam-shared cross-attention (section 4.2, Beam-Shared
//                           KV Caching): one workgroup owns a block of beams of one
//                           (request, head); the context K/V tile is staged in LDS
//                           once and reused by every beam of the block.  MFMA, online
//                           softmax.
//  * cross_attn_simple<T>   one wavefront per (beam row, head), any shape; float32
//                           path and fallback.
//  * context_attn_flash_bf16  the lazy layers' cross-attention in absorbed form
//                           (keys = values = the raw context rows, one query of
//                           width d per (position, head)): one pass over the
//                           context, MFMA, online softmax.
//  * context_scores / context_sums  the same for few requests, tiles side by side.
//  * self_attn_step<T>      autoregressive self-attention of the new position over
//                           the beam path's earlier positions (at most T keys), read
//                           in place from the buffers their levels wrote, through
//                           the beams' ancestor table (no reorder copy).
//  * trunk_self_attn<T>     causal self-attention over the T trunk positions.
#include <stdlib.h>

#include <type_traits>

#include "common.h"

// ---------------------------------------------------------------------------
// simple cross-attention: wave per (row, head)
// ---------------------------------------------------------------------------
// AHEAD (heads of at most 64 columns): with few workgroups a wavefront's time is a few memory latencies, so the keys and values of a tile of 64 keys are requested
// together, before the scores are formed.  Otherwise the values follow the softmax, 16 keys at a time, and keys past the end cost nothing: the rule is at the
// launch.
template <typename T, bool AHEAD>
__global__ __launch_bounds__(256) void cross_attn_simple(const T *__restrict__ q, int64_t ldq, const T *__restrict__ kv,
                                                         const int32_t *__restrict__ ctx_len, T *__restrict__ out, int64_t ldo,
                                                         int64_t rows, int n, int q_stride, int S, int d, int H) {
    __shared__ __attribute__((aligned(16))) float sq[4][128];
    __shared__ float sp[4][64];
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
    const int64_t wid = (int64_t)blockIdx.x * 4 + wv;
    if (wid >= rows * H) return;
    const int64_t row = wid / H;
    const int h = (int)(wid % H);
    const int64_t b = row / n;
    const int dh = d / H;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const float scale = 1.0f / sqrtf((float)dh);
    const T *qr = q + (row - b * (n - q_stride)) * ldq + h * dh;
    const float q0 = AHEAD && lane < dh ? to_f(qr[lane]) : 0.0f;  // (put down once the first tile's loads are on their way)
    if (!AHEAD)
        for (int c = lane; c < dh; c += 64) sq[wv][c] = to_f(qr[c]) * scale;
    const T *kbase = kv + b * (int64_t)S * 2 * d + h * dh;  // key j at kbase + j*2d, value at + d
    constexpr int E = 16 / sizeof(T), U = 32 / E;           // values of a 16-byte load; loads of 32 columns
    const bool vec = ((uintptr_t)kbase % 16) == 0 && (2 * d) % E == 0 && dh % E == 0;
    float m = -INFINITY, l = 0.0f, acc[2] = {0.0f, 0.0f};
    constexpr int G = AHEAD ? 64 : 16;  // keys whose values are in flight
    for (int j0 = 0; j0 < len; j0 += 64) {
        const int j = j0 + lane, cnt = (len - j0) < 64 ? (len - j0) : 64;
        float v0[G], v1[AHEAD ? 1 : G];
        auto load_values = [&](int j1) {  // (keys past the tile's last re-read it and count as zero: 0 * v is no zero where v is infinite)
#pragma unroll
            for (int u = 0; u < G; u++) {
                const T *vr = kbase + (int64_t)(j0 + (j1 + u < cnt ? j1 + u : cnt - 1)) * 2 * d + d;
                v0[u] = lane < dh ? to_f(vr[lane]) : 0.0f;
                if constexpr (!AHEAD) v1[u] = lane + 64 < dh ? to_f(vr[lane + 64]) : 0.0f;
            }
        };
        const T *kr = kbase + (int64_t)(j < len ? j : len - 1) * 2 * d;
        float s = 0.0f;
        if (AHEAD ? vec : vec && j < len) {  // 16 bytes per load, same order of additions
            if constexpr (AHEAD) {
                uint4 raw[U];
#pragma unroll
                for (int u = 0; u < U; u++) raw[u] = *(const uint4 *)(kr + (u * E < dh ? u * E : 0));
                load_values(0);
                __builtin_amdgcn_sched_barrier(0);
                if (j0 == 0) sq[wv][lane] = q0 * scale;
#pragma unroll
                for (int u = 0; u < U; u++)
#pragma unroll
                    for (int e = 0; e < E; e++)
                        if (u * E < dh) s = fmaf(sq[wv][u * E + e], to_f(((const T *)&raw[u])[e]), s);
            }
#pragma unroll 4
            for (int c = AHEAD ? 32 : 0; c < dh; c += E) {
                const uint4 more = *(const uint4 *)(kr + c);
#pragma unroll
                for (int e = 0; e < E; e++) s = fmaf(sq[wv][c + e], to_f(((const T *)&more)[e]), s);
            }
        } else if (AHEAD || j < len) {
            if constexpr (AHEAD) {
                load_values(0);
                if (j0 == 0) sq[wv][lane] = q0 * scale;
            }
            for (int c = 0; c < dh; c++) s = fmaf(sq[wv][c], to_f(kr[c]), s);
        }
        if (j >= len) s = -INFINITY;
        const float mnew = fmaxf(m, wave_max(s));
        const float p = (j < len) ? __expf(s - mnew) : 0.0f;
        const float alpha = __expf(m - mnew);  // m = -inf on the first tile gives 0
        l = l * alpha + wave_sum(p);
        m = mnew;
        sp[wv][lane] = p;
        acc[0] *= alpha;
        acc[1] *= alpha;
        for (int j1 = 0; j1 < cnt; j1 += G) {
            if constexpr (!AHEAD) load_values(j1);
            if (j1 + G > cnt) {
#pragma unroll
                for (int u = 0; u < G; u++)
                    if (j1 + u >= cnt) {
                        v0[u] = 0.0f;
                        if constexpr (!AHEAD) v1[u] = 0.0f;
                    }
            }
#pragma unroll
            for (int u = 0; u < G; u++) {
                const float pj = j1 + u < cnt ? sp[wv][j1 + u] : 0.0f;
                acc[0] = fmaf(pj, v0[u], acc[0]);
                if constexpr (!AHEAD) acc[1] = fmaf(pj, v1[u], acc[1]);
            }
        }
    }
    const float inv = 1.0f / l;
    if (lane < dh) out[row * ldo + h * dh + lane] = from_f<T>(acc[0] * inv);
    if (lane + 64 < dh) out[row * ldo + h * dh + lane + 64] = from_f<T>(acc[1] * inv);
}

// ---------------------------------------------------------------------------
// beam-shared flash cross-attention on the matrix cores (bf16)
// ---------------------------------------------------------------------------
// Values transposed per (request, head): vt[b][h][c][s] = V[b][s][h*dh+c] for s < len_b, 0 beyond
// (s runs to Spad = S rounded up to 64), so a tile of V^T is row-major like a tile of K.
__global__ __launch_bounds__(256) void v_transpose_kernel(const bf16 *__restrict__ kv, const int32_t *__restrict__ ctx_len,
                                                          bf16 *__restrict__ vt, int S, int Spad, int d, int src_pitch, int src_col0) {
    __shared__ bf16 tile[64][66];
    const int b = blockIdx.z, c0 = blockIdx.y * 64, s0 = blockIdx.x * 64;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const int tid = threadIdx.x;
    for (int i = tid; i < 64 * 8; i += 256) {  // 64 rows (s) x 8 chunks of 8 columns
        const int r = i / 8, ch = i % 8, s = s0 + r;
        uint4 raw = make_uint4(0, 0, 0, 0);
        if (s < len) raw = *(const uint4 *)(kv + ((int64_t)b * S + s) * src_pitch + src_col0 + c0 + ch * 8);
        const bf16 *e = (const bf16 *)&raw;
#pragma unroll
        for (int k = 0; k < 8; k++) tile[r][ch * 8 + k] = e[k];
    }
    __syncthreads();
    for (int i = tid; i < 64 * 8; i += 256) {  // 64 rows (c) x 8 chunks of 8 positions
        const int r = i / 8, ch = i % 8;
        uint4 raw;
        bf16 *e = (bf16 *)&raw;
#pragma unroll
        for (int k = 0; k < 8; k++) e[k] = tile[ch * 8 + k][r];
        *(uint4 *)(vt + ((int64_t)b * d + c0 + r) * Spad + s0 + ch * 8) = raw;
    }
}

// One workgroup: NW wavefronts of 32 beams each of one (request, head).  The context streams through LDS in tiles of 64 keys (K [64 x DH] and
// V^T [DH x 64]), filled by direct global->LDS loads (no staging registers); every beam of the block reuses them.
// LD = 0: the wavefronts load what they use, two tiles double-buffered, one barrier per tile: in between, the wavefronts that share a SIMD drift
// apart, so one's softmax (vector instructions, the larger part) overlaps the other's MFMAs.  For launches that fill the chip many times.
// LD > 0: LD wavefronts of their own load, three tiles in LDS.  With few blocks per compute unit a wavefront's own chain is what counts, and its share
// of a tile's loads (address arithmetic, 25 to 35 cycles to issue each) is a fifth to a third of it: 1 request of 512 keys, d = 512, 1 / 128 / 256 beams 12.1 / 13.1 /
// 13.7 -> 8.3 / 9.2 / 9.3 us; 32 requests, 128 beams 16.2 -> 11.8; 8 requests of 1024 keys, d = 1024, 256 beams 24.9 -> 16.9; 128 such, 128 beams 129 -> 109; head
// width 32, 64 requests of 256 keys, 64 beams 9.0 -> 7.4, of 512 keys, 512 beams 74 -> 67 (before: pairs of tiles double-buffered; head width 32 with up to 64 beams
// to a wavefront).
// Both products are computed transposed,
//   S^T = K Q^T  (keys x beams)   and   O^T = V^T P^T  (head dims x beams),
// so that each lane owns one beam: its running max / sum are lane-local, P^T leaves the
// accumulators of the first product already in the operand layout of the second, and the
// only cross-lane step is one exchange between the two half-waves.  Key rows enter the
// first product with index bits 2 and 3 swapped, which makes the 8 keys a lane holds for
// one MFMA k-step consecutive (one 16-byte chunk of a V^T row).
template <int DH, int NW, int LD>
__global__ __launch_bounds__((NW + LD) * 64, 4) void cross_attn_flash_bf16(const bf16 *__restrict__ q, int64_t ldq, const bf16 *__restrict__ kv, int64_t ldk,
                                                                 const bf16 *__restrict__ vt, int64_t vt_req, const int32_t *__restrict__ ctx_len,
                                                                 bf16 *__restrict__ out, int64_t ldo, int n, int S, int Spad, int H,
                                                                 float scale_log2e, int beam_blocks, int64_t total_blocks,
                                                                 const int32_t *__restrict__ q_first, const int32_t *__restrict__ q_count, int q_stride) {
    constexpr int KCH = DH / 8;                   // 16-byte chunks per K row
    constexpr int K_CHUNKS = 64 * KCH, V_CHUNKS = DH * 8;
    constexpr int STAGE = K_CHUNKS + V_CHUNKS;    // one 64-key tile
    constexpr int BUFS = LD ? 3 : 2;              // tiles in LDS
    constexpr int KSTEPS = DH / 16, MT = DH / 32;
    // A tile is K_CHUNKS/64 wave loads of K rows and V_CHUNKS/64 of V^T rows, dealt in turn to the NLW wavefronts that load.  A wave load fills 64
    // consecutive 16-byte slots; slot p of row r holds chunk p ^ swizzle(r), applied on the global side.  Keys past the context end re-read its last
    // row (masked later); V^T is zero beyond the length.
    constexpr int KI = K_CHUNKS / 64, NLW = LD ? LD : NW, NL = STAGE / 64 / NLW;
    static_assert(STAGE / 64 % NLW == 0, "every loading wavefront issues the same number of loads");
    extern __shared__ bf16x8 smem[];              // BUFS * STAGE chunks
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    // Workgroup ids are dealt to the 8 XCDs in turn, each with an L2 of its own.  The beam blocks of one (request, head) read the
    // same keys and values, so they get consecutive slots of ONE XCD: XCD x owns the contiguous range [x*per, (x+1)*per) of the
    // logical blocks (beam block fastest, then head, then request) and its blocks of one (request, head) start together.
    const int64_t per_xcd = (total_blocks + 7) / 8;
    const int64_t logical = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (logical >= total_blocks) return;
    int beam_block = (int)(logical % beam_blocks);
    int h = (int)((logical / beam_blocks) % H);
    const int b = (int)(logical / ((int64_t)beam_blocks * H));
    if (q_count) {
        // Requests have fewer rows than the launch allows for and their last blocks find no work.  Idle blocks in a short regular pattern
        // starve some of the XCD's shader engines (workgroups are dealt to those in turn), so here the head runs fastest: a request's blocks
        // with work are consecutive.  (1024 requests, 512 beams of which about 20 % distinct: 1.35 ms -> 0.76 ms.)
        const int in = (int)(logical - (int64_t)b * beam_blocks * H);
        h = in % H;
        beam_block = in / H;
    }
    const int frow = lane % 32, hf = lane / 32;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const int ntiles = (len + 63) / 64;
    const int q0 = (beam_block * NW + wave) * 32;
    int64_t req_row = (int64_t)b * n;
    if (q_count) {  // rows packed over the requests
        req_row = q_first[b];
        n = q_count[b];
        if (beam_block * (NW * 32) >= n) return;
    }
    auto meet = [&]() {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    const bf16 *kbase = kv + (int64_t)b * S * ldk + h * DH;
    const bf16 *vbase = vt + (int64_t)b * vt_req + (int64_t)h * DH * Spad;
    auto k_source = [&](int tile, int w) {  // what this lane loads of a tile with load w < KI
        const int id = w * 64 + lane, r = id / KCH, key = tile * 64 + r;
        return kbase + (int64_t)(key < S ? key : S - 1) * ldk + ((id % KCH) ^ ((KCH == 8 ? (r >> 1) : (r >> 2)) & (KCH - 1))) * 8;
    };
    auto v_source = [&](int tile, int w) {  // w >= KI
        const int id = (w - KI) * 64 + lane, r = id / 8;
        return vbase + (int64_t)r * Spad + tile * 64 + ((id % 8) ^ ((r >> 1) & 7)) * 8;
    };
    auto load = [&](const bf16 *src, int buf, int w) {
        __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                         (void __attribute__((address_space(3))) *)(smem + buf * STAGE + w * 64), 16, 0, 0);
    };
    if constexpr (LD > 0) {
        if (wave >= NW) {
            const int me = wave - NW;
            auto issue = [&](int tile, int buf) {
#pragma unroll
                for (int i = 0; i < NL; i++) {
                    const int w = i * LD + me;  // wave-uniform
                    load(w < KI ? k_source(tile, w) : v_source(tile, w), buf, w);
                }
            };
            auto landed = [&](auto k) {  // this loader's share of all but the newest k tiles is there
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(k.value * NL) : "memory");
                meet();
            };
            auto rest = [&](auto self, auto k) {  // the last k + 1 tiles
                if constexpr (k.value >= 0) {
                    if (ntiles > k.value) landed(k);
                    self(self, std::integral_constant<int, k.value - 1>());
                }
            };
            for (int t = 0; t < BUFS && t < ntiles; t++) issue(t, t);
            if (ntiles >= BUFS) {
                landed(std::integral_constant<int, BUFS - 1>());
                int buf = 0;
                for (int t = BUFS; t < ntiles; t++) {  // past the barrier of tile t - BUFS + 1 tile t - BUFS has been read
                    landed(std::integral_constant<int, BUFS - 2>());
                    issue(t, buf);
                    buf = buf + 1 == BUFS ? 0 : buf + 1;
                }
            }
            rest(rest, std::integral_constant<int, BUFS - 2>());
            return;
        }
    }
    // LD = 0: tiles are requested in ascending order, so each of a wavefront's NL loads keeps a running per-lane source address that advances by a
    // fixed step per tile; only a tile that reaches past row S-1 of the keys (the last one, when S is not a multiple of 64) computes clamped
    // addresses.
    const bf16 *lsrc[NL];
    auto issue = [&](int tile, int buf) {  // tile = 0, 1, 2, ... in this order
#pragma unroll
        for (int i = 0; i < NL; i++) {
            const int w = i * NW + wave;
            const bf16 *src = lsrc[i];
            lsrc[i] += w < KI ? 64 * ldk : 64;
            if (w < KI && tile * 64 + 63 > S - 1) src = k_source(tile, w);
            load(src, buf, w);
        }
    };
    if constexpr (LD == 0) {
#pragma unroll
        for (int i = 0; i < NL; i++) {
            const int w = i * NW + wave;
            if (w < KI) {
                const int id = w * 64 + lane, r = id / KCH;
                lsrc[i] = kbase + (int64_t)r * ldk + ((id % KCH) ^ ((KCH == 8 ? (r >> 1) : (r >> 2)) & (KCH - 1))) * 8;
            } else {
                lsrc[i] = v_source(0, w);
            }
        }
    }

    // query fragments stay in registers for the whole kernel
    bf16x8 qf[KSTEPS];
    {
        int row = q0 + frow;
        if (row > n - 1) row = n - 1;  // rows past the end are computed and dropped
        const bf16 *qr = q + ((q_count ? req_row : (int64_t)b * q_stride) + row) * ldq + h * DH;  // (q_stride 0: the same queries for every request)
#pragma unroll
        for (int s = 0; s < KSTEPS; s++) qf[s] = *(const bf16x8 *)(qr + 16 * s + 8 * hf);
    }
    float m_run = -INFINITY, l_run = 0.0f;
    floatx16 o[MT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int v = 0; v < 16; v++) o[mt][v] = 0.0f;
    // key row read by this lane in the first product: bits 2 and 3 of the row index swapped
    const int krow = (frow & 0x13) | ((frow & 4) << 1) | ((frow & 8) >> 1);

    if constexpr (LD == 0) {
        issue(0, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        meet();
        if (ntiles > 1) issue(1, 1);
    }
    int buf = 0;  // the tile's
    for (int tile = 0; tile < ntiles; tile++) {
        if constexpr (LD > 0) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile before is read out; once everybody meets, this one has landed
            meet();
            if (tile > 0) buf = buf + 1 == BUFS ? 0 : buf + 1;
        } else if (tile > 0) {
            // the previous tile is read out and this wave's share of the current one has landed: meet, then refill the free buffer
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            meet();
            if (tile + 1 < ntiles) issue(tile + 1, buf);
            buf ^= 1;
        }
        if (q0 >= n) continue;  // a wavefront without beams
        const bf16x8 *sk = smem + buf * STAGE, *sv = sk + K_CHUNKS;
        // first product: the two 32-key halves are independent accumulation chains, issued in turn; the key fragments of
        // k-step st+1 are read while step st multiplies
        floatx16 s[2];
#pragma unroll
        for (int sub = 0; sub < 2; sub++)
#pragma unroll
            for (int v = 0; v < 16; v++) s[sub][v] = 0.0f;
        auto key_frag = [&](int sub, int st) {
            const int r = sub * 32 + krow;
            return sk[r * KCH + ((2 * st + hf) ^ ((KCH == 8 ? (r >> 1) : (r >> 2)) & (KCH - 1)))];
        };
        bf16x8 kf[2][2];
        kf[0][0] = key_frag(0, 0);
        kf[0][1] = key_frag(1, 0);
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) {
            if (st + 1 < KSTEPS) {
                kf[(st + 1) & 1][0] = key_frag(0, st + 1);
                kf[(st + 1) & 1][1] = key_frag(1, st + 1);
            }
#pragma unroll
            for (int sub = 0; sub < 2; sub++) s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st & 1][sub], qf[st], s[sub], 0, 0, 0);
        }
        // this lane holds, for beam frow, keys tile*64 + 32*sub + 16*(v/8) + 8*hf + v%8.
        // The softmax is the instruction-bound part of the kernel (about three vector instructions per MFMA flop-cycle),
        // so it is kept lean: scores stay raw and the scale enters through one fused multiply-add per element; only a
        // partial last tile is masked; and the running maximum is refreshed lazily -- as long as no score exceeds the
        // maximum in use by more than 2^8 the old one stays, p <= 256 is harmless in fp32 sums and bf16 operands, and
        // the rescaling of O (one multiply per score element) is skipped.
        const int key0 = tile * 64 + 8 * hf;
        bf16x8 pf[4];
        if (tile * 64 + 64 > len) {
#pragma unroll
            for (int sub = 0; sub < 2; sub++)
#pragma unroll
                for (int v = 0; v < 16; v++)
                    if (key0 + 32 * sub + 16 * (v / 8) + (v % 8) >= len) s[sub][v] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int sub = 0; sub < 2; sub++)
#pragma unroll
            for (int v = 0; v < 16; v++) mx = fmaxf(mx, s[sub][v]);
        mx = halves_max(mx) * scale_log2e;  // finite: every tile holds at least one valid key
        if (__builtin_amdgcn_ballot_w64(mx > m_run + 8.0f) != 0) {  // some beam of the wave outgrew its maximum
            const float mnew = mx > m_run + 8.0f ? mx : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - mnew);  // m_run = -inf on the first tile gives 0
            m_run = mnew;
            l_run *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int v = 0; v < 16; v++) o[mt][v] *= alpha;
        }
        const float neg_m = -m_run;
        float lsum = 0.0f;
#pragma unroll
        for (int sub = 0; sub < 2; sub++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[sub][v], scale_log2e, neg_m));
                lsum += pv;
                pf[2 * sub + v / 8][v % 8] = (bf16)pv;  // k-step 2*sub + v/8 of the second product
            }
        l_run += lsum;  // per half-wave partial sum, joined at the end
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                const int r = mt * 32 + frow;
                const bf16x8 vf = sv[r * 8 + ((2 * ks + hf) ^ ((r >> 1) & 7))];
                o[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ks], o[mt], 0, 0, 0);
            }
    }
    const float l = halves_sum(l_run);
    const float inv = 1.0f / l;
    const int row = q0 + frow;
    if (row < n) {
        bf16 *orow = out + (req_row + row) * ldo + h * DH;
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                bf16x4 pk;
#pragma unroll
                for (int j = 0; j < 4; j++) pk[j] = (bf16)(o[mt][4 * g + j] * inv);
                *(bf16x4 *)(orow + mt * 32 + 8 * g + 4 * hf) = pk;
            }
    }
}

size_t cross_attention_workspace_bytes(gr4ad_dtype dtype, int B, int S, int d, int H) {
    const int dh = d / H;
    if (dtype != GR4AD_BF16 || (dh != 32 && dh != 64) || d % 64) return 0;
    const int64_t Spad = (S + 63) / 64 * 64;
    return (size_t)B * d * Spad * sizeof(bf16);
}

int launch_cross_attention_prepare(gr4ad_dtype dtype, const void *kv, const int32_t *ctx_len, void *vt, int B, int S, int d, int H,
                                   hipStream_t st) {
    if (cross_attention_workspace_bytes(dtype, B, S, d, H) == 0) return GR4AD_OK;  // plain kernel reads kv directly
    if (!vt || ((uintptr_t)vt % 16) || ((uintptr_t)kv % 16)) return GR4AD_EWORKSPACE;
    const int Spad = (S + 63) / 64 * 64;
    if (B > 65535 || d / 64 > 65535) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_V_TRANSPOSE, st, 0.0, 2.0 * B * (double)S * d * sizeof(bf16));
    hipLaunchKernelGGL(v_transpose_kernel, dim3(Spad / 64, d / 64, B), dim3(256), 0, st, (const bf16 *)kv, ctx_len, (bf16 *)vt, S, Spad, d, 2 * d,
                       d);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// xt[b][c][s] = x[b][s][c] for s < len_b, zero beyond (s up to the padded length): the operand layout of the
// P*X product of the lazy layers' cross-attention in absorbed form.  x: [B, S, d] bf16, d % 64 == 0.
int launch_context_transpose(const void *x, const int32_t *ctx_len, void *xt, int B, int S, int d, hipStream_t st) {
    const int Spad = (S + 63) / 64 * 64;
    if (B < 1 || S < 1 || d < 64 || d % 64 || B > 65535 || d / 64 > 65535) return GR4AD_EUNSUPPORTED;
    if (!x || !xt || ((uintptr_t)x % 16) || ((uintptr_t)xt % 16)) return GR4AD_EINVAL;
    ProfScope ps(KC_V_TRANSPOSE, st, 0.0, 2.0 * B * (double)S * d * sizeof(bf16));
    hipLaunchKernelGGL(v_transpose_kernel, dim3(Spad / 64, d / 64, B), dim3(256), 0, st, (const bf16 *)x, ctx_len, (bf16 *)xt, S, Spad, d, d, 0);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// Row softmax over the valid keys of a request: one wavefront per row of raw scores sc [rows, ld] (float32);
// row r belongs to request r / rows_per_req.  p[r, s] = softmax_s(scale * sc[r, s]) over s < len, exactly zero
// for len <= s < ld (the product with the values then runs over whole tiles without a mask).
__global__ __launch_bounds__(256) void masked_softmax_rows(const float *__restrict__ sc, bf16 *__restrict__ p, const int32_t *__restrict__ ctx_len,
                                                           int64_t rows, int rows_per_req, int S, int ld, float scale_log2e) {
    const int lane = threadIdx.x % 64;
    const int64_t r = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (r >= rows) return;
    int len = ctx_len ? ctx_len[r / rows_per_req] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const float *row = sc + r * ld;
    bf16 *out = p + r * ld;
    const int full = len & ~3;  // whole float4 groups below len
    float mx = -INFINITY;
    for (int s = lane * 4; s < full; s += 256) {
        const float4 v = *(const float4 *)(row + s);
        mx = fmaxf(fmaxf(mx, fmaxf(v.x, v.y)), fmaxf(v.z, v.w));
    }
    for (int s = full + lane; s < len; s += 64) mx = fmaxf(mx, row[s]);
    mx = wave_max(mx) * scale_log2e;  // scale > 0: the max commutes with it
    float sum = 0.f;
    for (int s = lane * 4; s < full; s += 256) {
        const float4 v = *(const float4 *)(row + s);
        sum += exp2f(fmaf(v.x, scale_log2e, -mx)) + exp2f(fmaf(v.y, scale_log2e, -mx)) + exp2f(fmaf(v.z, scale_log2e, -mx)) +
               exp2f(fmaf(v.w, scale_log2e, -mx));
    }
    for (int s = full + lane; s < len; s += 64) sum += exp2f(fmaf(row[s], scale_log2e, -mx));
    const float inv = 1.f / wave_sum(sum);
    for (int s = lane * 4; s < ld; s += 256) {  // ld % 4 == 0
        float e[4] = {0.f, 0.f, 0.f, 0.f};
        if (s + 3 < len) {
            const float4 v = *(const float4 *)(row + s);
            e[0] = v.x; e[1] = v.y; e[2] = v.z; e[3] = v.w;
#pragma unroll
            for (int k = 0; k < 4; k++) e[k] = exp2f(fmaf(e[k], scale_log2e, -mx)) * inv;
        } else {
#pragma unroll
            for (int k = 0; k < 4; k++)
                if (s + k < len) e[k] = exp2f(fmaf(row[s + k], scale_log2e, -mx)) * inv;
        }
        bf16x4 o;
#pragma unroll
        for (int k = 0; k < 4; k++) o[k] = (bf16)e[k];
        *(bf16x4 *)(out + s) = o;
    }
}

int launch_masked_softmax(const float *sc, void *p, const int32_t *ctx_len, int64_t rows, int rows_per_req, int S, int ld, float scale,
                          hipStream_t st) {
    if (rows < 1 || rows_per_req < 1 || S < 1 || ld < S || ld % 4 || !sc || !p || ((uintptr_t)sc % 16) || ((uintptr_t)p % 8)) return GR4AD_EINVAL;
    const int64_t grid = ceil_div64(rows, 4);
    if (grid > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_SOFTMAX, st, 0.0, (double)rows * S * (sizeof(float) + sizeof(bf16)));
    hipLaunchKernelGGL(masked_softmax_rows, dim3((unsigned)grid), dim3(256), 0, st, sc, (bf16 *)p, ctx_len, rows, rows_per_req, S, ld,
                       scale * 1.4426950408889634f);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// ---------------------------------------------------------------------------
// Lazy layers, cross-attention in absorbed form, one pass over the context.  In that form (eq. trunk with
// q_h . (W_k,h x_s) = (W_k,h^T q_h) . x_s and sum_s p_s W_v,h x_s = W_v,h sum_s p_s x_s) every (position, head) of a
// request is a query q' of width D over keys AND values that are the raw context rows:
//     z[b, i, :] = sum_{s < len_b} softmax_s(scale * q'[b, i, :] . x[b, s, :]) x[b, s, :],      i < RQ = positions * heads.
// One workgroup of 8 wavefronts owns a request and streams its rows once, in double-buffered tiles of 32 rows filled
// by direct global->LDS loads (16-byte piece c of tile row r at position c ^ swz(r), applied on the global side).
// Per tile:
//   1. scores^T [32 rows x 32*QT queries]: the contraction over D is split over the 8/QT wavefronts that share a query
//      tile, each with its slice of q' in registers; all but the first leave their partial sums in LDS;
//   2. the first wavefront of each query tile adds the partials in a fixed order and does the online softmax with
//      lane-local running maximum and sum (a lane owns one query), as the beam-shared kernel above does: raw scores,
//      a maximum that is refreshed only when outgrown by 2^8, unrounded terms in the sum, bf16 terms in the product;
//      it leaves P [queries x 32] and the rescale factor of each query in LDS;
//   3. z^T += x^T P^T: every wavefront owns D/8 columns of z for all queries.  The operand x^T (8 rows of one column
//      per lane) comes from the row-major tile through the transposing LDS read (ds_read_b64_tr_b16: of 16 lanes that
//      pass the addresses of a 4 x 16 block of 16-bit words, four words a lane, lane i receives column i).
// Rows past the length re-read the last valid row (finite) and enter with p = 0.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int ctx_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }  // 16 rows -> 16 values; 4 rows -> 4 groups of 64 bytes

template <int D, int QT>
__global__ __launch_bounds__(512) void context_attn_flash_bf16(const bf16 *__restrict__ qp, const bf16 *__restrict__ x,
                                                               const int32_t *__restrict__ ctx_len, bf16 *__restrict__ z, int RQ, int q_stride, int rq_stride,
                                                               int S, float scale_log2e) {
    constexpr int ROWB = D * 2, CH = D / 8, TILE = 32 * ROWB;  // bytes per row, 16-byte pieces per row, bytes per tile
    constexpr int KSPLIT = 8 / QT, KSL = D / KSPLIT, KSTEPS = KSL / 16;
    constexpr int CW = D / 8, MT = CW / 32;  // columns of z per wavefront
    constexpr int NL = D / 128;              // wave loads per wavefront and tile (32 * CH / 64 dealt to 8 wavefronts)
    constexpr int NPART = QT * (KSPLIT - 1);
    constexpr int PART = 2 * TILE, PBUF = PART + NPART * 4096, ABUF = PBUF + QT * 2048;
    extern __shared__ __attribute__((aligned(16))) char ctx_lds[];  // 2 tiles | partial scores | P | per-query factor
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int b = blockIdx.x;
    const int r32 = lane % 32, g = lane / 32;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const int ntiles = (len + 31) / 32;
    const bf16 *xb = x + (int64_t)b * S * D;

    // (Everything a lane derives from its id for addressing is recomputed per tile from a value the compiler cannot see through:
    // hoisted out of the tile loop these addresses cost some 50 registers on top of the 192 that hold q' and z, and the spills
    // that follow are scratch loads whose waits drain the tile loads in flight.)
    auto issue_tile = [&](int tile, int buf) {
        unsigned lv = lane;
        asm volatile("" : "+v"(lv));
#pragma unroll
        for (int i = 0; i < NL; i++) {
            const int idx = i * 8 + wave;  // wave-uniform: 64 consecutive 16-byte slots of the tile
            const unsigned id = idx * 64 + lv;
            const int r = id / CH, pos = id % CH;
            int row = tile * 32 + r;
            if (row > len - 1) row = len - 1;
            const bf16 *src = xb + (int64_t)row * D + (pos ^ ctx_swz(r)) * 8;
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)src,
                                             (void __attribute__((address_space(3))) *)(ctx_lds + buf * TILE + idx * 1024), 16, 0, 0);
        }
    };

    // first product: wavefront = (query tile qh, slice kq of the contraction)
    const int kq = wave % KSPLIT, qh = wave / KSPLIT;
    bf16x8 qf[KSTEPS];
    {
        int qrow = qh * 32 + r32;
        if (qrow > RQ - 1) qrow = RQ - 1;  // queries past the end are computed and dropped
        const bf16 *qr = qp + ((int64_t)b * q_stride + qrow) * D + kq * KSL + 8 * g;
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) qf[st] = *(const bf16x8 *)(qr + 16 * st);
    }
    float m_run = -INFINITY, l_run = 0.0f;

    // second product: wavefront = columns [wave*CW, wave*CW + CW) of z
    floatx16 o[QT][MT];
#pragma unroll
    for (int qt = 0; qt < QT; qt++)
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int v = 0; v < 16; v++) o[qt][mt][v] = 0.0f;
    issue_tile(0, 0);
    issue_tile(1, 1);  // (unconditional, so that the wait for q' is a count the compiler knows: past the length it re-reads the last row)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    for (int tile = 0; tile < ntiles; tile++) {
        char *xt = ctx_lds + (tile & 1) * TILE;
        const uint32_t xt0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ctx_lds + (tile & 1) * TILE;
        unsigned lv = lane;
        asm volatile("" : "+v"(lv));
        const int r32 = lv % 32, g = lv / 32;
        const int xrow_off = r32 * ROWB, xswz = ctx_swz(r32);
        char *part_w = ctx_lds + PART + (qh * (KSPLIT - 1) + (kq > 0 ? kq - 1 : 0)) * 4096 + r32 * 128;  // this wavefront's partial tile (kq > 0)
        const int prow = qh * 32 + r32;                                                                 // P row of this lane's query
        char *p_w = ctx_lds + PBUF + prow * 64 + g * 8;
        // ---- 1. partial scores^T of this wavefront's slice ----
        floatx16 sacc;
#pragma unroll
        for (int v = 0; v < 16; v++) sacc[v] = 0.0f;
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) {
            const bf16x8 xf = *(const bf16x8 *)(xt + xrow_off + (((kq * (KSL / 8) + 2 * st + g) ^ xswz) * 16));
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, qf[st], sacc, 0, 0, 0);
        }
        // this lane: query r32 of the tile, rows 8i + 4g + e at sacc[4i + e]
        if (kq > 0) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                floatx4 pk;
#pragma unroll
                for (int e = 0; e < 4; e++) pk[e] = sacc[4 * i + e];
                *(floatx4 *)(part_w + (((2 * i + g) ^ (r32 & 7)) * 16)) = pk;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // ---- 2. online softmax (first wavefront of each query tile) ----
        if (kq == 0) {
#pragma unroll
            for (int k = 0; k < KSPLIT - 1; k++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const floatx4 pk = *(const floatx4 *)(part_w + k * 4096 + (((2 * i + g) ^ (r32 & 7)) * 16));
#pragma unroll
                    for (int e = 0; e < 4; e++) sacc[4 * i + e] += pk[e];
                }
            if (tile * 32 + 32 > len) {
#pragma unroll
                for (int v = 0; v < 16; v++)
                    if (tile * 32 + 8 * (v / 4) + 4 * g + (v % 4) >= len) sacc[v] = -INFINITY;
            }
            float mx = -INFINITY;
#pragma unroll
            for (int v = 0; v < 16; v++) mx = fmaxf(mx, sacc[v]);
            mx = halves_max(mx) * scale_log2e;  // finite: every tile holds at least one valid row
            float alpha = 1.0f;
            if (mx > m_run + 8.0f) {
                alpha = __builtin_amdgcn_exp2f(m_run - mx);  // m_run = -inf on the first tile gives 0
                m_run = mx;
                l_run *= alpha;
            }
            const float neg_m = -m_run;
            float lsum = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * i + e], scale_log2e, neg_m));
                    lsum += pv;
                    pk[e] = (bf16)pv;
                }
                *(bf16x4 *)(p_w + ((i ^ ((prow >> 2) & 3)) * 16)) = pk;  // rows 8i + 4g .. + 3: half g of 16-byte piece i
            }
            l_run += lsum;  // per half-wave partial sum, joined at the end
            if (g == 0) *(float *)(ctx_lds + ABUF + prow * 4) = alpha;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // ---- 3. z^T += x^T P^T ----
        // the 8-byte piece this lane passes to the transposing read h (rows 8g + 4h + i16/4 of a 16-row k-step), before the column tile
        const int i16 = lv % 16, b1 = (lv / 16) & 1;
        int tr_off[2], tr_swz[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int sr = 8 * g + 4 * h + i16 / 4;
            tr_off[h] = sr * ROWB + (i16 & 1) * 8;
            tr_swz[h] = ctx_swz(sr);  // (rows 16 apart share the value)
        }
        const int tr_piece = wave * (CW / 8) + 2 * b1 + (i16 % 4) / 2;
#pragma unroll
        for (int qt = 0; qt < QT; qt++) {
            const float a = *(const float *)(ctx_lds + ABUF + (qt * 32 + r32) * 4);
            if (__builtin_amdgcn_ballot_w64(a != 1.0f) != 0) {
#pragma unroll
                for (int mt = 0; mt < MT; mt++)
#pragma unroll
                    for (int v = 0; v < 16; v++) o[qt][mt][v] *= a;
            }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            bf16x8 pf[QT];
#pragma unroll
            for (int qt = 0; qt < QT; qt++) {
                const int q = qt * 32 + r32;
                pf[qt] = *(const bf16x8 *)(ctx_lds + PBUF + q * 64 + (((2 * ks + g) ^ ((q >> 2) & 3)) * 16));
            }
            // (The transposing reads are inline assembly: issued through the builtin, each would be preceded by a wait for every
            // tile load in flight.  The wait below carries them as operands so that the MFMAs stay behind it.)
            intx2 t[MT][2];
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const uint32_t addr = xt0 + ks * 16 * ROWB + tr_off[h] + (((tr_piece + mt * 4) ^ tr_swz[h]) * 16);
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(t[mt][h]) : "v"(addr));
                }
            if (MT == 4)
                asm volatile("s_waitcnt lgkmcnt(0)"
                             : "+v"(t[0][0]), "+v"(t[0][1]), "+v"(t[1][0]), "+v"(t[1][1]), "+v"(t[MT - 2][0]), "+v"(t[MT - 2][1]), "+v"(t[MT - 1][0]),
                               "+v"(t[MT - 1][1]));
            else
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(t[0][0]), "+v"(t[0][1]), "+v"(t[1][0]), "+v"(t[1][1]));
#pragma unroll
            for (int mt = 0; mt < MT; mt++) {
                const intx4 both = __builtin_shufflevector(t[mt][0], t[mt][1], 0, 1, 2, 3);
                const bf16x8 xf = __builtin_bit_cast(bf16x8, both);
#pragma unroll
                for (int qt = 0; qt < QT; qt++) o[qt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf, pf[qt], o[qt][mt], 0, 0, 0);
            }
        }
        // ---- the tile is consumed: refill its buffer two tiles ahead, then wait for the next one ----
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (tile + 2 < ntiles) issue_tile(tile + 2, tile & 1);
        if (tile + 1 < ntiles) {
            if (tile + 2 < ntiles) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (a one-tile request never waited for its second buffer: no load may outlive the workgroup's LDS)
    // 1 / sum of every query through LDS (the last barrier of the loop is behind every read of the factors)
    const float l_tot = halves_sum(l_run);  // (all lanes: the exchange needs both half-waves)
    if (kq == 0 && g == 0) *(float *)(ctx_lds + ABUF + (qh * 32 + r32) * 4) = 1.0f / l_tot;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int qt = 0; qt < QT; qt++) {
        const int q = qt * 32 + r32;
        const float inv = *(const float *)(ctx_lds + ABUF + q * 4);
        if (q < RQ) {
            bf16 *zr = z + ((int64_t)b * rq_stride + q) * D + wave * CW + 4 * g;
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    bf16x4 pk;
#pragma unroll
                    for (int e = 0; e < 4; e++) pk[e] = (bf16)(o[qt][mt][4 * i + e] * inv);
                    *(bf16x4 *)(zr + mt * 32 + 8 * i) = pk;
                }
        }
    }
}

// (more than 64 queries per request run as two launches, each reading the context: beyond 128 the stored-score form moves fewer bytes)
bool context_attention_covers(gr4ad_dtype dtype, int RQ, int d) { return dtype == GR4AD_BF16 && (d == 512 || d == 1024) && RQ >= 1 && RQ <= 128; }

template <int D, int QT>
static int launch_context_flash(const bf16 *qp, const bf16 *x, const int32_t *ctx_len, bf16 *z, int B, int RQ, int q_stride, int rq_stride, int S, float scale,
                                hipStream_t st) {  // RQ <= 32 * QT queries per request, rows rq_stride apart from one request to the next
    auto kern = context_attn_flash_bf16<D, QT>;
    constexpr int LDS_BYTES = 2 * 32 * D * 2 + QT * (8 / QT - 1) * 4096 + QT * 2048 + QT * 128;
    static_assert(LDS_BYTES <= 160 * 1024, "the workgroup's LDS");
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    // flops on the padded length S, both products; bytes: the context once, queries and sums once
    ProfScope ps(KC_CONTEXT_ATTN, st, 4.0 * B * (double)RQ * S * D, (2.0 * B * (double)RQ * D + B * (double)S * D) * sizeof(bf16));
    hipLaunchKernelGGL(kern, dim3((unsigned)B), dim3(512), LDS_BYTES, st, qp, x, ctx_len, z, RQ, q_stride, rq_stride, S, scale * 1.4426950408889634f);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// ---------------------------------------------------------------------------
// The same for few requests: the tiles of a request side by side.  One workgroup per request leaves most of the chip idle below some
// hundred requests and walks its tiles one after the other, 2.9 us each (8 requests of 1024 rows: 93 us).  Here context_scores
// computes the scores of every tile at once, with one workgroup per compute unit dealt to the requests (it keeps its fragments of the
// queries over its tiles, and contexts far shorter than S leave few idle workgroups), and context_sums gives every request D / 64 workgroups (D / 128, with one
// query tile D / 256, where those would outnumber the compute units), one per slice of the columns of z: they repeat the cheap part, the running maxima over the tile
// maxima and the exponentials, and walk the tiles only for their product.  Every sum keeps the order of the one-pass kernel (partial
// scores of the same slices of D, the lazily refreshed maximum tile by tile, the normaliser per half wavefront, z over the rows), so
// the two give the same bits.  8 requests of up to 1024 rows, d = 1024, 64 queries: 93 us in one pass, now 26 (slices of 128 columns 29); one of 512 rows, d = 512: 40, now 12
// (slices of 256 columns, each tile's operands read after the product before: 15).
// ---------------------------------------------------------------------------
#define CTX_CHUNK 8  // tiles whose probabilities are formed together
#define CTX_STAGE (32 * 1024)
#define CTX_SCORE_GROUPS 256  // workgroups of context_scores; more than the most requests

// sc: [B][ntiles][QT][4][64 lanes][4] raw scores as a wavefront holds them; mxs: [B][ntiles][QT][32] scaled maximum of each tile's valid rows
template <int D, int QT>
__global__ __launch_bounds__(512) void context_scores(const bf16 *__restrict__ qp, const bf16 *__restrict__ x, const int32_t *__restrict__ ctx_len,
                                                      float *__restrict__ sc, float *__restrict__ mxs, int RQ, int q_stride, int S, int ntiles, float scale_log2e) {
    constexpr int KSPLIT = 8 / QT, KSL = D / KSPLIT, KSTEPS = KSL / 16;
    constexpr int PART = QT * (KSPLIT - 1) * 4096;
    __shared__ __attribute__((aligned(16))) char parts[2 * PART];  // (two tiles: one barrier each)
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int b = blockIdx.y;
    const int r32 = lane % 32, g = lane / 32, kq = wave % KSPLIT, qh = wave / KSPLIT;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    if ((int)blockIdx.x * 32 >= len) return;
    const int qrow = qh * 32 + r32 < RQ ? qh * 32 + r32 : RQ - 1;
    const bf16 *qr = qp + ((int64_t)b * q_stride + qrow) * D + kq * KSL + 8 * g;
    bf16x8 qf[KSTEPS];
#pragma unroll
    for (int st = 0; st < KSTEPS; st++) qf[st] = *(const bf16x8 *)(qr + 16 * st);
    char *part = parts;
    for (int tile = blockIdx.x; tile * 32 < len; tile += gridDim.x, part = part == parts ? parts + PART : parts) {
        const int row = tile * 32 + r32 < len ? tile * 32 + r32 : len - 1;
        const bf16 *xr = x + ((int64_t)b * S + row) * D + kq * KSL + 8 * g;
        bf16x8 xf[KSTEPS];
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) xf[st] = *(const bf16x8 *)(xr + 16 * st);
        __builtin_amdgcn_sched_barrier(0);  // (every load on its way before the first product: one latency)
        floatx16 s;
#pragma unroll
        for (int v = 0; v < 16; v++) s[v] = 0.0f;
#pragma unroll
        for (int st = 0; st < KSTEPS; st++) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[st], qf[st], s, 0, 0, 0);
        if (kq > 0) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                floatx4 pk;
#pragma unroll
                for (int e = 0; e < 4; e++) pk[e] = s[4 * i + e];
                *(floatx4 *)(part + (qh * (KSPLIT - 1) + kq - 1) * 4096 + (i * 64 + lane) * 16) = pk;
            }
        }
        __syncthreads();
        if (kq > 0) continue;
#pragma unroll
        for (int k = 0; k < KSPLIT - 1; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const floatx4 pk = *(const floatx4 *)(part + (qh * (KSPLIT - 1) + k) * 4096 + (i * 64 + lane) * 16);
#pragma unroll
                for (int e = 0; e < 4; e++) s[4 * i + e] += pk[e];
            }
        const int64_t unit = ((int64_t)b * ntiles + tile) * QT + qh;
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            floatx4 pk;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                pk[e] = s[4 * i + e];
                if (tile * 32 + 8 * i + 4 * g + e < len) mx = fmaxf(mx, pk[e]);
            }
            *(floatx4 *)(sc + unit * 1024 + (i * 64 + lane) * 4) = pk;
        }
        mx = halves_max(mx) * scale_log2e;
        if (g == 0) mxs[unit * 32 + r32] = mx;
    }
}

template <int D, int QT, int COLS>
__global__ __launch_bounds__(512) void context_sums(const bf16 *__restrict__ x, const int32_t *__restrict__ ctx_len, const float *__restrict__ sc,
                                                    const float *__restrict__ mxs, bf16 *__restrict__ z, int RQ, int rq_stride, int S, int nt_max,
                                                    float scale_log2e) {
    constexpr int ROWB = COLS * 2, CH = COLS / 8;                   // bytes and 16-byte pieces of a staged row
    constexpr int TS = CTX_STAGE / (32 * ROWB);                     // tiles per stage (2, 4 or 8)
    static_assert(CTX_CHUNK % TS == 0 && QT * (COLS / 32) <= 8, "a chunk is whole stages, a wavefront has 32 queries and 32 columns");
    constexpr int UPW = CTX_CHUNK * QT / 8;                         // (tile, query tile) units of probabilities per wavefront and chunk
    constexpr int PB = 3 * CTX_STAGE, MB = PB + CTX_CHUNK * QT * 2048, AB = MB + CTX_CHUNK * QT * 128, LB = AB + 2 * CTX_CHUNK * QT * 128,
                  IB = LB + CTX_CHUNK * QT * 256;
    extern __shared__ __attribute__((aligned(16))) char ctx_lds[];  // 3 stages | P | maxima in use | rescale factors (two chunks) | sums | 1/l
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int b = blockIdx.y, slice = blockIdx.x;
    const int r32 = lane % 32, g = lane / 32;
    int len = ctx_len ? ctx_len[b] : S;
    len = len < 1 ? 1 : (len > S ? S : len);
    const int ntiles = (len + 31) / 32, nstages = (ntiles + TS - 1) / TS;
    const bf16 *xb = x + (int64_t)b * S * D + slice * COLS;
    const float *scb = sc + (int64_t)b * nt_max * QT * 1024, *mxb = mxs + (int64_t)b * nt_max * QT * 32;

    auto swz = [](int r) { return CH >= 16 ? ctx_swz(r) : ((r & 3) << 1) | ((r >> 2) & 1); };
    auto issue_stage = [&](int st) {  // rows st*TS*32 .. of this workgroup's columns (past the length: the last valid row again)
        char *dst = ctx_lds + (st % 3) * CTX_STAGE;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int id = (i * 8 + wave) * 64 + lane, r = id / CH, pos = id % CH;
            int row = st * TS * 32 + r;
            if (row > len - 1) row = len - 1;
            __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)(xb + (int64_t)row * D + (pos ^ swz(r)) * 8),
                                             (void __attribute__((address_space(3))) *)(dst + (i * 8 + wave) * 1024), 16, 0, 0);
        }
    };
    // scores of this wavefront's units and, in the first QT wavefronts, the tile maxima of the chunk from tile c0 on, a chunk ahead
    floatx4 sreg[UPW][4];
    float mreg[CTX_CHUNK];
    auto load_chunk = [&](int c0) {
#pragma unroll
        for (int k = 0; k < UPW; k++) {
            const int u = wave + k * 8;
            int t = c0 + u / QT;
            if (t > ntiles - 1) t = ntiles - 1;
#pragma unroll
            for (int i = 0; i < 4; i++) sreg[k][i] = *(const floatx4 *)(scb + ((int64_t)t * QT + u % QT) * 1024 + (i * 64 + lane) * 4);
        }
        if (wave < QT) {
#pragma unroll
            for (int t = 0; t < CTX_CHUNK; t++) mreg[t] = mxb[((c0 + t < ntiles ? c0 + t : ntiles - 1) * QT + wave) * 32 + r32];
        }
    };
    load_chunk(0);
    issue_stage(0);
    if (nstages > 1) issue_stage(1);

    float m_run = -INFINITY, l_run = 0.0f, areg[CTX_CHUNK];  // (first QT wavefronts: lane = query r32, half g)
    const int qt = wave / (COLS / 32), ct = wave % (COLS / 32);  // second product: query tile, 32 columns (wavefronts past the last query tile load and wait)
    floatx16 o;
#pragma unroll
    for (int v = 0; v < 16; v++) o[v] = 0.0f;
    // transposing reads: see context_attn_flash_bf16
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ctx_lds;
    const int i16 = lane % 16, piece = ct * 4 + 2 * ((lane / 16) & 1) + (i16 % 4) / 2;
    uint32_t tr_off[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int sr = 8 * g + 4 * h + i16 / 4;
        tr_off[h] = (uint32_t)(sr * ROWB + (i16 & 1) * 8 + ((piece ^ swz(sr)) * 16));
    }
    int par = 0;
    for (int c0 = 0; c0 < ntiles; c0 += CTX_CHUNK, par ^= 1) {
        float *mA = (float *)(ctx_lds + MB), *aA = (float *)(ctx_lds + AB) + par * CTX_CHUNK * QT * 32, *lS = (float *)(ctx_lds + LB);
        // ---- the maximum in use at every tile of the chunk ----
        if (wave < QT) {
#pragma unroll
            for (int t = 0; t < CTX_CHUNK; t++) {
                const float mx = mreg[t];
                float alpha = 1.0f;
                if (c0 + t < ntiles && mx > m_run + 8.0f) {
                    alpha = __builtin_amdgcn_exp2f(m_run - mx);
                    m_run = mx;
                }
                areg[t] = alpha;
                if (g == 0) { mA[(t * QT + wave) * 32 + r32] = m_run; aA[(t * QT + wave) * 32 + r32] = alpha; }
            }
        }
        __syncthreads();
        // ---- probabilities ----
#pragma unroll
        for (int k = 0; k < UPW; k++) {
            const int u = wave + k * 8, t = u / QT, q = (u % QT) * 32 + r32;
            if (c0 + t < ntiles) {
                const float neg_m = -mA[u * 32 + r32];
                float lsum = 0.0f;
                char *p_w = ctx_lds + PB + t * (QT * 2048) + q * 64 + g * 8;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    bf16x4 pk;
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const float s = (c0 + t) * 32 + 8 * i + 4 * g + e < len ? sreg[k][i][e] : -INFINITY;
                        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s, scale_log2e, neg_m));
                        lsum += pv;
                        pk[e] = (bf16)pv;
                    }
                    *(bf16x4 *)(p_w + ((i ^ ((q >> 2) & 3)) * 16)) = pk;
                }
                lS[u * 64 + lane] = lsum;
            }
        }
        __syncthreads();
        if (wave < QT) {
#pragma clang fp contract(off)
#pragma unroll
            for (int t = 0; t < CTX_CHUNK; t++)
                if (c0 + t < ntiles) {
                    l_run *= areg[t];
                    l_run += lS[(t * QT + wave) * 64 + lane];
                }
        }
        if (c0 + CTX_CHUNK < ntiles) load_chunk(c0 + CTX_CHUNK);
        // ---- z^T += x^T P^T over the chunk's stages ----
        float alpha[CTX_CHUNK];  // rescale factors of the chunk's tiles
#pragma unroll
        for (int t = 0; t < CTX_CHUNK; t++) alpha[t] = qt < QT ? aA[(t * QT + qt) * 32 + r32] : 1.0f;
        struct Fragments { intx2 w[2][2]; intx4 p[2]; };
        Fragments f0, f1;
#pragma unroll
        for (int s = 0; s < CTX_CHUNK / TS; s++) {
            const int st = c0 / TS + s;
            if (st >= nstages) break;
            // this wavefront's share of the stage has landed (the next stage's loads, and younger ones, may be in flight); after the
            // barrier everybody's has, and the stage before it is read out: its buffer takes stage st + 2
            if (st + 1 < nstages) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (st + 2 < nstages) issue_stage(st + 2);
            if (qt >= QT) continue;
            // the six reads of a tile are on their way under the products of the one before
            auto read = [&](Fragments &f, int tt) {
                const int q = qt * 32 + r32;
                const uint32_t xa = lds0 + (st % 3) * CTX_STAGE + tt * 32 * ROWB, pa = lds0 + PB + (s * TS + tt) * (QT * 2048) + q * 64;
#pragma unroll
                for (int ks = 0; ks < 2; ks++) {
                    asm volatile("ds_read_b128 %0, %1" : "=v"(f.p[ks]) : "v"(pa + (((2 * ks + g) ^ ((q >> 2) & 3)) * 16)));
#pragma unroll
                    for (int h = 0; h < 2; h++) asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(f.w[ks][h]) : "v"(xa + ks * 16 * ROWB + tr_off[h]));
                }
            };
            auto multiply = [&](Fragments &f, int tt, bool behind) {
                __builtin_amdgcn_sched_barrier(0);
                if (behind) asm volatile("s_waitcnt lgkmcnt(6)" ::: "memory");  // (before the copies that the next lines' operands may take)
                else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                if (behind) asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(f.w[0][0]), "+v"(f.w[0][1]), "+v"(f.w[1][0]), "+v"(f.w[1][1]), "+v"(f.p[0]), "+v"(f.p[1]));
                else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.w[0][0]), "+v"(f.w[0][1]), "+v"(f.w[1][0]), "+v"(f.w[1][1]), "+v"(f.p[0]), "+v"(f.p[1]));
                __builtin_amdgcn_sched_barrier(0);
                const float a = alpha[s * TS + tt];
                if (__builtin_amdgcn_ballot_w64(a != 1.0f) != 0) {
#pragma unroll
                    for (int v = 0; v < 16; v++) o[v] *= a;
                }
#pragma unroll
                for (int ks = 0; ks < 2; ks++) {
                    const intx4 both = __builtin_shufflevector(f.w[ks][0], f.w[ks][1], 0, 1, 2, 3);
                    o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), __builtin_bit_cast(bf16x8, f.p[ks]), o, 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // (a read and the wait for it stand in one block: a copy of its registers between the two would be of what they held before)
            const int left = ntiles - st * TS;  // tiles of this stage and later ones, at least one
            if (left >= TS) {
                read(f0, 0);
#pragma unroll
                for (int tt = 0; tt < TS; tt += 2) {
                    read(f1, tt + 1);
                    multiply(f0, tt, true);
                    if (tt + 2 < TS) read(f0, tt + 2);
                    multiply(f1, tt + 1, tt + 2 < TS);
                }
            } else {
#pragma unroll
                for (int tt = 0; tt < TS; tt += 2) {
                    if (tt + 1 < left) {
                        read(f0, tt);
                        read(f1, tt + 1);
                        multiply(f0, tt, true);
                        multiply(f1, tt + 1, false);
                    } else if (tt < left) {
                        read(f0, tt);
                        multiply(f0, tt, false);
                    }
                }
            }
        }
    }
    const float l_tot = halves_sum(l_run);
    float *inv_l = (float *)(ctx_lds + IB);
    if (wave < QT && g == 0) inv_l[wave * 32 + r32] = 1.0f / l_tot;
    __syncthreads();
    const int q = qt * 32 + r32;
    if (qt < QT && q < RQ) {
        const float inv = inv_l[q];
        bf16 *zr = z + ((int64_t)b * rq_stride + q) * D + slice * COLS + ct * 32 + 4 * g;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            bf16x4 pk;
#pragma unroll
            for (int e = 0; e < 4; e++) pk[e] = (bf16)(o[4 * i + e] * inv);
            *(bf16x4 *)(zr + 8 * i) = pk;
        }
    }
}

// Requests up to which the tiles run side by side.  The line lies where the workgroups of context_sums outnumber the compute units (one fits a
// unit, D * QT / 256 to a request); at d = 1024 and two query tiles a little beyond.  Decodes with six lazy layers, one-pass kernel and side by
// side, 1024 context rows: d = 512, 24 queries, 128 requests 1382 and 1225 us; 40 queries, 64 requests 1340 and 1236, 80 requests 1495 and 1521;
// d = 1024, 64 queries, 48 requests 1802 and 1689, 64 requests of 256 rows 1142 and 1150.
static int context_split_most(int RQ, int d) { return RQ <= 32 ? 65536 / d : (d == 512 ? 64 : 48); }
// (more requests than that need none of it; they are told the same size as the most that do, so that a larger batch's scratch serves a smaller one)
size_t context_attention_workspace_bytes(gr4ad_dtype dtype, int B, int RQ, int S, int d) {
    if (!context_attention_covers(dtype, RQ, d)) return 0;
    const int most = context_split_most(RQ, d);
    return (size_t)(B < most ? B : most) * ((S + 31) / 32) * (RQ > 32 ? 2 : 1) * (1024 + 32) * sizeof(float);
}

template <int D, int QT, int COLS>
static int launch_context_split_as(const bf16 *qp, const bf16 *x, const int32_t *ctx_len, bf16 *z, int B, int RQ, int q_stride, int rq_stride, int S, float scale,
                                float *ws, hipStream_t st) {
    auto sums = context_sums<D, QT, COLS>;
    constexpr int LDS_BYTES = 3 * CTX_STAGE + CTX_CHUNK * QT * (2048 + 128 + 256 + 256) + QT * 128;
    static_assert(LDS_BYTES <= 160 * 1024, "the workgroup's LDS");
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)sums, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const int nt = (S + 31) / 32;
    float *mxs = ws + (size_t)B * nt * QT * 1024;
    ProfScope ps(KC_CONTEXT_ATTN, st, 4.0 * B * (double)RQ * S * D, (2.0 * B * (double)RQ * D + B * (double)S * D) * sizeof(bf16));
    const int per_request = nt * B <= CTX_SCORE_GROUPS ? nt : CTX_SCORE_GROUPS / B;
    hipLaunchKernelGGL((context_scores<D, QT>), dim3(per_request, B), dim3(512), 0, st, qp, x, ctx_len, ws, mxs, RQ, q_stride, S, nt,
                       scale * 1.4426950408889634f);
    GR4AD_LAUNCH_CHECK();
    hipLaunchKernelGGL(sums, dim3(D / COLS, B), dim3(512), LDS_BYTES, st, x, ctx_len, (const float *)ws, (const float *)mxs, z, RQ, rq_stride, S, nt,
                       scale * 1.4426950408889634f);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// Slices of 64 columns of z while their workgroups fit the compute units: a quarter (half) of the context's bytes to each.
template <int D, int QT>
static int launch_context_split(const bf16 *qp, const bf16 *x, const int32_t *ctx_len, bf16 *z, int B, int RQ, int q_stride, int rq_stride, int S, float scale,
                                float *ws, hipStream_t st) {
    if (B * (D / 64) <= 256) return launch_context_split_as<D, QT, 64>(qp, x, ctx_len, z, B, RQ, q_stride, rq_stride, S, scale, ws, st);
    return launch_context_split_as<D, QT, 256 / QT>(qp, x, ctx_len, z, B, RQ, q_stride, rq_stride, S, scale, ws, st);
}

// z [B, RQ, d] = attention of the queries qp [B, RQ, d] over the context rows x [B, S, d] as keys and values (above).
int launch_context_attention(gr4ad_dtype dtype, const void *qp, const void *x, const int32_t *ctx_len, void *z, int B, int RQ, int S, int d,
                             float scale, void *ws, hipStream_t st, bool shared_q) {
    if (!context_attention_covers(dtype, RQ, d) || B < 1 || S < 1) return GR4AD_EUNSUPPORTED;
    if (!qp || !x || !z || ((uintptr_t)qp % 16) || ((uintptr_t)x % 16) || ((uintptr_t)z % 8) || ((uintptr_t)ws % 16)) return GR4AD_EINVAL;
    const bf16 *xx = (const bf16 *)x;
    for (int q0 = 0; q0 < RQ; q0 += 64) {  // 64 queries of every request per launch
        const bf16 *q = (const bf16 *)qp + (int64_t)q0 * d;
        bf16 *zz = (bf16 *)z + (int64_t)q0 * d;
        const int nq = RQ - q0 < 64 ? RQ - q0 : 64, qs = shared_q ? 0 : RQ;
        int s;
        if (ws && B <= context_split_most(RQ, d)) {
            float *w = (float *)ws;
            if (d == 1024) s = nq > 32 ? launch_context_split<1024, 2>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, w, st)
                                       : launch_context_split<1024, 1>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, w, st);
            else s = nq > 32 ? launch_context_split<512, 2>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, w, st)
                             : launch_context_split<512, 1>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, w, st);
        } else if (d == 1024) {
            s = nq > 32 ? launch_context_flash<1024, 2>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, st)
                        : launch_context_flash<1024, 1>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, st);
        } else {
            s = nq > 32 ? launch_context_flash<512, 2>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, st)
                        : launch_context_flash<512, 1>(q, xx, ctx_len, zz, B, nq, qs, RQ, S, scale, st);
        }
        if (s) return s;
    }
    return GR4AD_OK;
}

template <int DH, int NW, int LD>
static int launch_flash(const bf16 *q, int64_t ldq, const bf16 *kv, int64_t ldk, const bf16 *vt, int64_t vt_req, const int32_t *ctx_len, bf16 *out, int64_t ldo, int B,
                        int n, int S, int d, int H, hipStream_t st, const DistinctRows *dr, int q_stride) {
    auto kern = cross_attn_flash_bf16<DH, NW, LD>;
    constexpr int LDS_BYTES = (LD ? 3 : 2) * (64 * (DH / 8) + DH * 8) * 16;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const int per_block = NW * 32;
    const int beam_blocks = (n + per_block - 1) / per_block;
    const int64_t total_blocks = (int64_t)beam_blocks * H * B;
    const int64_t grid = (total_blocks + 7) / 8 * 8;
    if (grid > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)DH);
    // flops on the padded length S; bytes: queries and outputs once, keys and values once per request (beam-shared)
    ProfScope ps(KC_XATTN_FLASH, st, 4.0 * B * (double)n * S * d, (2.0 * B * n * d + 2.0 * B * (double)S * d) * sizeof(bf16));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((NW + LD) * 64), LDS_BYTES, st, q, ldq, kv, ldk, vt, vt_req, ctx_len, out, ldo, n, S, (S + 63) / 64 * 64, H, scale_log2e,
                       beam_blocks, total_blocks, dr ? dr->first : nullptr, dr ? dr->count : nullptr, q_stride);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

int launch_cross_attention(gr4ad_dtype dtype, const void *q, int64_t ldq, const void *kv, int64_t ldk, const void *vt, int64_t vt_req, const int32_t *ctx_len,
                           void *out, int64_t ldo, int B, int n, int S, int d, int H, hipStream_t st, const DistinctRows *dr, bool shared_q) {
    if (B <= 0 || n <= 0 || S <= 0 || d <= 0 || H <= 0 || d % H) return GR4AD_EINVAL;
    const int dh = d / H, q_stride = shared_q ? 0 : n;
    if (dh > 128 || (shared_q && dr)) return GR4AD_EUNSUPPORTED;
    if (vt && cross_attention_workspace_bytes(dtype, B, S, d, H) && ldq % 8 == 0 && ldk % 8 == 0 && ldo % 4 == 0 && ((uintptr_t)q % 16) == 0 &&
        ((uintptr_t)out % 8) == 0) {
        const bf16 *qq = (const bf16 *)q, *kk = (const bf16 *)kv, *vv = (const bf16 *)vt;
        bf16 *oo = (bf16 *)out;
        // Where the lines lie, in us, 8 wavefronts that load for themselves / 4 that do / 4 with 4 loaders (blocks of 256 / 128 / 128 beams; one card, others differ by
        // up to 8 %): 1 request of 512 keys, d = 512, 256 beams 13.8 / 10.6 / 9.5; 32 of them 18.4 / 18.7 / 17.5 (512 blocks of 128 beams); 45 of 389 keys, 512 beams 37.1 / 33.9 /
        // 35.7 (1440); 128 of 512 keys, 256 beams 55.1 / 53.9 / 59.3 (2048); 128 of 1024 keys, d = 1024, 256 beams 170 / 174 / 180 and 64 with 512 157 / 164 / 171 (4096).  Many
        // blocks: occupancy hides LDS, barrier and dependent-MFMA latencies, and a staged tile serves twice as many beams.  At most 128 beams: 128
        // requests of 1024 keys, d = 1024, 64 beams 97 / 97 / 95, 128 beams 117 / 113 / 113.  (Distinct rows: n is a bound, most blocks find less.)
        // One or two tiles of keys leave the loaders nothing to run ahead on: 32 requests of 64 keys, d = 1024, 256 beams 12.6 / 14.2 / 12.7 (1024 blocks).  Blocks that at most 64 beams fill by
        // half are better alone, where many share a unit: 128 requests of 100 keys, d = 512, 33 beams (4 without loaders / with) 8.3 / 10.6, 128 beams 18.8 / 16.8.  At head width 32 a tile is half as
        // much work for the same loads: 128 requests, d = 1024, 64 keys, 64 beams 15.3 / 20.9 and 256 beams 33.5 / 41.6; 1024 keys, 64 beams 114 / 127 and 256 beams 250 / 266.
        const int64_t blocks = (int64_t)((n + 127) / 128) * H * B;
        if (dh == 32) {
            if (blocks <= 768 || (n > 64 && n <= 128 && S > 192)) return launch_flash<32, 4, 4>(qq, ldq, kk, ldk, vv, vt_req, ctx_len, oo, ldo, B, n, S, d, H, st, dr, q_stride);
            return launch_flash<32, 4, 0>(qq, ldq, kk, ldk, vv, vt_req, ctx_len, oo, ldo, B, n, S, d, H, st, dr, q_stride);
        }
        if (blocks <= 768 || (n <= 128 && (n > 64 || S > 256))) return launch_flash<64, 4, 4>(qq, ldq, kk, ldk, vv, vt_req, ctx_len, oo, ldo, B, n, S, d, H, st, dr, q_stride);
        if (n <= 128 || (blocks <= 2048 && S > 128) || (n + 255) / 256 * 256 != (n + 127) / 128 * 128)
            return launch_flash<64, 4, 0>(qq, ldq, kk, ldk, vv, vt_req, ctx_len, oo, ldo, B, n, S, d, H, st, dr, q_stride);
        return launch_flash<64, 8, 0>(qq, ldq, kk, ldk, vv, vt_req, ctx_len, oo, ldo, B, n, S, d, H, st, dr, q_stride);
    }
    if (dr) return GR4AD_EUNSUPPORTED;
    const int64_t rows = (int64_t)B * n;
    const int64_t grid = ceil_div64(rows * H, 4);
    if (grid > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_XATTN_SIMPLE, st, 4.0 * B * (double)n * S * d, (2.0 * B * n * d + 2.0 * B * (double)S * d) * (dtype == GR4AD_BF16 ? 2 : 4));
    // Ahead where most of the tiles' 64 keys exist and the registers (three wavefronts per SIMD) suffice: head width 32, 64 keys, up to 512 workgroups 9.5 us, 7.5 ahead,
    // 16384 workgroups 140, 156 ahead; 65 keys, 512 workgroups 12.4, 14.4 ahead; 5 keys, 512 workgroups 6.9, 10.8 ahead.
    const bool ahead = dh <= 64 && (S <= 64 ? S > 32 : 5 * (int64_t)S > 3 * (((int64_t)S + 63) / 64 * 64)) && grid < 1024;
#define SIMPLE_(T, AHEAD) hipLaunchKernelGGL((cross_attn_simple<T, AHEAD>), dim3((unsigned)grid), dim3(256), 0, st, (const T *)q, ldq, (const T *)kv, ctx_len, (T *)out, ldo, rows, n, q_stride, S, d, H)
    if (dtype == GR4AD_BF16) { if (ahead) SIMPLE_(bf16, true); else SIMPLE_(bf16, false); }
    else if (ahead) SIMPLE_(float, true);
    else SIMPLE_(float, false);
#undef SIMPLE_
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// ---------------------------------------------------------------------------
// self-attention of the new position over the beam path's earlier positions
// ---------------------------------------------------------------------------
// qkv [rows,3d] of the new position; position p < pos of row r is row anc[r*T + p]
// of the [*,3d] buffer level p wrote (keys at column d, values at 2d); the
// query attends to 0..pos.  Beams that share an ancestor read the same row.
// One thread owns 8 consecutive channels of one row (16-byte accesses in bf16); the
// dh/8 threads of a head are neighbouring lanes and join their partial dot products
// with moves between lanes, so every access of a wavefront is one contiguous stretch.
// The positions are a template parameter, so that no branch stands between the loads: the ancestors' numbers, then all keys and values, then the
// sums.  With a branch, and so a wait, per position the eight calls of 1024 requests x 512 beams x 4 positions (d 1024) took 4.92 ms; now 3.93,
// where the last two positions move their bytes (the new rows once, 4.3 GB) at the rate of a large copy.
template <typename T> struct Chunk8;
template <> struct Chunk8<bf16> {
    bf16x8 v;
    __device__ __forceinline__ void load(const bf16 *p) { v = *(const bf16x8 *)p; }
    __device__ __forceinline__ float operator[](int i) const { return (float)v[i]; }
    static __device__ __forceinline__ void store(bf16 *p, const float *o) {
        bf16x8 v;
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = (bf16)o[i];
        *(bf16x8 *)p = v;
    }
};
template <> struct Chunk8<float> {
    floatx4 v[2];
    __device__ __forceinline__ void load(const float *p) {
        v[0] = *(const floatx4 *)p;
        v[1] = *(const floatx4 *)(p + 4);
    }
    __device__ __forceinline__ float operator[](int i) const { return v[i / 4][i % 4]; }
    static __device__ __forceinline__ void store(float *p, const float *o) {
        floatx4 a, b;
#pragma unroll
        for (int i = 0; i < 4; i++) { a[i] = o[i]; b[i] = o[4 + i]; }
        *(floatx4 *)p = a;
        *(floatx4 *)(p + 4) = b;
    }
};

struct LevelRows { const void *p[GR4AD_MAX_LEVELS]; };
struct NoMaps {};
template <typename T, typename MAPS, int POS>
__global__ __launch_bounds__(256) void self_attn_step(const T *__restrict__ qkv, const int32_t *__restrict__ anc, T *__restrict__ out, int64_t rows,
                                                      int Tlev, int d, int H, LevelRows prev, MAPS maps) {
#pragma clang fp contract(off)  // the scaled score is rounded before the maximum is taken off, at every number of positions
    constexpr bool MAPPED = sizeof(MAPS) > sizeof(NoMaps);  // some of the buffers hold distinct rows
    const int cpr = d / 8;        // chunks per row
    const int lph = (d / H) / 8;  // lanes per head: 2, 4, 8 or 16
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool live = gid < rows * cpr;
    const int64_t quot = rows * cpr <= 0x7fffffffLL ? (int64_t)((uint32_t)gid / (uint32_t)cpr) : gid / cpr;  // (a 64-bit division is a hundred instructions)
    const int64_t row = live ? quot : rows - 1;  // idle lanes shadow the last row and store nothing
    const int ch = live ? (int)(gid - quot * cpr) : 0;
    const float scale = 1.0f / sqrtf((float)(d / H));
    int64_t r[POS + 1];
#pragma unroll
    for (int p = 0; p < POS; p++) r[p] = anc[row * Tlev + p];
    r[POS] = row;
    if constexpr (MAPPED) {
#pragma unroll
        for (int p = 0; p <= POS; p++)
            if (maps.map[p]) r[p] = maps.map[p][r[p]];
    }
    Chunk8<T> q, k[POS + 1], v[POS + 1];
#pragma unroll
    for (int i = 0; i <= POS; i++) {
        const int p = i == 0 ? POS : i - 1;  // (the new row's address is known first)
        const T *kvp = (p == POS ? qkv : (const T *)prev.p[p]) + r[p] * 3 * d + ch * 8;
        if (p == POS) q.load(kvp);
        k[p].load(kvp + d);
        v[p].load(kvp + 2 * d);
    }
    __builtin_amdgcn_sched_barrier(0);
    float s[POS + 1];
    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p <= POS; p++) {
        float part = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; i++) part = fmaf(q[i], k[p][i], part);
        // over the head's lph lanes: lane ^ 1, 2, 4, 8 (the mirrors of 8 and of 16 lanes, whose quads and halves agree by then)
        if (lph > 1) part += lane_xor1(part);
        if (lph > 2) part += lane_xor2(part);
        if (lph > 4) part += dpp_move<0x141, 0xF>(part, part);
        if (lph > 8) part += dpp_move<0x140, 0xF>(part, part);
        s[p] = part * scale;
        mx = fmaxf(mx, s[p]);
    }
    float den = 0.0f;
#pragma unroll
    for (int p = 0; p <= POS; p++) { s[p] = __expf(s[p] - mx); den += s[p]; }
    const float inv = 1.0f / den;
    float o8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p <= POS; p++) {
        const float w = s[p] * inv;
#pragma unroll
        for (int i = 0; i < 8; i++) o8[i] = fmaf(w, v[p][i], o8[i]);
    }
    if (live) Chunk8<T>::store(out + row * d + ch * 8, o8);
}

template <typename T, typename MAPS>
static void launch_self_step(int pos, dim3 grid, hipStream_t st, const void *qkv, const int32_t *anc, void *out, int64_t rows, int T_, int d, int H,
                             const LevelRows &lr, const MAPS &maps) {
#define POS_(p) case p: hipLaunchKernelGGL((self_attn_step<T, MAPS, p>), grid, dim3(256), 0, st, (const T *)qkv, anc, (T *)out, rows, T_, d, H, lr, maps); break;
    static_assert(GR4AD_MAX_LEVELS == 8, "one case per position");
    switch (pos) { POS_(0) POS_(1) POS_(2) POS_(3) POS_(4) POS_(5) POS_(6) POS_(7) }
#undef POS_
}

int launch_self_attention_step(gr4ad_dtype dtype, const void *qkv, const LevelBuffers &prev, const int32_t *anc, void *out, int64_t rows,
                               int pos, int T, int d, int H, hipStream_t st, const LevelMaps *maps) {
    // T is the row stride of anc: positions 0..pos-1 are read from it, so pos == T (a step after the last level) is allowed
    if (rows <= 0 || pos < 0 || pos > T || pos >= GR4AD_MAX_LEVELS || T > GR4AD_MAX_LEVELS || d % H) return GR4AD_EINVAL;
    if ((pos > 0 && !anc) || (maps && dtype != GR4AD_BF16)) return GR4AD_EINVAL;
    for (int p = 0; p < pos; p++)
        if (!prev.p[p] || ((uintptr_t)prev.p[p] % 32) || prev.rows[p] < 1) return GR4AD_EINVAL;
    const int dh = d / H;
    if (dh != 16 && dh != 32 && dh != 64 && dh != 128) return GR4AD_EUNSUPPORTED;
    if (((uintptr_t)qkv % 32) || ((uintptr_t)out % 32)) return GR4AD_EUNSUPPORTED;
    const int64_t grid = ceil_div64(rows * (d / 8), 256);
    if (grid > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    // reads q,k,v of the new position and the pos earlier (k,v) pairs of the beam's path, writes the output
    // (beams that share an ancestor share its row: an earlier level contributes at most its own size)
    double units = 4.0 * rows;
    for (int p = 0; p < pos; p++) units += 2.0 * (double)(prev.rows[p] > 0 && prev.rows[p] < rows ? prev.rows[p] : rows);
    ProfScope ps(KC_SELF_STEP, st, 4.0 * rows * (double)(pos + 1) * d, units * d * (dtype == GR4AD_BF16 ? 2 : 4));
    LevelRows lr;
    for (int p = 0; p < GR4AD_MAX_LEVELS; p++) lr.p[p] = p < pos ? prev.p[p] : nullptr;
    const dim3 g((unsigned)grid);
    if (dtype != GR4AD_BF16) launch_self_step<float>(pos, g, st, qkv, anc, out, rows, T, d, H, lr, NoMaps{});
    else if (maps) launch_self_step<bf16>(pos, g, st, qkv, anc, out, rows, T, d, H, lr, *maps);
    else launch_self_step<bf16>(pos, g, st, qkv, anc, out, rows, T, d, H, lr, NoMaps{});
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// ---------------------------------------------------------------------------
// causal self-attention over the trunk positions (lazy layers, eq. trunk)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void trunk_self_attn(const T *__restrict__ qkv, T *__restrict__ out, int64_t rows, int Tlev, int d, int H) {
#pragma clang fp contract(off)  // (as in self_attn_step)
    const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
    const int64_t wid = (int64_t)blockIdx.x * 4 + wv;
    if (wid >= rows * H) return;
    const int64_t row = wid / H;  // b*T + tau
    const int h = (int)(wid % H);
    const int tau = (int)(row % Tlev);
    const int64_t first = row - tau;  // row of position 0 of this request
    const int dh = d / H;
    const float scale = 1.0f / sqrtf((float)dh);
    // All keys and values at once; positions past this one re-read its row and are not used.  (One by one, each behind the sum before it: 55.7 us
    // for 16384 blocks, 6.0 for 6; now 45.0 and 4.6.)
    float qv[2], kv[GR4AD_MAX_LEVELS][2], vv[GR4AD_MAX_LEVELS][2];
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const int c = lane + 64 * e;
        qv[e] = c < dh ? to_f(qkv[row * 3 * d + h * dh + c]) : 0.0f;
#pragma unroll
        for (int p = 0; p < GR4AD_MAX_LEVELS; p++)
            if (p < Tlev && c < dh) {
                const T *src = qkv + (first + (p < tau ? p : tau)) * 3 * d + h * dh + c;
                kv[p][e] = to_f(src[d]);
                vv[p][e] = to_f(src[2 * d]);
            }
    }
    __builtin_amdgcn_sched_barrier(0);
    float s[GR4AD_MAX_LEVELS];
    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < GR4AD_MAX_LEVELS; p++) {
        if (p <= tau) {
            float part = 0.0f;
#pragma unroll
            for (int e = 0; e < 2; e++)
                if (lane + 64 * e < dh) part = fmaf(qv[e], kv[p][e], part);
            s[p] = wave_sum(part) * scale;
            mx = fmaxf(mx, s[p]);
        }
    }
    float den = 0.0f;
#pragma unroll
    for (int p = 0; p < GR4AD_MAX_LEVELS; p++)
        if (p <= tau) { s[p] = __expf(s[p] - mx); den += s[p]; }
    const float inv = 1.0f / den;
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const int c = lane + 64 * e;
        if (c < dh) {
            float o = 0.0f;
#pragma unroll
            for (int p = 0; p < GR4AD_MAX_LEVELS; p++)
                if (p <= tau) o = fmaf(s[p] * inv, vv[p][e], o);
            out[row * d + h * dh + c] = from_f<T>(o);
        }
    }
}

int launch_trunk_self_attention(gr4ad_dtype dtype, const void *qkv, void *out, int B, int T, int d, int H, hipStream_t st) {
    if (B <= 0 || T <= 0 || T > GR4AD_MAX_LEVELS || d % H) return GR4AD_EINVAL;
    if (d / H > 128) return GR4AD_EUNSUPPORTED;
    const int64_t rows = (int64_t)B * T;
    const int64_t grid = ceil_div64(rows * H, 4);
    if (grid > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_TRUNK_SELF, st, 0.0, (double)rows * d * 4 * (dtype == GR4AD_BF16 ? 2 : 4));
    if (dtype == GR4AD_BF16)
        hipLaunchKernelGGL(trunk_self_attn<bf16>, dim3((unsigned)grid), dim3(256), 0, st, (const bf16 *)qkv, (bf16 *)out, rows, T, d, H);
    else
        hipLaunchKernelGGL(trunk_self_attn<float>, dim3((unsigned)grid), dim3(256), 0, st, (const float *)qkv, (float *)out, rows, T, d, H);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}
