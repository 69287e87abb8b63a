// GEMM kernels: C[M,N] = A[M,K] * W[N,K]^T with fused epilogue.
//
// Every linear map of the decoder (section 3.2: the projections of the
// cross-/self-attention and feed-forward sub-layers, the Fuse projection
// and the per-level classifier W_t) is this contraction: activations are
// row-major with the reduction index contiguous, and so are the weights
// ([out,in]), so both MFMA operands stream K-contiguous 16-byte chunks.
//
//  * gemm_simple<T>      64x64 tile, plain FMA, any shape; fallback.
//  * gemm_f32_mfma<T>    float32 operands on the matrix cores.
//  * gemm_bf16_tile<..>  bf16 operands, fp32 accumulation on the matrix cores with
//                        v_mfma_f32_32x32x16_bf16; 32x32 to 128x128 tiles for the
//                        small and middle shapes, operands streamed into LDS,
//                        by wavefronts of their own where tiles are few.
//  * gemm_bf16_panel<..> the small products behind an RMSNorm, a gate or the trunk's
//                        self-attention: the workgroup forms the rows it multiplies.
//  * gemm_bf16_ring<..>  the kernel of the large shapes: persistent, 256x256 tiles,
//                        operands stream global -> LDS without passing registers.
#include <string.h>

#include <algorithm>

#include <type_traits>

#include "common.h"

// An FP8 operand byte (OCP E4M3: sign, 4 exponent bits with bias 7, 3 mantissa bits), decoded in software by the plain kernel.
struct fp8e4m3 { uint8_t v; };
__device__ __forceinline__ float to_f(fp8e4m3 x) {
    const int e = (x.v >> 3) & 15, m = x.v & 7;
    const float a = e ? ldexpf((float)(8 + m), e - 10) : ldexpf((float)m, -9);
    return (x.v & 0x80) ? -a : a;
}

// ---------------------------------------------------------------------------
// epilogue of one element (plain kernel)
// ---------------------------------------------------------------------------
struct Addends { float bias, table, resid; };  // what the epilogue adds to an element
__device__ __forceinline__ Addends epilogue_addends(const GemmEpilogue &e, int64_t row, int col, int N) {
    Addends a = {0.0f, 0.0f, 0.0f};
    if (e.bias) a.bias = e.bias[col];
    if (e.table) a.table = e.table[(e.tok ? (int64_t)e.tok[row] : 0) * N + col];
    if (e.resid) a.resid = e.resid[row * e.ldr + col];
    return a;
}
// a: the element's addends where they were requested ahead (NULL: they are read here; both reading and asking again cost a 64x64 float32 tile 0.9 us)
template <typename T>
__device__ __forceinline__ void epilogue_store(const GemmEpilogue &e, int64_t row, int col, int N, float v, const Addends *a = nullptr) {
    if (e.bias) v += a ? a->bias : e.bias[col];
    if (e.table) v += a ? a->table : e.table[(e.tok ? (int64_t)e.tok[row] : 0) * N + col];
    if (e.act == ACT_SILU) v = v / (1.0f + __expf(-v));
    if (e.resid) v += a ? a->resid : e.resid[row * e.ldr + col];
    if (e.out_f32)
        ((float *)e.C)[row * e.ldc + col] = v;
    else
        ((T *)e.C)[row * e.ldc + col] = from_f<T>(v);
}

// ---------------------------------------------------------------------------
// plain FMA kernel
// ---------------------------------------------------------------------------
// T: operand type; TO: type of C when it is not float32.  FP8 operands: the product row is scaled by a_scale[row] * w_scale.
template <typename T, typename TO = T>
__global__ __launch_bounds__(256) void gemm_simple(const T *__restrict__ A, int64_t lda, const T *__restrict__ W, int64_t ldw,
                                                   int64_t M, int N, int K, GemmEpilogue epi) {
    __shared__ float As[16][65], Ws[16][65];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    const int64_t m0 = (int64_t)blockIdx.x * 64;
    const int n0 = blockIdx.y * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            int idx = tid + i * 256, r = idx / 16, kk = idx % 16;
            int64_t gr = m0 + r;
            int gk = k0 + kk;
            As[kk][r] = (gr < M && gk < K) ? to_f(A[gr * lda + gk]) : 0.0f;
            int gn = n0 + r;
            Ws[kk][r] = (gn < N && gk < K) ? to_f(W[(int64_t)gn * ldw + gk]) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 16; kk++) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; i++) { a[i] = As[kk][ty * 4 + i]; w[i] = Ws[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            int64_t row = m0 + ty * 4 + i;
            int col = n0 + tx * 4 + j;
            if (row < M && col < N) {
                float v = acc[i][j];
                if (epi.a_scale) v *= epi.a_scale[row] * epi.w_scale;
                epilogue_store<TO>(epi, row, col, N, v);
            }
        }
}

// ---------------------------------------------------------------------------
// float32 kernel on the matrix cores (v_mfma_f32_*: float32 operands and sums)
// ---------------------------------------------------------------------------
// The float32 decodes are small (a few to a few thousand rows, K of a few hundred), so a launch is bound by latency: of the loads, and
// of the chain of MFMAs over K.  Fragments come straight from global memory (a lane reads 4 consecutive k of its row, 16 bytes; the
// L1 serves the sharing), with all loads of an unrolled block in flight.  T = 16: a workgroup owns a 16x16 tile and its four
// wavefronts split K, joined through LDS in a fixed order - 12 x 512 x 128 runs on 32 compute units for a chain of 8 MFMAs.
// T = 32: four wavefronts own a 64x64 tile, 32x32 each, for shapes with enough tiles to fill the chip (twice the flops per byte).
// A request's result must not depend on its batch, so both add in one order: the same instruction (v_mfma_f32_16x16x4_f32: T = 32 has four
// accumulators per wavefront, at the rate of one v_mfma_f32_32x32x2_f32) over the same quarters of K, joined in the same way; a wavefront with
// 32x32 elements walks the quarters in turn.
// Replaces 64x64 FMA tiles staged through LDS value by value: 27 us on average for the products of a decode of 4 requests at d = 128,
// now 2.8 to 4 us (64 x 128 x 512 with a residual 4.0, 64 x 512 x 128 behind a norm 4.1; 1024 x 1024 x 512 on 64x64 tiles 19.2).  Needs K % 4 == 0 and 16-byte aligned rows.
template <int T>
__global__ __launch_bounds__(256) void gemm_f32_mfma(const float *__restrict__ A, int64_t lda, const float *__restrict__ W, int64_t ldw, int64_t M,
                                                     int N, int K, GemmEpilogue epi) {
    constexpr int G = T / 16, KB = 16;            // 16x16 tiles of a wavefront each way; k values of one 16-byte load per lane
    constexpr int UN = T == 16 ? 8 : 2;           // blocks of KB whose loads are in flight (2 UN G per lane)
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int64_t m0 = T == 16 ? (int64_t)blockIdx.x * 16 : (int64_t)blockIdx.x * 64 + (wave / 2) * 32;
    const int n0 = T == 16 ? blockIdx.y * 16 : blockIdx.y * 64 + (wave % 2) * 32;
    const int k4 = (lane / 16) * 4;
    const float *a[G], *w[G];
#pragma unroll
    for (int g = 0; g < G; g++) {  // (rows past the edge: never stored)
        const int64_t ar = m0 + g * 16 + lane % 16;
        const int wr = n0 + g * 16 + lane % 16;
        a[g] = A + (ar < M ? ar : M - 1) * lda + k4;
        w[g] = W + (int64_t)(wr < N ? wr : N - 1) * ldw + k4;
    }
    __shared__ float rinv[16];
    __shared__ __attribute__((aligned(16))) float gain[1024];  // its first 1024 values (a read from memory between the norm and the first MFMA is a latency more)
    const int nb = (K + KB - 1) / KB, per = (nb + 3) / 4;  // blocks of KB values of k; blocks in a quarter
    struct Blocks { floatx4 a[UN][G], w[UN][G]; };
    auto load = [&](Blocks &x, int b, int b1) {
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int k = (b + u) * KB + k4;
#pragma unroll
            for (int g = 0; g < G; g++) {
                x.a[u][g] = x.w[u][g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                if (b + u < b1 && k < K) {
                    x.a[u][g] = *(const floatx4 *)(a[g] + (int64_t)(b + u) * KB);
                    x.w[u][g] = *(const floatx4 *)(w[g] + (int64_t)(b + u) * KB);
                }
            }
        }
    };
    auto scale = [&](Blocks &x, int b, int b1) {  // A = RMSNorm(pre_x)
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int k = (b + u) * KB + k4;
            if (b + u < b1 && k < K) x.a[u][0] = *(const floatx4 *)(k < 1024 ? gain + k : (const float *)epi.pre_gain + k) * x.a[u][0] * rinv[lane % 16];
        }
    };
    auto multiply = [&](const Blocks &x, floatx4 (&acc)[G][G]) {
#pragma unroll
        for (int u = 0; u < UN; u++)
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int i = 0; i < G; i++)
#pragma unroll
                    for (int j = 0; j < G; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.a[u][i][e], x.w[u][j][e], acc[i][j], 0, 0, 0);
    };
    auto quarter = [&](int s, floatx4 (&acc)[G][G], Blocks &x, bool loaded) {  // loaded: x holds its first blocks
        const int b0 = s * per, b1 = b0 + per < nb ? b0 + per : nb;
#pragma unroll
        for (int i = 0; i < G; i++)
#pragma unroll
            for (int j = 0; j < G; j++) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int b = b0; b < b1; b += UN) {
            if (!loaded || b > b0) {
                load(x, b, b1);
                if constexpr (T == 16)
                    if (epi.pre_x) scale(x, b, b1);
            }
            multiply(x, acc);
        }
    };
    floatx4 acc[G][G];
    // accumulators: column lane % 16, row 4 * (lane / 16) + v
    if constexpr (T == 16) {
        // Every memory latency of the tile at once: the first operand blocks and what the epilogue adds are requested before the rows are summed up.
        const int64_t row = m0 + threadIdx.x / 16;
        const int col = n0 + threadIdx.x % 16, b0 = wave * per;
        const int g4 = (int)threadIdx.x * 4;
        floatx4 first_gain = {0.0f, 0.0f, 0.0f, 0.0f};
        if (epi.pre_x && g4 < K) first_gain = *(const floatx4 *)((const float *)epi.pre_gain + g4);
        Blocks x;
        Addends add = {0.0f, 0.0f, 0.0f};
        load(x, b0, b0 + per < nb ? b0 + per : nb);
        if (row < M && col < N) add = epilogue_addends(epi, row, col, N);
        if (epi.pre_x) {  // 1/rms of the tile's rows, four per wavefront, as rmsnorm_kernel has it
            *(floatx4 *)(gain + g4) = first_gain;
            float ss[4] = {};
            for (int k = lane * 4; k < K; k += 256)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int64_t r = m0 + wave + 4 * q;
                    const floatx4 v = *(const floatx4 *)(epi.pre_x + (r < M ? r : M - 1) * lda + k);
                    ss[q] += sum_sq4(v[0], v[1], v[2], v[3]);
                }
#pragma unroll
            for (int q = 0; q < 4; q++) ss[q] = wave_sum_dpp(ss[q]);
            const float mine = (lane & 2) ? ((lane & 1) ? ss[3] : ss[2]) : (lane & 1) ? ss[1] : ss[0];  // (one root and two divisions for the four rows)
            const float inv = rms_inv(mine, K, epi.pre_eps);
            if (lane < 4) rinv[wave + 4 * lane] = inv;
            __syncthreads();
            scale(x, b0, b0 + per < nb ? b0 + per : nb);
        }
        quarter(wave, acc, x, true);
        __shared__ float part[4][256];
#pragma unroll
        for (int v = 0; v < 4; v++) part[wave][(4 * (lane / 16) + v) * 16 + lane % 16] = acc[0][0][v];
        __syncthreads();
        const int t = threadIdx.x;
        if (row < M && col < N) epilogue_store<float>(epi, row, col, N, (part[0][t] + part[1][t]) + (part[2][t] + part[3][t]), &add);
    } else {
        floatx4 low[G][G], high[G][G];
        auto join = [&](floatx4 (&sum)[G][G]) {
#pragma unroll
            for (int i = 0; i < G; i++)
#pragma unroll
                for (int j = 0; j < G; j++) sum[i][j] += acc[i][j];
        };
        auto walk = [&](int s, floatx4 (&sum)[G][G]) {  // (blocks of its own: kept over the quarters they went to scratch, 1024 x 1024 x 512 19.3 us to 30.6)
            Blocks x;
            quarter(s, sum, x, false);
        };
        walk(0, low);
        walk(1, acc);
        join(low);
        walk(2, high);
        walk(3, acc);
        join(high);
#pragma unroll
        for (int i = 0; i < G; i++)
#pragma unroll
            for (int j = 0; j < G; j++)
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int64_t row = m0 + i * 16 + 4 * (lane / 16) + v;
                    const int col = n0 + j * 16 + lane % 16;
                    if (row < M && col < N) epilogue_store<float>(epi, row, col, N, low[i][j][v] + high[i][j][v]);
                }
    }
}

// 64x64 tiles once they give every compute unit one (below that the finer tiles and the split of K win)
static bool f32_big_tiles(int64_t M, int N) { return ceil_div64(M, 64) * ceil_div64(N, 64) >= 256; }

static int launch_f32(const float *A, int64_t lda, const float *W, int64_t ldw, int64_t M, int N, int K, const GemmEpilogue &epi, hipStream_t st) {
    const bool big = f32_big_tiles(M, N);
    const int64_t gx = ceil_div64(M, big ? 64 : 16), gy = ceil_div64(N, big ? 64 : 16);
    if (gx > 0x7fffffffLL || gy > 65535) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_GEMM_SIMPLE, st, 2.0 * (double)M * N * K);
    if (big) hipLaunchKernelGGL(gemm_f32_mfma<32>, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, st, A, lda, W, ldw, M, N, K, epi);
    else hipLaunchKernelGGL(gemm_f32_mfma<16>, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, st, A, lda, W, ldw, M, N, K, epi);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// What a matrix-core kernel does with a product.  EPI_VT: transposed per request (context values); EPI_SILU / EPI_SILU_DIV: the
// activation through the hardware reciprocal / through a division (they differ in the last bits; the row count of a product
// decides, see launch_gemm, never the kernel that happens to run it).
enum { EPI_STORE = 0, EPI_SILU, EPI_F32, EPI_F32_RESID, EPI_F32_TABLE, EPI_VT, EPI_SILU_DIV };
__host__ __device__ constexpr bool kind_f32(int kind) { return kind == EPI_F32 || kind == EPI_F32_RESID || kind == EPI_F32_TABLE; }

// bytes a bf16 GEMM must move once: both operands, the output, and the residual it adds
static double gemm_bytes(int64_t M, int N, int K, bool out_f32, bool resid) {
    return 2.0 * ((double)M * K + (double)N * K) + (double)M * N * ((out_f32 ? 4 : 2) + (resid ? 4 : 0));
}

// ---------------------------------------------------------------------------
// Persistent MFMA kernel: 256x256 block tile, BK = 64, ring of five 32 KB half-tiles in LDS
// ---------------------------------------------------------------------------
// One workgroup (8 wavefronts, 2 x 4, wave tile 128 x 64) per compute unit walks a list of output tiles.
// A k-tile is two half-tiles of 256 rows x 128 bytes (one full cache line per row): A(g) and W(g).  The ring holds
// five half-tiles, filled by global_load_lds_dwordx4 (every lane moves 16 bytes straight into LDS; one wave
// instruction fills 8 rows; chunk c of row r sits at position c ^ ((r >> 1) & 7), which keeps both the 1 KB
// writes and the fragment reads conflict-free, and the swizzle is applied on the global side).  In item order
// A0 W0 A1 W1 A2 ... item q lives in slot q % 5.  The bf16 loop requests A(g+2) under the first MFMAs of k-tile g (into
// the slot W(g-1) left at the previous barrier) and W(g+2) under the MFMAs that follow the barrier ending k-tile g (into
// the slot A(g) just left), one load after every second MFMA: a burst of eight loads per wave right after the barrier
// holds up the MFMAs queued behind it.  (The FP8 loop requests W(g+2) and A(g+3) under the four MFMAs after the barrier.)
// The item stream runs on into the next tile of the workgroup, so a tile's first operands arrive while the previous
// tile is still being multiplied and stored.
// Per k-tile: four k-steps of 8 MFMAs; the fragments of step s+1 are read while step s multiplies.  Fragment
// reads are inline assembly so that their waits can be exact (lgkmcnt(6): the six reads just issued may still
// be in flight); one bare s_barrier per k-tile separates "every wave has read A(g), W(g)" from "everybody's
// share of A(g+1), W(g+1) has landed" (each wave waits for its own loads with vmcnt first).
// The MFMA operands are swapped (W fragment first), so a lane owns one row of C and, per group of four
// accumulator registers, four consecutive columns: the epilogue writes 8/16-byte pieces into the two slots the
// last k-tile released (8 KB per wave, rows swizzled) and reads them back as full rows, so C leaves in 16-byte
// pieces with whole cache lines per row.
#define RING_SLOTS 5
#define SLOT_CHUNKS 2048  // 256 rows x 8 chunks of 16 bytes
#define RING_LDS_BYTES (RING_SLOTS * SLOT_CHUNKS * 16)

__device__ __forceinline__ void ring_dma16(const char *g, bf16x8 *lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1))) *)g,
                                     (void __attribute__((address_space(3))) *)lds_wave_base, 16, 0, 0);
}

__device__ __forceinline__ float fast_silu(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x)); }

// F8: the operands are FP8 (E4M3) bytes instead of bf16.  The byte geometry is unchanged - a k-tile is still 128 bytes per
// row, now 128 values of k - so loads, ring and epilogue are shared; the main loop issues v_mfma_f32_32x32x64_f8f6f4, whose
// 32-byte operand per lane is the two 16-byte fragments the bf16 loop reads for two consecutive k-steps.  (Which of the 64
// values of k a lane holds does not matter as long as both operands agree, and they are read the same way.)  lda, ldw and K
// count elements (bytes).  The product row is scaled by a_scale[row] * w_scale before the epilogue.
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));

template <int KIND, bool F8 = false>
__global__ __launch_bounds__(512) void gemm_bf16_ring(const bf16 *__restrict__ A, int64_t lda, const bf16 *__restrict__ W, int64_t ldw,
                                                      int64_t M, int N, int K, int64_t tiles_m, int tiles_n, int group_m, GemmEpilogue epi) {
    extern __shared__ bf16x8 smem[];
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int wm = wave / 4, wn = wave % 4;
    const int frow = lane % 32, hf = lane / 32;
    const int KT = F8 ? K / 128 : K / 64;
    static_assert(!(F8 && KIND == EPI_VT), "the transposed epilogue has no FP8 form");
    if (epi.skip_len && !epi.skip_S) {  // the row count is known on the device only; M is its bound
        M = epi.skip_len[0];
        tiles_m = (M + 255) / 256;
    }

    // ---- tile schedule: every XCD (workgroup id % 8) owns a contiguous range of logical tiles and its workgroups walk it
    // with stride nslots; inside a group of group_m row blocks the row index runs fastest, so the workgroups of an XCD
    // share a few A blocks and a few W blocks through their L2 at any time ----
    const int64_t total = tiles_m * tiles_n;
    const int nslots = gridDim.x / 8;
    const int xcd = blockIdx.x % 8, wslot = blockIdx.x / 8;
    const int64_t per_xcd = (total + 7) / 8;
    const int64_t xcd_end = (xcd + 1) * per_xcd < total ? (xcd + 1) * per_xcd : total;
    const uint32_t gsz = (uint32_t)group_m * (uint32_t)tiles_n;
    auto tile_coords = [&](int64_t l64, int64_t &m0, int &n0) {  // fewer than 2^31 tiles: 32-bit division
        const uint32_t l = (uint32_t)l64;
        const uint32_t grp = l / gsz, in = l - grp * gsz;
        const uint32_t first_m = grp * (uint32_t)group_m;
        const uint32_t left = (uint32_t)tiles_m - first_m;
        const uint32_t gm = left < (uint32_t)group_m ? left : (uint32_t)group_m;
        const uint32_t nn = in / gm;
        m0 = (int64_t)(first_m + (in - nn * gm)) * 256;
        n0 = (int)nn * 256;
    };
    // Rows of A beyond a request's valid length (epi.skip_len[b] of every skip_S rows) are padding nobody reads the product
    // of: a tile whose 256 rows all lie in one request's padding is passed over.
    auto tile_live = [&](int64_t l) -> bool {
        if (!epi.skip_len || !epi.skip_S) return true;
        int64_t tm0;
        int tn0;
        tile_coords(l, tm0, tn0);
        const uint32_t r0 = (uint32_t)tm0, rows_per = (uint32_t)epi.skip_S;
        const uint32_t b0 = r0 / rows_per, b1 = (r0 + 255u) / rows_per;
        if (b0 != b1) return true;  // straddles two requests
        int len = epi.skip_len[b0];
        len = len < 1 ? 1 : len;
        return r0 - b0 * rows_per < (uint32_t)len;
    };
    auto next_live = [&](int64_t l) {
        while (l < xcd_end && !tile_live(l)) l += nslots;
        return l;
    };
    int64_t L = next_live(xcd * per_xcd + wslot);
    if (L >= xcd_end) return;

    // ---- loads: load j of this wave fills rows (wave*4+j)*8 .. +7 of a half-tile, lane -> row lane/8, position lane%8.
    // The chunk that lives at position p of row r is p ^ ((r >> 1) & 7), and (r >> 1) & 7 = 4*(j&1) + (lane/8 >> 1).
    // Per tile: a wave-uniform base pointer (row block; a k-tile adds 128 bytes) and the last valid row of the block (rows
    // past the matrix edge re-read it).  The lane's byte offset - clamped row times the pitch plus the chunk - is computed
    // when the load is issued (three vector instructions that run beside the MFMAs) instead of being kept per tile. ----
    const int dma_row0 = wave * 32 + lane / 8;
    const uint32_t cb0 = (uint32_t)(((lane % 8) ^ ((lane / 8) >> 1)) * 16), cb1 = cb0 ^ 64u;
    const uint32_t lda2 = (uint32_t)lda * (F8 ? 1 : 2), ldw2 = (uint32_t)ldw * (F8 ? 1 : 2);  // row pitches in bytes
    int64_t m0, m0n = 0;
    int n0, n0n = 0;
    tile_coords(L, m0, n0);
    int64_t Lnext = next_live(L + nslots);
    bool has_next = Lnext < xcd_end;
    if (has_next) tile_coords(Lnext, m0n, n0n);
    const char *baseA, *baseW, *baseAn, *baseWn;
    int maxa, maxw, maxan, maxwn;
    auto tile_sources = [&](int64_t tm0, int tn0, const char *&bA, const char *&bW, int &mA, int &mW) {
        bW = (const char *)W + (int64_t)tn0 * ldw2;
        mW = N - 1 - tn0 < 255 ? N - 1 - tn0 : 255;
        if (KIND == EPI_VT) {
            // the rows count every request's vt_rows tokens up to vt_S, a multiple of 64: a wavefront's 32 rows lie in one request, those past its
            // last token (and past the last request) re-read it
            const uint32_t row = (uint32_t)tm0 + wave * 32, v = row < (uint32_t)M ? row : (uint32_t)M - 1;
            const uint32_t b = v / (uint32_t)epi.vt_S, s = v - b * (uint32_t)epi.vt_S, last = (uint32_t)epi.vt_rows - 1, at = s < last ? s : last;
            bA = (const char *)A + ((int64_t)b * epi.vt_rows + at - wave * 32) * lda2;
            mA = wave * 32 + (int)(last - at < 31 ? last - at : 31);
            return;
        }
        bA = (const char *)A + tm0 * lda2;
        mA = (int)(M - 1 - tm0 < 255 ? M - 1 - tm0 : 255);
    };
    tile_sources(m0, n0, baseA, baseW, maxa, maxw);
    // Without a next tile the loads that would fetch its first k-tiles re-read the current tile's instead (valid memory, into
    // slots nobody reads again and the epilogue does not stage in; all of them have landed at the tile's last barrier): the
    // load sequence stays free of branches, which the register allocation of this kernel depends on.
    baseAn = baseA; baseWn = baseW; maxan = maxa; maxwn = maxw;
    if (has_next) tile_sources(m0n, n0n, baseAn, baseWn, maxan, maxwn);
    // piece j (8 rows) of this wave's share of a half-tile
    auto load_piece = [&](const char *base, int mx, uint32_t pitch, bf16x8 *dst, int j) {
        const int r = dma_row0 + j * 8;
        const uint32_t off = (uint32_t)(r < mx ? r : mx) * pitch + ((j & 1) ? cb1 : cb0);
        ring_dma16(base + off, dst + j * 64);
    };
    // k-tile gk of the current tile (gk < KT) or of the workgroup's next tile (gk >= KT)
    auto issue_a = [&](int gk, int slot) {
        const bool cur = gk < KT;
        const char *base = cur ? baseA + gk * 128 : baseAn + (gk - KT) * 128;
        const int mx = cur ? maxa : maxan;
        bf16x8 *dst = smem + slot * SLOT_CHUNKS + wave * 256;
#pragma unroll
        for (int j = 0; j < 4; j++) load_piece(base, mx, lda2, dst, j);
    };
    auto issue_w = [&](int gk, int slot) {
        const bool cur = gk < KT;
        const char *base = cur ? baseW + gk * 128 : baseWn + (gk - KT) * 128;
        const int mx = cur ? maxw : maxwn;
        bf16x8 *dst = smem + slot * SLOT_CHUNKS + wave * 256;
#pragma unroll
        for (int j = 0; j < 4; j++) load_piece(base, mx, ldw2, dst, j);
    };

    // ---- fragments: lane reads row frow of a 32-row block, chunk 2s + hf of k-step s, i.e. position (hf ^ fx) ^ 2s ----
    const int fx = (frow >> 1) & 7;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const uint32_t a_lane = lds0 + (uint32_t)((wm * 128 + frow) * 8 + (hf ^ fx)) * 16;
    const uint32_t w_lane = lds0 + (uint32_t)((wn * 64 + frow) * 8 + (hf ^ fx)) * 16;
    auto read_frags = [&](bf16x8 (&af)[4], bf16x8 (&wf)[2], int slot_a, int slot_w, int s) {
        const uint32_t pa = (a_lane ^ (uint32_t)(s << 5)) + (uint32_t)slot_a * 32768u;
        const uint32_t pw = (w_lane ^ (uint32_t)(s << 5)) + (uint32_t)slot_w * 32768u;
        asm volatile("ds_read_b128 %0, %1" : "=v"(af[0]) : "v"(pa));
        asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(af[1]) : "v"(pa));
        asm volatile("ds_read_b128 %0, %1 offset:8192" : "=v"(af[2]) : "v"(pa));
        asm volatile("ds_read_b128 %0, %1 offset:12288" : "=v"(af[3]) : "v"(pa));
        asm volatile("ds_read_b128 %0, %1" : "=v"(wf[0]) : "v"(pw));
        asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(wf[1]) : "v"(pw));
    };
    // the fragments are operands of the wait, so nothing that uses them can move above it
    auto wait_frags = [&](bf16x8 (&af)[4], bf16x8 (&wf)[2], bool all) {
        if (all) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(af[0]), "+v"(af[1]), "+v"(af[2]), "+v"(af[3]), "+v"(wf[0]), "+v"(wf[1]));
        else asm volatile("s_waitcnt lgkmcnt(6)" : "+v"(af[0]), "+v"(af[1]), "+v"(af[2]), "+v"(af[3]), "+v"(wf[0]), "+v"(wf[1]));
    };
    floatx16 acc[4][2];
    auto mma = [&](const bf16x8 (&af)[4], const bf16x8 (&wf)[2]) {
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 2; j++) {
                // EPI_VT wants C transposed: with the operands in natural order a lane owns one column of C and four consecutive rows
                if (KIND == EPI_VT) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], wf[j], acc[i][j], 0, 0, 0);
                else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
            }
    };

    // the eight MFMAs of a step with the four direct loads of one half-tile between them, one after every second MFMA: a burst of
    // loads right after the barrier would hold up the MFMAs behind it while the loads queue
    auto mma_dma = [&](const bf16x8 (&af)[4], const bf16x8 (&wf)[2], bool doit, const char *base, int mx, uint32_t pitch, bf16x8 *dst) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
#pragma unroll
            for (int j = 0; j < 2; j++) {
                if (KIND == EPI_VT) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], wf[j], acc[i][j], 0, 0, 0);
                else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (doit) load_piece(base, mx, pitch, dst, i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // ---- FP8 main loop pieces.  One register set: operand i of A (rows i*32..) and j of W are 32 bytes per lane, the chunks
    // 2u and 2u+1 of k-step u (two per k-tile).  The MFMAs of a step run W-block-major, (0,0) (1,0) (2,0) (3,0) (0,1) .. (3,1);
    // as soon as the last MFMA that uses an operand has been issued its registers take the next step's data, so the twelve
    // reads of a step are spread under the step before it: W0 after (3,0), A_i after (i,1), W1 after (3,1). ----
    intx8 A8[4], W8[2];
#define LD8(dst, base, u, OFF)                                                                                     \
    do {                                                                                                           \
        intx4 lo_, hi_;                                                                                            \
        asm volatile("ds_read_b128 %0, %1 offset:" #OFF : "=v"(lo_) : "v"((base) ^ (uint32_t)((u) << 6)));          \
        asm volatile("ds_read_b128 %0, %1 offset:" #OFF : "=v"(hi_) : "v"((base) ^ (uint32_t)(((u) << 6) | 32))); \
        dst = __builtin_shufflevector(lo_, hi_, 0, 1, 2, 3, 4, 5, 6, 7);                                           \
    } while (0)
#define WAIT8(N, a, w) asm volatile("s_waitcnt lgkmcnt(" #N ")" : "+v"(a), "+v"(w))
#define MMA8(i, j) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(W8[j], A8[i], acc[i][j], 0, 0, 0, 0, 0, 0)
    auto load_step8 = [&](int slot_a, int slot_w, int u) {  // all twelve reads of a step, in the order the waits of a step assume
        const uint32_t pa = a_lane + (uint32_t)slot_a * 32768u, pw = w_lane + (uint32_t)slot_w * 32768u;
        LD8(W8[0], pw, u, 0);
        LD8(A8[0], pa, u, 0);
        LD8(A8[1], pa, u, 4096);
        LD8(A8[2], pa, u, 8192);
        LD8(A8[3], pa, u, 12288);
        LD8(W8[1], pw, u, 4096);
    };

    // ---- prologue: A(0) W(0) A(1) W(1) (and A(2) for the FP8 loop) into slots 0..4 (at least three k-tiles, so all belong to the first tile) ----
    issue_a(0, 0);
    issue_w(0, 1);
    issue_a(1, 2);
    issue_w(1, 3);
    if (F8) {
        issue_a(2, 4);
        asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    } else {  // (the bf16 loop requests A(2) under its first MFMAs)
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8 fa0[4], fw0[2], fa1[4], fw1[2];
    int sa = 0;  // slot of A(g); W(g) sits in the next slot
    if (F8) load_step8(0, 1, 0);
    else read_frags(fa0, fw0, 0, 1, 0);

#define SB __builtin_amdgcn_sched_barrier(0)
    for (;;) {  // tiles of this workgroup
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
        float rinv[4] = {1.0f, 1.0f, 1.0f, 1.0f};
        floatx4 bias4 = {0.0f, 0.0f, 0.0f, 0.0f};  // EPI_F32: bias of this lane's four columns in the epilogue's read-back layout
        if (KIND != EPI_VT && (F8 || epi.row_inv)) {
            const float *rs = F8 ? epi.a_scale : epi.row_inv;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int64_t row = m0 + wm * 128 + i * 32 + frow;
                rinv[i] = rs[row < M ? row : M - 1] * (F8 ? epi.w_scale : 1.0f);
            }
        }
        if (F8) {
            for (int kt = 0; kt < KT; kt++) {
                const int sw = sa + 1 >= RING_SLOTS ? sa + 1 - RING_SLOTS : sa + 1;
                const uint32_t pa = a_lane + (uint32_t)sa * 32768u, pw = w_lane + (uint32_t)sw * 32768u;
                // step 0: its reads are in flight in the order W0 A0 A1 A2 A3 W1 (two each)
                SB; WAIT8(8, A8[0], W8[0]); MMA8(0, 0); SB;
                WAIT8(6, A8[1], W8[0]); MMA8(1, 0); SB;
                WAIT8(4, A8[2], W8[0]); MMA8(2, 0); SB;
                WAIT8(2, A8[3], W8[0]); MMA8(3, 0); SB;
                LD8(W8[0], pw, 1, 0); SB;
                WAIT8(2, A8[0], W8[1]); MMA8(0, 1); SB;
                LD8(A8[0], pa, 1, 0); SB;
                MMA8(1, 1); SB;
                LD8(A8[1], pa, 1, 4096); SB;
                MMA8(2, 1); SB;
                LD8(A8[2], pa, 1, 8192); SB;
                MMA8(3, 1); SB;
                LD8(A8[3], pa, 1, 12288);
                LD8(W8[1], pw, 1, 4096); SB;
                // step 1
                WAIT8(8, A8[0], W8[0]); MMA8(0, 0); SB;
                WAIT8(6, A8[1], W8[0]); MMA8(1, 0); SB;
                WAIT8(4, A8[2], W8[0]); MMA8(2, 0); SB;
                WAIT8(2, A8[3], W8[0]); MMA8(3, 0); SB;
                // every read of A(g), W(g) has been issued; once they have returned and this wave's share of A(g+1), W(g+1) has
                // landed, the barrier releases the two slots (only A(g+2) may stay in flight)
                WAIT8(0, A8[0], W8[1]);
                if (kt + 2 < KT || has_next) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                const int sa1 = sa + 2 >= RING_SLOTS ? sa + 2 - RING_SLOTS : sa + 2;
                const int sw1 = sa + 3 >= RING_SLOTS ? sa + 3 - RING_SLOTS : sa + 3;
                const uint32_t pa1 = a_lane + (uint32_t)sa1 * 32768u, pw1 = w_lane + (uint32_t)sw1 * 32768u;
                const bool more = kt + 1 < KT;  // (a next tile's first operands are read after the epilogue: it needs the registers)
                SB; if (more) LD8(W8[0], pw1, 0, 0); SB;
                if (KIND == EPI_F32 && kt + 2 == KT && epi.bias) {  // see the bf16 loop
                    const int c0 = n0 + wn * 64 + (lane % 16) * 4;
                    const float *src = epi.bias + (c0 + 3 < N ? c0 : 0);
                    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(bias4) : "v"(src) : "memory");
                }
                // the two slots just released take W(g+2) and A(g+3), two loads after each MFMA (not in one burst, which would hold
                // up the MFMAs queued behind it)
                const int gw = kt + 2, ga = kt + 3;
                const char *srcw = gw < KT ? baseW + gw * 128 : baseWn + (gw - KT) * 128;
                const char *srca = ga < KT ? baseA + ga * 128 : baseAn + (ga - KT) * 128;
                const int mxw = gw < KT ? maxw : maxwn, mxa = ga < KT ? maxa : maxan;
                bf16x8 *dstw = smem + sa * SLOT_CHUNKS + wave * 256, *dsta = smem + sw * SLOT_CHUNKS + wave * 256;
                SB; MMA8(0, 1); SB;
                if (more) { LD8(A8[0], pa1, 0, 0); load_piece(srcw, mxw, ldw2, dstw, 0); load_piece(srcw, mxw, ldw2, dstw, 1); } SB;
                MMA8(1, 1); SB;
                if (more) { LD8(A8[1], pa1, 0, 4096); load_piece(srcw, mxw, ldw2, dstw, 2); load_piece(srcw, mxw, ldw2, dstw, 3); } SB;
                MMA8(2, 1); SB;
                if (more) { LD8(A8[2], pa1, 0, 8192); load_piece(srca, mxa, lda2, dsta, 0); load_piece(srca, mxa, lda2, dsta, 1); } SB;
                MMA8(3, 1); SB;
                if (more) { LD8(A8[3], pa1, 0, 12288); LD8(W8[1], pw1, 0, 4096); load_piece(srca, mxa, lda2, dsta, 2); load_piece(srca, mxa, lda2, dsta, 3); } SB;
                if (more) sa = sa1;
            }
        } else
        for (int kt = 0; kt < KT; kt++) {
            const int sw = sa + 1 >= RING_SLOTS ? sa + 1 - RING_SLOTS : sa + 1;
            SB; read_frags(fa1, fw1, sa, sw, 1); wait_frags(fa0, fw0, false); SB;
            {   // A(g+2) into the slot W(g-1) left at the previous barrier
                const int gk = kt + 2;
                const bool cur = gk < KT;
                mma_dma(fa0, fw0, true, cur ? baseA + gk * 128 : baseAn + (gk - KT) * 128, cur ? maxa : maxan, lda2,
                        smem + (sa == 0 ? RING_SLOTS - 1 : sa - 1) * SLOT_CHUNKS + wave * 256);
            }
            SB;
            read_frags(fa0, fw0, sa, sw, 2); wait_frags(fa1, fw1, false); SB;
            mma(fa1, fw1); SB;
            read_frags(fa1, fw1, sa, sw, 3); wait_frags(fa0, fw0, false); SB;
            mma(fa0, fw0); SB;
            // every read of A(g), W(g) has returned; this wave's share of A(g+1), W(g+1) has landed (only A(g+2) may stay in flight)
            wait_frags(fa1, fw1, true);
            if (kt + 2 < KT || has_next) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int sa1 = sa + 2 >= RING_SLOTS ? sa + 2 - RING_SLOTS : sa + 2;
            const int sw1 = sa + 3 >= RING_SLOTS ? sa + 3 - RING_SLOTS : sa + 3;
            SB; if (kt + 1 < KT) read_frags(fa0, fw0, sa1, sw1, 0); SB;  // (a next tile's first fragments are read after the epilogue: it needs the registers)
            if (KIND == EPI_F32 && kt + 2 == KT && epi.bias) {
                // The bias of this lane's four columns (read-back layout of the epilogue) is requested here, just before the
                // tile's last operand loads, by a load the compiler does not track: the wait that ends the last k-tile (all but
                // the four newest loads have landed) covers it.  A tracked load in the epilogue would make the compiler guard
                // the reuse of its registers with a full drain of outstanding loads inside the k-loop.
                const int c0 = n0 + wn * 64 + (lane % 16) * 4;
                const float *src = epi.bias + (c0 + 3 < N ? c0 : 0);
                asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(bias4) : "v"(src) : "memory");
            }
            {   // the slot A(g) left takes W(g+2); after a tile's last k-tile the released slots first stage C
                const int gk = kt + 2;
                const bool cur = gk < KT;
                SB;
                mma_dma(fa1, fw1, kt + 1 < KT, cur ? baseW + gk * 128 : baseWn + (gk - KT) * 128, cur ? maxw : maxwn, ldw2,
                        smem + sa * SLOT_CHUNKS + wave * 256);
                SB;
            }
            if (kt + 1 < KT) sa = sa1;
        }
        // ---- epilogue: slots sa (waves 0..3) and sa+1 (waves 4..7) are free, 8 KB per wave ----
        const int sw = sa + 1 >= RING_SLOTS ? sa + 1 - RING_SLOTS : sa + 1;
        {
            constexpr bool OUT_F32 = kind_f32(KIND);
            char *stage = (char *)(smem + (wave < 4 ? sa : sw) * SLOT_CHUNKS) + (wave % 4) * 8192;
            const int64_t wrow0 = m0 + wm * 128;
            const int wcol0 = n0 + wn * 64;
            if (KIND != EPI_VT && (F8 || epi.row_inv)) {
                // folded RMSNorm, reader side: the A operand was gain * x, not yet divided by rms(x); a lane owns row frow of
                // each 32-row block (factors requested at the start of the tile).  FP8 operands: the scales of the row and of W.
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++)
#pragma unroll
                        for (int v = 0; v < 16; v++) acc[i][j][v] *= rinv[i];
            }
            if (KIND == EPI_VT) {
                // C^T per request: out[(b*N + n) * ldc + s] = C[b*vt_S + s][n] for s < len_b, 0 beyond (values of the context, transposed
                // per head for the attention kernel's second product).  vt_S is a multiple of 64, so the 64 rows of a pass share one request.
                // Two passes of 64 rows: staged as 64 columns x 64 rows (128-byte lines of 8 chunks, chunk c of line r at c ^ (r & 7)).
#pragma unroll
                for (int pass = 0; pass < 2; pass++) {
#pragma unroll
                    for (int ii = 0; ii < 2; ii++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            const int r = j * 32 + frow;
#pragma unroll
                            for (int g = 0; g < 4; g++) {
                                bf16x4 pk;
#pragma unroll
                                for (int e = 0; e < 4; e++) pk[e] = (bf16)acc[pass * 2 + ii][j][4 * g + e];
                                const int c = ii * 4 + g;
                                *(bf16x4 *)(stage + r * 128 + ((c ^ (r & 7)) * 16) + hf * 8) = pk;
                            }
                        }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    const int64_t t0 = wrow0 + pass * 64;  // first of the 64 rows (tokens) of this pass
                    if (t0 < M) {
                        const uint32_t b = (uint32_t)t0 / (uint32_t)epi.vt_S;
                        const int s0 = (int)((uint32_t)t0 - b * (uint32_t)epi.vt_S);
                        int len = epi.ctx_len ? epi.ctx_len[b] : epi.vt_rows;
                        len = len < 1 ? 1 : (len > epi.vt_rows ? epi.vt_rows : len);
#pragma unroll 4
                        for (int it = 0; it < 8; it++) {
                            const int r = it * 8 + lane / 8, c = lane % 8;
                            bf16x8 x = *(const bf16x8 *)(stage + r * 128 + ((c ^ (r & 7)) * 16));
                            const int col = wcol0 + r, s = s0 + c * 8;
#pragma unroll
                            for (int e = 0; e < 8; e++) if (s + e >= len) x[e] = (bf16)0.0f;
                            if (col < N) __builtin_nontemporal_store(x, (bf16x8 *)((bf16 *)epi.C + ((int64_t)b * N + col) * epi.ldc + s));
                        }
                    }
                    if (pass == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
            } else if (!OUT_F32) {
                // two passes of 64 rows x 64 columns: 128-byte rows of 8 chunks, chunk c of row r at position c ^ (r & 7)
#pragma unroll
                for (int pass = 0; pass < 2; pass++) {
#pragma unroll
                    for (int ii = 0; ii < 2; ii++) {
                        const int r = ii * 32 + frow;
#pragma unroll
                        for (int j = 0; j < 2; j++)
#pragma unroll
                            for (int g = 0; g < 4; g++) {
                                bf16x4 pk;
#pragma unroll
                                for (int e = 0; e < 4; e++) {
                                    const float x = acc[pass * 2 + ii][j][4 * g + e];
                                    pk[e] = (bf16)(KIND == EPI_SILU ? fast_silu(x) : KIND == EPI_SILU_DIV ? x / (1.0f + __expf(-x)) : x);
                                }
                                const int c = j * 4 + g;
                                *(bf16x4 *)(stage + r * 128 + ((c ^ (r & 7)) * 16) + hf * 8) = pk;
                            }
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // wave-private region: no barrier needed
                    if (wrow0 + 128 <= M && wcol0 + 64 <= N) {
                        // the wave's block lies inside C (all but the last row and column of tiles): no bounds tests, one running
                        // address, LDS offsets that are instruction immediates (rows it*8 + lane/8: the swizzle only sees lane/8)
                        const char *rd = stage + (lane / 8) * 128 + (((lane % 8) ^ ((lane / 8) & 7)) * 16);
                        bf16 *wr = (bf16 *)epi.C + (wrow0 + pass * 64 + lane / 8) * epi.ldc + wcol0 + (lane % 8) * 8;
#pragma unroll
                        for (int it = 0; it < 8; it++) {
                            __builtin_nontemporal_store(*(const bf16x8 *)(rd + it * 1024), (bf16x8 *)wr);  // C streams out: not re-read before it leaves the caches
                            wr += 8 * epi.ldc;
                        }
                    } else {
#pragma unroll 4
                        for (int it = 0; it < 8; it++) {
                            const int r = it * 8 + lane / 8, c = lane % 8;
                            const bf16x8 x = *(const bf16x8 *)(stage + r * 128 + ((c ^ (r & 7)) * 16));
                            const int64_t row = wrow0 + pass * 64 + r;
                            const int col = wcol0 + c * 8;
                            if (row < M && col < N) {
                                if (col + 7 < N) __builtin_nontemporal_store(x, (bf16x8 *)((bf16 *)epi.C + row * epi.ldc + col));
                                else for (int e = 0; e < 8 && col + e < N; e++) ((bf16 *)epi.C)[row * epi.ldc + col + e] = x[e];
                            }
                        }
                    }
                    if (pass == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
            } else {
                // four passes of 32 rows x 64 columns: 256-byte rows of 16 chunks, chunk c of row r at position c ^ (r & 15).
                // What a pass adds (residual rows, table rows) is requested before its accumulators are staged, all eight
                // 16-byte pieces at once.  (Requesting them a pass ahead changes nothing: at N = K = 1024 these launches move
                // 12-14 bytes per output element and run at the memory system's mixed read/write rate.)
                constexpr bool HAS_ADD = KIND == EPI_F32_RESID || KIND == EPI_F32_TABLE;  // per-row addends; a bias is one vector per lane
                const int erow = lane / 16, ecol = wcol0 + (lane % 16) * 4;
                // folded RMSNorm, writer side (N % 256 == 0: every column exists)
                const bool emit = HAS_ADD && epi.norm_out != nullptr;
                floatx4 gain4 = {0.0f, 0.0f, 0.0f, 0.0f};
                if (emit) {
                    const bf16x4 g4 = *(const bf16x4 *)((const bf16 *)epi.norm_gain + ecol);
#pragma unroll
                    for (int e = 0; e < 4; e++) gain4[e] = (float)g4[e];
                }
                // the wave's block lies inside C (all but the last row and column of tiles): no bounds tests and running addresses
                const bool interior = wrow0 + 128 <= M && wcol0 + 64 <= N;
                // table rows: a lane fetches the selectors of two of the wave's 128 rows, the others take them from it (one memory
                // latency per tile in front of the table's own instead of one per pass: 524288 x 1024 x 1024 with rows through a map 1.97 -> 1.54 ms)
                uint32_t sel[2] = {0, 0};
                if (KIND == EPI_F32_TABLE && epi.tok)
#pragma unroll
                    for (int i = 0; i < 2; i++) {
                        const int64_t row = wrow0 + i * 64 + lane;
                        sel[i] = (uint32_t)epi.tok[row < M ? row : M - 1];
                    }
                auto table_row = [&](int pass, int it) {
                    return epi.table + (uint64_t)(uint32_t)__shfl((int)sel[pass / 2], (pass % 2) * 32 + it * 4 + erow, 64) * (uint32_t)N;
                };
#pragma unroll
                for (int pass = 0; pass < 4; pass++) {
                    floatx4 adds[8];
                    if (HAS_ADD && interior) {
                        const int64_t row0 = wrow0 + pass * 32 + erow;
                        if (KIND == EPI_F32_RESID) {
                            const float *rp = epi.resid + row0 * epi.ldr + ecol;
#pragma unroll
                            for (int it = 0; it < 8; it++) adds[it] = *(const floatx4 *)(rp + (int64_t)(it * 4) * epi.ldr);
                        } else {
#pragma unroll
                            for (int it = 0; it < 8; it++)
                                adds[it] = *(const floatx4 *)(table_row(pass, it) + ecol);
                        }
                    } else if (HAS_ADD) {
#pragma unroll
                        for (int it = 0; it < 8; it++) {
                            const int64_t row = wrow0 + pass * 32 + it * 4 + erow;
                            adds[it] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                            if (row < M && ecol + 3 < N) {
                                if (KIND == EPI_F32_RESID) adds[it] = *(const floatx4 *)(epi.resid + row * epi.ldr + ecol);
                                if (KIND == EPI_F32_TABLE) adds[it] = *(const floatx4 *)(epi.table + (epi.tok ? (int64_t)epi.tok[row] : 0) * N + ecol);
                            }
                        }
                    }
                    const int r = frow;
#pragma unroll
                    for (int j = 0; j < 2; j++)
#pragma unroll
                        for (int g = 0; g < 4; g++) {
                            floatx4 pk;
#pragma unroll
                            for (int e = 0; e < 4; e++) pk[e] = acc[pass][j][4 * g + e];
                            const int c = j * 8 + g * 2 + hf;
                            *(floatx4 *)(stage + r * 256 + ((c ^ (r & 15)) * 16)) = pk;
                        }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    if (interior) {
                        const int64_t row0 = wrow0 + pass * 32 + erow;
                        char *cp = (char *)epi.C + (row0 * epi.ldc + ecol) * (KIND == EPI_F32 && epi.out_f16 ? 2 : 4);
                        const int64_t cstep = (int64_t)4 * epi.ldc * (KIND == EPI_F32 && epi.out_f16 ? 2 : 4);
                        bf16 *np = emit ? (bf16 *)epi.norm_out + row0 * epi.norm_ld + ecol : nullptr;
                        float *ssp = emit ? epi.norm_ss + row0 * (N / 64) + (wcol0 >> 6) : nullptr;
#pragma unroll
                        for (int it = 0; it < 8; it++) {  // (fully unrolled: the addends must stay in registers)
                            const int rr = it * 4 + erow, c = lane % 16;
                            floatx4 x = *(const floatx4 *)(stage + rr * 256 + ((c ^ (rr & 15)) * 16));
                            if (HAS_ADD) x += adds[it];
                            if (emit) {  // (as below)
                                float sq = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
                                sq += lane_xor1(sq);
                                sq += lane_xor2(sq);
                                sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x114, 0xf, 0xf, true));
                                sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x118, 0xf, 0xf, true));
                                if (lane % 16 == 15) ssp[(int64_t)(it * 4) * (N / 64)] = sq;
                            }
                            if (KIND == EPI_F32) x += bias4;
                            if (KIND == EPI_F32 && epi.out_f16) {
                                halfx4 hx;
#pragma unroll
                                for (int e = 0; e < 4; e++) hx[e] = (_Float16)x[e];
                                __builtin_nontemporal_store(hx, (halfx4 *)(cp + it * cstep));
                            } else {
                                __builtin_nontemporal_store(x, (floatx4 *)(cp + it * cstep));
                            }
                            if (emit) {
                                bf16x4 nb;
#pragma unroll
                                for (int e = 0; e < 4; e++) nb[e] = (bf16)(x[e] * gain4[e]);
                                *(bf16x4 *)(np + (int64_t)(it * 4) * epi.norm_ld) = nb;
                            }
                        }
                    } else
#pragma unroll
                    for (int it = 0; it < 8; it++) {  // (fully unrolled: the addends must stay in registers)
                        const int rr = it * 4 + erow, c = lane % 16;
                        floatx4 x = *(const floatx4 *)(stage + rr * 256 + ((c ^ (rr & 15)) * 16));
                        const int64_t row = wrow0 + pass * 32 + rr;
                        const int col = ecol;
                        if (HAS_ADD) x += adds[it];  // (zero where the lane stores nothing or takes the slow path below)
                        if (emit) {  // sum of squares over the row's 64 columns in this wave: the 16 lanes of a DPP row
                            float sq = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
                            sq += lane_xor1(sq);
                            sq += lane_xor2(sq);  // every lane: its quad's sum
                            // row_shr:4 then row_shr:8 (lane i takes lane i-4 / i-8 of its row, 0 if there is none): lane 15 of the
                            // row ends with all four quads
                            sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x114, 0xf, 0xf, true));
                            sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x118, 0xf, 0xf, true));
                            if (lane % 16 == 15 && row < M) epi.norm_ss[row * (N / 64) + (wcol0 >> 6)] = sq;
                        }
                        if (row < M && col < N) {
                            if (col + 3 < N) {
                                if (KIND == EPI_F32) x += bias4;
                                if (KIND == EPI_F32 && epi.out_f16) {  // logits for the selection: half precision, 8 bytes per lane, 128 per row
                                    halfx4 hx;
#pragma unroll
                                    for (int e = 0; e < 4; e++) hx[e] = (_Float16)x[e];
                                    __builtin_nontemporal_store(hx, (halfx4 *)((_Float16 *)epi.C + row * epi.ldc + col));
                                } else
                                __builtin_nontemporal_store(x, (floatx4 *)((float *)epi.C + row * epi.ldc + col));
                                if (emit) {
                                    bf16x4 nb;
#pragma unroll
                                    for (int e = 0; e < 4; e++) nb[e] = (bf16)(x[e] * gain4[e]);
                                    *(bf16x4 *)((bf16 *)epi.norm_out + row * epi.norm_ld + col) = nb;
                                }
                            } else {
                                for (int e = 0; e < 4 && col + e < N; e++) {
                                    float y = x[e];
                                    if (KIND == EPI_F32 && epi.bias) y += epi.bias[col + e];
                                    if (KIND == EPI_F32_RESID) y += epi.resid[row * epi.ldr + col + e];
                                    if (KIND == EPI_F32_TABLE) y += epi.table[(epi.tok ? (int64_t)epi.tok[row] : 0) * N + col + e];
                                    if (KIND == EPI_F32 && epi.out_f16) ((_Float16 *)epi.C)[row * epi.ldc + col + e] = (_Float16)y;
                                    else ((float *)epi.C)[row * epi.ldc + col + e] = y;
                                }
                            }
                        }
                    }
                    if (pass < 3) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
            }
        }
        if (!has_next) break;
        // ---- the next tile becomes current; the staging slots take its W(1) and A(2) ----
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();  // every wave has read its staged rows back before the slots are overwritten
        asm volatile("" ::: "memory");
        L = Lnext;
        m0 = m0n; n0 = n0n; baseA = baseAn; baseW = baseWn;
        maxa = maxan; maxw = maxwn;
        Lnext = next_live(L + nslots);
        has_next = Lnext < xcd_end;
        if (has_next) {  // (else the "next" sources stay on what is now the current tile)
            tile_coords(Lnext, m0n, n0n);
            tile_sources(m0n, n0n, baseAn, baseWn, maxan, maxwn);
        }
        issue_w(1, sa);
        if (F8) issue_a(2, sw);
        sa = sa + 2 >= RING_SLOTS ? sa + 2 - RING_SLOTS : sa + 2;
        // A(0), W(0) of the new tile landed before its predecessor's last barrier
        if (F8) load_step8(sa, sa + 1 >= RING_SLOTS ? sa + 1 - RING_SLOTS : sa + 1, 0);
        else read_frags(fa0, fw0, sa, sa + 1 >= RING_SLOTS ? sa + 1 - RING_SLOTS : sa + 1, 0);
    }
#undef SB
#undef LD8
#undef WAIT8
#undef MMA8
}

template <int KIND, bool F8 = false>
static int launch_ring_kind(const bf16 *A, int64_t lda, const bf16 *W, int64_t ldw, int64_t M, int N, int K, const GemmEpilogue &epi,
                            hipStream_t st) {
    auto kern = gemm_bf16_ring<KIND, F8>;
    static bool attr_done = false;
    static int n_cu = 0;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, RING_LDS_BYTES) != hipSuccess) return GR4AD_EHIP;
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return GR4AD_EHIP;
        n_cu = prop.multiProcessorCount;
        attr_done = true;
    }
    const int64_t tiles_m = ceil_div64(M, 256);
    const int tiles_n = (N + 255) / 256;
    const int64_t total = tiles_m * tiles_n;
    if (total > 0x7fffffffLL) return GR4AD_EUNSUPPORTED;
    // one workgroup per compute unit (the ring takes the whole LDS), a multiple of the 8 XCDs
    int64_t grid = n_cu / 8 * 8;
    if (grid < 8) grid = 8;
    if (total < grid) grid = ceil_div64(total, 8) * 8;
    {
        const double operand_bytes = F8 ? ((double)M * K + (double)N * K) : 0.0;  // FP8 operands are half the bytes gemm_bytes counts
        ProfScope ps(F8 ? KC_GEMM_RING_F8 : KC_GEMM_RING, st, 2.0 * (double)M * N * K,
                     gemm_bytes(M, N, K, kind_f32(KIND) && !epi.out_f16, KIND == EPI_F32_RESID) - operand_bytes);
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), RING_LDS_BYTES, st, A, lda, W, ldw, M, N, K, tiles_m, tiles_n, 4, epi);
    }
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// The persistent kernel stores 16-byte pieces: it needs 16-byte aligned rows of C (and of what the epilogue adds),
// at least three k-tiles, and row pitches whose byte offsets inside a 256-row block fit 32 bits.
static bool ring_ok(int kind, int N, int K, int64_t lda, int64_t ldw, const GemmEpilogue &e) {
    const bool f32 = kind_f32(kind);
    if (e.skip_len && e.skip_S < 0) return false;
    if (K < 192 || lda >= (1 << 22) || ldw >= (1 << 22)) return false;
    if (e.out_f16 && kind != EPI_F32) return false;
    if (e.ldc % (f32 ? 4 : 8) || ((uintptr_t)e.C % 16)) return false;
    if (kind == EPI_F32 && e.bias && ((uintptr_t)e.bias % 16)) return false;
    if (kind == EPI_F32_RESID && (e.ldr % 4 || ((uintptr_t)e.resid % 16))) return false;
    if (kind == EPI_F32_TABLE && (N % 4 || ((uintptr_t)e.table % 16))) return false;
    if (e.norm_out) {  // folded RMSNorm, producer side
        if ((kind != EPI_F32_RESID && kind != EPI_F32_TABLE) || N % 256 || !e.norm_gain || !e.norm_ss) return false;
        if (e.norm_ld % 4 || ((uintptr_t)e.norm_out % 8) || ((uintptr_t)e.norm_gain % 8)) return false;
    }
    if (e.row_inv && kind == EPI_VT) return false;  // reader side
    return true;
}

// the staged epilogue of the tile kernel stores 16-byte pieces like the persistent kernel's
static bool tile_staged_ok(int kind, int N, const GemmEpilogue &e) {
    const bool f32 = kind_f32(kind);
    if (e.ldc % (f32 ? 4 : 8) || ((uintptr_t)e.C % 16) || N % (f32 ? 4 : 8)) return false;
    if (kind == EPI_F32 && e.bias && ((uintptr_t)e.bias % 16)) return false;
    if (kind == EPI_F32_RESID && (e.ldr % 4 || ((uintptr_t)e.resid % 16))) return false;
    return kind != EPI_F32_TABLE || ((uintptr_t)e.table % 16) == 0;
}

static int launch_ring(const bf16 *A, int64_t lda, const bf16 *W, int64_t ldw, int64_t M, int N, int K, int kind, const GemmEpilogue &epi,
                       hipStream_t st) {
    switch (kind) {
        case EPI_STORE: return launch_ring_kind<EPI_STORE>(A, lda, W, ldw, M, N, K, epi, st);
        case EPI_SILU: return launch_ring_kind<EPI_SILU>(A, lda, W, ldw, M, N, K, epi, st);
        case EPI_F32: return launch_ring_kind<EPI_F32>(A, lda, W, ldw, M, N, K, epi, st);
        case EPI_F32_RESID: return launch_ring_kind<EPI_F32_RESID>(A, lda, W, ldw, M, N, K, epi, st);
        case EPI_VT: return launch_ring_kind<EPI_VT>(A, lda, W, ldw, M, N, K, epi, st);
        case EPI_SILU_DIV: return launch_ring_kind<EPI_SILU_DIV>(A, lda, W, ldw, M, N, K, epi, st);
        default: return launch_ring_kind<EPI_F32_TABLE>(A, lda, W, ldw, M, N, K, epi, st);
    }
}

// Which fused epilogues the MFMA kernel covers; anything else runs on the plain kernel.
static int epilogue_kind(const GemmEpilogue &e) {
    const bool extra = e.bias || e.table || e.resid || e.act != ACT_NONE;
    if (!e.out_f32 && !extra) return EPI_STORE;
    if (!e.out_f32 && e.act == ACT_SILU && !e.bias && !e.table && !e.resid) return EPI_SILU;
    if (e.out_f32 && !e.table && !e.resid && e.act == ACT_NONE) return EPI_F32;
    if (e.out_f32 && e.resid && !e.bias && !e.table && e.act == ACT_NONE) return EPI_F32_RESID;
    if (e.out_f32 && e.table && !e.bias && !e.resid && e.act == ACT_NONE) return EPI_F32_TABLE;
    return -1;
}

// ---------------------------------------------------------------------------
// MFMA kernel of the small and middle shapes: one output tile per workgroup, ring of ST k-tiles in LDS
// ---------------------------------------------------------------------------
// The persistent kernel needs about one 256x256 tile per compute unit; a decode of a few requests has products of 1 to a few
// thousand rows, whose time is the latency of one tile.  So the tiles are small (32x32 to 128x128) to spread over the chip, and the work of a
// workgroup is divided: wavefronts of their own (NL loaders) stream the operands from global memory into an LDS ring of ST k-tiles (64 values of
// k) and the others multiply.  A wavefront issues a 1 KB load every 25 to 35 cycles while its data comes from beyond the L1, so a wavefront that
// multiplied and loaded spent more cycles issuing the eight loads of its k-tile (264) than on its four MFMAs (144), and none of its MFMAs ran before
// the first ST k-tiles were requested: M = 32, N = K = 512 took 4.0 us with the loads between the MFMAs of 32x64 tiles, now 3.3 (an empty kernel: 2.35);
// N = K = 1024 5.3, now 4.0; N = 1024, K = 4096 17.1, now 8.5 to 10.8; on 128x128 tiles M = 4096, N = K = 1024 13.5, now 12.2.
// NL = 0: every wavefront loads its share of the k-tiles itself, and two (128x128, 64 KB of LDS) or three (64x64) workgroups share a compute unit: one's
// epilogue runs beside another's k-loop.  For launches of several rounds, where the loaders' one workgroup per unit has nothing beside its epilogue: 8192 x 1024 x 1024 with a
// residual 36.6 us with loaders, 27.6 without; sixteen batches of 8192 x 1024 x 64 105 and 71; 64x64 tiles 8000 x 1024 x 1024 float32 32.5 and 30.4.  LDS is
// only asked for the k-tiles that exist (K = 64: one).
// Same LDS geometry as the persistent kernel: 128-byte rows, chunk c of row r at position c ^ ((r >> 1) & 7).  One barrier per k-tile: the loaders
// pass it when the k-tile has landed, the others when the one before (32x32 blocks: the one before that) has left LDS.  A product of one C
// element is the same sequence of v_mfma_f32_32x32x16 over k as in the persistent kernel: the two give the same bits.
// STAGED (WN = 64, N and C aligned): operands swapped, C leaves through LDS in 16-byte pieces of whole rows, with everything the
// persistent kernel's epilogue offers.  Otherwise a lane stores the 16 rows of its column directly (64 or 128 bytes per half
// wavefront and register), any N and pitch; EPI_VT swaps the operands so that these are 32 consecutive tokens of a column.
// The addends of 32 rows in the read-back layout of the staged epilogue: piece it is row it*4 + lane/16, columns
// (lane%16)*4 .. +3 (zero outside C).  Requested before the operands, they arrive under the main loop; requested in the epilogue
// each pass waits for them (8192 x 512 x 512: 14.2 us, now 11).
template <int KIND>
__device__ __forceinline__ void staged_addends(floatx4 (&adds)[8], int64_t row0, int wcol0, int64_t M, int N, const GemmEpilogue &epi, int lane) {
    if (KIND != EPI_F32_RESID && KIND != EPI_F32_TABLE) return;
    const int ecol = wcol0 + (lane % 16) * 4;
#pragma unroll
    for (int it = 0; it < 8; it++) {
        const int64_t row = row0 + it * 4 + lane / 16;
        adds[it] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        if (row < M && ecol < N) {
            if (KIND == EPI_F32_RESID) adds[it] = *(const floatx4 *)(epi.resid + row * epi.ldr + ecol);
            else adds[it] = *(const floatx4 *)(epi.table + (epi.tok ? (int64_t)epi.tok[row] : 0) * N + ecol);
        }
    }
}

template <int KIND, int TM>
__device__ __forceinline__ void staged_epilogue(floatx16 (&acc)[TM][2], const floatx4 (&adds)[TM][8], char *stage, int64_t wrow0, int wcol0, int64_t M, int N,
                                                const GemmEpilogue &epi, int lane) {
    const int frow = lane % 32, hf = lane / 32;
    if (epi.row_inv) {  // folded RMSNorm, reader side: a lane owns row frow of each 32-row block
#pragma unroll
        for (int i = 0; i < TM; i++) {
            const int64_t row = wrow0 + i * 32 + frow;
            const float f = epi.row_inv[row < M ? row : M - 1];
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int v = 0; v < 16; v++) acc[i][j][v] *= f;
        }
    }
    if (!kind_f32(KIND)) {
        // passes of 64 rows x 64 columns: 128-byte rows of 8 chunks, chunk c of row r at position c ^ (r & 7)
#pragma unroll
        for (int pass = 0; pass < TM / 2; pass++) {
#pragma unroll
            for (int ii = 0; ii < 2; ii++) {
                const int r = ii * 32 + frow;
#pragma unroll
                for (int j = 0; j < 2; j++)
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        bf16x4 pk;
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const float x = acc[pass * 2 + ii][j][4 * g + e];
                            pk[e] = (bf16)(KIND == EPI_SILU ? fast_silu(x) : KIND == EPI_SILU_DIV ? x / (1.0f + __expf(-x)) : x);
                        }
                        const int c = j * 4 + g;
                        *(bf16x4 *)(stage + r * 128 + ((c ^ (r & 7)) * 16) + hf * 8) = pk;
                    }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // wave-private region: no barrier needed
            const char *rd = stage + (lane / 8) * 128 + (((lane % 8) ^ ((lane / 8) & 7)) * 16);
            const int64_t row0 = wrow0 + pass * 64 + lane / 8;
            const int col = wcol0 + (lane % 8) * 8;
            bf16 *wr = (bf16 *)epi.C + row0 * epi.ldc + col;
#pragma unroll
            for (int it = 0; it < 8; it++)
                if (row0 + it * 8 < M && col < N) *(bf16x8 *)(wr + (int64_t)(it * 8) * epi.ldc) = *(const bf16x8 *)(rd + it * 1024);
            if (pass + 1 < TM / 2) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    } else {
        // passes of 32 rows x 64 columns: 256-byte rows of 16 chunks, chunk c of row r at position c ^ (r & 15)
        const int erow = lane / 16, ecol = wcol0 + (lane % 16) * 4;
        const bool emit = KIND != EPI_F32 && epi.norm_out != nullptr;  // folded RMSNorm, writer side (N % 256 == 0)
        floatx4 bias4 = {0.0f, 0.0f, 0.0f, 0.0f}, gain4 = {0.0f, 0.0f, 0.0f, 0.0f};
        if (KIND == EPI_F32 && epi.bias && ecol < N) bias4 = *(const floatx4 *)(epi.bias + ecol);
        if (emit) {
            const bf16x4 g4 = *(const bf16x4 *)((const bf16 *)epi.norm_gain + ecol);
#pragma unroll
            for (int e = 0; e < 4; e++) gain4[e] = (float)g4[e];
        }
#pragma unroll
        for (int pass = 0; pass < TM; pass++) {
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    floatx4 pk;
#pragma unroll
                    for (int e = 0; e < 4; e++) pk[e] = acc[pass][j][4 * g + e];
                    const int c = j * 8 + g * 2 + hf;
                    *(floatx4 *)(stage + frow * 256 + ((c ^ (frow & 15)) * 16)) = pk;
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int it = 0; it < 8; it++) {
                const int rr = it * 4 + erow, c = lane % 16;
                floatx4 x = *(const floatx4 *)(stage + rr * 256 + ((c ^ (rr & 15)) * 16));
                const int64_t row = wrow0 + pass * 32 + rr;
                if (KIND != EPI_F32) x += adds[pass][it];
                if (emit) {  // sum of squares over the row's 64 columns of this wavefront: the same tree as in the persistent kernel
                    float sq = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
                    sq += lane_xor1(sq);
                    sq += lane_xor2(sq);
                    sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x114, 0xf, 0xf, true));
                    sq += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, sq), 0x118, 0xf, 0xf, true));
                    if (lane % 16 == 15 && row < M) epi.norm_ss[row * (N / 64) + (wcol0 >> 6)] = sq;
                }
                if (row < M && ecol < N) {
                    if (KIND == EPI_F32) x += bias4;
                    if (KIND == EPI_F32 && epi.out_f16) {
                        halfx4 hx;
#pragma unroll
                        for (int e = 0; e < 4; e++) hx[e] = (_Float16)x[e];
                        *(halfx4 *)((_Float16 *)epi.C + row * epi.ldc + ecol) = hx;
                    } else {
                        *(floatx4 *)((float *)epi.C + row * epi.ldc + ecol) = x;
                    }
                    if (emit) {
                        bf16x4 nb;
#pragma unroll
                        for (int e = 0; e < 4; e++) nb[e] = (bf16)(x[e] * gain4[e]);
                        *(bf16x4 *)((bf16 *)epi.norm_out + row * epi.norm_ld + ecol) = nb;
                    }
                }
            }
            if (pass < TM - 1) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    }
}

template <typename T> __device__ __forceinline__ void step_ptr(T *&p, int64_t by) {
    p += by;
    asm volatile("" : "+v"(p));  // (keeps the compiler from forming every address anew: a 64-bit multiply-add is three quarter-rate instructions)
}

// One wave tile of 32 x 32 accumulators at (row0, col0), operands in natural order (a lane owns column lane % 32 and, per register v,
// row 8 * (v / 4) + 4 * (lane / 32) + v % 4); EPI_VT: swapped (a lane owns row lane % 32 and 16 columns).  The addresses run: formed one
// by one they cost 0.3 us of a small product each way.
template <typename T> __device__ __forceinline__ void next_row(T *&p, int v, int64_t ld) { step_ptr(p, v % 4 == 3 ? 5 * ld : ld); }  // register v to v + 1
// What the epilogue adds to the 16 elements of a lane; rows and columns past the edge read inside the arrays and are dropped.
template <int KIND>
__device__ __forceinline__ void direct_addends(float (&add)[16], int64_t row0, int col0, int64_t M, int N, const GemmEpilogue &epi, int lane) {
    if (KIND != EPI_F32_RESID && KIND != EPI_F32_TABLE) return;
    const int hf = lane / 32, c = col0 + lane % 32, col = c < N ? c : N - 1;
    if (row0 >= M) row0 = M - 1;  // (a block wholly past the edge)
    const int last = M - 1 - row0 < 31 ? (int)(M - 1 - row0) : 31;  // last row of the block inside C, 0 .. 31
    if (KIND == EPI_F32_RESID) {
        const float *p = epi.resid + (row0 + 4 * hf) * epi.ldr + col, *end = epi.resid + (row0 + last) * epi.ldr + col;
#pragma unroll
        for (int v = 0; v < 16; v++) {
            add[v] = *(last == 31 || p < end ? p : end);
            next_row(p, v, epi.ldr);
        }
    } else {
        uint32_t sel[16];
        if (epi.tok) {
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int r = 8 * (v / 4) + v % 4 + 4 * hf;
                sel[v] = (uint32_t)(epi.tok + row0)[r < last ? r : last];
            }
        } else {
#pragma unroll
            for (int v = 0; v < 16; v++) sel[v] = 0;
        }
#pragma unroll
        for (int v = 0; v < 16; v++) add[v] = (epi.table + col)[(uint64_t)sel[v] * (uint32_t)N];
    }
}

template <int KIND>
__device__ __forceinline__ void direct_epilogue(const floatx16 &acc, const float (&add)[16], int64_t row0, int col0, int64_t M, int N,
                                                const GemmEpilogue &epi, int lane) {
    const int frow = lane % 32, hf = lane / 32;
    if (KIND == EPI_VT) {
        // out[(b*N + n) * ldc + s] for token s of request b: zero from the request's length on
        const int64_t row = row0 + frow;
        if (row >= M) return;
        const uint32_t b = (uint32_t)row / (uint32_t)epi.vt_S;  // (fewer than 2^31 rows)
        const int s = (int)((uint32_t)row - b * (uint32_t)epi.vt_S);
        int len = epi.ctx_len ? epi.ctx_len[b] : epi.vt_rows;
        len = len < 1 ? 1 : (len > epi.vt_rows ? epi.vt_rows : len);
        bf16 *o = (bf16 *)epi.C + ((int64_t)b * N + col0 + 4 * hf) * epi.ldc + s;
#pragma unroll
        for (int v = 0; v < 16; v++) {
            if (col0 + 4 * hf + 8 * (v / 4) + v % 4 < N) *o = s < len ? (bf16)acc[v] : (bf16)0.0f;
            next_row(o, v, epi.ldc);
        }
        return;
    }
    const int col = col0 + frow;
    if (col >= N) return;
    const float bias = (KIND == EPI_F32 && epi.bias) ? epi.bias[col] : 0.0f;
    constexpr int E = kind_f32(KIND) ? 4 : 2;
    char *p = (char *)epi.C + ((row0 + 4 * hf) * epi.ldc + col) * E;
    auto store = [&](int v) {
        const float x = acc[v];
        if (KIND == EPI_STORE) *(bf16 *)p = (bf16)x;
        else if (KIND == EPI_SILU) *(bf16 *)p = (bf16)fast_silu(x);
        else if (KIND == EPI_SILU_DIV) *(bf16 *)p = (bf16)(x / (1.0f + __expf(-x)));
        else if (KIND == EPI_F32) *(float *)p = x + bias;
        else *(float *)p = x + add[v];
    };
    const int rows = M - row0 < 32 ? (int)(M - row0) : 32;
    if (rows == 32) {
#pragma unroll
        for (int v = 0; v < 16; v++) {
            store(v);
            next_row(p, v, epi.ldc * E);
        }
    } else {
#pragma unroll
        for (int v = 0; v < 16; v++) {
            if (4 * hf + 8 * (v / 4) + v % 4 < rows) store(v);
            next_row(p, v, epi.ldc * E);
        }
    }
}

template <int BM, int BN, int WM, int WN, int NL, int ST, int KIND, bool STAGED, bool BATCHED>
__global__ __launch_bounds__(((BM / WM) * (BN / WN) + NL) * 64) void gemm_bf16_tile(const bf16 *__restrict__ A, int64_t lda, const bf16 *__restrict__ W,
                                                                                    int64_t ldw, int64_t M, int N, int K, int tiles_m, int tiles_n,
                                                                                    GemmEpilogue epi, int64_t batch_a, int64_t batch_w, int64_t batch_c) {
    constexpr int WAVES_N = BN / WN, NC = (BM / WM) * WAVES_N, TM = WM / 32, TN = WN / 32;
    constexpr bool OWN = NL == 0;                     // the wavefronts load what they multiply
    constexpr int NLW = OWN ? NC : NL;                // wavefronts that load
    constexpr int LPW = (BM + BN) / 8 / NLW;          // loads of each per k-tile (1 KB each: 8 rows)
    constexpr int STAGE = (BM + BN) * 128;            // bytes of a k-tile
    constexpr bool SWAP = STAGED || KIND == EPI_VT;   // W fragment first
    constexpr bool ONE = TM * TN == 1 && !OWN;        // one 32x32 block per wavefront: a whole k-tile of fragments ahead
    constexpr int LAG = ONE ? 2 : 1;                  // past barrier j the slots of k-tiles up to j - LAG are free
    constexpr int LA = BM / 8 / NLW;                  // the first of them fetch rows of A, the others rows of W
    static_assert(BM / 8 % NLW == 0 && BN / 8 % NLW == 0 && (ST - 1) * LPW <= 63 && ST > LAG && (!OWN || ST <= 3), "load counts");
    static_assert(!STAGED || WN == 64, "the staged epilogue takes wave tiles of 64 columns");
    extern __shared__ bf16x8 smem[];
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // blockIdx.y: batch index; the operands and the output of batch i start batch_a/w/c elements further on
    if (BATCHED) {
        A += (int64_t)blockIdx.y * batch_a;
        W += (int64_t)blockIdx.y * batch_w;
        epi.C = (char *)epi.C + (int64_t)blockIdx.y * batch_c * (kind_f32(KIND) ? 4 : 2);
    }
    if (!BATCHED && KIND != EPI_VT && STAGED && epi.skip_len && !epi.skip_S) {  // the row count is known on the device only; M is its bound
        M = epi.skip_len[0];
        tiles_m = (int)((M + BM - 1) / BM);
    }
    // XCD-aware order: consecutive workgroup ids land on different XCDs (each with its own L2), so every XCD gets a contiguous range
    // of tiles, walked in groups of 8 row blocks (rows fastest): the tiles in flight on an XCD share their A and W blocks
    const uint32_t total = (uint32_t)tiles_m * (uint32_t)tiles_n, per_xcd = (total + 7) / 8;
    const uint32_t l = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || l >= total) return;
    const uint32_t gsz = 8u * (uint32_t)tiles_n, grp = l / gsz, in = l - grp * gsz;
    const uint32_t left = (uint32_t)tiles_m - grp * 8, gm = left < 8 ? left : 8;
    const int64_t m0 = (int64_t)(grp * 8 + in % gm) * BM;
    const int n0 = (int)(in / gm) * BN;
    if (BATCHED && epi.batch_len) {  // a valid length per batch: bounds the columns of C that are needed (1) or K (2)
        int len = epi.batch_len[blockIdx.y];
        len = len < 1 ? 1 : len;
        if (epi.len_bounds == 1 && n0 >= len) return;
        if (epi.len_bounds == 2 && len < K) K = (len + 63) / 64 * 64;
    }
    if (!BATCHED && (KIND == EPI_STORE || KIND == EPI_VT) && epi.skip_len && epi.skip_S) {
        // all rows of the tile in one request's padding, past the 64-row block of its last valid row: nobody reads the product
        const uint32_t r0 = (uint32_t)m0, S = (uint32_t)epi.skip_S, b0 = r0 / S;
        if (b0 == (r0 + BM - 1) / S) {
            const int len = epi.skip_len[b0];
            if (r0 - b0 * S >= (uint32_t)(len < 1 ? 64 : (len + 63) / 64 * 64)) return;
        }
    }
    const int KT = K / 64;
    auto bar = [&]() {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // ---- loads: piece p = i * NLW + me fills rows 8p .. 8p+7 of the k-tile's BM rows of A and BN rows of W, lane -> row lane/8,
    // position lane%8 (rows past the matrix edge re-read its last row) ----
    // A lane's byte offset in its operand block stays, the two block addresses move on: no vector arithmetic per k-tile.
    const int me = OWN ? wave : wave - NC;
    const char *base_a, *base_w;
    uint32_t off[LPW];
    auto start = [&]() {
        auto source = [&](int64_t row) -> int64_t {  // row of A behind row `row` of C
            const int64_t r = row < M ? row : M - 1;
            if (KIND != EPI_VT) return r;
            const uint32_t b = (uint32_t)r / (uint32_t)epi.vt_S, t = (uint32_t)r - b * (uint32_t)epi.vt_S;  // (see the persistent kernel)
            return (int64_t)b * epi.vt_rows + (t < (uint32_t)epi.vt_rows ? t : (uint32_t)epi.vt_rows - 1);
        };
        const int64_t first_row = source(m0);
        base_a = (const char *)(A + first_row * lda);
        base_w = (const char *)(W + (int64_t)n0 * ldw);
#pragma unroll
        for (int i = 0; i < LPW; i++) {
            const int p = i * NLW + me, r = p * 8 + lane / 8, chunk = (lane % 8) ^ ((4 * (p & 1)) ^ (lane / 16));
            if (i < LA) off[i] = (uint32_t)(source(m0 + r) - first_row) * ((uint32_t)lda * 2) + chunk * 16;
            else off[i] = (uint32_t)(n0 + r - BM < N ? r - BM : N - 1 - n0) * ((uint32_t)ldw * 2) + chunk * 16;
        }
    };
    auto issue = [&](uint32_t at) {  // k-tiles are requested in ascending order; at: byte offset of the slot
#pragma unroll
        for (int i = 0; i < LPW; i++)
            ring_dma16((i < LA ? base_a : base_w) + off[i], (bf16x8 *)((char *)smem + at + (i * NLW + me) * 1024));
        base_a += 128;
        base_w += 128;
    };
    auto landed = [&](auto n) {  // this wavefront's share of all but the newest n k-tiles is there; past the barrier everybody's is
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n.value * LPW) : "memory");
        bar();
    };
    const int first = KT < ST ? KT : ST;
    if (!OWN && wave >= NC) {  // ---- loader ----
        start();
        auto rest = [&](auto self, auto n) {  // the last n + 1 k-tiles
            if constexpr (n.value >= 0) {
                if (KT > n.value) landed(n);
                self(self, std::integral_constant<int, n.value - 1>());
            }
        };
        for (int t = 0; t < first; t++) issue((uint32_t)(t * STAGE));
        if (KT >= ST) {
            landed(std::integral_constant<int, ST - 1>());
            if constexpr (LAG == 2) landed(std::integral_constant<int, ST - 2>());
            uint32_t at = 0;
            for (int t = ST; t < KT; t++) {  // past the barrier of k-tile t - ST + LAG the slot of k-tile t - ST is free
                landed(std::integral_constant<int, ST - 1 - LAG>());
                issue(at);
                at = at + STAGE == (uint32_t)(ST * STAGE) ? 0u : at + (uint32_t)STAGE;
            }
            rest(rest, std::integral_constant<int, ST - 1 - LAG>());
        } else {
            rest(rest, std::integral_constant<int, ST - 2>());
        }
        return;
    }

    // ---- fragments: lane reads row frow of a 32-row block, chunk 2s + hf of k-step s, i.e. position (hf ^ fx) ^ 2s ----
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int64_t wrow0 = m0 + wm * WM;
    const int wcol0 = n0 + wn * WN;
    float add[16];
    floatx4 adds[TM][8];
    // (on their way before the operands)
    if constexpr (STAGED) {
#pragma unroll
        for (int i = 0; i < TM; i++) staged_addends<KIND>(adds[i], wrow0 + i * 32, wcol0, M, N, epi, lane);
    } else if (TM * TN == 1) direct_addends<KIND>(add, wrow0, wcol0, M, N, epi, lane);
    if (OWN) {
        start();
        for (int t = 0; t < first; t++) issue((uint32_t)(t * STAGE));
    }
    const int frow = lane % 32, hf = lane / 32, fx = (frow >> 1) & 7;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const uint32_t a_lane = lds0 + (uint32_t)((wm * WM + frow) * 8 + (hf ^ fx)) * 16;
    const uint32_t w_lane = lds0 + (uint32_t)((BM + wn * WN + frow) * 8 + (hf ^ fx)) * 16;
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.0f;
    uint32_t at = 0;
    auto advance = [&]() { at = at + STAGE == (uint32_t)(ST * STAGE) ? 0u : at + (uint32_t)STAGE; };
#define SB __builtin_amdgcn_sched_barrier(0)
    if constexpr (ONE) {
        // The k-tile is one chain of four MFMAs (144 cycles), shorter than an LDS read takes: the fragments of a k-tile are read under the
        // MFMAs of the one before the last.
        bf16x8 af[2][4], wf[2][4];
        auto read = [&](auto p) {  // the next k-tile's fragments into set p
            bar();
#pragma unroll
            for (int s = 0; s < 4; s++) {
                asm volatile("ds_read_b128 %0, %1" : "=v"(af[p.value][s]) : "v"((a_lane ^ (uint32_t)(s << 5)) + at));
                asm volatile("ds_read_b128 %0, %1" : "=v"(wf[p.value][s]) : "v"((w_lane ^ (uint32_t)(s << 5)) + at));
            }
            advance();
        };
        auto mma = [&](auto p, auto behind) {  // behind: reads issued after set p's
            bf16x8(&a)[4] = af[p.value], (&w)[4] = wf[p.value];
            SB;
            asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(behind.value) : "memory");  // (before the copies that the next line's operands may take)
            SB;
            asm volatile("s_waitcnt lgkmcnt(%8)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]) : "n"(behind.value));
            SB;
#pragma unroll
            for (int s = 0; s < 4; s++)
                acc[0][0] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[s], a[s], acc[0][0], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], w[s], acc[0][0], 0, 0, 0);
            SB;
        };
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, 1> c1{};
        constexpr std::integral_constant<int, 8> c8{};
        read(c0);
        int kt = 1;
        for (; kt + 1 < KT; kt += 2) {
            read(c1);
            mma(c0, c8);
            read(c0);
            mma(c1, c8);
        }
        if (kt < KT) {
            read(c1);
            mma(c0, c8);
            mma(c1, c0);
        } else {
            mma(c0, c0);
        }
    } else {
        // One barrier per k-tile, in its middle: the fragments of k-steps 2 and 3 have been read by then, so the slot is free, and the
        // first fragments of the next k-tile are read under the MFMAs of steps 2 and 3.
        bf16x8 af[4][TM], wf[4][TN];
        constexpr int R = TM + TN;  // reads of a k-step
        auto read = [&](int s) {
            const uint32_t pa = (a_lane ^ (uint32_t)(s << 5)) + at, pw = (w_lane ^ (uint32_t)(s << 5)) + at;
            asm volatile("ds_read_b128 %0, %1" : "=v"(af[s][0]) : "v"(pa));
            if constexpr (TM > 1) asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(af[s][TM - 1]) : "v"(pa));
            asm volatile("ds_read_b128 %0, %1" : "=v"(wf[s][0]) : "v"(pw));
            if constexpr (TN > 1) asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(wf[s][TN - 1]) : "v"(pw));
        };
        auto wait = [&](int s, auto n) {  // the fragments of step s are there, the newest n reads may still be on the way
            static_assert(TM == TN && TM <= 2, "wave tiles");
            bf16x8(&fa)[TM] = af[s], (&fw)[TN] = wf[s];
            if constexpr (TM == 2) asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(fa[0]), "+v"(fa[TM - 1]), "+v"(fw[0]), "+v"(fw[TN - 1]) : "n"(n.value));
            else asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(fa[0]), "+v"(fw[0]) : "n"(n.value));
        };
        auto mma = [&](int s) {
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++)
                    acc[i][j] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s][j], af[s][i], acc[i][j], 0, 0, 0)
                                     : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[s][i], wf[s][j], acc[i][j], 0, 0, 0);
        };
        constexpr std::integral_constant<int, 0> c0{};
        constexpr std::integral_constant<int, 2 * R> c2{};
        constexpr std::integral_constant<int, 3 * R> c3{};
        // One k-tile.  ahead (OWN): k-tiles that may be in flight beyond the next one (-1: this is the last); refill: k-tile kt + ST goes into its slot.
        auto step = [&](auto ahead, auto refill) {
            SB; read(2); read(3);
            wait(0, c3); SB; mma(0); SB;
            wait(1, c2); SB; mma(1); SB;
            wait(2, c0); wait(3, c0); SB;
            if constexpr (ahead.value >= 0) {
                if constexpr (OWN) landed(ahead);
                else bar();
                if constexpr (refill.value) issue(at);
                advance();
                SB; read(0); read(1); SB;
            }
            mma(2); mma(3);
        };
        constexpr std::integral_constant<int, -1> last{};
        if constexpr (OWN) {
            if (KT < ST) landed(c0);
            else landed(std::integral_constant<int, ST - 1>());
        } else bar();
        read(0);
        read(1);
        if constexpr (OWN) {
            for (int kt = ST; kt < KT; kt++) step(std::integral_constant<int, ST - 2>(), std::true_type());
            if constexpr (ST >= 3)
                if (KT >= 3) step(std::integral_constant<int, 1>(), std::false_type());
            if (KT >= 2) step(c0, std::false_type());
        } else {
            for (int kt = 1; kt < KT; kt++) step(c0, std::false_type());
        }
        step(last, std::false_type());
    }
#undef SB
    if constexpr (STAGED) {
        bar();  // every wavefront has read its last fragments: LDS becomes the staging area
        staged_epilogue<KIND, TM>(acc, adds, (char *)smem + wave * 8192, wrow0, wcol0, M, N, epi, lane);
    } else {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++) {
                if (TM * TN > 1) direct_addends<KIND>(add, wrow0 + i * 32, wcol0 + j * 32, M, N, epi, lane);
                direct_epilogue<KIND>(acc[i][j], add, wrow0 + i * 32, wcol0 + j * 32, M, N, epi, lane);
            }
    }
}

template <int BM, int BN, int WM, int WN, int NL, int ST, int KIND, bool STAGED, bool BATCHED = false>
static int launch_tile_kind(const bf16 *A, int64_t lda, const bf16 *W, int64_t ldw, int64_t M, int N, int K, const GemmEpilogue &epi,
                            hipStream_t st, int batch = 1, int64_t batch_a = 0, int64_t batch_w = 0, int64_t batch_c = 0) {
    constexpr int NT = ((BM / WM) * (BN / WN) + NL) * 64;
    constexpr int STAGE = (BM + BN) * 128, STAGING = STAGED ? (BM / WM) * (BN / WN) * 8192 : 0;  // bytes of a k-tile, and of the staged epilogue
    auto kern = gemm_bf16_tile<BM, BN, WM, WN, NL, ST, KIND, STAGED, BATCHED>;
    static bool attr_done = false;  // one attribute call per instantiation is enough (value never changes)
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, std::max(ST * STAGE, STAGING)) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const int smem = std::max((K / 64 < ST ? K / 64 : ST) * STAGE, STAGING);
    const int64_t tiles_m = ceil_div64(M, BM), tiles_n = (N + BN - 1) / BN, total = tiles_m * tiles_n;
    if (total > 0x7ffffff0LL || batch < 1 || batch > 65535 || lda >= (1 << 23) || ldw >= (1 << 23)) return GR4AD_EUNSUPPORTED;
    if (epi.skip_len && M > 0x7fffff00LL) return GR4AD_EUNSUPPORTED;
    {
        ProfScope ps(KC_GEMM_TILE, st, 2.0 * (double)M * N * K * batch, batch * gemm_bytes(M, N, K, kind_f32(KIND) && !epi.out_f16, KIND == EPI_F32_RESID));
        hipLaunchKernelGGL(kern, dim3((unsigned)(ceil_div64(total, 8) * 8), (unsigned)batch), dim3(NT), smem, st, A, lda, W, ldw, M, N, K, (int)tiles_m,
                           (int)tiles_n, epi, batch_a, batch_w, batch_c);
    }
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

template <int BM, int BN, int WM, int WN, int NL, int ST, bool STAGED>
static int launch_tile_cfg(const bf16 *A, int64_t lda, const bf16 *W, int64_t ldw, int64_t M, int N, int K, int kind, const GemmEpilogue &epi,
                           hipStream_t st, int batch, int64_t ba, int64_t bw, int64_t bc) {
#define KIND_(k) case k: return launch_tile_kind<BM, BN, WM, WN, NL, ST, k, STAGED>(A, lda, W, ldw, M, N, K, epi, st);
    if (batch > 1) {
        if (kind == EPI_STORE) return launch_tile_kind<BM, BN, WM, WN, NL, ST, EPI_STORE, STAGED, true>(A, lda, W, ldw, M, N, K, epi, st, batch, ba, bw, bc);
        if (kind == EPI_F32) return launch_tile_kind<BM, BN, WM, WN, NL, ST, EPI_F32, STAGED, true>(A, lda, W, ldw, M, N, K, epi, st, batch, ba, bw, bc);
        return GR4AD_EUNSUPPORTED;
    }
    switch (kind) {
        KIND_(EPI_STORE) KIND_(EPI_SILU_DIV) KIND_(EPI_F32) KIND_(EPI_F32_RESID) KIND_(EPI_F32_TABLE)
        case EPI_SILU: if constexpr (STAGED) return launch_tile_kind<BM, BN, WM, WN, NL, ST, EPI_SILU, STAGED>(A, lda, W, ldw, M, N, K, epi, st);
            return GR4AD_EUNSUPPORTED;
        case EPI_VT: if constexpr (!STAGED) return launch_tile_kind<BM, BN, WM, WN, NL, ST, EPI_VT, STAGED>(A, lda, W, ldw, M, N, K, epi, st);
            return GR4AD_EUNSUPPORTED;
    }
#undef KIND_
    return GR4AD_EUNSUPPORTED;
}

// Which kernel runs a product: the least of these estimates of its time in microseconds (all give the same bits).  Fitted to every kernel's time on 5300 products on
// MI355X: 64 <= M <= 32768, 256 <= N <= 8192, 64 <= K <= 4096, each epilogue, transposed values, and batches of 1 to 256 products of 1 to 12288 rows (rms error of an
// estimate 4 to 12 %; the kernel it picks takes 0.8 % longer than the best one in the mean, 1.4 times as long at worst).  A tile of the first round costs first[kind] +
// kt * k_first (kt: k-tiles of 64), every further round of 256 tiles more[kind] + kt * k_more, of which the second costs k_second.
// Where the lines lie (us, this kernel against the next best): 1024 x 512 x 512 32x64 4.2, 32x32 4.4; 256 x 3072 x 1024 64x64 6.0, 128x128 9.7; 2048 x 512 x 4096
// 64x64 15, 128x128 19; 4096 x 1024 x 1024 128x128 with loaders 12, 64x64 15; 8192 x 1024 x 1024 with a residual 128x128 in pairs 27.6, 256x256 33, 128x128 with
// loaders 37; 4096 x 3072 x 1024 256x256 26, 128x128 32; sixteen batches of 8192 x 1024 x 64 128x128 in pairs 71, with loaders 105.
enum { RUN_TILE32 = 0, RUN_TILE32X64, RUN_TILE64, RUN_TILE64_OWN, RUN_TILE128, RUN_TILE128_OWN, RUN_RING };
static int pick_kernel(int64_t M, int N, int K, int kind, int batch, bool tile64, bool tile128, bool ring) {
    struct Cost { int bm, bn; float start, first[6], more[6], k_first, k_second, k_more; };  // (kinds: bf16, SiLU, float32, residual, table, transposed)
    static const Cost cost[RUN_RING] = {
        {32, 32, 2.73f, {0.06f, 0.19f, 0.17f, 0.0f, 0.02f, 0.72f}, {0.14f, 0.18f, 0.18f, 0.22f, 0.23f, 0.09f}, 0.11f, 0.06f, 0.11f},
        {32, 64, 2.83f, {0.09f, 0.29f, 0.21f, 0.0f, 0.09f, 0.77f}, {0.22f, 0.33f, 0.27f, 0.4f, 0.42f, 0.35f}, 0.12f, 0.18f, 0.18f},
        {64, 64, 2.84f, {0.0f, 0.29f, 0.3f, 0.17f, 0.18f, 0.73f}, {0.7f, 0.78f, 0.74f, 1.1f, 1.06f, 0.68f}, 0.16f, 0.25f, 0.22f},
        {64, 64, 2.86f, {0.0f, 0.07f, 0.16f, 0.32f, 0.26f, 0.43f}, {0.36f, 0.58f, 0.54f, 1.07f, 1.05f, 0.44f}, 0.19f, 0.15f, 0.17f},
        {128, 128, 3.51f, {0.0f, 2.01f, 2.85f, 2.21f, 4.75f, 2.46f}, {1.69f, 2.47f, 3.09f, 7.33f, 8.75f, 3.64f}, 0.43f, 0.6f, 0.55f},
        {128, 128, 3.39f, {0.0f, 2.0f, 2.59f, 2.61f, 4.72f, 2.2f}, {1.28f, 1.95f, 2.45f, 5.46f, 5.85f, 2.03f}, 0.55f, 0.4f, 0.51f},
    };
    const int kc = kind == EPI_STORE ? 0 : kind == EPI_SILU || kind == EPI_SILU_DIV ? 1 : kind == EPI_F32 ? 2 : kind == EPI_F32_RESID ? 3 : kind == EPI_F32_TABLE ? 4 : 5;
    const float kt = (float)(K / 64);
    // Batches stream operands that no other batch reads, and eight k-tiles of LDS leave one workgroup per compute unit to ask for them (45 batches of 16 x 1024 x 512
    // 15.4 us on 32x64 tiles, 11.0 on 64x64 in threes)
    const bool stream = batch > 1 && ceil_div64(M, 64) * ceil_div64(N, 64) * batch > 256;
    float best = 1e30f;
    int run = RUN_TILE128;
    for (int r = stream ? RUN_TILE64_OWN : RUN_TILE32; r < RUN_RING; r++) {
        const Cost &c = cost[r];
        if (!(c.bm < 128 ? tile64 : tile128)) continue;
        int64_t tiles = ceil_div64(M, c.bm) * ceil_div64(N, c.bn);
        if (batch > 1) tiles = (tiles + 7) / 8 * 8 * batch;  // (a batch's tiles are dealt to the eight XCDs from the first on)
        const float more = (float)(ceil_div64(tiles, 256) - 1);
        const float t = c.start + c.first[kc] + kt * c.k_first + more * c.more[kc] + (more > 0.0f ? kt * (c.k_second + (more - 1.0f) * c.k_more) : 0.0f);
        if (t < best) { best = t; run = r; }
    }
    if (ring) {  // 256x256 tiles: full rounds, and a last one whose clock falls as it fills the chip
        static const float full[6] = {5.4f, 7.3f, 10.8f, 20.4f, 20.3f, 6.4f}, any[6] = {1.45f, 7.25f, 3.15f, 4.4f, 8.0f, 3.4f},
                           part[6] = {2.4f, 0.0f, 5.6f, 12.3f, 12.2f, 0.4f};
        const int64_t tiles = ceil_div64(M, 256) * ceil_div64(N, 256);
        const float f = (float)(tiles / 256), rest = (float)(tiles % 256) / 256.0f;
        const float t = 3.3f + f * (full[kc] + 1.49f * kt) + (rest > 0.0f ? any[kc] + 1.05f * kt + rest * (part[kc] + 0.44f * rest * kt) : 0.0f);
        if (t < best) run = RUN_RING;
    }
    return run;
}

static int launch_tile(int run, const bf16 *A, int64_t lda, const bf16 *W, int64_t ldw, int64_t M, int N, int K, int kind, const GemmEpilogue &epi,
                       hipStream_t st, int batch = 1, int64_t ba = 0, int64_t bw = 0, int64_t bc = 0) {
    const bool staged = kind != EPI_VT && tile_staged_ok(kind, N, epi);
    switch (run) {
        // with loaders: eight k-tiles in LDS, three of the large tiles; without: three and two, so that three and two workgroups share a compute unit
        case RUN_TILE32: return launch_tile_cfg<32, 32, 32, 32, 2, 8, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
        case RUN_TILE32X64: return launch_tile_cfg<32, 64, 32, 32, 2, 8, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
        case RUN_TILE64:  // (up to eight k-tiles: four, requested sooner: 256 x 3072 x 512 4.4 us, 4.1)
            if (K <= 512) return launch_tile_cfg<64, 64, 32, 32, 4, 4, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
            return launch_tile_cfg<64, 64, 32, 32, 4, 8, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
        case RUN_TILE64_OWN: return launch_tile_cfg<64, 64, 32, 32, 0, 3, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
        case RUN_TILE128_OWN:
            if (staged) return launch_tile_cfg<128, 128, 64, 64, 0, 2, true>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
            return launch_tile_cfg<128, 128, 64, 64, 0, 2, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
    }
    if (staged) return launch_tile_cfg<128, 128, 64, 64, 4, 3, true>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
    return launch_tile_cfg<128, 128, 64, 64, 4, 3, false>(A, lda, W, ldw, M, N, K, kind, epi, st, batch, ba, bw, bc);
}

// ---------------------------------------------------------------------------
// MFMA kernel of the small products behind an RMSNorm, Fuse's gate or the trunk's self-attention: the rows of A are formed by the workgroup that multiplies them
// ---------------------------------------------------------------------------
// Where launches are short a norm of its own is a launch of 1.7 to 4.7 us whose rows the product then waits for again.  Here a workgroup (8 wavefronts) requests
// its rows of x (float32, all K columns) and every k-tile of W it will multiply at once, normalises the rows while W is on the way, leaves them in LDS as the
// tile kernel's operand (bf16, rounded as the norm kernel rounds them) and multiplies: BM x BN / 1024 wavefronts, 32x32 each, one chain of MFMAs over K without a barrier.
// The price is that each column of tiles forms the rows anew, so it is for few tiles: the rule is at panel_shape.  Same order of every sum as rmsnorm_kernel
// and gemm_bf16_tile: same bits.
// LDS: BM x K values of A (a k-tile of 64 values: BM rows of 128 bytes), then BN x K of W.
// V: 16-byte pieces of a row per lane (1: K <= 512, 2: K <= 1024), 0: K <= 256, two rows to a wavefront.
// J: steps a wavefront takes its rows in (fewer than BM has: rows beyond them are past the last one).
// SRC: what the rows are: norms; products of a trunk row and a gate table's (Fuse); the trunk's causal self-attention - each as the kernel of its own forms it.
enum { ROWS_NORM = 0, ROWS_GATED, ROWS_TRUNK };
struct PanelRows {
    const float *x;       // ROWS_NORM: rows, gains and epsilon; ROWS_GATED: trunk row of request b at x + b * x_req
    const bf16 *gain;
    float eps;
    int n;                // ROWS_GATED: rows of a request; ROWS_TRUNK: its positions
    int64_t x_req;
    const float *table;   // ROWS_GATED: row tok[r] (0 if NULL)
    const int32_t *tok;
    const bf16 *qkv;      // ROWS_TRUNK: [rows, 3K]
    int lanes_per_head;   // K / heads / 8: 2, 4 or 8
};
struct PanelOut { void *C; int64_t ldc; const float *bias, *resid, *table; const int32_t *tok; int64_t ldr; };
// eight channels of one trunk row (as trunk_self_attn, whose lanes hold a channel each: its sums over lane ^ 32, ^ 16, ^ 8 are over lanes ^ 4, ^ 2, ^ 1 here, those over lane ^ 4, ^ 2, ^ 1 over
// a lane's own values)
__device__ __forceinline__ float lane_xor4(float v) { return dpp_move<0x1B, 0xF>(0.0f, dpp_move<0x141, 0xF>(0.0f, v)); }  // 7 - lane, then 3 - lane of the quad
__device__ __forceinline__ bf16x8 trunk_attended(const bf16x8 &q, const bf16x8 (&k)[4], const bf16x8 (&v)[4], int tau, int lph) {
#pragma clang fp contract(off)
    const float scale = 1.0f / sqrtf((float)(8 * lph));
    float s[4], mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < 4; p++) {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            e[i] = (float)q[i] * (float)k[p][i];
            if (lph > 4) e[i] += lane_xor4(e[i]);
            if (lph > 2) e[i] += lane_xor2(e[i]);
            e[i] += lane_xor1(e[i]);
        }
        const float sum = ((e[0] + e[4]) + (e[2] + e[6])) + ((e[1] + e[5]) + (e[3] + e[7]));
        s[p] = sum * scale;
        if (p <= tau) mx = fmaxf(mx, s[p]);
    }
    float den = 0.0f;
#pragma unroll
    for (int p = 0; p < 4; p++)
        if (p <= tau) { s[p] = __expf(s[p] - mx); den += s[p]; }
    const float inv = 1.0f / den;
    bf16x8 y;
#pragma unroll
    for (int i = 0; i < 8; i++) {
        float o = 0.0f;
#pragma unroll
        for (int p = 0; p < 4; p++)
            if (p <= tau) o = fmaf(s[p] * inv, (float)v[p][i], o);
        y[i] = (bf16)o;
    }
    return y;
}
template <int BM, int BN, int V, int J, int SRC, int KIND>
__global__ __launch_bounds__(512, 4) void gemm_bf16_panel(PanelRows rows, const bf16 *__restrict__ W, int64_t ldw, int M, int N, int K, int tiles_m, int tiles_n, PanelOut out) {
    constexpr int WAVES_N = BN / 32, NC = BM / 32 * WAVES_N, WTILE = BN * 128, PIECES = BN / 8;
    constexpr int VEC = V == 2 ? 2 : 1, KMAX = V == 0 ? 256 : 512 * V;
    static_assert(J * (V == 0 ? 16 : 8) <= BM, "rows of the tile");
    extern __shared__ bf16x8 smem[];
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // (the tile order of gemm_bf16_tile)
    const uint32_t total = (uint32_t)tiles_m * (uint32_t)tiles_n, per_xcd = (total + 7) / 8;
    const uint32_t l = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || l >= total) return;
    const uint32_t gsz = 8u * (uint32_t)tiles_n, grp = l / gsz, in = l - grp * gsz;
    const uint32_t left = (uint32_t)tiles_m - grp * 8, gm = left < 8 ? left : 8;
    const int m0 = (int)(grp * 8 + in % gm) * BM;
    const int n0 = (int)(in / gm) * BN;
    const int KT = K / 64;
    char *const panel = (char *)smem, *const slots = panel + BM * K * 2;

    // ---- what the rows are formed from: requested first, it is needed first.  Rows are dealt to the wavefronts in turn, those past the edge re-read the last one.
    // No branch between these loads and those of W, so that the compiler can count them and wait for the rows alone ----
    const int nvec = K / 8, pos = V == 0 ? lane % 32 : lane, half = V == 0 ? lane / 32 : 0;
    auto row_of = [&](int j) { return (j * 8 + wave) * (V == 0 ? 2 : 1) + half; };
    auto inside = [&](int j) { return m0 + row_of(j) < M ? m0 + row_of(j) : M - 1; };
    auto piece = [&](int i) { return pos + 64 * i < nvec ? pos + 64 * i : nvec - 1; };
    auto load8 = [](float *v, const float *p) {
        *(floatx4 *)v = *(const floatx4 *)p;
        *(floatx4 *)(v + 4) = *(const floatx4 *)(p + 4);
    };
    float v[J][VEC][8], u[J][VEC][8];
    bf16x8 g[VEC], q[J][VEC], k[J][VEC][4], w[J][VEC][4];
    int tau[J];
    if constexpr (SRC == ROWS_NORM) {
#pragma unroll
        for (int i = 0; i < VEC; i++) g[i] = *(const bf16x8 *)(rows.gain + piece(i) * 8);
        const float *xr = rows.x + (int64_t)m0 * K;  // (rows and columns of the block by 32-bit offsets)
#pragma unroll
        for (int j = 0; j < J; j++) {
            const int off = (inside(j) - m0) * K;
#pragma unroll
            for (int i = 0; i < VEC; i++) load8(v[j][i], xr + off + piece(i) * 8);
        }
    } else if constexpr (SRC == ROWS_GATED) {
        uint32_t sel[J];
#pragma unroll
        for (int j = 0; j < J; j++) sel[j] = rows.tok ? (uint32_t)rows.tok[inside(j)] : 0u;
#pragma unroll
        for (int j = 0; j < J; j++) {
            const float *mr = rows.x + (int64_t)((uint32_t)inside(j) / (uint32_t)rows.n) * rows.x_req, *gr = rows.table + (uint64_t)sel[j] * (uint32_t)K;
#pragma unroll
            for (int i = 0; i < VEC; i++) {
                load8(v[j][i], mr + piece(i) * 8);
                load8(u[j][i], gr + piece(i) * 8);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < J; j++) {
            const int r = inside(j);
            tau[j] = r % rows.n;
#pragma unroll
            for (int i = 0; i < VEC; i++) {
                const bf16 *src = rows.qkv + (int64_t)r * 3 * K + piece(i) * 8;
                q[j][i] = *(const bf16x8 *)src;
#pragma unroll
                for (int p = 0; p < 4; p++) {  // (positions past this row's re-read its own and are not used)
                    const bf16 *at = src - (int64_t)(p < tau[j] ? tau[j] - p : 0) * 3 * K;
                    k[j][i][p] = *(const bf16x8 *)(at + K);
                    w[j][i][p] = *(const bf16x8 *)(at + 2 * K);
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- W: piece p of a k-tile is its rows 8p .. 8p+7 (rows past the edge re-read the last one).  A wavefront has one piece of every k-tile (of every other one);
    // past the last k-tile it loads its last piece again ----
    auto source = [&](int pc, int t) {
        const int r = n0 + pc * 8 + lane / 8;
        return (const char *)(W + (int64_t)(r < N ? r : N - 1) * ldw) + t * 128 + ((lane % 8) ^ ((4 * (pc & 1)) ^ (lane / 16))) * 16;
    };
    {
        constexpr int EVERY = 8 / PIECES, LOADS = KMAX / 64 / EVERY;  // k-tiles from one of a wavefront's loads to the next; its loads
        const int t0 = wave / PIECES, last = KT > t0 ? (KT - 1 - t0) / EVERY : 0;  // (one k-tile, and none for this wavefront: it loads what another does)
        const char *src = source(wave % PIECES, KT > t0 ? t0 : 0);
        char *dst = slots + (KT > t0 ? wave : wave % PIECES) * 1024;
#pragma unroll
        for (int i = 0; i < LOADS; i++) {
            const int at = i < last ? i : last;
            ring_dma16(src + at * (EVERY * 128), (bf16x8 *)(dst + at * 8192));
        }
    }
    GemmEpilogue epi = {};
    epi.C = out.C;
    epi.ldc = out.ldc;
    epi.bias = out.bias;
    epi.resid = out.resid;
    epi.ldr = out.ldr;
    epi.table = out.table;
    epi.tok = out.tok;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int wrow0 = m0 + wm * 32, wcol0 = n0 + wn * 32;
    float add[16];
    if ((KIND == EPI_F32_RESID || KIND == EPI_F32_TABLE) && wave < NC) direct_addends<KIND>(add, wrow0, wcol0, M, N, epi, lane);
    __builtin_amdgcn_sched_barrier(0);
    auto put = [&](int j, int i, const bf16x8 &y) {
        const int r = row_of(j), c = pos + 64 * i;
        if (c < nvec) *(bf16x8 *)(panel + (c / 8) * (BM * 128) + r * 128 + ((c % 8) ^ ((r >> 1) & 7)) * 16) = y;
    };
    if constexpr (SRC == ROWS_NORM) {
        // ---- RMSNorm: four steps' factors at once, one in each lane of a quad (a division and a root are some fifty instructions) ----
        float ss[J], inv[J];
#pragma unroll
        for (int j = 0; j < J; j++) {
            const float one = first_squares(v[j][0]);
            ss[j] = pos < nvec ? one : 0.0f;
            if constexpr (VEC == 2) {
                const float two = more_squares(ss[j], v[j][1]);
                if (pos + 64 < nvec) ss[j] = two;
            }
        }
#pragma unroll
        for (int j = 0; j < J; j++) ss[j] = V == 0 ? half_wave_sum(ss[j]) : wave_sum(ss[j]);
#pragma unroll
        for (int j = 0; j < J; j += 4) {
            float mine = ss[j];
            if constexpr (J >= 2) mine = (lane & 1) ? ss[j + 1] : mine;
            if constexpr (J >= 4) mine = (lane & 2) ? ((lane & 1) ? ss[j + 3] : ss[j + 2]) : mine;
            const float f = rms_inv(mine, K, rows.eps);
            inv[j] = dpp_move<0x00, 0xF>(f, f);  // quad_perm: one lane of the quad to all four
            if constexpr (J >= 2) inv[j + 1] = dpp_move<0x55, 0xF>(f, f);
            if constexpr (J >= 4) {
                inv[j + 2] = dpp_move<0xAA, 0xF>(f, f);
                inv[j + 3] = dpp_move<0xFF, 0xF>(f, f);
            }
        }
#pragma unroll
        for (int j = 0; j < J; j++)
#pragma unroll
            for (int i = 0; i < VEC; i++) {
                bf16x8 y;
#pragma unroll
                for (int e = 0; e < 8; e++) y[e] = (bf16)((float)g[i][e] * v[j][i][e] * inv[j]);
                put(j, i, y);
            }
    } else if constexpr (SRC == ROWS_GATED) {
#pragma unroll
        for (int j = 0; j < J; j++)
#pragma unroll
            for (int i = 0; i < VEC; i++) {
                bf16x8 y;
#pragma unroll
                for (int e = 0; e < 8; e++) y[e] = (bf16)(v[j][i][e] * u[j][i][e]);
                put(j, i, y);
            }
    } else {
#pragma unroll
        for (int j = 0; j < J; j++)
#pragma unroll
            for (int i = 0; i < VEC; i++) put(j, i, trunk_attended(q[j][i], k[j][i], w[j][i], tau[j], rows.lanes_per_head));
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (wave >= NC) return;
    // ---- products: fragments as in gemm_bf16_tile, a k-tile ahead ----
    const int frow = lane % 32, hf = lane / 32, fx = (frow >> 1) & 7;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const uint32_t a_lane = lds0 + (uint32_t)((wm * 32 + frow) * 8 + (hf ^ fx)) * 16;
    const uint32_t w_lane = lds0 + (uint32_t)(BM * K * 2) + (uint32_t)((wn * 32 + frow) * 8 + (hf ^ fx)) * 16;
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; v++) acc[v] = 0.0f;
    struct Fragments { bf16x8 a[4], w[4]; };
    Fragments f0, f1;
    auto read = [&](Fragments &f, int t) {
        const uint32_t pa = a_lane + (uint32_t)(t * BM * 128), pw = w_lane + (uint32_t)(t * WTILE);
#pragma unroll
        for (int s = 0; s < 4; s++) {
            asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[s]) : "v"(pa ^ (uint32_t)(s << 5)));
            asm volatile("ds_read_b128 %0, %1" : "=v"(f.w[s]) : "v"(pw ^ (uint32_t)(s << 5)));
        }
    };
    auto mma = [&](Fragments &f, bool behind) {  // behind: the other set's eight reads were issued after this one's
        __builtin_amdgcn_sched_barrier(0);
        if (behind) asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");  // (before the copies that the next lines' operands may take)
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (behind) asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.w[0]), "+v"(f.w[1]), "+v"(f.w[2]), "+v"(f.w[3]));
        else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.a[2]), "+v"(f.a[3]), "+v"(f.w[0]), "+v"(f.w[1]), "+v"(f.w[2]), "+v"(f.w[3]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; s++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[s], f.w[s], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    read(f0, 0);
    int t = 1;
    for (; t + 1 < KT; t += 2) {
        read(f1, t);
        mma(f0, true);
        read(f0, t + 1);
        mma(f1, true);
    }
    if (t < KT) {
        read(f1, t);
        mma(f0, true);
        mma(f1, false);
    } else {
        mma(f0, false);
    }
    direct_epilogue<KIND>(acc, add, wrow0, wcol0, M, N, epi, lane);
}

template <int BM, int BN, int V, int J, int SRC, int KIND>
static int launch_panel_kind(const PanelRows &rows, const bf16 *W, int64_t ldw, int64_t M, int N, int K, const GemmEpilogue &epi, hipStream_t st) {
    auto kern = gemm_bf16_panel<BM, BN, V, J, SRC, KIND>;
    constexpr int KMAX = V == 0 ? 256 : 512 * V;
    auto bytes = [](int k) { return (BM + BN) * k * 2; };
    static_assert(KMAX * (BM + BN) * 2 <= 160 * 1024, "the workgroup's LDS");
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes(KMAX)) != hipSuccess) return GR4AD_EHIP;
        attr_done = true;
    }
    const int64_t tiles_m = ceil_div64(M, BM), tiles_n = (N + BN - 1) / BN, total = tiles_m * tiles_n;
    const PanelOut out = {epi.C, epi.ldc, epi.bias, epi.resid, epi.table, epi.tok, epi.ldr};
    {
        ProfScope ps(KC_GEMM_TILE, st, 2.0 * (double)M * N * K, gemm_bytes(M, N, K, kind_f32(KIND), KIND == EPI_F32_RESID) + 2.0 * M * K);
        hipLaunchKernelGGL(kern, dim3((unsigned)(ceil_div64(total, 8) * 8)), dim3(512), bytes(K), st, rows, W, ldw, (int)M, N, K, (int)tiles_m, (int)tiles_n, out);
    }
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

template <int BM, int BN, int V, int J>
static int launch_panel_cfg(int src, const PanelRows &rows, const bf16 *W, int64_t ldw, int64_t M, int N, int K, int kind, const GemmEpilogue &epi, hipStream_t st) {
#define KIND_(s, k) if (src == s && kind == k) return launch_panel_kind<BM, BN, V, J, s, k>(rows, W, ldw, M, N, K, epi, st)
    KIND_(ROWS_NORM, EPI_STORE);
    KIND_(ROWS_NORM, EPI_SILU_DIV);
    KIND_(ROWS_NORM, EPI_F32);
    KIND_(ROWS_GATED, EPI_F32_TABLE);
    if constexpr (J * (V == 2 ? 2 : 1) <= 2) KIND_(ROWS_TRUNK, EPI_F32_RESID);  // (two pieces of a row to a lane: see launch_gemm_trunk_attended)
#undef KIND_
    return GR4AD_EUNSUPPORTED;
}

// Where the lines lie (us, norm kernel and product / this kernel, calls in a row on weights in turn): K = 256: 64 x 1024 5.4 / 4.2, 512 x 768 5.5 / 4.0 (32x64 tiles, 4.7 on
// 32x32), 1024 x 1024 6.3 / 5.5 (64x64 tiles, 6.0 on 32x64), 4096 x 256 6.8 / 4.9, 2048 x 1024 7.6 / 7.5 (512 tiles), 4096 x 768 9.1 / 9.9.  K = 512: 64 x 512 5.7 / 4.7,
// 256 x 2048 6.6 / 6.0 (32x64 tiles, 7.4 on 32x32), 192 x 4096 6.9 / 9.6 (384 tiles), 512 x 1536 on 64x64 tiles 7.0 / 7.3.  K = 1024: 8 x 1024 6.7 / 5.4, but 32 x 1024 6.7 / 6.9:
// every column of tiles forms the rows anew, 0.85 us of vector arithmetic and 128 KB of x for 32 of them.  Decodes of one request, d = 512, 619 -> 585 us; of 64, d = 256, 577 -> 548; gates and
// the trunk's attention as well 551 -> 544 and 524 -> 515.
enum { PANEL_NONE = 0, PANEL_32, PANEL_32X64, PANEL_64, PANEL_FEW };  // few: at most 16 rows of 32x32 tiles
static int panel_shape(int64_t M, int N, int K) {
    if (K > 1024) return PANEL_NONE;
    auto tiles = [&](int bm, int bn) { return ceil_div64(M, bm) * ((N + bn - 1) / bn); };
    if (M <= 16) return tiles(32, 32) <= 256 ? PANEL_FEW : PANEL_NONE;
    if (K > 512) return PANEL_NONE;
    if (tiles(32, 32) <= (K <= 256 ? 256 : 192)) return PANEL_32;
    if (tiles(32, 64) <= 256) return PANEL_32X64;
    return K <= 256 && tiles(64, 64) <= 384 ? PANEL_64 : PANEL_NONE;
}

static int launch_panel(int shape, int src, const PanelRows &rows, const bf16 *W, int64_t ldw, int64_t M, int N, int K, int kind, const GemmEpilogue &epi, hipStream_t st) {
#define PANEL_(bm, bn, v, j) return launch_panel_cfg<bm, bn, v, j>(src, rows, W, ldw, M, N, K, kind, epi, st)
    if (shape == PANEL_FEW) {
        if (K <= 256) PANEL_(32, 32, 0, 1);
        if (M <= 8) {
            if (K <= 512) PANEL_(32, 32, 1, 1);
            PANEL_(32, 32, 2, 1);
        }
        if (K <= 512) PANEL_(32, 32, 1, 2);
        PANEL_(32, 32, 2, 2);
    }
    if (shape == PANEL_32) {
        if (K <= 256) PANEL_(32, 32, 0, 2);
        PANEL_(32, 32, 1, 4);
    }
    if (shape == PANEL_32X64) {
        if (K <= 256) PANEL_(32, 64, 0, 2);
        PANEL_(32, 64, 1, 4);
    }
    PANEL_(64, 64, 0, 4);
#undef PANEL_
}

// Batched product on the tile kernels: for i < batch, C_i[M,N] = A_i[M,K] * W_i[N,K]^T with A_i = A + i*batch_a elements etc.
// bf16 operands; C bf16 or (out_f32) float.  Used by the lazy layers' cross-attention in absorbed form (many small products).
// batch_len (may be NULL), len_bounds: 1 = batch i only needs columns n < batch_len[i] of C_i (the rest may stay unwritten),
// 2 = A_i and W_i are zero from column batch_len[i] (rounded up to 64) on, so the K loop stops there.
int launch_gemm_batched(const void *A, int64_t lda, int64_t batch_a, const void *W, int64_t ldw, int64_t batch_w, void *C, int64_t ldc,
                        int64_t batch_c, int out_f32, int64_t M, int N, int K, int batch, const int32_t *batch_len, int len_bounds,
                        hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0 || K % 64 || lda % 8 || ldw % 8 || batch_a % 8 || batch_w % 8 || ((uintptr_t)A % 16) || ((uintptr_t)W % 16))
        return GR4AD_EUNSUPPORTED;
    GemmEpilogue e;
    memset(&e, 0, sizeof(e));
    e.C = C;
    e.ldc = ldc;
    e.out_f32 = out_f32;
    e.batch_len = batch_len;
    e.len_bounds = batch_len ? len_bounds : 0;
    const bf16 *a = (const bf16 *)A, *w = (const bf16 *)W;
    const int kind = out_f32 ? EPI_F32 : EPI_STORE;
    return launch_tile(pick_kernel(M, N, K, kind, batch, true, true, false), a, lda, w, ldw, M, N, K, kind, e, st, batch, batch_a, batch_w, batch_c);
}

// Transposed-per-request product for the context values: out[(b*N + n) * ld_out + s] = sum_k A[b*S + s][k] * W[n][k] for
// s < len_b, 0 for len_b <= s < ld_out (ld_out = S rounded up to 64).  The kernels see requests of ld_out rows, so that no 64 rows straddle two
// requests and the transposed lines are written in whole aligned pieces at every S (32 requests of 500 rows, N = K = 1024: 64 us on 128x128 tiles
// that scattered single values, now 30 as a third of 3072 columns).  false = shape not covered.
bool gemm_vt_supported(gr4ad_dtype dtype, const void *A, int64_t lda, const void *W, int64_t ldw, int64_t M, int N, int K, int S,
                       const void *out, int64_t ld_out) {
    if (dtype != GR4AD_BF16 || K % 64 || S < 1 || M % S || lda % 8 || ldw % 8 || ((uintptr_t)A % 16) || ((uintptr_t)W % 16) || ((uintptr_t)out % 16)) return false;
    return ld_out == (S + 63) / 64 * 64 && M / S * ld_out <= 0x7fffff00LL;
}
int launch_gemm_vt(const void *A, int64_t lda, const void *W, int64_t ldw, int64_t M, int N, int K, int S, const int32_t *ctx_len, void *out,
                   int64_t ld_out, hipStream_t st) {
    if (!gemm_vt_supported(GR4AD_BF16, A, lda, W, ldw, M, N, K, S, out, ld_out)) return GR4AD_EUNSUPPORTED;
    GemmEpilogue e;
    memset(&e, 0, sizeof(e));
    e.C = out;
    e.ldc = ld_out;
    e.ctx_len = ctx_len;
    e.vt_S = (int)ld_out;
    e.vt_rows = S;
    e.skip_len = ctx_len;  // key tiles beyond ceil(len / 64) * 64 are never read by the attention kernel
    e.skip_S = (int)ld_out;
    const int64_t rows = M / S * ld_out;
    const bool ring = K >= 192 && rows >= 256 && N >= 256 && lda < (1 << 22) && ldw < (1 << 22);
    const int run = pick_kernel(rows, N, K, EPI_VT, 1, true, true, ring);
    if (run == RUN_RING) return launch_ring((const bf16 *)A, lda, (const bf16 *)W, ldw, rows, N, K, EPI_VT, e, st);
    return launch_tile(run, (const bf16 *)A, lda, (const bf16 *)W, ldw, rows, N, K, EPI_VT, e, st);
}

// ---------------------------------------------------------------------------
// FP8 products: C = (a_scale[row] * w_scale) * Aq Wq^T with the same epilogues (Aq, Wq: E4M3 bytes; C bf16 or float32)
// ---------------------------------------------------------------------------
static bool ring_f8_ok(int kind, int64_t M, int N, int K, int64_t lda, int64_t ldw, const void *A, const void *W, const GemmEpilogue &e) {
    if (kind < 0 || kind == EPI_VT || e.norm_out || e.row_inv) return false;
    // (there is no mid-size FP8 kernel: a few 256-row tiles on the persistent kernel still beat the plain kernel by far)
    if (M < 64 || N < 256 || K % 128 || K < 384 || lda % 16 || ldw % 16 || ((uintptr_t)A % 16) || ((uintptr_t)W % 16)) return false;
    return ring_ok(kind, N, K, lda, ldw, e);
}

bool gemm_f8_on_persistent_kernel(const void *A, int64_t lda, const void *W, int64_t ldw, int64_t M, int N, int K, const GemmEpilogue &epi) {
    return ring_f8_ok(epilogue_kind(epi), M, N, K, lda, ldw, A, W, epi);
}

int launch_gemm_f8(const void *A, int64_t lda, const float *a_scale, const void *W, int64_t ldw, float w_scale, int64_t M, int N, int K,
                   const GemmEpilogue &epi_in, hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0 || !A || !W || !a_scale || !(w_scale > 0.0f)) return GR4AD_EINVAL;
    if (epi_in.norm_out || epi_in.row_inv) return GR4AD_EUNSUPPORTED;
    if (epi_in.out_f16 && !gemm_f8_on_persistent_kernel(A, lda, W, ldw, M, N, K, epi_in)) return GR4AD_EUNSUPPORTED;
    GemmEpilogue epi = epi_in;
    epi.a_scale = a_scale;
    epi.w_scale = w_scale;
    const int kind = epilogue_kind(epi);
    if (gemm_f8_on_persistent_kernel(A, lda, W, ldw, M, N, K, epi)) {
        const bf16 *a = (const bf16 *)A, *w = (const bf16 *)W;  // (the kernel's pointer type; it addresses bytes)
        switch (kind) {
            case EPI_STORE: return launch_ring_kind<EPI_STORE, true>(a, lda, w, ldw, M, N, K, epi, st);
            case EPI_SILU: return launch_ring_kind<EPI_SILU, true>(a, lda, w, ldw, M, N, K, epi, st);
            case EPI_F32: return launch_ring_kind<EPI_F32, true>(a, lda, w, ldw, M, N, K, epi, st);
            case EPI_F32_RESID: return launch_ring_kind<EPI_F32_RESID, true>(a, lda, w, ldw, M, N, K, epi, st);
            default: return launch_ring_kind<EPI_F32_TABLE, true>(a, lda, w, ldw, M, N, K, epi, st);
        }
    }
    dim3 grid((unsigned)ceil_div64(M, 64), (unsigned)((N + 63) / 64));
    if (ceil_div64(M, 64) > 0x7fffffffLL || grid.y > 65535) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_GEMM_SIMPLE, st, 2.0 * (double)M * N * K);
    hipLaunchKernelGGL((gemm_simple<fp8e4m3, bf16>), grid, dim3(256), 0, st, (const fp8e4m3 *)A, lda, (const fp8e4m3 *)W, ldw, M, N, K, epi);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

static bool f32_mfma_ok(const void *A, int64_t lda, const void *W, int64_t ldw, int K) {
    return K % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)W % 16) == 0;
}

// bf16 products with 16-byte aligned, K-contiguous operands run on the matrix cores, everything else on the plain kernel.  Products
// of at least 8192 rows and 256 columns with aligned rows form a class of their own: they may fold the RMSNorm into their
// epilogues, leave half-precision logits and use the hardware reciprocal in SiLU.  What a product computes depends on that class alone;
// inside it (and below it) pick_kernel is free to choose.
static bool mfma_ok(gr4ad_dtype dtype, const void *A, int64_t lda, const void *W, int64_t ldw, int K, int kind) {
    return dtype == GR4AD_BF16 && kind >= 0 && K % 64 == 0 && lda % 8 == 0 && ldw % 8 == 0 && lda < (1 << 23) && ldw < (1 << 23) && ((uintptr_t)A % 16) == 0 && ((uintptr_t)W % 16) == 0;
}

bool gemm_large_class(gr4ad_dtype dtype, const void *A, int64_t lda, const void *W, int64_t ldw, int64_t M, int N, int K,
                               const GemmEpilogue &epi) {
    const int kind = epilogue_kind(epi);
    if (M <= 0 || N <= 0 || K <= 0 || !mfma_ok(dtype, A, lda, W, ldw, K, kind)) return false;
    if (epi.skip_len && M > 0x7fffff00LL) return false;  // (the tile test works on 32-bit row numbers)
    return M >= 8192 && N >= 256 && ring_ok(kind, N, K, lda, ldw, epi);
}

int launch_gemm(gr4ad_dtype dtype, const void *A, int64_t lda, const void *W, int64_t ldw, int64_t M, int N, int K,
                const GemmEpilogue &epi, hipStream_t st) {
    if (M <= 0 || N <= 0 || K <= 0) return GR4AD_EINVAL;
    const int kind = epilogue_kind(epi);
    // only products of the large class fold the RMSNorm or write half-precision logits: never drop such a request silently
    if ((epi.norm_out || epi.row_inv || epi.out_f16) && !gemm_large_class(dtype, A, lda, W, ldw, M, N, K, epi)) return GR4AD_EUNSUPPORTED;
    if (epi.pre_x) {
        if (lda != K || !epi.pre_gain) return GR4AD_EINVAL;
        if (dtype == GR4AD_F32 && !f32_big_tiles(M, N) && f32_mfma_ok(epi.pre_x, lda, W, ldw, K) && ((uintptr_t)epi.pre_gain % 16) == 0)
            return launch_f32(epi.pre_x, lda, (const float *)W, ldw, M, N, K, epi, st);
        const int kd = kind == EPI_SILU ? EPI_SILU_DIV : kind;
        if (M < 8192 && !epi.skip_len && (kd == EPI_STORE || kd == EPI_SILU_DIV || kd == EPI_F32) && mfma_ok(dtype, A, lda, W, ldw, K, kind) && ((uintptr_t)epi.pre_x % 16) == 0 &&
            ((uintptr_t)epi.pre_gain % 16) == 0) {  // (the epilogues that launch_panel_cfg has behind a norm)
            const int shape = panel_shape(M, N, K);
            PanelRows rows = {};
            rows.x = epi.pre_x;
            rows.gain = (const bf16 *)epi.pre_gain;
            rows.eps = epi.pre_eps;
            if (shape != PANEL_NONE) return launch_panel(shape, ROWS_NORM, rows, (const bf16 *)W, ldw, M, N, K, kd, epi, st);
        }
        const int s = launch_rmsnorm(dtype, epi.pre_x, epi.pre_gain, (void *)A, M, K, epi.pre_eps, st, epi.skip_len && !epi.skip_S ? epi.skip_len : nullptr);
        if (s) return s;
        GemmEpilogue plain = epi;
        plain.pre_x = nullptr;
        return launch_gemm(dtype, A, lda, W, ldw, M, N, K, plain, st);
    }
    if (mfma_ok(dtype, A, lda, W, ldw, K, kind)) {
        const bf16 *a = (const bf16 *)A, *w = (const bf16 *)W;
        if (gemm_large_class(dtype, A, lda, W, ldw, M, N, K, epi)) {
            const int run = pick_kernel(M, N, K, kind, 1, false, tile_staged_ok(kind, N, epi), true);
            return run == RUN_RING ? launch_ring(a, lda, w, ldw, M, N, K, kind, epi, st) : launch_tile(run, a, lda, w, ldw, M, N, K, kind, epi, st);
        }
        const int k = kind == EPI_SILU ? EPI_SILU_DIV : kind;
        const int run = pick_kernel(M, N, K, k, 1, true, true, N >= 256 && ring_ok(k, N, K, lda, ldw, epi));
        return run == RUN_RING ? launch_ring(a, lda, w, ldw, M, N, K, k, epi, st) : launch_tile(run, a, lda, w, ldw, M, N, K, k, epi, st);
    }
    if (dtype == GR4AD_F32 && f32_mfma_ok(A, lda, W, ldw, K))
        return launch_f32((const float *)A, lda, (const float *)W, ldw, M, N, K, epi, st);
    dim3 grid((unsigned)ceil_div64(M, 64), (unsigned)((N + 63) / 64));
    if (ceil_div64(M, 64) > 0x7fffffffLL || grid.y > 65535) return GR4AD_EUNSUPPORTED;
    ProfScope ps(KC_GEMM_SIMPLE, st, 2.0 * (double)M * N * K);
    if (dtype == GR4AD_BF16)
        hipLaunchKernelGGL(gemm_simple<bf16>, grid, dim3(256), 0, st, (const bf16 *)A, lda, (const bf16 *)W, ldw, M, N, K, epi);
    else
        hipLaunchKernelGGL(gemm_simple<float>, grid, dim3(256), 0, st, (const float *)A, lda, (const float *)W, ldw, M, N, K, epi);
    GR4AD_LAUNCH_CHECK();
    return GR4AD_OK;
}

// A = the gated rows of Fuse (launch_fuse_gate), formed by the product where it has few tiles, else by a launch of their own into `gated`
int launch_gemm_gated(gr4ad_dtype dtype, const float *m, int64_t m_req_stride, const float *G, int64_t table_rows, const int32_t *tok, void *gated, int B, int n, const void *W, int N,
                      int d, const GemmEpilogue &epi, hipStream_t st) {
    const int64_t M = (int64_t)B * n;
    const int kind = epilogue_kind(epi);
    if (M < 8192 && kind == EPI_F32_TABLE && !epi.skip_len && !epi.norm_out && mfma_ok(dtype, gated, d, W, d, d, kind) && ((uintptr_t)m % 16) == 0 && m_req_stride % 4 == 0 && ((uintptr_t)G % 16) == 0) {
        const int shape = panel_shape(M, N, d);
        if (shape != PANEL_NONE) {
            PanelRows rows = {};
            rows.x = m;
            rows.x_req = m_req_stride;
            rows.table = G;
            rows.tok = tok;
            rows.n = n;
            return launch_panel(shape, ROWS_GATED, rows, (const bf16 *)W, d, M, N, d, kind, epi, st);
        }
    }
    const int s = launch_fuse_gate(dtype, m, m_req_stride, G, table_rows, tok, gated, B, n, d, st);
    return s ? s : launch_gemm(dtype, gated, d, W, d, M, N, d, epi, st);
}

// A = the trunk's self-attention over qkv [B*T, 3d] (launch_trunk_self_attention), formed by the product where it has few rows, else by a launch of its own into `o`
int launch_gemm_trunk_attended(gr4ad_dtype dtype, const void *qkv, void *o, int B, int T, int H, const void *W, int N, int d, const GemmEpilogue &epi, hipStream_t st) {
    const int64_t M = (int64_t)B * T;
    const int kind = epilogue_kind(epi), dh = d / H;
    // (up to four positions and head widths 16, 32 and 64; a wavefront holds nine pieces of a row in registers, so two rows of at most 512 columns or one of 1024)
    if (M < 8192 && kind == EPI_F32_RESID && T <= 4 && (dh == 16 || dh == 32 || dh == 64) && !epi.norm_out && mfma_ok(dtype, o, d, W, d, d, kind) && ((uintptr_t)qkv % 16) == 0) {
        const int shape = panel_shape(M, N, d);
        if ((shape == PANEL_FEW && (M <= 8 || d <= 512)) || (d <= 256 && (shape == PANEL_32 || shape == PANEL_32X64))) {
            PanelRows rows = {};
            rows.qkv = (const bf16 *)qkv;
            rows.n = T;
            rows.lanes_per_head = dh / 8;
            return launch_panel(shape, ROWS_TRUNK, rows, (const bf16 *)W, d, M, N, d, kind, epi, st);
        }
    }
    const int s = launch_trunk_self_attention(dtype, qkv, o, B, T, d, H, st);
    return s ? s : launch_gemm(dtype, o, d, W, d, M, N, d, epi, st);
}
