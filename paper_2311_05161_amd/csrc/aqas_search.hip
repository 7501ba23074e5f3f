// AQAS scale search (Sec. 3.2, Eq. 1: the scale vector s minimizes the squared error of the quantized
// layer's output against the unquantized product on calibration activations; App. A.4: maximum
// magnitude per input channel as the representative of activations and weights, a grid search, then
// weight clipping).  One candidate at a time, the inner loop is the layer itself: the layer's activation and weight
// quantizers, packing and w4a8_gemm; several at a time, the same definitions in kernels with a candidate index (below and in
// weight_quant.hip, gemm_i8.hip, gemm_prefill.hip), whose fp32 sums may run in another order.  The kernels below supply the
// representatives, the scale family, the unquantized product and the error sums.  Everything stays on
// the stream: the best grid point is picked on the device and the final scale is computed from it there.
//
// Scale family: s_k(j) = ax_k^(j/16) / aw_k^(1 - j/16), j = 0..16.  A sixteenth power is a chain of
// correctly rounded square roots, so the whole family is a fixed sequence of IEEE binary32 operations
// (this file is compiled without mul+add contraction).
#include "w4a8_common.hpp"

namespace w4a8 {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int AQ_GRID = 16;
constexpr int AQ_CLIP_STEPS = 11;

// ---- representatives: out[k] = max_r |A[r,k]| (out zeroed beforehand; non-negative floats order
// like their bit patterns, so an integer atomic max is exact and order-independent) ----------------
template <typename T>
__global__ __launch_bounds__(256) void channel_absmax_kernel(const T *__restrict__ A, int64_t R,
                                                             int64_t K, int64_t lda, int rows_per_block,
                                                             float *__restrict__ out)
{
    __shared__ float part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * 64 + lane;
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_block;
    const int64_t r1 = min(R, r0 + rows_per_block);
    float m = 0.0f;
    if (k < K) {
        // eight loads in flight (rows past the end repeat the last one)
        for (int64_t r = r0 + wave; r < r1; r += 32) {
            T a[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) a[i] = A[min(r + 4 * i, r1 - 1) * lda + k];
#pragma unroll
            for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(to_f32(a[i])));
        }
    }
    part[wave][lane] = m;
    __syncthreads();
    if (wave == 0 && k < K) {
        m = fmaxf(fmaxf(part[0][lane], part[1][lane]), fmaxf(part[2][lane], part[3][lane]));
        atomicMax(reinterpret_cast<unsigned int *>(out) + k, __float_as_uint(m));
    }
}

__global__ __launch_bounds__(256) void fill_f32_kernel(float *p, int64_t n, float v)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

int launch_channel_absmax(const void *A, int dtype, int64_t R, int64_t K, int64_t lda, float *out,
                          hipStream_t st)
{
    hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, out, K, 0.0f);
    if (R == 0) return hip_status(hipGetLastError());
    // Rows per block: few enough to fill the chip, many enough that a channel's atomics do not queue up (one row at a
    // time and always 256 of them: 512 x 4096 28 us, 4096 x 4096 21 us).
    const int64_t blocks128 = (K + 63) / 64 * ((R + 127) / 128);
    const int rpb = blocks128 < 512 ? 32 : R > 65535 * 128LL ? 256 : 128;
    const dim3 grid((unsigned)((K + 63) / 64), (unsigned)((R + rpb - 1) / rpb));
    switch (dtype) {
        case W4A8_F32:
            hipLaunchKernelGGL((channel_absmax_kernel<float>), grid, dim3(256), 0, st, (const float *)A, R, K, lda, rpb, out);
            break;
        case W4A8_F16:
            hipLaunchKernelGGL((channel_absmax_kernel<__half>), grid, dim3(256), 0, st, (const __half *)A, R, K, lda, rpb, out);
            break;
        case W4A8_BF16:
            hipLaunchKernelGGL((channel_absmax_kernel<bf16_t>), grid, dim3(256), 0, st, (const bf16_t *)A, R, K, lda, rpb, out);
            break;
        default: return W4A8_ERR_DTYPE;
    }
    return hip_status(hipGetLastError());
}

// ---- scale family -------------------------------------------------------------------------------
__device__ __forceinline__ float pow_sixteenths(float x, int j)
{
    if (j == AQ_GRID) return x;
    float out = 1.0f, r = x;
#pragma unroll
    for (int bit = 3; bit >= 0; --bit) {   // x^(1/2), x^(1/4), x^(1/8), x^(1/16)
        r = sqrtf(r);   // correctly rounded (hipcc default for binary32 sqrt and division)
        if ((j >> bit) & 1) out = out * r;
    }
    return out;
}

__device__ __forceinline__ float scale_at(float x, float w, int j)
{
    if (x == 0.0f || w == 0.0f) return 1.0f;
    const float v = pow_sixteenths(x, j) / pow_sixteenths(w, AQ_GRID - j);
    return fminf(fmaxf(v, 1e-4f), 1e4f);
}

__global__ __launch_bounds__(256) void aqas_scale_kernel(const float *__restrict__ ax,
                                                         const float *__restrict__ aw, int64_t K, int j,
                                                         float *__restrict__ s)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < K) s[k] = scale_at(ax[k], aw[k], j);
}

int launch_aqas_scale(const float *ax, const float *aw, int64_t K, int j, float *s, hipStream_t st)
{
    hipLaunchKernelGGL(aqas_scale_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, ax, aw, K, j, s);
    return hip_status(hipGetLastError());
}

// ---- the unquantized product Yref[m,n] = sum_k X[m,k] W[n,k] in fp32 on the matrix cores ----------
// 16-bit inputs, rows 16-byte aligned and K % 128 == 0: products of 16-bit numbers are exact in fp32, so the 16-bit matrix
// instructions (32 x 32 x 16) lose nothing against widened operands.  A block makes a 64 x 128 tile with RG_PHASES x 4 waves:
// wave (p, w) the columns 32 w .. + 31 of all 64 rows over every RG_PHASES-th step of 64 columns of K.  A round of RG_PHASES
// steps lies in one of RG_RING LDS buffers (rows of 128 bytes in 16-byte chunks, chunk index XORed with half the row so that
// the reads of 16 rows at one chunk cover all banks -- on the global side, as a copy lands in lane order), filled by direct
// copies RG_RING - 1 rounds ahead; the phases' sums meet in LDS at the end, in their order.
// At 512 x 4096 x 4096 the grid is one block per CU, and what bounds it is the way of the tiles through the CU's memory pipe
// (48 KB per round: 768 clocks).  us there: one wave per 32 x 32 tile straight from global memory 127; four waves, through
// registers to LDS, 39.5; two phases and copies straight to LDS 28.9 (medians of a trace of searches one candidate at a time; side by side,
// where the weights come from further away, 33) (97 x 3072 x 2000 26 / 19, 2048 x 4096 x 4096 106 / 103; rms error against
// 64 bits 8.1e-7 / 1.8e-7 with two shorter chains).
constexpr int RG_BM = 64, RG_BN = 128, RG_BK = 64, RG_PHASES = 2, RG_RING = 3;
constexpr int RG_THREADS = RG_PHASES * 256;
constexpr int RG_ROWS = RG_BM + RG_BN;                    // rows of X, then rows of W
constexpr int RG_STEP = RG_ROWS * RG_BK * 2;              // bytes of a step in LDS (24 KB)

// FAR: rows too far apart for the 32-bit offsets of a buffer descriptor (eight of its rows below 2^31 bytes): the same copies
// by 64-bit addresses.  (64 x 4096 x 128, rows 2^26 + 8 elements apart: clipping choice 95 us; with the kernel below 1760.)
template <typename T, bool FAR>
__global__ __launch_bounds__(RG_THREADS) void ref_gemm16_kernel(const T *__restrict__ X, int64_t M, int64_t K, int64_t ldx,
                                                                const T *__restrict__ W, int64_t N, int64_t ldw,
                                                                float *__restrict__ Y, uint32_t grid_n)
{
    constexpr int COPIES = RG_ROWS / 8 / 4;               // of eight rows, per wave and round (6)
    extern __shared__ __attribute__((aligned(16))) uint8_t rg_lds[];   // [RG_RING][RG_PHASES][RG_STEP]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3), phase = __builtin_amdgcn_readfirstlane(tid >> 8);
    const uint32_t bm = blockIdx.x / grid_n, bn = blockIdx.x - bm * grid_n;
    const int64_t m0 = (int64_t)bm * RG_BM, n0 = (int64_t)bn * RG_BN;
    const int r32 = lane & 31, kh = lane >> 5;
    // Copy i of a wave: rows 8 (4 i + wave) .. + 7 of its phase's step, eight lanes a row.  (Rows past the end repeat the last one;
    // they are not stored.  A descriptor starts at the first of the eight rows.)
    v4i rsrc[FAR ? 1 : COPIES];
    int voff[FAR ? 1 : COPIES];
    const T *far[FAR ? COPIES : 1];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
        const int row0 = 8 * (4 * i + wave), row = row0 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        const bool is_x = row0 < RG_BM;   // (RG_BM % 8 == 0: uniform)
        const int64_t last = is_x ? M - 1 : N - 1, at = is_x ? m0 : n0 - RG_BM, ld = is_x ? ldx : ldw;
        if constexpr (FAR) {
            far[i] = (is_x ? X : W) + min(at + row, last) * ld + c * 8;
        } else {
            const int64_t first = min(at + row0, last);
            const uint64_t base = (uint64_t)((is_x ? X : W) + first * ld);
            rsrc[i] = v4i{(int)(uint32_t)base, (int)((base >> 32) & 0xffffu), 0x7fffffff, 0x00020000};
            voff[i] = (int)((min(at + row, last) - first) * ld * 2) + c * 16;
        }
    }
    v16f acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.0f;
    const int steps = (int)(K / RG_BK), rounds = steps / RG_PHASES;   // (K is a multiple of the columns of a round)
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)rg_lds;
    auto copy_round = [&](int round, int slot) {
        const int step = min(round * RG_PHASES + phase, steps - 1);   // (past the end: the last step, unused)
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            const int at = (slot * RG_PHASES + phase) * RG_STEP + (4 * i + wave) * 1024;
            if constexpr (FAR)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(uintptr_t)(far[i] + (int64_t)step * RG_BK),
                                                 (__attribute__((address_space(3))) void *)(rg_lds + at), 16, 0, 0);
            else
                dma_b128(rsrc[i], voff[i], step * (RG_BK * 2), lds_base + (uint32_t)at);
        }
    };
#pragma unroll
    for (int i = 0; i < RG_RING - 1; ++i) copy_round(i, i);
    int slot = 0;
    for (int round = 0; round < rounds; ++round) {
        // this round's copies have landed, the next ones' are on their way; behind the barrier everyone's have, and the slot
        // of the round before is free
        static_assert(RG_RING == 3 && COPIES == 6, "the wait counts the copies of one round");
        asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        __syncthreads();
        copy_round(round + RG_RING - 1, slot == 0 ? RG_RING - 1 : slot - 1);
        const v4u *t = reinterpret_cast<const v4u *>(rg_lds + (slot * RG_PHASES + phase) * RG_STEP);
#pragma unroll
        for (int q = 0; q < RG_BK / 16; ++q) {   // lane (r32, kh) holds 8 consecutive k of its row, as both operands agree on
            const int c = (2 * q + kh) ^ ((r32 >> 1) & 7);
            const v4u wv = t[(RG_BM + wave * 32 + r32) * 8 + c];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const v4u xv = t[(h * 32 + r32) * 8 + c];
                if constexpr (__is_same(T, bf16_t))
                    acc[h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, xv),
                                                                     __builtin_bit_cast(v8bf, wv), acc[h], 0, 0, 0);
                else
                    acc[h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, xv),
                                                                    __builtin_bit_cast(v8h, wv), acc[h], 0, 0, 0);
            }
        }
        slot = slot + 1 == RG_RING ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (copies past the end: the buffers are used again below)
    // the phases' sums: phase 1 .. hand theirs over, phase 0 adds them in order and stores
    __syncthreads();
    v4f *red = reinterpret_cast<v4f *>(rg_lds);   // [phase - 1][wave][half][quarter][lane]
    auto at = [&](int p, int h, int i) { return (((p - 1) * 4 + wave) * 8 + h * 4 + i) * 64 + lane; };
    if (phase > 0) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                red[at(phase, h, i)] = v4f{acc[h][4 * i], acc[h][4 * i + 1], acc[h][4 * i + 2], acc[h][4 * i + 3]};
    }
    __syncthreads();
    if (phase > 0) return;
#pragma unroll
    for (int p = 1; p < RG_PHASES; ++p)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v4f o = red[at(p, h, i)];
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[h][4 * i + r] += o[r];
            }
    // D[i][j], A = tokens, B = channels: lane holds channel n0 + 32 wave + r32, tokens 8 (r / 4) + 4 kh + r % 4
    const int64_t n = n0 + wave * 32 + r32;
    if (n < N) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = m0 + 32 * h + 8 * (r >> 2) + 4 * kh + (r & 3);
                if (m < M) Y[m * N + n] = acc[h][r];
            }
    }
}

// Binary32, and bfloat16 off the 16-byte alignment (fp16 rows have to have it): one wave per 32 x 32 output tile, operands
// straight from global memory, widened exactly, v_mfma_f32_32x32x2_f32.
template <typename T>
__global__ __launch_bounds__(256) void ref_gemm_kernel(const T *__restrict__ X, int64_t M, int64_t K,
                                                       int64_t ldx, const T *__restrict__ W, int64_t N,
                                                       int64_t ldw, float *__restrict__ Y)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t m0 = ((int64_t)blockIdx.y * 2 + (wave >> 1)) * 32;
    const int64_t n0 = ((int64_t)blockIdx.x * 2 + (wave & 1)) * 32;
    if (m0 >= M || n0 >= N) return;   // whole wave
    const int r32 = lane & 31, kh = lane >> 5;
    const T *xr = X + min(m0 + r32, M - 1) * ldx;   // rows past the end recompute the last row (not stored)
    const T *wr = W + min(n0 + r32, N - 1) * ldw;
    v16f acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (int64_t k = 0; k < K; k += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(to_f32(xr[k + kh]), to_f32(wr[k + kh]), acc, 0, 0, 0);
    // D[i][j] = sum_k A[i][k] B[k][j], A = tokens, B = channels: lane holds channel n0 + r32 and the
    // tokens m0 + 8 (r / 4) + 4 kh + r % 4
    const int64_t n = n0 + r32;
    if (n < N) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t m = m0 + 8 * (r >> 2) + 4 * kh + (r & 3);
            if (m < M) Y[m * N + n] = acc[r];
        }
    }
}

int launch_ref_gemm(const void *X, const void *W, int dtype, int64_t M, int64_t N, int64_t K,
                    int64_t ldx, int64_t ldw, float *Y, hipStream_t st)
{
    const int64_t gn16 = (N + RG_BN - 1) / RG_BN, blocks16 = (M + RG_BM - 1) / RG_BM * gn16;
    if (dtype != W4A8_F32 && K % (RG_BK * RG_PHASES) == 0 && (uintptr_t)X % 16 == 0 && (uintptr_t)W % 16 == 0 && ldx % 8 == 0 &&
        ldw % 8 == 0 && blocks16 <= 0x7fffffffLL) {
        const bool far = ldx > (1 << 26) || ldw > (1 << 26);
        const dim3 grid16((unsigned)blocks16);
        constexpr int lds_bytes = RG_RING * RG_PHASES * RG_STEP;   // 144 KB
#define W4A8_RG(T_, FAR_)                                                                                                   \
    do {                                                                                                                    \
        static std::atomic<uint64_t> lds_opted{0};                                                                          \
        if (opt_in_dynamic_lds((const void *)ref_gemm16_kernel<T_, FAR_>, lds_bytes, lds_opted) != W4A8_OK)                 \
            return W4A8_ERR_HIP;                                                                                            \
        hipLaunchKernelGGL((ref_gemm16_kernel<T_, FAR_>), grid16, dim3(RG_THREADS), lds_bytes, st, (const T_ *)X, M, K, ldx, \
                           (const T_ *)W, N, ldw, Y, (uint32_t)gn16);                                                       \
    } while (0)
        if (dtype == W4A8_F16) {
            if (far) W4A8_RG(__half, true);
            else W4A8_RG(__half, false);
        } else {
            if (far) W4A8_RG(bf16_t, true);
            else W4A8_RG(bf16_t, false);
        }
#undef W4A8_RG
        return hip_status(hipGetLastError());
    }
    const dim3 grid((unsigned)((N + 63) / 64), (unsigned)((M + 63) / 64));
    switch (dtype) {
        case W4A8_F16: return W4A8_ERR_SHAPE;   // (all that the callers accept went above)
        case W4A8_BF16:
            hipLaunchKernelGGL((ref_gemm_kernel<bf16_t>), grid, dim3(256), 0, st, (const bf16_t *)X, M, K, ldx,
                               (const bf16_t *)W, N, ldw, Y);
            break;
        case W4A8_F32:
            hipLaunchKernelGGL((ref_gemm_kernel<float>), grid, dim3(256), 0, st, (const float *)X, M, K, ldx,
                               (const float *)W, N, ldw, Y);
            break;
        default: return W4A8_ERR_DTYPE;
    }
    return hip_status(hipGetLastError());
}

// ---- error sums ---------------------------------------------------------------------------------
// err[n] = sum_m (Y[m,n] - Yref[m,n])^2; the difference in binary32, squares and sums in binary64, in a
// fixed order (deterministic).  Bound by the read of Y and Yref (6 bytes per output, mostly from the
// caches: both were just written).  A block of 1024 threads takes 16 channels of all tokens: a thread four
// channels of every 256th token (one 8-byte and one 16-byte load), then the 16 lanes of a wave with the
// same channels and the 16 waves meet.  (One lane per channel over all tokens left all but N / 256 CUs
// idle and waited for every load in turn: 512 x 4096: 139 us, now 7.2 us.)
// The clipping search's bookkeeping rides along: candidate i replaces a channel's incumbent only if strictly
// better (so ties keep the larger range); err_table (may be null) keeps every candidate's errors.
struct ClipState {
    int i;
    double *best_err;      // null: the search of the scale, which wants err itself
    int32_t *best_idx;
    double *err_table;
};

constexpr int SQ_THREADS = 1024;
constexpr int SQ_CHANNELS = 16;

__global__ __launch_bounds__(SQ_THREADS) void output_sq_error_kernel(const uint16_t *__restrict__ Y, int y_dtype,
                                                                     const float *__restrict__ Yref, int64_t M,
                                                                     int64_t N, double *__restrict__ err,
                                                                     ClipState clip)
{
    __shared__ double part[SQ_THREADS / WAVE][SQ_CHANNELS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = (int64_t)blockIdx.x * SQ_CHANNELS + (tid & 3) * 4;   // N % 16 == 0
    Y += blockIdx.y * M * N;   // (several candidates' outputs against one reference)
    err += blockIdx.y * N;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t m = tid >> 2; m < M; m += SQ_THREADS / 4) {
        const ushort4 b = *reinterpret_cast<const ushort4 *>(Y + m * N + n);
        const float4 r = *reinterpret_cast<const float4 *>(Yref + m * N + n);
        const uint16_t bits[4] = {b.x, b.y, b.z, b.w};
        const float ref[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float y = (y_dtype == W4A8_F16) ? __half2float(__ushort_as_half(bits[c]))
                                                  : __uint_as_float((uint32_t)bits[c] << 16);
            const float d = y - ref[c];
            sum[c] += (double)d * (double)d;
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int off = 4; off <= 32; off <<= 1) sum[c] += __shfl_xor(sum[c], off, WAVE);
    if (lane < 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) part[wave][lane * 4 + c] = sum[c];
    }
    __syncthreads();
    if (tid < SQ_CHANNELS) {
        double e = 0.0;
#pragma unroll
        for (int w = 0; w < SQ_THREADS / WAVE; ++w) e += part[w][tid];
        const int64_t ch = (int64_t)blockIdx.x * SQ_CHANNELS + tid;
        if (clip.best_err == nullptr) {
            err[ch] = e;
        } else {
            if (clip.err_table != nullptr) clip.err_table[(int64_t)clip.i * N + ch] = e;
            if (clip.i == 0 || e < clip.best_err[ch]) {
                clip.best_err[ch] = e;
                clip.best_idx[ch] = clip.i;
            }
        }
    }
}

// sum_n err[n] in every thread's return value: 256 partial sums and one fixed tree, whatever the size of the
// workgroup (256 or more threads, part: 256 doubles).  All losses are compared with each other, so all go
// through this one order: equal errors give equal losses, and the first grid point wins a tie.
constexpr int LOSS_LANES = 256;
__device__ __forceinline__ double loss_sum(const double *__restrict__ err, int64_t N, double *part)
{
    const int tid = (int)threadIdx.x;
    if (tid < LOSS_LANES) {
        double s = 0.0;
        for (int64_t n = tid; n < N; n += LOSS_LANES) s += err[n];
        part[tid] = s;
    }
    __syncthreads();
    for (int w = LOSS_LANES / 2; w >= 1; w >>= 1) {
        if (tid < w) part[tid] += part[tid + w];
        __syncthreads();
    }
    return part[0];
}

// Between two grid points: losses[j - 1] from the errors of the point just evaluated (the last block;
// j = 0: nothing to sum) and the scale of point j.  Neither depends on the other; two launches cost twice
// the launch time, which is all either takes.
__global__ __launch_bounds__(256) void aqas_next_point_kernel(const float *__restrict__ ax,
                                                              const float *__restrict__ aw, int64_t K, int j,
                                                              float *__restrict__ s,
                                                              const double *__restrict__ err, int64_t N,
                                                              double *__restrict__ losses)
{
    __shared__ double part[LOSS_LANES];
    if (blockIdx.x + 1 == gridDim.x) {
        if (j == 0) return;
        const double sum = loss_sum(err, N, part);
        if (threadIdx.x == 0) losses[j - 1] = sum;
        return;
    }
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < K) s[k] = scale_at(ax[k], aw[k], j);
}

// After the last grid point: its loss, the first minimum of all of them, the scale there.  With err one block; without it
// (all losses are there) every block looks for the minimum and takes its share of the scales (one block of 1024 threads
// for 4096 channels: 8.0 us, sixteen of 256 4.9).
__global__ __launch_bounds__(1024) void aqas_finish_kernel(const float *__restrict__ ax,
                                                           const float *__restrict__ aw, int64_t K,
                                                           float *__restrict__ s,
                                                           const double *__restrict__ err, int64_t N,
                                                           double *__restrict__ losses, int32_t *__restrict__ best)
{
    __shared__ double part[LOSS_LANES];
    __shared__ int s_best;
    // (err null: all losses are there)
    const double last = err != nullptr ? loss_sum(err, N, part) : losses[AQ_GRID];
    if (threadIdx.x == 0) {
        if (err != nullptr) losses[AQ_GRID] = last;
        double l[AQ_GRID + 1];   // (all on their way together)
#pragma unroll
        for (int i = 0; i <= AQ_GRID; ++i) l[i] = i == AQ_GRID ? last : losses[i];
        int b = 0;
        double at_b = l[0];
#pragma unroll
        for (int i = 1; i <= AQ_GRID; ++i) {
            if (l[i] < at_b) {
                b = i;
                at_b = l[i];
            }
        }
        if (blockIdx.x == 0) *best = b;
        s_best = b;
    }
    __syncthreads();
    const int j = s_best;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x)
        s[k] = scale_at(ax[k], aw[k], j);
}

// Y and Yref [M, N] dense, N % 16 == 0, both 16-byte aligned.  best_err null: err[n] is written; else the
// clipping bookkeeping of candidate i.
int launch_output_sq_error(const void *Y, int y_dtype, const float *Yref, int64_t M, int64_t N, double *err,
                           int i, double *best_err, int32_t *best_idx, double *err_table, hipStream_t st)
{
    hipLaunchKernelGGL(output_sq_error_kernel, dim3((unsigned)(N / SQ_CHANNELS)), dim3(SQ_THREADS), 0, st,
                       (const uint16_t *)Y, y_dtype, Yref, M, N, err, ClipState{i, best_err, best_idx, err_table});
    return hip_status(hipGetLastError());
}
int launch_aqas_next_point(const float *ax, const float *aw, int64_t K, int j, float *s, const double *err,
                           int64_t N, double *losses, hipStream_t st)
{
    hipLaunchKernelGGL(aqas_next_point_kernel, dim3((unsigned)((K + 255) / 256 + 1)), dim3(256), 0, st, ax, aw, K,
                       j, s, err, N, losses);
    return hip_status(hipGetLastError());
}
int launch_aqas_finish(const float *ax, const float *aw, int64_t K, float *s, const double *err, int64_t N,
                       double *losses, int32_t *best, hipStream_t st)
{
    hipLaunchKernelGGL(aqas_finish_kernel, dim3(1), dim3(1024), 0, st, ax, aw, K, s, err, N, losses, best);
    return hip_status(hipGetLastError());
}

// ---- several candidates per launch ----------------------------------------------------------------
// One candidate at a time, a layer of 4096 x 4096 on 512 tokens is five launches of 4 to 22 us per grid point: the product
// has one workgroup per CU, the others wait for one memory round trip after the other.  With the candidates of a
// search side by side every launch fills the chip several times over.

// s[j][k] and 1 / s[j][k] of all grid points
__global__ __launch_bounds__(256) void aqas_all_scales_kernel(const float *__restrict__ ax, const float *__restrict__ aw,
                                                              int64_t K, float *__restrict__ s, float *__restrict__ r)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    const float v = scale_at(ax[k], aw[k], blockIdx.y);
    s[blockIdx.y * K + k] = v;
    r[blockIdx.y * K + k] = 1.0f / v;
}

// Symmetric activation quantizer (the definition's operations, one binary32 rounding each, as in the layer's own kernels)
// for `count` candidates: a workgroup loads a token row once and keeps it in registers, four consecutive elements
// per thread and chunk, then takes the candidates one by one, each with its reciprocal scales from the cache.
template <typename T, int NC>
__global__ __launch_bounds__(256) void aqas_act_quant_kernel(const T *__restrict__ X, int64_t M, int K, int64_t ldx,
                                                             const float *__restrict__ r, int8_t *__restrict__ Xq,
                                                             float *__restrict__ sx, int count, int per_block)
{
    __shared__ float red[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m = blockIdx.x;
    const T *x = X + m * ldx;
    float v[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int k = (tid + 256 * c) * 4;   // K % 4 == 0
#pragma unroll
        for (int i = 0; i < 4; ++i) v[c][i] = k < K ? to_f32(x[k + i]) : 0.0f;
    }
    const int first = blockIdx.y * per_block, last = min(count, first + per_block);
    for (int j = first; j < last; ++j) {
        const float *rj = r + (int64_t)j * K;
        float t[NC][4], a = 0.0f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int k = (tid + 256 * c) * 4;
            float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k < K) q = *reinterpret_cast<const float4 *>(rj + k);
            t[c][0] = v[c][0] * q.x; t[c][1] = v[c][1] * q.y; t[c][2] = v[c][2] * q.z; t[c][3] = v[c][3] * q.w;
#pragma unroll
            for (int i = 0; i < 4; ++i) a = fmaxf(a, fabsf(t[c][i]));
        }
        a = wave_max(a);
        float *part = red[j & 1];   // (two sets: a wave a candidate ahead writes the other one)
        if (lane == 0) part[wave] = a;
        __syncthreads();
        a = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
        float inv = 127.0f / a;
        const bool zero_row = !(inv <= 3.402823466e+38f);   // a == 0, or so small that 127 / a overflows
        if (zero_row) inv = 0.0f;
        if (tid == 0) sx[(int64_t)j * M + m] = zero_row ? 1.0f : a / 127.0f;
        uint32_t *out = reinterpret_cast<uint32_t *>(Xq + ((int64_t)j * M + m) * K);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int k = (tid + 256 * c) * 4;
            uint32_t b[4];
            // rne and the conversion in one addition (|t inv| <= 127 (1 + 2^-23): the low byte is the code)
#pragma unroll
            for (int i = 0; i < 4; ++i) b[i] = __float_as_uint(t[c][i] * inv + 12582912.0f);
            if (k < K)
                out[k / 4] = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
        }
    }
}

bool aqas_act_quant_applies(int64_t K) { return K % 4 == 0 && K <= 8 * 1024; }

// losses[j] = sum of err[j][0 .. n - 1], all through one order (1024 partial sums, four loads in flight, one tree)
__global__ __launch_bounds__(1024) void aqas_losses_kernel(const double *__restrict__ err, int64_t n,
                                                           double *__restrict__ losses)
{
    __shared__ double part[1024];
    const int tid = threadIdx.x;
    const double *e = err + blockIdx.x * n;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = tid; i < n; i += 4096) {
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] += i + c * 1024 < n ? e[i + c * 1024] : 0.0;
    }
    part[tid] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (tid < w) part[tid] += part[tid + w];
        __syncthreads();
    }
    if (tid == 0) losses[blockIdx.x] = part[0];
}

// a candidate replaces a channel's incumbent only if strictly better (ties keep the larger range); the candidates'
// sums of a token tile are loaded together
__global__ __launch_bounds__(64) void clip_pick_kernel(const double *__restrict__ err, int parts, int64_t N, int i0, int count,
                                                       double *__restrict__ best_err, int32_t *__restrict__ best_idx,
                                                       double *__restrict__ err_table)
{
    const int64_t n = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (n >= N) return;
    double e[AQ_CLIP_STEPS];
#pragma unroll
    for (int c = 0; c < AQ_CLIP_STEPS; ++c) e[c] = 0.0;
    // (one thread per channel: what counts is the memory latency, so four token tiles' sums are on their way at a time;
    // 4096 channels, 4 tiles: 15.9 -> 5.3 us)
    constexpr int AHEAD = 4;
    for (int i = 0; i < parts; i += AHEAD) {
        double t[AHEAD][AQ_CLIP_STEPS];
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
#pragma unroll
            for (int c = 0; c < AQ_CLIP_STEPS; ++c)
                t[a][c] = err[((int64_t)min(c, count - 1) * parts + min(i + a, parts - 1)) * N + n];   // (past the end: not added)
#pragma unroll
        for (int a = 0; a < AHEAD; ++a)
#pragma unroll
            for (int c = 0; c < AQ_CLIP_STEPS; ++c)
                if (i + a < parts && c < count) e[c] += t[a][c];
    }
    double best = 0.0;
    int32_t idx = 0;
    if (i0 > 0) {
        best = best_err[n];
        idx = best_idx[n];
    }
#pragma unroll
    for (int c = 0; c < AQ_CLIP_STEPS; ++c) {
        if (c >= count) break;
        if (err_table != nullptr) err_table[(i0 + c) * N + n] = e[c];
        if (i0 + c == 0 || e[c] < best) {
            best = e[c];
            idx = i0 + c;
        }
    }
    best_err[n] = best;
    best_idx[n] = idx;
}

int launch_aqas_all_scales(const float *ax, const float *aw, int64_t K, float *s, float *r, hipStream_t st)
{
    hipLaunchKernelGGL(aqas_all_scales_kernel, dim3((unsigned)((K + 255) / 256), AQ_GRID + 1), dim3(256), 0, st, ax, aw,
                       K, s, r);
    return hip_status(hipGetLastError());
}

template <typename T>
static int launch_aqas_act_quant_t(const T *X, int64_t M, int64_t K, int64_t ldx, const float *r, int8_t *Xq, float *sx,
                                   int count, hipStream_t st)
{
    // (all candidates in the workgroup that has the row, unless that leaves CUs without work)
    int per_block = (int)(M * count / 1024);
    if (per_block < 1) per_block = 1;
    if (per_block > count) per_block = count;
    const dim3 grid((unsigned)M, (unsigned)((count + per_block - 1) / per_block));
#define W4A8_AAQ(NC_)                                                                                                  \
    if (K <= NC_ * 1024) {                                                                                             \
        hipLaunchKernelGGL((aqas_act_quant_kernel<T, NC_>), grid, dim3(256), 0, st, X, M, (int)K, ldx, r, Xq, sx, count, \
                           per_block);                                                                                 \
        return hip_status(hipGetLastError());                                                                          \
    }
    W4A8_AAQ(1) W4A8_AAQ(2) W4A8_AAQ(4) W4A8_AAQ(8)
#undef W4A8_AAQ
    return W4A8_ERR_SHAPE;
}

int launch_aqas_act_quant(const void *X, int dtype, int64_t M, int64_t K, int64_t ldx, const float *r, int8_t *Xq,
                          float *sx, int count, hipStream_t st)
{
    if (!aqas_act_quant_applies(K)) return W4A8_ERR_SHAPE;
    switch (dtype) {
        case W4A8_F32: return launch_aqas_act_quant_t((const float *)X, M, K, ldx, r, Xq, sx, count, st);
        case W4A8_F16: return launch_aqas_act_quant_t((const __half *)X, M, K, ldx, r, Xq, sx, count, st);
        case W4A8_BF16: return launch_aqas_act_quant_t((const bf16_t *)X, M, K, ldx, r, Xq, sx, count, st);
        default: return W4A8_ERR_DTYPE;
    }
}

int launch_aqas_finish_all(const float *ax, const float *aw, int64_t K, float *s, const double *err, int parts,
                           int64_t N, double *losses, int32_t *best, hipStream_t st)
{
    hipLaunchKernelGGL(aqas_losses_kernel, dim3(AQ_GRID + 1), dim3(1024), 0, st, err, parts * N, losses);
    hipLaunchKernelGGL(aqas_finish_kernel, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, ax, aw, K, s, (const double *)nullptr, N,
                       losses, best);
    return hip_status(hipGetLastError());
}

int launch_clip_pick(const double *err, int parts, int64_t N, int i0, int count, double *best_err, int32_t *best_idx,
                     double *err_table, hipStream_t st)
{
    hipLaunchKernelGGL(clip_pick_kernel, dim3((unsigned)((N + 63) / 64)), dim3(64), 0, st, err, parts, N, i0, count, best_err,
                       best_idx, err_table);
    return hip_status(hipGetLastError());
}

// err[v][n] of `count` candidates against one reference (M <= 64 R): as output_sq_error_kernel, but a block takes 64
// channels (whole 128-byte lines of the outputs: with 16, and as many passes over Yref as candidates, 17 x 512 x 4096
// took 65 us), keeps its share of Yref in registers and takes its candidates one after the other, the next one's
// outputs on their way meanwhile.  A wave's four sums per lane meet by halving: two doubles, then one, cross the
// lanes that hold the other channels.
constexpr int SQM_CHANNELS = 64;

template <int R>
__global__ __launch_bounds__(SQ_THREADS) void sq_error_many_kernel(const uint16_t *__restrict__ Y,
                                                                   const float *__restrict__ Yref, int64_t M, int64_t N,
                                                                   double *__restrict__ err, int count, int per_block)
{
    __shared__ double part[2][SQ_THREADS / WAVE][SQM_CHANNELS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t nb = (int64_t)blockIdx.x * SQM_CHANNELS;
    const int64_t n = min(nb + (tid & 15) * 4, N - 4);   // (N % 16 == 0; channels past the end are not stored)
    const int64_t m0 = tid >> 4;
    const int first = blockIdx.y * per_block, last = min(count, first + per_block);
    v2u b[R];
    auto load = [&](int v) {
#pragma unroll
        for (int i = 0; i < R; ++i)   // (rows past the end repeat the last one; they are not added)
            b[i] = *reinterpret_cast<const v2u *>(Y + (v * M + min(m0 + 64 * i, M - 1)) * N + n);
    };
    load(first);
    v4f ref[R];
#pragma unroll
    for (int i = 0; i < R; ++i) ref[i] = *reinterpret_cast<const v4f *>(Yref + min(m0 + 64 * i, M - 1) * N + n);
    for (int v = first; v < last; ++v) {
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint16_t bits[4] = {(uint16_t)b[i].x, (uint16_t)(b[i].x >> 16), (uint16_t)b[i].y, (uint16_t)(b[i].y >> 16)};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float d = __half2float(__ushort_as_half(bits[c])) - ref[i][c];
                if (m0 + 64 * i < M) sum[c] += (double)d * (double)d;
            }
        }
        if (v + 1 < last) load(v + 1);
        const bool up = lane & 32, up2 = lane & 16;   // lanes 16 apart hold the same channels
        double a0 = up ? sum[2] : sum[0], a1 = up ? sum[3] : sum[1];
        a0 += __shfl_xor(up ? sum[0] : sum[2], 32, WAVE);
        a1 += __shfl_xor(up ? sum[1] : sum[3], 32, WAVE);
        double a = up2 ? a1 : a0;
        a += __shfl_xor(up2 ? a0 : a1, 16, WAVE);
        part[v & 1][wave][(lane & 15) * 4 + (up ? 2 : 0) + (up2 ? 1 : 0)] = a;
        __syncthreads();
        if (tid < SQM_CHANNELS && nb + tid < N) {   // (the two sets of sums take turns: one barrier per candidate)
            double e = 0.0;
#pragma unroll
            for (int w = 0; w < SQ_THREADS / WAVE; ++w) e += part[v & 1][w][tid];
            err[v * N + nb + tid] = e;
        }
    }
}

// fp16 outputs Y [count][M][N] against Yref [M][N], N % 16 == 0, both 16-byte aligned
int launch_sq_error_many(const void *Y, const float *Yref, int64_t M, int64_t N, double *err, int count, hipStream_t st)
{
    const int64_t blocks = (N + SQM_CHANNELS - 1) / SQM_CHANNELS;
    int per_block = (int)(blocks * count / 512);   // all of a block's candidates in turn, unless that leaves CUs idle
    per_block = per_block < 1 ? 1 : per_block > count ? count : per_block;
    const dim3 grid((unsigned)blocks, (unsigned)((count + per_block - 1) / per_block));
#define W4A8_SQM(R_)                                                                                                   \
    if (M <= 64 * R_) {                                                                                                \
        hipLaunchKernelGGL((sq_error_many_kernel<R_>), grid, dim3(SQ_THREADS), 0, st, (const uint16_t *)Y, Yref, M, N, err, \
                           count, per_block);                                                                          \
        return hip_status(hipGetLastError());                                                                          \
    }
    W4A8_SQM(1) W4A8_SQM(2) W4A8_SQM(4) W4A8_SQM(8)
#undef W4A8_SQM
    // (longer columns than a block's registers hold)
    hipLaunchKernelGGL(output_sq_error_kernel, dim3((unsigned)(N / SQ_CHANNELS), (unsigned)count), dim3(SQ_THREADS), 0, st,
                       (const uint16_t *)Y, (int)W4A8_F16, Yref, M, N, err, ClipState{0, nullptr, nullptr, nullptr});
    return hip_status(hipGetLastError());
}

// ---- the error split of Sec. 4.1 (Eq. 4) ---------------------------------------------------------
// delta = Wq - W diag(s) per weight, written to du where the quantized value is zero (underflow) and
// to dr otherwise (rounding); the other array gets 0.
template <typename T>
__global__ __launch_bounds__(256) void error_split_kernel(const T *__restrict__ W, int64_t N, int64_t K,
                                                          int64_t ldw, const float *__restrict__ s, int64_t G,
                                                          int special, const uint8_t *__restrict__ codes,
                                                          const float *__restrict__ step,
                                                          const uint8_t *__restrict__ zero,
                                                          float *__restrict__ du, float *__restrict__ dr)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N * K) return;
    const int64_t n = i / K, k = i - n * K;
    const int64_t pi = n * (K / G) + k / G;
    const float w = to_f32(W[n * ldw + k]);
    const float wp = s ? w * s[k] : w;
    // special: 0 = no special levels, t = 1..3: codes 14 / 15 are +-step / 2^t
    const int code = codes[i] & 15, z = zero[pi];
    const int t = special ? special : 1;
    const int d = (special && code >= 14) ? (code == 14 ? 1 : -1) : (code - z) * (1 << t);   // units of step / 2^t
    const float unit = step[pi] * (t == 1 ? 0.5f : (t == 2 ? 0.25f : 0.125f));
    const float wq = (float)d * unit;
    const float delta = wq - wp;
    du[i] = d == 0 ? delta : 0.0f;
    dr[i] = d == 0 ? 0.0f : delta;
}

template <typename T>
__global__ __launch_bounds__(256) void scale_activations_kernel(const T *__restrict__ X, int64_t M, int64_t K,
                                                                int64_t ldx, const float *__restrict__ s,
                                                                float *__restrict__ xs)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= M * K) return;
    const int64_t m = i / K, k = i - m * K;
    const float x = to_f32(X[m * ldx + k]);
    xs[i] = s ? x * (1.0f / s[k]) : x;
}

// terms = {sum pu^2, sum pr^2, sum 2 pu pr, number of non-zero entries of du}; one workgroup, fixed order
__global__ __launch_bounds__(256) void error_terms_kernel(const float *__restrict__ pu,
                                                          const float *__restrict__ pr, int64_t n,
                                                          const float *__restrict__ du, int64_t nw,
                                                          double *__restrict__ terms)
{
    __shared__ double part[4][256];
    double a = 0.0, b = 0.0, c = 0.0, u = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double x = pu[i], y = pr[i];
        a += x * x;
        b += y * y;
        c += 2.0 * x * y;
    }
    for (int64_t i = threadIdx.x; i < nw; i += 256) u += du[i] != 0.0f ? 1.0 : 0.0;
    part[0][threadIdx.x] = a;
    part[1][threadIdx.x] = b;
    part[2][threadIdx.x] = c;
    part[3][threadIdx.x] = u;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int t = 0; t < 4; ++t) part[t][threadIdx.x] += part[t][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 4) terms[threadIdx.x] = part[threadIdx.x][0];
}

int launch_error_split(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw, const float *s,
                       int64_t G, int special, const uint8_t *codes, const float *step,
                       const uint8_t *zero, float *du, float *dr, hipStream_t st)
{
    const dim3 grid((unsigned)((N * K + 255) / 256));
#define W4A8_ES_LAUNCH(T_)                                                                             \
    hipLaunchKernelGGL((error_split_kernel<T_>), grid, dim3(256), 0, st, (const T_ *)W, N, K, ldw, s, G, \
                       special, codes, step, zero, du, dr)
    switch (w_dtype) {
        case W4A8_F32: W4A8_ES_LAUNCH(float); break;
        case W4A8_F16: W4A8_ES_LAUNCH(__half); break;
        case W4A8_BF16: W4A8_ES_LAUNCH(bf16_t); break;
        default: return W4A8_ERR_DTYPE;
    }
#undef W4A8_ES_LAUNCH
    return hip_status(hipGetLastError());
}

int launch_scale_activations(const void *X, int x_dtype, int64_t M, int64_t K, int64_t ldx,
                             const float *s, float *xs, hipStream_t st)
{
    const dim3 grid((unsigned)((M * K + 255) / 256));
#define W4A8_SA_LAUNCH(T_) \
    hipLaunchKernelGGL((scale_activations_kernel<T_>), grid, dim3(256), 0, st, (const T_ *)X, M, K, ldx, s, xs)
    switch (x_dtype) {
        case W4A8_F32: W4A8_SA_LAUNCH(float); break;
        case W4A8_F16: W4A8_SA_LAUNCH(__half); break;
        case W4A8_BF16: W4A8_SA_LAUNCH(bf16_t); break;
        default: return W4A8_ERR_DTYPE;
    }
#undef W4A8_SA_LAUNCH
    return hip_status(hipGetLastError());
}

int launch_error_terms(const float *pu, const float *pr, int64_t n, const float *du, int64_t nw,
                       double *terms, hipStream_t st)
{
    hipLaunchKernelGGL(error_terms_kernel, dim3(1), dim3(256), 0, st, pu, pr, n, du, nw, terms);
    return hip_status(hipGetLastError());
}

}  // namespace w4a8
