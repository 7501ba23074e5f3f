// Group-wise product on weights decoded to int8 beforehand.
//
// What bounds the group-wise tile kernel (gemm_prefill.hip) is the vector ALU together with the matrix cores: per 128-wide
// group and wave, 16 matrix instructions (32 clocks each), 128 operations that rescale the accumulators (a conversion and a
// fused multiply-add each, 4 clocks) and 88 that decode the packed weights; two waves of a SIMD overlap hardly any of it
// (with neither memory nor LDS in the loop, matrix and vector clocks still add up to the measured time).  The decode is the
// same for every token tile and goes out of the loop here: once per call for products of many tokens
// (decode_i8_kernel), or the quantizer writes int8 itself (calibration).
// Integer operands and group sums are those of the tile kernel; so is the order of the fp32 sums of a product's outputs,
// which are the same bits.
#include <type_traits>

#include "w4a8_common.hpp"

namespace w4a8 {

typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int I8_BM = 128, I8_BN = 128, I8_THREADS = 256, I8_MS = I8_BM / 32;
constexpr int I8_TILE = I8_BM * TILE_K;   // bytes of one activation k-tile in LDS

// Activation tiles in LDS: one is read, one has landed or is about to, the others are on their way.
template <bool ERR> struct I8Ring { static constexpr int RING = 4; };
template <> struct I8Ring<true> { static constexpr int RING = 3; };   // (with 24 KB of block sums beside it, twice on a CU)
constexpr int I8_CHUNK = 8;      // ERR: k-tiles per block of the running sums
constexpr int I8_LDS_SUMS = 6;   // ERR: quarters of 4 x 4 block sums per lane that lie in LDS (the last ones), of 16

// Packed tiles -> int8 blocks, 4 d per weight (the signed decode of the tile kernel).  A wave per tile and turn: lane l
// (row l % 16, 32-column quarter l / 16) decodes its 16 bytes to the two 16-byte pieces of steps 2 sp and 2 sp + 1.
// Bound by memory: 1.5 bytes per weight (57 M weights 15.6 us, with the scales of 71 M 24).
__global__ __launch_bounds__(256) void decode_i8_kernel(const v4u *__restrict__ Wt, const float *__restrict__ step,
                                                        const uint8_t *__restrict__ zero, uint32_t tiles, uint32_t KT,
                                                        uint32_t tiles_per_group, uint8_t *__restrict__ W8,
                                                        float *__restrict__ es8, int es_ld, int plain)
{
    const int lane = threadIdx.x & 63;
    const uint32_t ng = KT / tiles_per_group;
    for (uint32_t t = blockIdx.x * 4 + (threadIdx.x >> 6); t < tiles; t += gridDim.x * 4) {
        const uint32_t nt = t / KT, kt = t - nt * KT;
        const v4u p = __builtin_nontemporal_load(Wt + (size_t)t * 64 + lane);
        const int row = lane & 15, q = lane >> 4;
        const uint32_t n = nt * 16 + row, g = kt / tiles_per_group;
        const SignedLut lut = make_signed_lut(zero[(size_t)n * ng + g], plain != 0);
        if (q == 0 && kt == g * tiles_per_group) es8[(size_t)g * es_ld + n] = step[(size_t)n * ng + g] * 0.125f;
        int a, b;
        v4i lo, hi;
        decode_word_signed(p.x, lut, a, b); lo.x = a; lo.y = b;
        decode_word_signed(p.y, lut, a, b); lo.z = a; lo.w = b;
        decode_word_signed(p.z, lut, a, b); hi.x = a; hi.y = b;
        decode_word_signed(p.w, lut, a, b); hi.z = a; hi.w = b;
        v4i *out = reinterpret_cast<v4i *>(W8 + ((size_t)(nt >> 1) * KT + kt) * I8_BLOCK) + (q >> 1) * 128 + (q & 1) * 32 +
                   (nt & 1) * 16 + row;
        out[0] = lo;
        out[64] = hi;
    }
}

// 128 tokens x 128 channels, four waves of 128 x 32, two workgroups per CU that share no barrier.  Activations through a ring
// of LDS tiles filled by direct copies, weights straight to registers two k-tiles ahead (two register sets that take
// turns), group scales through LDS two groups ahead: the pipeline of gemm_kernel.  2048 x 13824 x 4096: 185 us there, 143 here.
// (One workgroup of eight waves per CU whose halves take turns at multiplying and rescaling was 4 % faster per k-tile, 1.25 against
// 1.30 us, and lost it to coarser tiles, and to prologues and epilogues that nothing covers.)
//
// partial != null: K in ranges of kt_per_split k-tiles over blockIdx.x (see gemm_kernel), fp32 sums of a range out.
// ERR (calibration): blockIdx.y is a candidate with weights, scales and (x_tokens = M) activations of its own, and what
// comes out is, per channel and token tile, the sum of squared differences between the fp16 outputs and Yref: the outputs
// themselves never leave the registers.  The running sums go in blocks of eight k-tiles there: one rounding per group at
// the size of a block's sum and one per block at the size of the whole (a chain of 32 groups rounds at the size of the
// whole 32 times, and more outputs fall on the other side of an fp16 tie); of the sixteen quarters of block sums of a lane, ten
// are kept in registers and six in LDS.
template <bool ERR>
__global__ __launch_bounds__(I8_THREADS, 2) void gemm_i8_kernel(
    const int8_t *__restrict__ Xq, const float *__restrict__ sx, int M, const uint8_t *__restrict__ W8,
    const float *__restrict__ es8, int N, int K, int tiles_per_group, uint16_t *__restrict__ Y, int y_dtype, int64_t ldy,
    int vec_store, int grid_m, int grid_n, int kt_per_split, float *__restrict__ partial, int es_ld, int64_t x_tokens,
    int64_t w_stride, const float *__restrict__ Yref, double *__restrict__ err)
{
    constexpr int RING = I8Ring<ERR>::RING;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];   // [RING][I8_TILE], ERR: [I8_LDS_SUMS][I8_THREADS] v4f
    __shared__ __attribute__((aligned(16))) float s_es[4][I8_BN];       // step / 8, a ring of four groups
    v4f *s_sum = reinterpret_cast<v4f *>(lds_raw + RING * I8_TILE) + threadIdx.x;
    if (ERR) {
        const int64_t v = blockIdx.y;
        Xq += v * x_tokens * K;
        sx += v * x_tokens;
        W8 += v * w_stride;
        es8 = reinterpret_cast<const float *>(reinterpret_cast<const uint8_t *>(es8) + v * w_stride);
        err += v * grid_m * N;
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, kh = lane >> 5;
    const int KT = K / TILE_K;
    const int tiles = grid_m * grid_n;
    const int split = ERR ? 0 : blockIdx.x / tiles;
    const int kt0 = split * kt_per_split, KTl = min(kt_per_split, KT - kt0);
    // (the tile numbering of gemm_kernel: an XCD has a contiguous range of tiles, down panels of four token tiles)
    int bid = blockIdx.x - split * tiles;
    {
        const int per = tiles / 8;
        if (bid < per * 8) bid = (bid & 7) * per + (bid >> 3);
    }
    constexpr int PANEL = 4;
    const int panel = bid / (PANEL * grid_n);
    const int pr = bid - panel * (PANEL * grid_n);
    const int ph = min(PANEL, grid_m - panel * PANEL);
    const int bn = pr / ph;
    const int bm = panel * PANEL + pr - bn * ph;
    const int m0 = bm * I8_BM, nb0 = bn * I8_BN, n0 = nb0 + wave * 32;

    __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc((void *)W8, 0, (int)((int64_t)(N + 31) / 32 * 32 * K), 0x00020000);
    const uint64_t xq_addr = (uint64_t)Xq;
    const v4i rx = {(int)(uint32_t)xq_addr, (int)((xq_addr >> 32) & 0xffffu), (int)((int64_t)M * K), 0x00020000};
    const int wblock = min(n0 / 32, (N + 31) / 32 - 1) * KT;   // (a wave past the end repeats the last block)
    v4u pa[4], pb[4];
    auto load_b = [&](int kt, v4u(&dst)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            dst[s] = __builtin_amdgcn_raw_buffer_load_b128(rw, lane * 16 + s * 1024, (wblock + kt0 + kt) * I8_BLOCK, 0);
    };
    int avoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (i * 4 + wave) * 8 + (lane >> 3);
        avoff[i] = (m0 + row) * K + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw;
    auto dma = [&](int kt, int slot) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dma_b128(rx, avoff[i], (kt0 + kt) * TILE_K, lds_base + (uint32_t)(slot * I8_TILE + (i * 4 + wave) * 1024));
    };
    // scales of the workgroup's channels (threads 0 .. 127), fetched three groups ahead
    const int g0 = kt0 / tiles_per_group, g_end = g0 + KTl / tiles_per_group;
    float gp_es = 0.f;
    auto fetch_group = [&](int g) {
        if (tid < I8_BN) gp_es = es8[(int64_t)g * es_ld + nb0 + tid];
    };
    auto publish_group = [&](int g) {
        if (tid < I8_BN) s_es[g & 3][tid] = gp_es;
    };

    v16i acc[I8_MS];
    float y[I8_MS][16];
#pragma unroll
    for (int ms = 0; ms < I8_MS; ++ms)
#pragma unroll
        for (int r = 0; r < 16; ++r) y[ms][r] = 0.f;
    // accumulator layout as in gemm_kernel: token 32 ms + r32, channels n0 + 8 b + 4 kh + r
    auto flush_group = [&](int g) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const v4f es = *reinterpret_cast<const v4f *>(&s_es[g & 3][wave * 32 + 8 * b + 4 * kh]);
#pragma unroll
            for (int ms = 0; ms < I8_MS; ++ms)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    y[ms][4 * b + r] = __builtin_fmaf(es[r], (float)acc[ms][4 * b + r], y[ms][4 * b + r]);
        }
    };
    int frag_off[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int chunk = 2 * (2 * (s >> 1) + kh) + (s & 1);
        frag_off[s] = r32 * TILE_K + ((chunk ^ ((r32 >> 1) & 7)) << 4);
    }
    auto read_a = [&](int slot, int s, int ms) {
        return *reinterpret_cast<const v4i *>(&lds_raw[slot * I8_TILE + ms * (32 * TILE_K) + frag_off[s]]);
    };

    const int ktl = KTl - 1;
#pragma unroll
    for (int i = 0; i < RING - 1; ++i) dma(min(i, ktl), i);
    load_b(0, pa);
    load_b(min(1, ktl), pb);
    fetch_group(g0);
    publish_group(g0);
    if (g0 + 1 < g_end) {
        fetch_group(g0 + 1);
        publish_group(g0 + 1);
    }
    if (g0 + 2 < g_end) fetch_group(g0 + 2);
    asm volatile("" : "+v"(pa[0]), "+v"(pa[1]), "+v"(pa[2]), "+v"(pa[3]));
    asm volatile("" : "+v"(pb[0]), "+v"(pb[1]), "+v"(pb[2]), "+v"(pb[3]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    v4i af[2][I8_MS];
#pragma unroll
    for (int ms = 0; ms < I8_MS; ++ms) af[0][ms] = read_a(0, 0, ms);

    // ERR: block sums of quarter i = 4 ms + b, the first ten here, the others in LDS
    constexpr int REG_SUMS = 16 - I8_LDS_SUMS;
    v4f bsum[ERR ? REG_SUMS : 1];
    if (ERR) {
#pragma unroll
        for (int i = 0; i < REG_SUMS; ++i) bsum[ERR ? i : 0] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < I8_LDS_SUMS; ++i) s_sum[i * I8_THREADS] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    auto close_block = [&]() {   // block sums += running sums, which start again
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            v4f t = i < REG_SUMS ? bsum[ERR && i < REG_SUMS ? i : 0] : s_sum[(i - REG_SUMS) * I8_THREADS];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] += y[i / 4][4 * (i & 3) + r];
                y[i / 4][4 * (i & 3) + r] = 0.f;
            }
            if (i < REG_SUMS) bsum[ERR && i < REG_SUMS ? i : 0] = t;
            else s_sum[(i - REG_SUMS) * I8_THREADS] = t;
        }
    };
    // One k-tile from LDS slot `slot`; P: its weights, PN: the next tile's.  second: the odd tiles, which alone end a block.
    // Order of the accesses: [4 loads into P for tile kt + 2] wait [4 copies of tile kt + RING - 1] [scales]; the copies'
    // slot is that of tile kt - 1, which every wave has left behind the last barrier.
    auto k_tile = [&](v4u(&P)[4], v4u(&PN)[4], int kt, int t, int g, int slot, auto second) __attribute__((always_inline)) {
        const int next = slot + 1 == RING ? 0 : slot + 1;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const v4i w = {(int)P[s].x, (int)P[s].y, (int)P[s].z, (int)P[s].w};
            const v16i z16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            if (s < 3) {
#pragma unroll
                for (int ms = 0; ms < I8_MS; ++ms) af[(s + 1) & 1][ms] = read_a(slot, s + 1, ms);
            }
            if (s == 0 && t == 0) {
#pragma unroll
                for (int ms = 0; ms < I8_MS; ++ms)
                    acc[ms] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, af[s & 1][ms], z16, 0, 0, 0);
            } else {
#pragma unroll
                for (int ms = 0; ms < I8_MS; ++ms)
                    acc[ms] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, af[s & 1][ms], acc[ms], 0, 0, 0);
            }
            if (s < 3) __builtin_amdgcn_sched_group_barrier(0x100, I8_MS, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, I8_MS, 0);
        }
        order_fence();
        load_b(min(kt + 2, ktl), P);
        order_fence();
        if (t == 0 && g + 2 < g_end) publish_group(g + 2);   // (read for group g - 2 last, a barrier ago)
        // everything but the loads into P has arrived: the next tile's weights, and the copies of tile kt + RING - 2 (the
        // uses of PN behind the wait keep the compiler from waiting again behind the copies that follow)
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        asm volatile("" : "+v"(PN[0]), "+v"(PN[1]), "+v"(PN[2]), "+v"(PN[3]));
        dma(min(kt + RING - 1, ktl), slot == 0 ? RING - 1 : slot - 1);
        if (t == 0 && g + 3 < g_end) fetch_group(g + 3);
        order_fence();
        __syncthreads();   // (waits for no copy: the compiler does not know of them)
        // the next tile's first fragments arrive under the rescale
#pragma unroll
        for (int ms = 0; ms < I8_MS; ++ms) af[0][ms] = read_a(next, 0, ms);
        order_fence();
        if (t == tiles_per_group - 1) flush_group(g);
        if constexpr (ERR && decltype(second)::value) {
            if ((kt & (I8_CHUNK - 1)) == I8_CHUNK - 1) close_block();
        }
    };
    {
        int kt = 0, t = 0, g = g0, slot = 0;
        auto advance = [&]() {
            ++kt;
            slot = slot + 1 == RING ? 0 : slot + 1;
            if (++t == tiles_per_group) {
                t = 0;
                ++g;
            }
        };
        while (kt + 2 <= KTl) {
            k_tile(pa, pb, kt, t, g, slot, std::false_type{});
            advance();
            k_tile(pb, pa, kt, t, g, slot, std::true_type{});
            advance();
        }
        if (kt < KTl) k_tile(pa, pb, kt, t, g, slot, std::false_type{});
        if (ERR) close_block();   // (an open block, or an empty one: adds zeros)
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // epilogue: Y[m, n .. n+3] = cast(sx[m] * y), staged through LDS where Y allows 16-byte stores (see gemm_kernel)
    float sxm[I8_MS];
#pragma unroll
    for (int ms = 0; ms < I8_MS; ++ms) sxm[ms] = sx[min(m0 + ms * 32 + r32, M - 1)];
    if constexpr (ERR) {
        // squared differences of the fp16 outputs, binary64, over this lane's four tokens, then the 32 lanes of a channel:
        // by halving, eight of the sixteen channels' sums cross to the lane that keeps them, then four, two, one
        double e[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int nn = min(n0 + 8 * b + 4 * kh, N - 4);   // (channels past the end are not stored)
#pragma unroll
            for (int ms = 0; ms < I8_MS; ++ms) {
                const int m = m0 + ms * 32 + r32;
                const v4f ref = *reinterpret_cast<const v4f *>(Yref + (int64_t)min(m, M - 1) * N + nn);
                const int i = 4 * ms + b;
                const v4f sum = i < REG_SUMS ? bsum[ERR && i < REG_SUMS ? i : 0] : s_sum[(i - REG_SUMS) * I8_THREADS];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float out = sxm[ms] * sum[r];
                    asm volatile("" : "+v"(out));
                    const float d = __half2float(__ushort_as_half(f32_to_f16_bits(out))) - ref[r];
                    if (m < M) e[4 * b + r] += (double)d * (double)d;
                }
            }
        }
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1) {   // lanes 2 w apart exchange halves of their 2 w sums
            const bool up = (lane & (2 * w)) != 0;
#pragma unroll
            for (int i = 0; i < w; ++i) {
                const double send = up ? e[i] : e[i + w], keep = up ? e[i + w] : e[i];
                e[i] = keep + __shfl_xor(send, 2 * w, WAVE);
            }
        }
        e[0] += __shfl_xor(e[0], 1, WAVE);
        // lane bits 4, 3, 2, 1 chose bits 3, 2, 1, 0 of the sum's index 4 b + r
        const int i = (lane >> 1) & 15, n = n0 + 8 * (i >> 2) + 4 * kh + (i & 3);
        if ((lane & 1) == 0 && n < N) err[(int64_t)bm * N + n] = e[0];
        return;
    }
    const bool staged = partial == nullptr && (vec_store & 2) != 0;   // uniform
    auto store = [&](auto f16_tag, auto staged_tag) __attribute__((always_inline)) {
        constexpr bool F16 = decltype(f16_tag)::value, STAGED = decltype(staged_tag)::value;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int nl = wave * 32 + 8 * b + 4 * kh, nn = nb0 + nl;
            if (!STAGED && n0 + 8 * b >= N) continue;   // (N % 16 == 0: uniform over the wave)
#pragma unroll
            for (int ms = 0; ms < I8_MS; ++ms) {
                uint16_t hh[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float out = sxm[ms] * y[ms][4 * b + r];   // binary32 product, then the cast (see gemm_kernel)
                    asm volatile("" : "+v"(out));
                    hh[r] = F16 ? f32_to_f16_bits(out) : f32_to_bf16_bits(out);
                }
                const uint2 h4 = make_uint2((uint32_t)hh[0] | ((uint32_t)hh[1] << 16), (uint32_t)hh[2] | ((uint32_t)hh[3] << 16));
                const int rl = ms * 32 + r32;
                if (STAGED) {
                    const int c8 = nl >> 2;
                    *reinterpret_cast<uint2 *>(lds_raw + rl * (2 * I8_BN) + ((((c8 >> 1) ^ (rl & 15)) << 4) | ((c8 & 1) << 3))) = h4;
                } else if (m0 + rl < M) {
                    uint16_t *yp = Y + (int64_t)(m0 + rl) * ldy + nn;
                    if (vec_store & 1) {
                        *reinterpret_cast<uint2 *>(yp) = h4;
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) yp[r] = hh[r];
                    }
                }
            }
        }
    };
    using T = std::true_type;
    using F = std::false_type;
    if (partial != nullptr) {   // K in ranges: the combine kernel applies sx and the cast
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int nn = n0 + 8 * b + 4 * kh;
            if (n0 + 8 * b >= N) continue;
#pragma unroll
            for (int ms = 0; ms < I8_MS; ++ms) {
                const int m = m0 + ms * 32 + r32;
                if (m < M)
                    *reinterpret_cast<v4f *>(&partial[((int64_t)split * M + m) * N + nn]) =
                        v4f{y[ms][4 * b], y[ms][4 * b + 1], y[ms][4 * b + 2], y[ms][4 * b + 3]};
            }
        }
        return;
    }
    if (y_dtype == W4A8_F16) {
        if (staged) store(T{}, T{});
        else store(T{}, F{});
    } else {
        if (staged) store(F{}, T{});
        else store(F{}, F{});
    }
    if (staged) {
        __syncthreads();
        constexpr int LPR = I8_BN / 8, RPW = 64 / LPR;   // lanes per row (16 bytes each), rows per wave and store
        for (int r = wave * RPW + lane / LPR; r < I8_BM; r += 4 * RPW) {
            const int c16 = lane % LPR, m = m0 + r, nn = nb0 + c16 * 8;
            if (m < M && nn < N) {
                const v4u v = *reinterpret_cast<const v4u *>(lds_raw + r * (2 * I8_BN) + ((c16 ^ (r & 15)) << 4));
                __builtin_nontemporal_store(v, reinterpret_cast<v4u *>(Y + (int64_t)m * ldy + nn));
            }
        }
    }
}

size_t gemm_i8_bytes(int64_t N, int64_t K) { return (size_t)i8_scales_offset(N, K) + (size_t)(K / TILE_K) * i8_es_ld((int)N) * 4; }

int launch_decode_i8(const uint8_t *Wt, const float *step, const uint8_t *zero, int64_t N, int64_t K, int64_t G, uint8_t *W8, int plain,
                     hipStream_t st)
{
    const int64_t tiles = N / TILE_N * (K / TILE_K);
    if (tiles > 0x7fffffffLL || (uintptr_t)W8 % 16 != 0) return W4A8_ERR_SHAPE;
    const int64_t blocks = (tiles + 3) / 4;
    hipLaunchKernelGGL(decode_i8_kernel, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st, (const v4u *)Wt,
                       step, zero, (uint32_t)tiles, (uint32_t)(K / TILE_K), (uint32_t)(G / TILE_K), W8,
                       (float *)(W8 + i8_scales_offset(N, K)), i8_es_ld((int)N), plain);
    return hip_status(hipGetLastError());
}

static int i8_shape_ok(int64_t M, int64_t N, int64_t K)
{
    return (M + I8_BM - 1) / I8_BM * ((N + I8_BN - 1) / I8_BN) <= 0x7fffffLL && M * K <= 0x7fffffffLL &&
           (N + 31) / 32 * 32 * K <= 0x7fffffffLL;
}

int launch_gemm_i8(const int8_t *Xq, const float *sx, int64_t M, const uint8_t *W8, int64_t N, int64_t n0, int64_t n, int64_t K,
                   int64_t G, void *Y, int y_dtype, int64_t ldy, int splits, int kt_per_split, float *partial, hipStream_t st)
{
    const int64_t grid_m = (M + I8_BM - 1) / I8_BM, grid_n = (n + I8_BN - 1) / I8_BN;
    if (!i8_shape_ok(M, N, K) || n0 % I8_BN != 0 || n < 1 || n0 + n > N) return W4A8_ERR_SHAPE;
    uint16_t *y = (uint16_t *)Y + n0;
    const int vec_store = ((((uintptr_t)y % 8 == 0) && (ldy % 4 == 0)) ? 1 : 0) |
                          ((((uintptr_t)y % 16 == 0) && (ldy % 8 == 0)) ? 2 : 0);
    constexpr int lds_bytes = I8Ring<false>::RING * I8_TILE;
    static std::atomic<uint64_t> lds_opted{0};
    if (opt_in_dynamic_lds((const void *)gemm_i8_kernel<false>, lds_bytes, lds_opted) != W4A8_OK) return W4A8_ERR_HIP;
    const float *es8 = (const float *)(W8 + i8_scales_offset(N, K)) + n0;
    hipLaunchKernelGGL((gemm_i8_kernel<false>), dim3((unsigned)(grid_m * grid_n * splits)), dim3(I8_THREADS), lds_bytes, st,
                       Xq, sx, (int)M, W8 + n0 * K, es8, (int)n, (int)K, (int)(G / TILE_K), y, y_dtype, ldy, vec_store,
                       (int)grid_m, (int)grid_n, kt_per_split, splits > 1 ? partial : nullptr, i8_es_ld((int)N), (int64_t)0,
                       (int64_t)0, (const float *)nullptr, (double *)nullptr);
    return hip_status(hipGetLastError());
}

int gemm_i8_token_tiles(int64_t M) { return (int)((M + I8_BM - 1) / I8_BM); }

int launch_gemm_i8_errors(const int8_t *Xq, const float *sx, int64_t M, const uint8_t *W8, int64_t w_stride, int64_t N,
                          int64_t K, int64_t G, const float *Yref, double *err, GemmBatch batch, hipStream_t st)
{
    const int64_t grid_m = (M + I8_BM - 1) / I8_BM, grid_n = (N + I8_BN - 1) / I8_BN;
    if (!i8_shape_ok(M, N, K) || batch.count < 1 || batch.count > 65535 || w_stride % 16 != 0) return W4A8_ERR_SHAPE;
    constexpr int lds_bytes = I8Ring<true>::RING * I8_TILE + I8_LDS_SUMS * I8_THREADS * 16;
    static std::atomic<uint64_t> lds_opted{0};
    if (opt_in_dynamic_lds((const void *)gemm_i8_kernel<true>, lds_bytes, lds_opted) != W4A8_OK) return W4A8_ERR_HIP;
    const float *es8 = (const float *)(W8 + i8_scales_offset(N, K));
    hipLaunchKernelGGL((gemm_i8_kernel<true>), dim3((unsigned)(grid_m * grid_n), (unsigned)batch.count), dim3(I8_THREADS),
                       lds_bytes, st, Xq, sx, (int)M, W8, es8, (int)N, (int)K, (int)(G / TILE_K), (uint16_t *)nullptr, (int)W4A8_F16,
                       (int64_t)0, 0, (int)grid_m, (int)grid_n, (int)(K / TILE_K), (float *)nullptr, i8_es_ld((int)N),
                       batch.tokens, w_stride,
                       Yref, err);
    return hip_status(hipGetLastError());
}

}  // namespace w4a8
