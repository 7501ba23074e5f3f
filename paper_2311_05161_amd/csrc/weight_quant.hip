// dINT4 weight quantization of W diag(s)  (Eq. 1 factor Q(W diag(s)); Sec. 4.2, Eq. 5 with b = 4,
// p = 13; min-max asymmetric ranges per output channel or per group of G input channels, App. A.1).
//
// Offline; bound by memory and the vector ALU about equally.  Groups of 128 and 256 and most segments of 1024 to 16384
// elements stay in registers between the range and the codes (one sweep over W); other lengths and
// unaligned rows take one wavefront per (row, group) and two sweeps, the second served by the cache.
// Range min / max of w' = W * s extended to contain zero, step = (hi - lo) / 13, 1/step and the
// zero-point z, then Eq. 5 per element.  Every floating-point step is one binary32 operation in the
// order of the definition (no contraction), divisions are IEEE.
#include <algorithm>

#include "w4a8_common.hpp"

namespace w4a8 {

constexpr int WQ_THREADS = 256;

template <typename T, int V>
__device__ __forceinline__ void loadv(const T *p, float (&v)[V])
{
    if constexpr (V == 1) {
        v[0] = to_f32(p[0]);
    } else if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < V; i += 2) {
            const float2 a = *reinterpret_cast<const float2 *>(p + i);
            v[i] = a.x;
            v[i + 1] = a.y;
        }
    } else if constexpr (V == 2) {
        const uint32_t a = *reinterpret_cast<const uint32_t *>(p);
        T e[2];
        __builtin_memcpy(e, &a, 4);
        v[0] = to_f32(e[0]);
        v[1] = to_f32(e[1]);
    } else {
        static_assert(V == 8, "vector width");
        const uint4 a = *reinterpret_cast<const uint4 *>(p);
        T e[8];
        __builtin_memcpy(e, &a, 16);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = to_f32(e[i]);
    }
}

// Format of the code space (Sec. 4.2): p uniform steps, with or without the two special levels
// +-c, c = step / 2^shift.  dINT4: p = 13, special, shift 1 (Eq. 5); dINT3: p = 5, special; plain
// INT4: p = 15, none; shift 2 / 3: the other special values of the sweep in App. A.5 (Table 9).
struct CodeFormat {
    int p;
    int special;
    int shift = 1;
};
__host__ __device__ constexpr CodeFormat dint4_format() { return CodeFormat{DINT4_P, 1}; }

// The code rule with everything that is constant over a (row, group).  The vector ALU is what bounds the
// quantizer kernels before memory does, and not all of its operations cost the same: two waves of a SIMD issue an addition,
// multiplication, fused multiply-add, shift or AND every 2.35 clocks, but only one med3, minimum, conversion, comparison, select, byte
// permute, left shift, three-operand integer operation (bitop3 apart), or any of the former with a scalar register, every 4.6
// (measured, 16 independent chains).  So the rule keeps to the
// former where it can: per weight three of the latter (med3, comparison, select) and five of the former, and four weights
// share the rest.  (With the band as a shift-and-add and an unsigned comparison and the special code by a bit-align five
// and three.)
struct CodeRule {
    float istep;
    float lo, hi;        // -z, p - z: clamping u there is clamping rne(u) + z to 0 .. p (the bounds are integers)
    int z;
    float magic;         // 1.5 * 2^23 + z rounded up to even: adding it rounds to nearest even and converts
    uint32_t special;    // 14, and one more where the magic number holds one more than z
    uint32_t odd;        // that one, in every byte
    float band_scale, band_magic;   // see in_band: constants, in vector registers
    float target;        // what in_band's sum is in the special bands (0: no special levels)
    uint32_t band_lo;    // other special values (code_byte): the bands (lo_t, hi_t] of |u|, on the bits of |u| shifted
    uint32_t band_span;  // left by one: a subtraction and one unsigned comparison (span 0: no special levels)
};

constexpr float ROUND_MAGIC = 12582912.0f;   // 1.5 * 2^23
// 2 (1 - 2^-24).  fma(|u|, BAND_SCALE, ROUND_MAGIC), rounded once, is ROUND_MAGIC + 1 exactly where 0.25 < |u| <= 0.75: the factor
// takes the ties 0.5 and 1.5 of 2 |u| downwards and nothing else across them (checked for every binary32 u).
constexpr float BAND_SCALE = 1.99999988079071044921875f;

__device__ __forceinline__ CodeRule make_rule(float istep, int z, CodeFormat f = dint4_format())
{
    // nearest level: the band of +c runs from the midpoint between 0 and c to the midpoint
    // between c and one step (0.25 .. 0.75 for c = step/2), ends as in Eq. 5; both bounds exact
    const float lo_t = f.shift == 1 ? 0.25f : (f.shift == 2 ? 0.125f : 0.0625f);
    const float hi_t = 0.5f + lo_t;
    CodeRule r;
    r.istep = istep;
    r.lo = (float)-z;
    r.hi = (float)(f.p - z);
    r.z = z;
    r.magic = ROUND_MAGIC + (float)(z + (z & 1));
    r.special = 14u + (uint32_t)(z & 1);
    r.odd = (uint32_t)(z & 1) * 0x01010101u;
    r.band_scale = BAND_SCALE;
    r.band_magic = ROUND_MAGIC;
    asm("" : "+v"(r.band_scale), "+v"(r.band_magic));
    r.target = f.special ? ROUND_MAGIC + 1.0f : 0.0f;
    r.band_lo = (__float_as_uint(lo_t) << 1) + 1u;
    r.band_span = f.special ? (__float_as_uint(hi_t) - __float_as_uint(lo_t)) << 1 : 0u;
    return r;
}

// Whether u = x / step lies in the bands of +-step / 2.
__device__ __forceinline__ bool in_band(float u, const CodeRule &r)
{
    return __builtin_fmaf(__builtin_fabsf(u), r.band_scale, r.band_magic) == r.target;
}
// The code of x, or that and one (r.odd), in the low byte; the upper bits are whatever the arithmetic left there.
// Special values +-step / 2 or none.
__device__ __forceinline__ uint32_t code_byte_odd(float u, const CodeRule &r)   // u = x / step
{
    const uint32_t c = __float_as_uint(__builtin_amdgcn_fmed3f(u, r.lo, r.hi) + r.magic);
    const uint32_t sp = (__float_as_uint(u) >> 31) + r.special;
    // (a select, not a branch: the lanes of a wave disagree all the time)
    return in_band(u, r) ? sp : c;
}
// The code of x in the low byte, any special value.
__device__ __forceinline__ uint32_t code_byte(float x, const CodeRule &r)
{
    const float u = x * r.istep;
    const uint32_t c = __float_as_uint(__builtin_amdgcn_fmed3f(u, r.lo, r.hi) + ROUND_MAGIC) + (uint32_t)r.z;
    const uint32_t bits = __float_as_uint(u);
    const uint32_t sp = __builtin_amdgcn_alignbit(7u, bits, 31u);   // 14 + the sign bit
    return (bits << 1) - r.band_lo < r.band_span ? sp : c;
}

// Four low bytes into one register, two byte permutes and an OR.
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    return __builtin_amdgcn_perm(b, a, 0x0c0c0400u) | __builtin_amdgcn_perm(d, c, 0x04000c0cu);
}

// Four codes (special values +-step / 2 or none): no byte is below the one that r.odd takes off, so nothing borrows.
__device__ __forceinline__ uint32_t codes4(float u0, float u1, float u2, float u3, const CodeRule &r)
{
    return pack_low_bytes(code_byte_odd(u0, r), code_byte_odd(u1, r), code_byte_odd(u2, r), code_byte_odd(u3, r)) - r.odd;
}
__device__ __forceinline__ uint2 codes8(const float (&x)[8], const CodeRule &r)
{
    const float i = r.istep;
    return make_uint2(codes4(x[0] * i, x[1] * i, x[2] * i, x[3] * i, r), codes4(x[4] * i, x[5] * i, x[6] * i, x[7] * i, r));
}
// HALF: special values +-step / 2 or none; else any.
template <bool HALF>
__device__ __forceinline__ uint2 codes8_of(const float (&x)[8], const CodeRule &r)
{
    if (HALF) return codes8(x, r);
    uint32_t q[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = code_byte(x[j], r);
    return make_uint2(pack_low_bytes(q[0], q[1], q[2], q[3]), pack_low_bytes(q[4], q[5], q[6], q[7]));
}

// Min-max asymmetric parameters of a range that contains zero: step = (hi - lo) / p,
// z = clamp(rne(-lo / step), 0, p); a degenerate range gives step 1, z 0.
__device__ __forceinline__ void range_params(float lo, float hi, float &st, float &istep, int &z,
                                             CodeFormat f = dint4_format())
{
    if (hi == lo) {
        st = 1.0f;
        istep = 1.0f;
        z = 0;
    } else {
        const float range = hi - lo;
        const float pf = (float)f.p;
        st = range / pf;
        istep = 1.0f / st;
        const float nlo = -lo;
        float zf = __builtin_rintf(nlo * istep);
        zf = fminf(fmaxf(zf, 0.0f), pf);
        z = (int)zf;
    }
}

// Factor of a row's ranges (App. A.4: after the scale search the weights are additionally clipped): the
// (zero-containing) ends are multiplied by it, one binary32 multiply each; values beyond saturate.
__device__ __forceinline__ float clip_factor(const Clipping &clip, int64_t n)
{
    return 1.0f - 0.05f * (float)(clip.idx ? clip.idx[n] : clip.uniform);
}

// blockIdx.z: candidates of a search, their scales and clipping a stride apart, their outputs densely stacked
__device__ __forceinline__ void take_candidate(Clipping &clip, int64_t N, int64_t K, int64_t ng,
                                               const float *__restrict__ &s, uint8_t *__restrict__ &codes,
                                               float *__restrict__ &step, uint8_t *__restrict__ &zero)
{
    if (gridDim.z == 1) return;
    const int64_t v = blockIdx.z;
    if (s != nullptr) s += v * clip.s_stride;
    if (codes != nullptr) codes += v * N * K;
    step += v * N * ng;
    zero += v * N * ng;
    clip.uniform += (int)v * clip.stride;
}

// The V scales of a lane's V consecutive columns (1 where there is no scale vector).  Eight of
// them with two 16-byte loads where the vector is aligned: eight dword loads strided by 32 bytes
// over the lanes cost the memory pipeline several times as many cycles.
template <int V>
__device__ __forceinline__ void load_scales(const float *sg, int64_t k, int s_vec, float (&sv)[V])
{
    if (sg == nullptr) {
#pragma unroll
        for (int j = 0; j < V; ++j) sv[j] = 1.0f;
    } else if (V == 8 && s_vec) {
        const float4 s0 = *reinterpret_cast<const float4 *>(sg + k);
        const float4 s1 = *reinterpret_cast<const float4 *>(sg + k + 4);
        sv[0] = s0.x; sv[1] = s0.y; sv[2] = s0.z; sv[3] = s0.w;
        sv[4 % V] = s1.x; sv[5 % V] = s1.y; sv[6 % V] = s1.z; sv[7 % V] = s1.w;
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) sv[j] = sg[k + j];
    }
}

// A wave per (row, group), two sweeps; V columns per lane and load, times 1 where there is no scale vector.
// HALF (V = 8): special values +-step / 2 or none -- an instance of its own, as the choice between the two rules in the loop cost
// a long row 3 to 7 % (300 x 16392 fp16, us: one rule for all 26.0, the choice 28.0, instances 25.4; 768 x 768 3.90 / 4.02 / 3.89;
// 4096 x 4096 in groups of 512 21.4 / 20.9 / 20.6).
template <typename T, int V, bool HALF>
__global__ __launch_bounds__(WQ_THREADS) void weight_quant_kernel(
    const T *__restrict__ W, int64_t N, int64_t K, int64_t ldw, const float *__restrict__ s,
    int64_t G, int use_given, uint8_t *__restrict__ codes, float *__restrict__ step,
    uint8_t *__restrict__ zero, CodeFormat fmt, int s_vec, Clipping clip)
{
    const int lane = threadIdx.x & 63;
    const int64_t ng = K / G;
    take_candidate(clip, N, K, ng, s, codes, step, zero);
    const int64_t seg = (int64_t)blockIdx.x * (WQ_THREADS / WAVE) + (threadIdx.x >> 6);
    if (seg >= N * ng) return;  // whole wave leaves together
    const int64_t n = seg / ng, g = seg % ng;
    const T *w = W + n * ldw + g * G;
    const float *sg = s ? s + g * G : nullptr;

    float st, istep;
    int z;
    if (use_given) {
        st = step[seg];
        z = zero[seg];
        istep = 1.0f / st;
    } else {
        float lo = 0.0f, hi = 0.0f;
        for (int64_t k = (int64_t)lane * V; k < G; k += (int64_t)WAVE * V) {
            float v[V], sv[V];
            loadv<T, V>(w + k, v);
            load_scales<V>(sg, k, s_vec, sv);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float x = v[j] * sv[j];
                lo = fminf(lo, x);
                hi = fmaxf(hi, x);
            }
        }
        const float rho = clip_factor(clip, n);
        lo = wave_min(lo) * rho;
        hi = wave_max(hi) * rho;
        range_params(lo, hi, st, istep, z, fmt);
        if (lane == 0) {
            step[seg] = st;
            zero[seg] = (uint8_t)z;
        }
    }
    if (codes == nullptr) return;

    const CodeRule rule = make_rule(istep, z, fmt);
    uint8_t *c = codes + n * K + g * G;
    for (int64_t k = (int64_t)lane * V; k < G; k += (int64_t)WAVE * V) {
        float v[V], sv[V];
        loadv<T, V>(w + k, v);
        load_scales<V>(sg, k, s_vec, sv);
        float x[V];
#pragma unroll
        for (int j = 0; j < V; ++j) x[j] = v[j] * sv[j];
        if constexpr (V == 8)
            *reinterpret_cast<uint2 *>(c + k) = codes8_of<HALF>(x, rule);
        else if constexpr (V == 2)
            *reinterpret_cast<uint16_t *>(c + k) =
                (uint16_t)pack_low_bytes(code_byte(x[0], rule), code_byte(x[1], rule), 0u, 0u);
        else
            c[k] = (uint8_t)code_byte(x[0], rule);
    }
}

// x[j] = v[j] * sv[j], the eight elements still in their storage type (no scale vector: times 1, exactly v[j]).
template <typename T>
__device__ __forceinline__ void scaled8(const T *e, const float (&sv)[8], float (&x)[8])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = to_f32(e[j]) * sv[j];
}

template <typename T>
struct Raw8 {   // eight elements as they come from memory
    uint4 w[sizeof(T) / 2];
    __device__ __forceinline__ void load(const T *p)
    {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(T) / 2); ++i) w[i] = reinterpret_cast<const uint4 *>(p)[i];
    }
    __device__ __forceinline__ void elements(T (&e)[8]) const { __builtin_memcpy(e, w, sizeof(w)); }
};

__device__ __forceinline__ void min_max8(const float (&x)[8], float &lo, float &hi)
{
#pragma unroll
    for (int j = 0; j < 8; j += 2) {   // (v_min3 / v_max3)
        lo = fminf(fminf(lo, x[j]), x[j + 1]);
        hi = fmaxf(fmaxf(hi, x[j]), x[j + 1]);
    }
}

// The larger of this lane's and another lane's value, and of ends of ranges as bits: hi >= 0 without its sign, lo <= 0 as it
// is, whose bits grow with its magnitude (and of the zeros either will do).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max_u32(uint32_t keep, uint32_t send)
{
    return max(keep, (uint32_t)dpp_i32<CTRL>((int)send));
}
__device__ __forceinline__ uint32_t hi_bits(float hi) { return __float_as_uint(hi) & 0x7fffffffu; }

// Groups of 128 or 256 columns: a wave takes 512 consecutive columns (8 per lane, one 16-byte load) of
// ROWS rows, i.e. 4 or 2 whole groups of each row, each reduced over its own LANES = G / 8 lanes; the
// elements stay in registers between the range and the codes, so W is read once.
// Bound by the vector ALU until some 17 operations per lane and weight are left, so whatever is not per weight is kept off it:
// the four waves of a block take four times ROWS rows of the same columns, which needs no division and leaves the row
// addresses to the scalar unit; the rows share the lane's eight AQAS scales (twice the
// bytes of fp16 weights) and the two IEEE divisions of a group (some 25 operations): the rows' ranges are reduced
// together, on bits, and end with row l % 4 in lane l, which computes its parameters, and the four lanes of a quad exchange them.
// 13824 x 5120, G = 128: 48 -> 41 us (5.1 TB/s; a plain pass of the same loads and stores takes 33), 8192 x 8192, G = 256: 46 -> 38.
// (Non-temporal loads of W: the same, fp32 8 % slower.)
// ROWS = 1: small matrices, for which four rows per wave leave most CUs idle (one / four rows, us: 768 x 768 3.5 / 4.3,
// 1024 x 1024 3.6 / 4.3, 512 x 4096 4.5 / 4.5, 1024 x 4096 6.2 / 5.8).
constexpr int SG_ROWS = 4;

template <int ROW>
__device__ __forceinline__ float quad_lane_f32(float v) { return dpp_f32<ROW * 0x55>(v); }
template <int ROW>
__device__ __forceinline__ CodeRule quad_lane_rule(const CodeRule &m, CodeFormat fmt)
{
    CodeRule r = m;
    r.istep = quad_lane_f32<ROW>(m.istep);
    r.lo = quad_lane_f32<ROW>(m.lo);
    r.hi = r.lo + (float)fmt.p;   // (whole numbers)
    r.magic = quad_lane_f32<ROW>(m.magic);
    r.odd = (uint32_t)dpp_i32<ROW * 0x55>((int)m.odd);
    r.special = 14u + (r.odd & 1u);
    r.z = (int)-r.lo;
    return r;
}

template <typename T, int LANES, int ROWS, bool HALF>
__global__ __launch_bounds__(WQ_THREADS) void weight_quant_small_groups_kernel(
    const T *__restrict__ W, int64_t N, int64_t K, int64_t ldw, const float *__restrict__ s,
    int use_given, uint8_t *__restrict__ codes, float *__restrict__ step, uint8_t *__restrict__ zero,
    CodeFormat fmt, int s_vec, Clipping clip)
{
    static_assert(ROWS == 1 || ROWS == 4, "the lanes of a quad share the work on four rows");
    constexpr int G = LANES * 8, WAVES = WQ_THREADS / WAVE;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // One row per wave, four chunks (1544 to 2048 columns): every four rows start one chunk on.  In their order each chunk lies on
    // the same two XCDs in all rows, which is the slower way there: 1024 x 2048 fp16 4.1 -> 3.65 us (with given parameters 3.7 -> 3.3;
    // blocks along a row 4.1 and 3.6), 900 x 1664 3.75 -> 3.6.  With two or eight chunks it is the faster one (512 x 4096 3.6, turned 3.75).
    const uint32_t chunk = ROWS == 1 && gridDim.x == 4 ? (blockIdx.x + blockIdx.y) & 3u : blockIdx.x;
    const int64_t k0 = (int64_t)chunk * 512;
    const int kl = lane * 8;
    if (k0 + kl >= K) return;   // whole groups of LANES lanes leave together (K % G == 0)
    float sv[8];
    load_scales<8>(s ? s + k0 : nullptr, kl, s_vec, sv);
    const int64_t ng = K / G;
    const int64_t g0 = k0 / G;
    const int gl = lane / LANES;
    const int mine = ROWS == 4 ? lane & 3 : 0;   // the row whose parameters this lane computes
    for (int64_t n0 = ((int64_t)blockIdx.y * WAVES + wave) * ROWS; n0 < N; n0 += (int64_t)gridDim.y * WAVES * ROWS) {
        Raw8<T> raw[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) raw[r].load(W + min(n0 + r, N - 1) * ldw + k0 + kl);   // (rows past the end: not stored)
        float x[ROWS][8];
        uint32_t lo[ROWS], hi[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            T e[8];
            raw[r].elements(e);
            scaled8(e, sv, x[r]);
            float l = 0.0f, h = 0.0f;
            min_max8(x[r], l, h);
            lo[r] = __float_as_uint(l);
            hi[r] = hi_bits(h);
        }
        float st, istep;
        int z;
        const int64_t pidx = min(n0 + mine, N - 1) * ng + g0 + gl;
        if (use_given) {
            st = step[pidx];
            z = zero[pidx];
            istep = 1.0f / st;
        } else {
            auto reduce = [&](uint32_t(&v)[ROWS]) {
                uint32_t m;
                if constexpr (ROWS == 4) {   // lanes that differ in bit 0, then bit 1, keep the rows with their bit
                    const bool b0 = lane & 1, b1 = lane & 2;
                    const uint32_t a = dpp_max_u32<DPP_QUAD_XOR1>(b0 ? v[1] : v[0], b0 ? v[0] : v[1]);
                    const uint32_t c = dpp_max_u32<DPP_QUAD_XOR1>(b0 ? v[3] : v[2], b0 ? v[2] : v[3]);
                    m = dpp_max_u32<DPP_QUAD_XOR2>(b1 ? c : a, b1 ? a : c);
                } else {
                    m = dpp_max_u32<DPP_QUAD_XOR1>(v[0], v[0]);
                    m = dpp_max_u32<DPP_QUAD_XOR2>(m, m);
                }
                m = dpp_max_u32<DPP_ROW_ROR4>(m, m);
                m = dpp_max_u32<DPP_ROW_ROR8>(m, m);
                if (LANES == 32) m = max(m, (uint32_t)__shfl_xor((int)m, 16, WAVE));
                return __uint_as_float(m);
            };
            const float rho = clip_factor(clip, min(n0 + mine, N - 1));
            range_params(reduce(lo) * rho, reduce(hi) * rho, st, istep, z, fmt);
            if ((lane & (LANES - 1)) < ROWS && n0 + mine < N) {
                step[pidx] = st;
                zero[pidx] = (uint8_t)z;
            }
        }
        if (codes == nullptr) continue;
        const CodeRule own = make_rule(istep, z, fmt);
        const CodeRule rule[4] = {ROWS == 4 ? quad_lane_rule<0>(own, fmt) : own, quad_lane_rule<1>(own, fmt),
                                  quad_lane_rule<2>(own, fmt), quad_lane_rule<3>(own, fmt)};   // (one row: every lane has its own)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint2 q = codes8_of<HALF>(x[r], rule[r]);
            if (n0 + r < N) *reinterpret_cast<uint2 *>(codes + (n0 + r) * K + k0 + kl) = q;
        }
    }
}

// Segments (a row, or a group of it) of 1024 to 16384 elements: a block takes SEG_ROWS rows' segments of the
// same columns, CH chunks of eight elements per thread and row, which stay in registers between the range
// and the codes: W is read once, and the AQAS scales once for both rows.  One barrier.  Bound by
// memory (3 bytes per fp16 weight) and the vector ALU.  The wave-per-segment kernel above sweeps W
// twice, and the second time much of it comes from beyond the L2.
// 36864 x 9216 per channel: 322 -> 217 -> 199 us (5.1 TB/s), the last by the cheaper code rule.  (Keeping the 16-bit
// elements instead of the scaled values, which are half the registers: 221.)
constexpr int SEG_ROWS = 2;
constexpr int SEG_MAX_CHUNKS = 8;

template <typename T, int CH, bool HALF>
__global__ __launch_bounds__(WQ_THREADS) void weight_quant_segment_kernel(
    const T *__restrict__ W, int64_t N, int64_t K, int64_t ldw, const float *__restrict__ s, int G,
    int use_given, uint8_t *__restrict__ codes, float *__restrict__ step, uint8_t *__restrict__ zero,
    CodeFormat fmt, int s_vec, Clipping clip)
{
    __shared__ float part[2 * SEG_ROWS][WQ_THREADS / WAVE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n0 = (int64_t)blockIdx.x * SEG_ROWS, g = blockIdx.y, ng = K / G;
    take_candidate(clip, N, K, ng, s, codes, step, zero);
    const int chunks = G / 8;
    const int64_t col = g * G;
    const bool second = n0 + 1 < N;   // (an odd last row is taken twice and stored once)
    const T *w[SEG_ROWS] = {W + n0 * ldw + col, W + (second ? n0 + 1 : n0) * ldw + col};
    float x[SEG_ROWS][CH][8];
    float lo[SEG_ROWS] = {0.0f, 0.0f}, hi[SEG_ROWS] = {0.0f, 0.0f};
    Raw8<T> raw[SEG_ROWS][CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        // (past the end: the last chunk again, which changes no range and is not stored)
        const int k = min(c * WQ_THREADS + tid, chunks - 1) * 8;
#pragma unroll
        for (int r = 0; r < SEG_ROWS; ++r) raw[r][c].load(w[r] + k);
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int k = min(c * WQ_THREADS + tid, chunks - 1) * 8;
        float sv[8];
        load_scales<8>(s ? s + col : nullptr, k, s_vec, sv);
#pragma unroll
        for (int r = 0; r < SEG_ROWS; ++r) {
            T e[8];
            raw[r][c].elements(e);
            scaled8(e, sv, x[r][c]);
            if (!use_given) min_max8(x[r][c], lo[r], hi[r]);
        }
    }
    CodeRule rule[SEG_ROWS];
    if (!use_given) {
#pragma unroll
        for (int r = 0; r < SEG_ROWS; ++r) {
            lo[r] = wave_min(lo[r]);
            hi[r] = wave_max(hi[r]);
            if (lane == 0) {
                part[2 * r][wave] = lo[r];
                part[2 * r + 1][wave] = hi[r];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < SEG_ROWS; ++r) {
        const int64_t n = r == 0 || second ? n0 + r : n0, pidx = n * ng + g;
        float st, istep;
        int z;
        if (use_given) {
            istep = 1.0f / step[pidx];
            z = zero[pidx];
        } else {
            const float l = fminf(fminf(part[2 * r][0], part[2 * r][1]), fminf(part[2 * r][2], part[2 * r][3]));
            const float h = fmaxf(fmaxf(part[2 * r + 1][0], part[2 * r + 1][1]),
                                  fmaxf(part[2 * r + 1][2], part[2 * r + 1][3]));
            const float rho = clip_factor(clip, n);
            range_params(l * rho, h * rho, st, istep, z, fmt);
            if (tid == 0 && (r == 0 || second)) {
                step[pidx] = st;
                zero[pidx] = (uint8_t)z;
            }
        }
        rule[r] = make_rule(istep, z, fmt);
    }
    if (codes == nullptr) return;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int at = c * WQ_THREADS + tid;
        if (at >= chunks) break;
#pragma unroll
        for (int r = 0; r < SEG_ROWS; ++r)
            if (r == 0 || second)
                *reinterpret_cast<uint2 *>(codes + (n0 + r) * K + col + (int64_t)at * 8) = codes8_of<HALF>(x[r][c], rule[r]);
    }
}

template <typename T>
static int launch_weight_quant_t(const T *W, int64_t N, int64_t K, int64_t ldw, const float *s,
                                 int64_t G, int use_given, uint8_t *codes, float *step,
                                 uint8_t *zero, CodeFormat fmt, hipStream_t st, Clipping clip)
{
    const int64_t segs = N * (K / G);
    if (segs == 0) return W4A8_OK;
    if (clip.count < 1 || clip.count > 65535) return W4A8_ERR_SHAPE;
    const int64_t blocks = (segs + (WQ_THREADS / WAVE) - 1) / (WQ_THREADS / WAVE);
    if (blocks > 0x7fffffffLL) return W4A8_ERR_SHAPE;
    const unsigned cands = (unsigned)clip.count;
    const int s_vec = (uintptr_t)s % 16 == 0 && clip.s_stride % 4 == 0;   // (G % 8 == 0 wherever eight scales are loaded at once)
    const auto aligned = [&](int v) {
        return G % v == 0 && K % v == 0 && (ldw * sizeof(T)) % (v * sizeof(T)) == 0 &&
               (uintptr_t)W % (v * sizeof(T)) == 0 && (uintptr_t)codes % v == 0 && ldw % v == 0;
    };
    // Segments of 1024 to 16384 elements (the elements of two rows fit in registers): the segment kernel, except where too many of
    // its threads have no chunk.  It works in rounds of 2048 elements, a wave of the wave-per-segment kernel in rounds of 512:
    // with three or fewer of the latter, or five, more than a quarter of a block idles.  Up to 1536 segments, 1024 of the shortest (latency), it wins at every
    // length, and in binary32 with five rounds, or three and more than 70 MiB of weights (the second sweep comes from memory).
    // Wave / segment kernel, us, fp16: 16384 x 1024 17.5 / 23.4, 4096 x 1536 8.1 / 9.0, 4096 x 1792 9.8 / 9.5, 4096 x 2304 11.8 / 12.3,
    // 16384 x 2816 37.9 / 35.2, 16384 x 4096 51.6 / 42.5, 1024 x 1280 4.9 / 4.6; binary32: 4096 x 1024 6.4 / 8.1, 4096 x 2304 12.9 / 12.6,
    // 16384 x 1280 26.5 / 23.3, 4096 x 8192 in groups of 1024 33.3 / 37.7.
    const auto segment_pays = [&] {
        const int64_t rounds = (G + WAVE * 8 - 1) / (WAVE * 8);
        return segs * cands <= (rounds >= 3 ? 1536 : 1024) || rounds == 4 || rounds >= 6 ||
               (sizeof(T) == 4 && (rounds == 5 || (rounds == 3 && N * K * 4 > (70 << 20))));
    };
#define W4A8_WQ_LAUNCH(V_, HALF_)                                                                 \
    hipLaunchKernelGGL((weight_quant_kernel<T, V_, HALF_>), dim3((unsigned)blocks, 1, cands), dim3(WQ_THREADS), 0, \
                       st, W, N, K, ldw, s, G, use_given, codes, step, zero, fmt, s_vec, clip)
    if ((G == 128 || G == 256) && aligned(8) && cands == 1) {   // (candidates: per-channel layers of 128 or 256 columns only)
        // (fewer rows than a block of four per wave has room for leave waves of it idle: one per wave up to 1.5 * 2^23 weights,
        // and of one or two rows always.  One / four, us: 4 x 2^20 5.4 / 6.5, 9 x 2^20 9.0 / 9.9, 1 x 2^24 22.6 / 30.3; 15 x 1118208 15.5 / 15.0, 12 x 5592064 49 / 44)
        const int rows = N * K <= (N < SG_ROWS * (WQ_THREADS / WAVE) ? 3 << 22 : 1 << 21) || N <= 2 ? 1 : SG_ROWS;
        const int64_t strips = (N + rows * (WQ_THREADS / WAVE) - 1) / (rows * (WQ_THREADS / WAVE)), chunks = (K + 511) / 512;
        if (chunks > 0x7fffffffLL) return W4A8_ERR_SHAPE;
        const dim3 grid((unsigned)chunks, (unsigned)(strips < 65535 ? strips : 65535));
#define W4A8_WQ_SMALL_F(LANES_, ROWS_, HALF_)                                                                     \
    hipLaunchKernelGGL((weight_quant_small_groups_kernel<T, LANES_, ROWS_, HALF_>), grid, dim3(WQ_THREADS), 0, st, \
                       W, N, K, ldw, s, use_given, codes, step, zero, fmt, s_vec, clip)
#define W4A8_WQ_SMALL(LANES_, ROWS_)                              \
    do {                                                          \
        if (fmt.shift == 1) W4A8_WQ_SMALL_F(LANES_, ROWS_, true); \
        else W4A8_WQ_SMALL_F(LANES_, ROWS_, false);               \
    } while (0)
        if (G == 128) {
            if (rows == 1) W4A8_WQ_SMALL(16, 1);
            else W4A8_WQ_SMALL(16, SG_ROWS);
        } else {
            if (rows == 1) W4A8_WQ_SMALL(32, 1);
            else W4A8_WQ_SMALL(32, SG_ROWS);
        }
#undef W4A8_WQ_SMALL
#undef W4A8_WQ_SMALL_F
    } else if (G >= 1024 && G <= SEG_MAX_CHUNKS * 8 * WQ_THREADS && aligned(8) && K / G <= 65535 &&
               N <= 0x7fffffffLL && segment_pays()) {
        const dim3 grid((unsigned)((N + SEG_ROWS - 1) / SEG_ROWS), (unsigned)(K / G), cands);
#define W4A8_WQ_SEGMENT_F(CH_, HALF_)                                                                            \
    hipLaunchKernelGGL((weight_quant_segment_kernel<T, CH_, HALF_>), grid, dim3(WQ_THREADS), 0, st, W, N, K, ldw, \
                       s, (int)G, use_given, codes, step, zero, fmt, s_vec, clip)
#define W4A8_WQ_SEGMENT(CH_)                                                                              \
    case CH_:                                                                                             \
        if (fmt.shift == 1) W4A8_WQ_SEGMENT_F(CH_, true);                                                  \
        else W4A8_WQ_SEGMENT_F(CH_, false);                                                                \
        break
        switch ((int)((G / 8 + WQ_THREADS - 1) / WQ_THREADS)) {
            W4A8_WQ_SEGMENT(1);
            W4A8_WQ_SEGMENT(2);
            W4A8_WQ_SEGMENT(3);
            W4A8_WQ_SEGMENT(4);
            W4A8_WQ_SEGMENT(5);
            W4A8_WQ_SEGMENT(6);
            W4A8_WQ_SEGMENT(7);
            W4A8_WQ_SEGMENT(8);
        }
#undef W4A8_WQ_SEGMENT
#undef W4A8_WQ_SEGMENT_F
    } else if (G >= 512 && aligned(8)) {
        if (fmt.shift == 1) W4A8_WQ_LAUNCH(8, true);
        else W4A8_WQ_LAUNCH(8, false);
    } else if (aligned(2)) {
        W4A8_WQ_LAUNCH(2, false);
    } else {
        W4A8_WQ_LAUNCH(1, false);
    }
#undef W4A8_WQ_LAUNCH
    return hip_status(hipGetLastError());
}

int launch_weight_quant(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw,
                        const float *s, int64_t G, int use_given, uint8_t *codes, float *step,
                        uint8_t *zero, int format, hipStream_t st, Clipping clip)
{
    CodeFormat fmt;
    switch (format) {
        case W4A8_FMT_DINT4: fmt = CodeFormat{13, 1}; break;
        case W4A8_FMT_INT4: fmt = CodeFormat{15, 0}; break;
        case W4A8_FMT_DINT3: fmt = CodeFormat{5, 1}; break;
        case W4A8_FMT_DINT4_C4: fmt = CodeFormat{13, 1, 2}; break;
        case W4A8_FMT_DINT4_C8: fmt = CodeFormat{13, 1, 3}; break;
        default: return W4A8_ERR_DTYPE;
    }
    switch (w_dtype) {
        case W4A8_F32:
            return launch_weight_quant_t((const float *)W, N, K, ldw, s, G, use_given, codes, step,
                                         zero, fmt, st, clip);
        case W4A8_F16:
            return launch_weight_quant_t((const __half *)W, N, K, ldw, s, G, use_given, codes, step,
                                         zero, fmt, st, clip);
        case W4A8_BF16:
            return launch_weight_quant_t((const bf16_t *)W, N, K, ldw, s, G, use_given, codes, step,
                                         zero, fmt, st, clip);
        default: return W4A8_ERR_DTYPE;
    }
}

// ---- quantized straight to the tiled packed form --------------------------------------------------
// dINT4 with groups of 128: a 16 x 128 tile of the packed form is 16 whole groups.  A wave takes WQT_TILES row tiles of
// the same columns (one): lane l holds row l % 16, columns 32 c + 8 (l / 16) .. + 7,
// c = 0..3, so that a load instruction reads 64 contiguous bytes of each row (32 consecutive columns per
// lane, which would make one 16-byte store, read 16-byte pieces and measured the same), the four
// lanes of a group meet in two shuffles, and codes 8 c' .. of quarter c are one word of the tile.
// Bound by the vector ALU (a candidate's weights: two multiplications, the range, the code rule) and the stores; more waves
// on a SIMD serve both better than scales that two tiles share: one tile per wave (int8 111 registers, packed 97) instead of two (163, 173).
// us, two tiles / one, 4096 x 4096 fp16: int8 (one also with streaming stores) of 17 scales 113 / 101, of 11 clipping factors 56 / 50 (without
// the code rule's arithmetic 68 and 33), packed 15.1 / 12.6; 2048 x 3072: 46 / 39, 28 / 22 and 8.2 / 6.5.
// The streaming hint of the int8 stores takes from the quantizer what it costs the product that reads them next: ten layers of 64 to 2048 calibration
// tokens, whole searches, 5 % faster to 4 % slower with it in no order of size, 0.8 % faster on average (512 x 4096 x 4096 401 with, 416
// without; 97 x 1920 x 3072 112 and 108).
constexpr int WQT_TILES = 1;

// Eight weights -> four times their value in half steps, as bytes: 8 (code - z), or +-4 for the special codes (the rule of
// code_byte without the zero-point).
__device__ __forceinline__ uint32_t level_byte(float x, const CodeRule &r)   // twice the level's quarter, in the low byte
{
    const float u = x * r.istep;
    uint32_t c = __float_as_uint(__builtin_amdgcn_fmed3f(u, r.lo, r.hi) + ROUND_MAGIC);
    asm("v_add_u32 %0, %1, %1" : "=v"(c) : "v"(c));   // (twice it; the compiler would shift, at half the rate)
    const uint32_t sp = __float_as_uint(__builtin_fmaf(u, r.band_scale, r.band_magic));   // +-1 in the bands
    return in_band(u, r) ? sp : c;
}
__device__ __forceinline__ uint2 levels8(const float (&x)[8], const CodeRule &r)
{
    uint32_t b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) b[j] = level_byte(x[j], r);
    return make_uint2((pack_low_bytes(b[0], b[1], b[2], b[3]) << 2) & 0xfcfcfcfcu,
                      (pack_low_bytes(b[4], b[5], b[6], b[7]) << 2) & 0xfcfcfcfcu);
}

template <typename T, bool I8>
__global__ __launch_bounds__(WQ_THREADS) void weight_quant_packed_kernel(
    const T *__restrict__ W, uint32_t NT, uint32_t KT, int64_t ldw, const float *__restrict__ s,
    uint32_t *__restrict__ packed, float *__restrict__ step, uint8_t *__restrict__ zero, int s_vec, Clipping clip,
    int per_block, int64_t w_stride, int64_t scales_offset, int es_ld)
{
    const int lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * (WQ_THREADS / WAVE) + (threadIdx.x >> 6);
    const uint32_t ntp = wave / KT, kt = wave - ntp * KT;   // (WQT_TILES row tiles, k-tile)
    if (ntp * WQT_TILES >= NT) return;                      // whole wave
    const int row = lane & 15;
    const int kb = lane >> 4;
    const int64_t k = (int64_t)kt * TILE_K + kb * 8;
    uint32_t nt[WQT_TILES];
    Raw8<T> raw[WQT_TILES][4];
#pragma unroll
    for (int i = 0; i < WQT_TILES; ++i) {
        nt[i] = min(ntp * WQT_TILES + i, NT - 1);   // (past the end: the last tile again, the same results)
        const T *w = W + ((int64_t)nt[i] * TILE_N + row) * ldw + k;
#pragma unroll
        for (int c = 0; c < 4; ++c) raw[i][c].load(w + 32 * c);
    }
    float x[WQT_TILES][4][8];
    float lo[WQT_TILES], hi[WQT_TILES];
    const int first = blockIdx.y * per_block, last = min(clip.count, first + per_block);
    for (int v = first; v < last; ++v) {   // (uniform)
        if (v == first || clip.s_stride != 0) {   // candidates with one scale differ in the clipping of the range only
            const float *sc = s != nullptr ? s + v * clip.s_stride : nullptr;
#pragma unroll
            for (int i = 0; i < WQT_TILES; ++i) lo[i] = hi[i] = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float sv[8];
                load_scales<8>(sc, k + 32 * c, s_vec, sv);
#pragma unroll
                for (int i = 0; i < WQT_TILES; ++i) {
                    T e[8];
                    raw[i][c].elements(e);
                    scaled8(e, sv, x[i][c]);
                    min_max8(x[i][c], lo[i], hi[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < WQT_TILES; ++i) {
                lo[i] = fminf(lo[i], __shfl_xor(lo[i], 16, WAVE));
                hi[i] = fmaxf(hi[i], __shfl_xor(hi[i], 16, WAVE));
                lo[i] = fminf(lo[i], __shfl_xor(lo[i], 32, WAVE));
                hi[i] = fmaxf(hi[i], __shfl_xor(hi[i], 32, WAVE));
            }
        }
        const float rho = clip_factor(Clipping{nullptr, clip.uniform + v * clip.stride}, 0);
        const int64_t tiles = (int64_t)v * NT * KT;   // of the candidates before this one
#pragma unroll
        for (int i = 0; i < WQT_TILES; ++i) {
            const int64_t n = (int64_t)nt[i] * TILE_N + row;
            float st, istep;
            int z;
            range_params(lo[i] * rho, hi[i] * rho, st, istep, z);
            const CodeRule rule = make_rule(istep, z);
            if constexpr (I8) {
                uint8_t *w8 = reinterpret_cast<uint8_t *>(packed) + v * w_stride;
                if (lane < 16) reinterpret_cast<float *>(w8 + scales_offset)[(int64_t)kt * es_ld + n] = st * 0.125f;
                // columns 32 c + 8 kb ..: k-step 2 (c / 2) + kb / 2, lanes of half c % 2, upper or lower eight bytes
                uint8_t *block = w8 + ((int64_t)(nt[i] >> 1) * KT + kt) * I8_BLOCK + (kb >> 1) * 1024 +
                                 ((nt[i] & 1) * 16 + row) * 16 + (kb & 1) * 8;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint2 q = levels8(x[i][c], rule);
                    __builtin_nontemporal_store(v2u{q.x, q.y}, reinterpret_cast<v2u *>(block + (c >> 1) * 2048 + (c & 1) * 512));
                }
            } else {
                if (lane < 16) {
                    step[tiles * TILE_N + n * KT + kt] = st;
                    zero[tiles * TILE_N + n * KT + kt] = (uint8_t)z;
                }
                uint32_t *tile = packed + (tiles + (int64_t)nt[i] * KT + kt) * (TILE_BYTES / 4) + row * 4 + kb;
#pragma unroll
                for (int c = 0; c < 4; ++c) {   // word kb of lane (row, quarter c): 256 contiguous bytes per store
                    const uint2 q = codes8(x[i][c], rule);
                    tile[c * 64] = recode8(q.x, q.y, 0x01010101u);
                }
            }
        }
    }
}

bool weight_quant_packs(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw, int64_t G)
{
    const int64_t es = w_dtype == W4A8_F32 ? 4 : 2;
    return G == TILE_K && N % TILE_N == 0 && K % TILE_K == 0 && (uintptr_t)W % 16 == 0 && ldw * es % 16 == 0 &&
           (N / TILE_N) * (K / TILE_K) <= 0x7fffffffLL;
}

template <bool I8>
static int launch_weight_quant_tiles(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw, const float *s,
                                     int64_t G, uint8_t *out, float *step, uint8_t *zero, Clipping clip, int64_t w_stride,
                                     hipStream_t st)
{
    const int count = clip.count;
    if (!weight_quant_packs(W, w_dtype, N, K, ldw, G) || (uintptr_t)out % 16 != 0 || w_stride % 16 != 0 || count < 1 ||
        clip.idx != nullptr)
        return W4A8_ERR_SHAPE;
    const uint32_t NT = (uint32_t)(N / TILE_N), KT = (uint32_t)(K / TILE_K);
    const int64_t waves = (int64_t)((NT + WQT_TILES - 1) / WQT_TILES) * KT;
    const int64_t blocks = (waves + WQ_THREADS / WAVE - 1) / (WQ_THREADS / WAVE);
    // all candidates in the block that has the weights, unless that leaves CUs without work
    const int per_block = (int)std::max<int64_t>(1, std::min<int64_t>(count, blocks * count / 1024));
    const dim3 grid((unsigned)blocks, (unsigned)((count + per_block - 1) / per_block));
    const int s_vec = (uintptr_t)s % 16 == 0 && clip.s_stride % 4 == 0;
#define W4A8_WQT_LAUNCH(T_)                                                                                    \
    hipLaunchKernelGGL((weight_quant_packed_kernel<T_, I8>), grid, dim3(WQ_THREADS), 0, st, (const T_ *)W, NT, KT, \
                       ldw, s, (uint32_t *)out, step, zero, s_vec, clip, per_block, w_stride, i8_scales_offset(N, K), \
                       i8_es_ld((int)N))
    switch (w_dtype) {
        case W4A8_F32: W4A8_WQT_LAUNCH(float); break;
        case W4A8_F16: W4A8_WQT_LAUNCH(__half); break;
        case W4A8_BF16: W4A8_WQT_LAUNCH(bf16_t); break;
        default: return W4A8_ERR_DTYPE;
    }
#undef W4A8_WQT_LAUNCH
    return hip_status(hipGetLastError());
}

int launch_weight_quant_packed(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw, const float *s,
                               int64_t G, uint8_t *packed, float *step, uint8_t *zero, Clipping clip, hipStream_t st)
{
    return launch_weight_quant_tiles<false>(W, w_dtype, N, K, ldw, s, G, packed, step, zero, clip, 0, st);
}

int launch_weight_quant_i8(const void *W, int w_dtype, int64_t N, int64_t K, int64_t ldw, const float *s, int64_t G,
                           uint8_t *W8, int64_t w_stride, Clipping clip, hipStream_t st)
{
    return launch_weight_quant_tiles<true>(W, w_dtype, N, K, ldw, s, G, W8, nullptr, nullptr, clip, w_stride, st);
}

// ---- 4-bit Value cache (Sec. 5.1; App. A.1: channel-wise along the dimension the product with the
// attention map accumulates over, i.e. the tokens) -------------------------------------------------
// V [batch, T, D] is stored token-major, as a cache is appended to; the product wants V^T.  A
// workgroup owns 64 channels of one (head, token group): lane = channel, so every load is 64
// consecutive elements of one token; the four waves split the tokens, their ranges meet in LDS,
// and the codes go through an LDS transpose so that each channel row is written 16 bytes at a time.
template <typename T>
__global__ __launch_bounds__(256) void value_quant_kernel(const T *__restrict__ V, int64_t Tn,
                                                          int64_t D, int64_t ld_t, int64_t ld_b,
                                                          int64_t G, uint8_t *__restrict__ codes,
                                                          float *__restrict__ step,
                                                          uint8_t *__restrict__ zero, int vec_ok)
{
    __shared__ float s_lo[4][64], s_hi[4][64];
    __shared__ uint32_t s_codes[64][17];   // [channel][16 words of 4 tokens], odd stride
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t b = blockIdx.z, g = blockIdx.y;
    const int64_t d = (int64_t)blockIdx.x * 64 + lane;
    const bool live = d < D;
    const T *v = V + b * ld_b + g * G * ld_t + (live ? d : 0);

    float lo = 0.0f, hi = 0.0f;
    if (live) {
        // eight loads in flight per lane; tokens past the group re-read its first token
        for (int64_t t = wave; t < G; t += 32) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = to_f32(v[(t + 4 * i < G ? t + 4 * i : 0) * ld_t]);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                lo = fminf(lo, x[i]);
                hi = fmaxf(hi, x[i]);
            }
        }
    }
    s_lo[wave][lane] = lo;
    s_hi[wave][lane] = hi;
    __syncthreads();
    lo = fminf(fminf(s_lo[0][lane], s_lo[1][lane]), fminf(s_lo[2][lane], s_lo[3][lane]));
    hi = fmaxf(fmaxf(s_hi[0][lane], s_hi[1][lane]), fmaxf(s_hi[2][lane], s_hi[3][lane]));
    float st, istep;
    int z;
    range_params(lo, hi, st, istep, z);
    const int64_t ng = Tn / G;
    if (wave == 0 && live) {
        step[(b * D + d) * ng + g] = st;
        zero[(b * D + d) * ng + g] = (uint8_t)z;
    }

    const CodeRule rule = make_rule(istep, z);
    const int r = threadIdx.x >> 2, q = threadIdx.x & 3;   // write side: channel row, 16-token quarter
    const int64_t dr = (int64_t)blockIdx.x * 64 + r;
    for (int64_t c0 = 0; c0 < G; c0 += 64) {
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t t = c0 + wave * 16 + i;
            x[i] = to_f32(v[(t < G ? t : 0) * ld_t]);   // all sixteen loads issued before any is used
        }
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            uint32_t word = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t t = c0 + wave * 16 + i4 * 4 + i;
                if (live && t < G) word |= (code_byte(x[i4 * 4 + i], rule) & 0xffu) << (8 * i);
            }
            s_codes[lane][wave * 4 + i4] = word;
        }
        __syncthreads();
        if (dr < D) {
            const int64_t t0 = c0 + q * 16;
            uint8_t *dst = codes + (b * D + dr) * Tn + g * G + t0;
            const uint32_t *w = &s_codes[r][q * 4];
            if (vec_ok && t0 + 16 <= G) {
                *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            } else {
                for (int i = 0; i < 16 && t0 + i < G; ++i) dst[i] = (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
            }
        }
        __syncthreads();
    }
}

// A channel's rule as 16 bytes of LDS, and back.  (Vectors and not float4: the compiler takes that struct apart, and its four
// reads of four bytes, eight channels a stride of 128 bytes apart, cost value_quant_vec_kernel 13 % of its time.)
__device__ __forceinline__ v4f rule_entry(const CodeRule &r)
{
    return v4f{r.istep, r.lo, r.magic, __uint_as_float(r.odd)};
}
__device__ __forceinline__ CodeRule rule_of(const v4f f)
{
    CodeRule r = make_rule(f.x, 0);
    r.lo = f.y;
    r.hi = f.y + (float)DINT4_P;
    r.magic = f.z;
    r.odd = __float_as_uint(f.w);
    r.special = 14u + (r.odd & 1u);
    return r;
}
// The same for 16-bit elements with everything 16-byte aligned (D % 8 == 0, G % 128 == 0): a thread
// loads eight consecutive channels of a token at once, so a wave instruction moves eight 128-byte
// row segments instead of one (the channel-per-lane kernel above moves 128 bytes per instruction).
// Thread (c8, t4) = (tid % 8, tid / 8) owns channels 8 c8 .. + 7 and, per block of 128 tokens, the
// four tokens 4 t4 .. + 3: exactly one 32-bit word of codes per channel, which goes through LDS to
// the thread that stores the channel's row segment.
// Four codes per channel and round are too few for the rule with the folded zero-point: what it takes off and makes up per
// channel is as much as it saves, and with few workgroups more (32 heads x 5248 tokens x 128 channels 82.9 us with
// code_byte, 84.5 with codes4; 256 x 4096 in groups of 128 the same, 96.0 and 96.4).
template <typename T>
__global__ __launch_bounds__(256) void value_quant_vec_kernel(const T *__restrict__ V, int64_t Tn,
                                                              int64_t D, int64_t ld_t, int64_t ld_b,
                                                              int64_t G, uint8_t *__restrict__ codes,
                                                              float *__restrict__ step,
                                                              uint8_t *__restrict__ zero)
{
    static_assert(sizeof(T) == 2, "16-bit elements");
    __shared__ float s_lo[4][64], s_hi[4][64];
    __shared__ v4f s_rule[64];             // 1 / step, -z, p - z, z of each channel
    __shared__ uint32_t s_codes[64][33];   // [channel][32 words of 4 tokens], odd stride
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c8 = tid & 7, t4 = tid >> 3;
    const int64_t b = blockIdx.z, g = blockIdx.y;
    const int64_t d0 = (int64_t)blockIdx.x * 64;
    const bool live = d0 + c8 * 8 < D;   // D % 8 == 0: the eight channels are valid together
    const T *v = V + b * ld_b + g * G * ld_t + (live ? d0 + c8 * 8 : 0);

    // ---- ranges: min / max of every channel over the group's tokens -------------------------------
    float lo[8], hi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) lo[j] = hi[j] = 0.0f;
    for (int64_t t0 = 0; t0 < G; t0 += 128) {
        float x[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) loadv<T, 8>(v + (t0 + 4 * t4 + i) * ld_t, x[i]);
#pragma unroll
        for (int i = 0; i < 4; i += 2)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                lo[j] = fminf(fminf(lo[j], x[i][j]), x[i + 1][j]);
                hi[j] = fmaxf(fmaxf(hi[j], x[i][j]), x[i + 1][j]);
            }
    }
    // over the eight lanes of the wave with the same channels (lane bits 3..5), then over the waves
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
        for (int off = 8; off <= 32; off <<= 1) {
            lo[j] = fminf(lo[j], __shfl_xor(lo[j], off, WAVE));
            hi[j] = fmaxf(hi[j], __shfl_xor(hi[j], off, WAVE));
        }
    }
    if (lane < 8) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            s_lo[wave][lane * 8 + j] = lo[j];
            s_hi[wave][lane * 8 + j] = hi[j];
        }
    }
    __syncthreads();
    const int64_t ng = Tn / G;
    if (tid < 64) {   // one thread per channel: step, zero-point
        const float l = fminf(fminf(s_lo[0][tid], s_lo[1][tid]), fminf(s_lo[2][tid], s_lo[3][tid]));
        const float h = fmaxf(fmaxf(s_hi[0][tid], s_hi[1][tid]), fmaxf(s_hi[2][tid], s_hi[3][tid]));
        float st, istep;
        int z;
        range_params(l, h, st, istep, z);
        const CodeRule r = make_rule(istep, z);
        s_rule[tid] = v4f{r.istep, r.lo, r.hi, __int_as_float(r.z)};
        if (d0 + tid < D) {
            step[(b * D + d0 + tid) * ng + g] = st;
            zero[(b * D + d0 + tid) * ng + g] = (uint8_t)z;
        }
    }
    __syncthreads();

    // ---- codes: 128 tokens per round, transposed through LDS to token-contiguous rows ------------
    const int r = tid >> 2, q = tid & 3;   // write side: channel row, 32-token quarter
    for (int64_t t0 = 0; t0 < G; t0 += 128) {
        Raw8<T> raw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[i].load(v + (t0 + 4 * t4 + i) * ld_t);
        T e[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[i].elements(e[i]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // (the channel's rule comes from LDS each time: eight of them in registers cost the kernel
            // a wave per SIMD and 6 % of its time)
            const v4f f = s_rule[c8 * 8 + j];
            CodeRule rule = make_rule(f.x, 0);
            rule.lo = f.y;
            rule.hi = f.z;
            rule.z = __float_as_int(f.w);
            s_codes[c8 * 8 + j][t4] = pack_low_bytes(code_byte(to_f32(e[0][j]), rule), code_byte(to_f32(e[1][j]), rule),
                                                     code_byte(to_f32(e[2][j]), rule), code_byte(to_f32(e[3][j]), rule));
        }
        __syncthreads();
        if (d0 + r < D) {
            uint8_t *dst = codes + (b * D + d0 + r) * Tn + g * G + t0 + q * 32;
            const uint32_t *w = &s_codes[r][q * 8];
            *reinterpret_cast<uint4 *>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
            *reinterpret_cast<uint4 *>(dst + 16) = make_uint4(w[4], w[5], w[6], w[7]);
        }
        __syncthreads();
    }
}

// Longer groups, 16-bit elements under the same conditions: the group's values of 32 channels stay in registers
// between the range and the codes (1024 threads, 16 R registers each), so V is read once -- the kernel above sweeps
// it twice, and beyond the last-level cache's reach the second sweep comes from memory again.
// Bound by memory: 3 bytes per value.  Thread (c4, t4) = (tid % 4, tid / 4) owns channels 8 c4 .. + 7 and the tokens
// 1024 r + 4 t4 .. + 3, r < R: one word of codes per channel and r, which goes through LDS (two buffers, one barrier
// per r) to the wave that stores 1024 tokens of the channel's row, a kilobyte per instruction.  A row of 32 channels is 64 bytes,
// half a cache line: the channel parts of a head run on one XCD, so that its L2 serves the other half -- unless the codes have
// pushed it out in the meantime, so many of them are stored with the streaming hint.
// 256 heads x 4096 tokens x 128 channels, kernel trace: 126 (two sweeps) -> 112 -> 102 us (3.9 TB/s; without the vector work 93, the
// loads alone 63); calls in a graph: 115 -> 100, 256 x 2048 48 -> 44, 64 x 4096 31 -> 26.  (Blocks that go on to the next group and load it under the
// codes of the one before were no faster, and with 2048 tokens slower, as two blocks of it no longer share a CU.)
constexpr int VR_THREADS = 1024, VR_CHANNELS = 32, VR_TOKENS = 1024;
constexpr int VR_STRIDE = VR_TOKENS / 4 + 4;   // words per channel row in LDS (16-byte aligned)

// STREAM: the codes are stored with the streaming hint (launch_value_quant).  (Of both stores behind a uniform branch the compiler
// makes one without it.)
template <typename T, int R, bool STREAM>
__global__ __launch_bounds__(VR_THREADS) void value_quant_resident_kernel(const T *__restrict__ V, uint32_t groups,
                                                                          uint32_t parts, uint32_t ng, int64_t Tn,
                                                                          int64_t D, int64_t ld_t, int64_t ld_b,
                                                                          int G, uint8_t *__restrict__ codes,
                                                                          float *__restrict__ step,
                                                                          uint8_t *__restrict__ zero)
{
    static_assert(sizeof(T) == 2, "16-bit elements");
    constexpr int WAVES = VR_THREADS / WAVE;
    __shared__ float s_lo[WAVES][VR_CHANNELS], s_hi[WAVES][VR_CHANNELS];
    __shared__ v4f s_rule[VR_CHANNELS];             // each channel's rule
    __shared__ __attribute__((aligned(16))) uint32_t s_codes[R > 1 ? 2 : 1][VR_CHANNELS * VR_STRIDE];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // block -> (head and group, channel part): the parts of one follow each other on one XCD (blocks go round-robin
    // over eight)
    const uint32_t xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    const uint32_t hg = seq / parts * 8 + xcd, part = seq % parts;
    if (hg >= groups) return;   // whole block
    const int64_t b = hg / ng, g = hg % ng;
    const int64_t d0 = (int64_t)part * VR_CHANNELS;
    const int c4 = tid & 3, t4 = tid >> 2;
    const bool live = d0 + c4 * 8 < D;   // D % 8 == 0: the eight channels are valid together
    const T *v = V + b * ld_b + g * G * ld_t + (live ? d0 + c4 * 8 : 0);

    v4u raw[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int t = r * VR_TOKENS + 4 * t4;
        const T *p = v + (int64_t)(t < G ? t : 0) * ld_t;   // (past the end, G % 4 == 0: the first four tokens again)
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[r][i] = *reinterpret_cast<const v4u *>(p + i * ld_t);
    }
    auto element = [](const v4u &w, int j) {
        const uint32_t h = (j & 1) ? w[j >> 1] >> 16 : w[j >> 1] & 0xffffu;
        if constexpr (__is_same(T, bf16_t)) return bf16_t{(uint16_t)h};
        else return __ushort_as_half((uint16_t)h);
    };
    // ---- ranges: the thread's tokens, the 16 lanes of the wave with the same channels, the waves
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float lo = 0.0f, hi = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float x0 = to_f32(element(raw[r][i], j)), x1 = to_f32(element(raw[r][i + 1], j));
                lo = fminf(fminf(lo, x0), x1);
                hi = fmaxf(fmaxf(hi, x0), x1);
            }
        lo = fminf(lo, dpp_f32<DPP_ROW_ROR4>(lo));
        hi = fmaxf(hi, dpp_f32<DPP_ROW_ROR4>(hi));
        lo = fminf(lo, dpp_f32<DPP_ROW_ROR8>(lo));
        hi = fmaxf(hi, dpp_f32<DPP_ROW_ROR8>(hi));
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, off, WAVE));
            hi = fmaxf(hi, __shfl_xor(hi, off, WAVE));
        }
        if (lane < 4) {
            s_lo[wave][lane * 8 + j] = lo;
            s_hi[wave][lane * 8 + j] = hi;
        }
        __builtin_amdgcn_sched_barrier(0);   // (channel by channel: interleaved, all of them are widened at once)
    }
    __syncthreads();
    if (tid < VR_CHANNELS) {   // one thread per channel: step, zero-point
        float l = 0.0f, h = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            l = fminf(l, s_lo[w][tid]);
            h = fmaxf(h, s_hi[w][tid]);
        }
        float st, istep;
        int z;
        range_params(l, h, st, istep, z);
        const CodeRule rule = make_rule(istep, z);
        s_rule[tid] = rule_entry(rule);
        if (d0 + tid < D) {
            step[(b * D + d0 + tid) * ng + g] = st;
            zero[(b * D + d0 + tid) * ng + g] = (uint8_t)z;
        }
    }
    __syncthreads();

    // (the values are widened again below: kept widened from the ranges they would be twice the registers)
#pragma unroll
    for (int r = 0; r < R; ++r) asm volatile("" : "+v"(raw[r][0]), "+v"(raw[r][1]), "+v"(raw[r][2]), "+v"(raw[r][3]));
    // ---- codes, transposed through LDS to token-contiguous rows
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t *buf = s_codes[R > 1 ? r & 1 : 0];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const CodeRule rule = rule_of(s_rule[c4 * 8 + j]);
            buf[(c4 * 8 + j) * VR_STRIDE + t4] =
                codes4(to_f32(element(raw[r][0], j)) * rule.istep, to_f32(element(raw[r][1], j)) * rule.istep,
                       to_f32(element(raw[r][2], j)) * rule.istep, to_f32(element(raw[r][3], j)) * rule.istep, rule);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();   // (a wave that is a round ahead writes the other buffer)
        const int t = r * VR_TOKENS + lane * 16;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = wave * 2 + i;
            if (d0 + row < D && t < G) {   // G % 16 == 0
                const v4u w = *reinterpret_cast<const v4u *>(buf + row * VR_STRIDE + lane * 4);
                v4u *dst = reinterpret_cast<v4u *>(codes + (b * D + d0 + row) * Tn + g * G + t);
                if constexpr (STREAM) __builtin_nontemporal_store(w, dst);
                else *dst = w;
            }
        }
    }
}

int launch_value_quant(const void *V, int v_dtype, int64_t batch, int64_t T, int64_t D, int64_t ld_t,
                       int64_t ld_b, int64_t G, uint8_t *codes, float *step, uint8_t *zero,
                       hipStream_t st)
{
    const dim3 grid((unsigned)((D + 63) / 64), (unsigned)(T / G), (unsigned)batch);
    const int vec_ok = (uintptr_t)codes % 16 == 0 && T % 16 == 0 && G % 16 == 0;
    // 16-bit elements, every row and every store 16-byte aligned: eight channels per load
    if (v_dtype != W4A8_F32 && vec_ok && G % 128 == 0 && D % 8 == 0 && ld_t % 8 == 0 && ld_b % 8 == 0 &&
        (uintptr_t)V % 16 == 0) {
        const int64_t parts = (D + VR_CHANNELS - 1) / VR_CHANNELS, groups = batch * (T / G);
        const int64_t blocks = (groups + 7) / 8 * 8 * parts;
        const int64_t rounds = (G + VR_TOKENS - 1) / VR_TOKENS;
        // Groups that fill at least three quarters of their rounds.  Measured before the streaming stores, the two-sweep kernel / this, us
        // (256 heads of 128 channels): 1024 tokens 30.8 / 27.1, 2048 62.8 / 45.7, 4096 146 / 122 (64 heads 60 / 27, 8 heads 47 / 18); but 512
        // tokens 19.2 / 23.7, 640 21.9 / 25.0 and 1152 33.4 / 36.4.
        if (G >= VR_TOKENS && rounds <= 5 && 4 * G >= 3 * rounds * VR_TOKENS && blocks <= 0x7fffffffLL) {
            // Codes of more than 6 MB are stored with the streaming hint.  Quantizer, packing and product, us, without / with it: 8
            // heads x 1024 tokens 14.87 / 15.08, 16 x 3072 25.6 / 26.0, 48 x 1024 (6 MB) 19.15 / 19.12, 32 x 2048 (8 MB) 23.2 / 22.4,
            // 32 x 4096 40.0 / 38.2, 256 x 4096 162 / 151.
            const bool stream = batch * D * T > (6 << 20);
#define W4A8_VR_LAUNCH(T_, R_, S_)                                                                                 \
    hipLaunchKernelGGL((value_quant_resident_kernel<T_, R_, S_>), dim3((unsigned)blocks), dim3(VR_THREADS), 0, st, \
                       (const T_ *)V, (uint32_t)groups, (uint32_t)parts, (uint32_t)(T / G), T, D, ld_t, ld_b, (int)G, \
                       codes, step, zero)
#define W4A8_VR_CASE(R_)                                                         \
    case R_:                                                                     \
        if (v_dtype == W4A8_F16 && stream) W4A8_VR_LAUNCH(__half, R_, true);     \
        else if (v_dtype == W4A8_F16) W4A8_VR_LAUNCH(__half, R_, false);         \
        else if (stream) W4A8_VR_LAUNCH(bf16_t, R_, true);                       \
        else W4A8_VR_LAUNCH(bf16_t, R_, false);                                  \
        break
            switch ((int)rounds) {
                W4A8_VR_CASE(1);
                W4A8_VR_CASE(2);
                W4A8_VR_CASE(3);
                W4A8_VR_CASE(4);
                W4A8_VR_CASE(5);
            }
#undef W4A8_VR_CASE
#undef W4A8_VR_LAUNCH
            return hip_status(hipGetLastError());
        }
        if (v_dtype == W4A8_F16)
            hipLaunchKernelGGL((value_quant_vec_kernel<__half>), grid, dim3(256), 0, st, (const __half *)V, T,
                               D, ld_t, ld_b, G, codes, step, zero);
        else
            hipLaunchKernelGGL((value_quant_vec_kernel<bf16_t>), grid, dim3(256), 0, st, (const bf16_t *)V, T,
                               D, ld_t, ld_b, G, codes, step, zero);
        return hip_status(hipGetLastError());
    }
#define W4A8_VQ_LAUNCH(T_)                                                                     \
    hipLaunchKernelGGL((value_quant_kernel<T_>), grid, dim3(256), 0, st, (const T_ *)V, T, D, \
                       ld_t, ld_b, G, codes, step, zero, vec_ok)
    switch (v_dtype) {
        case W4A8_F32: W4A8_VQ_LAUNCH(float); break;
        case W4A8_F16: W4A8_VQ_LAUNCH(__half); break;
        case W4A8_BF16: W4A8_VQ_LAUNCH(bf16_t); break;
        default: return W4A8_ERR_DTYPE;
    }
#undef W4A8_VQ_LAUNCH
    return hip_status(hipGetLastError());
}

// ---- sums of the quantized weights (needed to take a token zero-point out of the product) ------
// wsum[n,b] = sum_{k in block b} d[n,k], d in half steps (Eq. 5, second half), over blocks of T
// consecutive input channels (T divides the group size G): one wave per (row, block).  Serves the
// group sizes and alignments that weight_sums_tiles_kernel does not take.
__global__ __launch_bounds__(256) void weight_block_sums_kernel(const uint8_t *__restrict__ codes,
                                                                const uint8_t *__restrict__ zero,
                                                                int64_t N, int64_t K, int64_t G,
                                                                int64_t T, int32_t *__restrict__ wsum)
{
    const int lane = threadIdx.x & 63;
    const int64_t ng = K / G, nb = K / T;
    const int64_t seg = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // (row, block)
    if (seg >= N * nb) return;
    const int64_t n = seg / nb, b = seg - n * nb;
    const int z = zero[n * ng + (b * T) / G];
    const uint8_t *c = codes + n * K + b * T;
    int sum = 0;
    for (int64_t k = lane; k < T; k += WAVE) {
        const int code = c[k] & 15;
        sum += code <= DINT4_P ? 2 * (code - z) : (code == 14 ? 1 : -1);
    }
    sum = wave_sum_i32(sum);
    if (lane == 0) wsum[seg] = sum;
}

// Sum of d over 16 codes, four per register: with n14, n15 the numbers of special codes,
//     sum d = 2 sum(code) - 32 z + n14 (2 z - 27) + n15 (2 z - 31)
// (a special code counted as an integer level gives 2 (14 - z) resp. 2 (15 - z) instead of +-1).
__device__ __forceinline__ int sum16_half_steps(const uint4 &c, int z)
{
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
    uint32_t total = 0, special = 0, odd = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t v = w[i] & 0x0f0f0f0fu;
        total = __builtin_amdgcn_udot4(v, 0x01010101u, total, false);
        const uint32_t m = (v >> 3) & (v >> 2) & (v >> 1) & 0x01010101u;   // one bit per code >= 14
        special += m;
        odd += m & v;                                                      // one bit per code 15
    }
    const int n_sp = (int)__builtin_amdgcn_udot4(special, 0x01010101u, 0, false);
    const int n15 = (int)__builtin_amdgcn_udot4(odd, 0x01010101u, 0, false);
    return 2 * (int)total - 32 * z + n_sp * (2 * z - 27) - 4 * n15;
}

// wsum [N, K/G] and tsum [N, K/128] in one pass over the codes, G a multiple of 128 and every
// 16-code chunk aligned.  Bound by the read of the codes (one byte per weight): the wave-per-block
// kernel above read them twice, two bytes per lane and instruction, at 0.6 TB/s.  Rows are contiguous, so
// group gi is codes [gi G, (gi + 1) G) and no index needs a division.  LANES lanes (16 codes each)
// take a group: 8, 16 or 32 where the group is exactly that long (several groups per wave), else a
// whole wave that walks it, SUMS_ILP loads in flight.  Eight lanes make one 128-column sum.
// 13824 x 5120, G = 128: both sums 241 -> 13.1 us (5.4 TB/s); 32768 x 4096 per channel: 313 -> 24 us (5.6 TB/s).
constexpr int SUMS_ILP = 4;

__device__ __forceinline__ int sum8_lanes(int v)
{
    v += dpp_i32<DPP_QUAD_XOR1>(v);
    v += dpp_i32<DPP_QUAD_XOR2>(v);
    return v + dpp_i32<DPP_ROW_HALF_MIRROR>(v);
}

template <int LANES>
__global__ __launch_bounds__(256) void weight_sums_tiles_kernel(const uint8_t *__restrict__ codes,
                                                                const uint8_t *__restrict__ zero,
                                                                int64_t groups, int G,
                                                                int32_t *__restrict__ wsum,
                                                                int32_t *__restrict__ tsum)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const uint4 *src = reinterpret_cast<const uint4 *>(codes);
    if constexpr (LANES < 64) {
        constexpr int PER = 64 / LANES;   // groups of one wave load
        const int64_t g0 = wave * (PER * SUMS_ILP) + lane / LANES;
        uint4 c[SUMS_ILP];
        int z[SUMS_ILP];
#pragma unroll
        for (int i = 0; i < SUMS_ILP; ++i) {
            const int64_t g = min(g0 + i * PER, groups - 1);   // (past the end: the last group again, not stored)
            c[i] = src[g * LANES + (lane & (LANES - 1))];
            z[i] = zero[g];
        }
#pragma unroll
        for (int i = 0; i < SUMS_ILP; ++i) {
            const int64_t g = g0 + i * PER;
            int v = sum8_lanes(sum16_half_steps(c[i], z[i]));
            if (tsum != nullptr && (lane & 7) == 0 && g < groups)
                tsum[g * (LANES / 8) + ((lane & (LANES - 1)) >> 3)] = v;
            if (LANES > 8) v += __shfl_xor(v, 8, WAVE);
            if (LANES > 16) v += __shfl_xor(v, 16, WAVE);
            if ((lane & (LANES - 1)) == 0 && g < groups) wsum[g] = v;
        }
    } else {
        if (wave >= groups) return;   // whole wave
        const int z = zero[wave];
        const int chunks = G / 16;
        const uint4 *row = src + wave * chunks;
        int32_t *trow = tsum != nullptr ? tsum + wave * (chunks / 8) : nullptr;
        int sum = 0;
        for (int c0 = 0; c0 < chunks; c0 += 64 * SUMS_ILP) {
            uint4 c[SUMS_ILP];
#pragma unroll
            for (int i = 0; i < SUMS_ILP; ++i) c[i] = row[min(c0 + i * 64 + lane, chunks - 1)];
#pragma unroll
            for (int i = 0; i < SUMS_ILP; ++i) {
                const int at = c0 + i * 64 + lane;   // (chunks % 8 == 0: eight lanes are in range together)
                const int v = sum8_lanes(sum16_half_steps(c[i], z));
                if ((lane & 7) == 0 && at < chunks) {
                    if (trow != nullptr) trow[at >> 3] = v;
                    sum += v;
                }
            }
        }
        sum = wave_sum_i32(sum);   // (non-zero in every eighth lane)
        if (lane == 0) wsum[wave] = sum;
    }
}

int launch_weight_sums(const uint8_t *codes, const uint8_t *zero, int64_t N, int64_t K, int64_t G,
                       int32_t *wsum, int32_t *tsum, hipStream_t st)
{
    if (G % TILE_K == 0 && G <= 0x7fffffff && (uintptr_t)codes % 16 == 0) {
        const int64_t groups = N * (K / G);
#define W4A8_WS_LAUNCH(LANES_)                                                                       \
    do {                                                                                             \
        const int64_t per = LANES_ < 64 ? 4 * (64 / LANES_) * SUMS_ILP : 4;   /* groups per block */ \
        const int64_t blocks = (groups + per - 1) / per;                                             \
        if (blocks > 0x7fffffffLL) return W4A8_ERR_SHAPE;                                            \
        hipLaunchKernelGGL((weight_sums_tiles_kernel<LANES_>), dim3((unsigned)blocks), dim3(256), 0, \
                           st, codes, zero, groups, (int)G, wsum, tsum);                             \
    } while (0)
        if (G == 128) W4A8_WS_LAUNCH(8);
        else if (G == 256) W4A8_WS_LAUNCH(16);
        else if (G == 512) W4A8_WS_LAUNCH(32);
        else W4A8_WS_LAUNCH(64);
#undef W4A8_WS_LAUNCH
        return hip_status(hipGetLastError());
    }
    const int64_t segs = N * (K / G);
    hipLaunchKernelGGL(weight_block_sums_kernel, dim3((unsigned)((segs + 3) / 4)), dim3(256), 0, st,
                       codes, zero, N, K, G, G, wsum);
    if (tsum != nullptr) {
        const int64_t tsegs = N * (K / TILE_K);
        hipLaunchKernelGGL(weight_block_sums_kernel, dim3((unsigned)((tsegs + 3) / 4)), dim3(256), 0, st,
                           codes, zero, N, K, G, (int64_t)TILE_K, tsum);
    }
    return hip_status(hipGetLastError());
}

}  // namespace w4a8
