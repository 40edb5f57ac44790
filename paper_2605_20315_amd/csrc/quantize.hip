// NVFP4 quantizer kernels for gfx950: Eq. 2 (block scale) then Eq. 1 (element codes) of
// Section 3.3, plus the amax-based tensor-level scale.
//
// The quantizer is HBM-bound: per element it reads 2 bytes (BF16) and writes 0.5 byte of
// codes and 1/16 byte of scale.  One lane owns one 16-element block: two 128-bit loads, a
// packed 16-bit integer max for the block amax (|x| of a BF16 is its low 15 bits, and for
// non-NaN values integer order equals magnitude order), two IEEE binary32 divisions per
// block, then one multiply per element and one hardware FP32->FP4 pack per element pair.
//
// Hardware conversions used, with the behaviour measured on gfx950:
//   v_cvt_pk_fp8_f32           OCP E4M3, nearest-even, gradual underflow; overflow gives the
//                              NaN byte, so the argument is clamped to 448 first (exact).
//   v_cvt_pk_f32_fp8           exact decode of all 256 bytes.
//   v_cvt_scalef32_pk_fp4_f32  nearest-even onto the E2M1 grid, clips to +-6, keeps the sign
//                              of zero; first source -> low nibble, second -> high nibble of
//                              the selected byte; only the exponent of its scale operand is
//                              used, so the scale is passed as 1.0 and the multiply by
//                              1/(alpha*sigma) is done beforehand in FP32.
#include "mq_common.h"

namespace mq {

namespace {

constexpr int kThreads = 256;

// Non-temporal: the lines take no place in the last-level cache.  A pure stream from HBM then runs at 7.0 instead of 5.9 TB/s;
// what waits in that cache is read more slowly this way (the quantizer on a [8192, 4096] tensor just written 15.3 us, through the
// cache 13.5).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream(const uint4 *p)
{
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store_stream(uint4 *p, uint4 v)
{
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
}

__device__ __forceinline__ uint32_t amax16_bits(uint4 v0, uint4 v1)
{
    const uint32_t m = 0x7FFF7FFFu;
    u16x2 a = __builtin_bit_cast(u16x2, v0.x & m);
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v0.y & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v0.z & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v0.w & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v1.x & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v1.y & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v1.z & m));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v1.w & m));
    uint32_t lo = a[0], hi = a[1];
    return lo > hi ? lo : hi;
}

// Two BF16 in one dword (element 2i low, 2i+1 high) -> one byte of two E2M1 codes written
// into byte `SEL` of `packed`.
template <int SEL>
__device__ __forceinline__ uint32_t pack_pair(uint32_t packed, uint32_t w, float r)
{
    float y0 = __uint_as_float(w << 16) * r;          // Eq. 1 argument, element 2i
    float y1 = __uint_as_float(w & 0xFFFF0000u) * r;  // element 2i+1
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(packed, y0, y1, 1.0f, SEL);
}

// Eq. 2 then Eq. 1 for one block of 16 BF16 values (v0: elements 0..7, v1: 8..15, two per dword):
// scale byte and two dwords of packed codes.  Every step IEEE binary32, nearest-even, unfused.
__device__ __forceinline__ void quantize_block16(uint4 v0, uint4 v1, float alpha, float d6, uint32_t &c0,
                                                 uint32_t &c1, int &sb)
{
    const float amax = __uint_as_float(amax16_bits(v0, v1) << 16);
    float s = amax / d6;                                     // Eq. 2 argument (IEEE division)
    s = fminf(s, 448.0f);                                    // saturation of Pi_E4M3
    sb = __builtin_amdgcn_cvt_pk_fp8_f32(s, 0.0f, 0, false) & 0xFF;  // Pi_E4M3
    const float sigma = __builtin_amdgcn_cvt_pk_f32_fp8(sb, false)[0];
    const float t = alpha * sigma;
    const float r = (sigma == 0.0f) ? 0.0f : 1.0f / t;       // IEEE division
    c0 = c1 = 0;
    c0 = pack_pair<0>(c0, v0.x, r);
    c0 = pack_pair<1>(c0, v0.y, r);
    c0 = pack_pair<2>(c0, v0.z, r);
    c0 = pack_pair<3>(c0, v0.w, r);
    c1 = pack_pair<0>(c1, v1.x, r);
    c1 = pack_pair<1>(c1, v1.y, r);
    c1 = pack_pair<2>(c1, v1.z, r);
    c1 = pack_pair<3>(c1, v1.w, r);
}

// ---- where a block's 16 BF16 values come from ---------------------------------------------------

// A source fetches what a block needs (fetch: loads only, so that a thread can have several blocks' loads in
// flight) and turns it into the 16 values (values).

// The tensor itself.  STREAM: read past the last-level cache.
template <bool STREAM>
struct TensorSrc {
    const uint16_t *x;
    int64_t ldx;
    static constexpr int kBatch = 4;  // see quantize_ktile_kernel
    static int few_groups(int64_t rows, int64_t K) { return rows % 4 ? 960 : K < 8192 ? 1100 : 4096; }  // see ktile_rows
    struct Raw {
        uint4 v[2];
    };
    __device__ __forceinline__ Raw fetch(int64_t row, int64_t col) const
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(x + row * ldx + col);
        if constexpr (STREAM) return Raw{{load_stream(src), load_stream(src + 1)}};
        return Raw{{src[0], src[1]}};
    }
    __device__ __forceinline__ void values(const Raw &raw, int64_t, int64_t, uint4 &v0, uint4 &v1) const
    {
        v0 = raw.v[0];
        v1 = raw.v[1];
    }
};

using PlainSrc = TensorSrc<false>;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)  // nearest-even, element 2i in the low half
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// The gated-MLP activation silu(gate) * up of a [rows, 2K] tensor (gate = columns [0, K), up =
// columns [K, 2K)), computed in binary32 and rounded once to BF16: the tensor an unfused
// pipeline would have stored and read back.  silu(g) = g / (1 + exp(-g)) with the hardware
// exponential (about 1 ulp: far inside half a BF16 ulp except within 1e-4 of a rounding
// boundary) and an IEEE division, which keeps the tiny quotients of strongly negative gates
// (the approximate reciprocal flushes them to zero).  Below about -88 exp(-g) overflows and the
// result is -0.  p, when not null, receives the BF16 values (checking aid).
struct SiluMulSrc {
    const uint16_t *gu;
    int64_t ld, K;
    uint16_t *p;
    int64_t ldp;
    static __device__ __forceinline__ uint32_t pair(uint32_t g, uint32_t u)
    {
        const float g0 = __uint_as_float(g << 16), g1 = __uint_as_float(g & 0xFFFF0000u);
        const float u0 = __uint_as_float(u << 16), u1 = __uint_as_float(u & 0xFFFF0000u);
        const float s0 = g0 / (1.0f + __expf(-g0));
        const float s1 = g1 / (1.0f + __expf(-g1));
        return pack_bf16(s0 * u0, s1 * u1);
    }
    static constexpr int kBatch = 1;
    static int few_groups(int64_t rows, int64_t) { return rows % 4 == 0 ? 16384 : 10240; }
    struct Raw {
        uint4 g[2], u[2];
    };
    __device__ __forceinline__ Raw fetch(int64_t row, int64_t col) const
    {
        const uint4 *gs = reinterpret_cast<const uint4 *>(gu + row * ld + col);
        const uint4 *us = reinterpret_cast<const uint4 *>(gu + row * ld + K + col);
        return Raw{{gs[0], gs[1]}, {us[0], us[1]}};
    }
    __device__ __forceinline__ void values(const Raw &r, int64_t row, int64_t col, uint4 &v0, uint4 &v1) const
    {
        const uint4 g0 = r.g[0], g1 = r.g[1], u0 = r.u[0], u1 = r.u[1];
        v0 = make_uint4(pair(g0.x, u0.x), pair(g0.y, u0.y), pair(g0.z, u0.z), pair(g0.w, u0.w));
        v1 = make_uint4(pair(g1.x, u1.x), pair(g1.y, u1.y), pair(g1.z, u1.z), pair(g1.w, u1.w));
        if (p) {
            uint4 *dst = reinterpret_cast<uint4 *>(p + row * ldp + col);
            dst[0] = v0;
            dst[1] = v1;
        }
    }
};

// One lane per 16-element block, canonical (linear) output.
template <class Src>
__global__ __launch_bounds__(kThreads) void quantize_kernel(Src src, int64_t total_blocks, int blocks_per_row,
                                                            const float *__restrict__ alpha_p,
                                                            uint8_t *__restrict__ codes,
                                                            uint8_t *__restrict__ scales)
{
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= total_blocks) return;
    const float alpha = *alpha_p;
    const float d6 = 6.0f * alpha;  // alpha * q_max
    const int64_t row = g / blocks_per_row;
    const int64_t b = g - row * blocks_per_row;
    uint4 v0, v1;
    src.values(src.fetch(row, b * kBlock), row, b * kBlock, v0, v1);
    uint32_t c0, c1;
    int sb;
    quantize_block16(v0, v1, alpha, d6, c0, c1, sb);
    reinterpret_cast<uint2 *>(codes)[g] = make_uint2(c0, c1);  // dense [rows, K/2]: 8 bytes per block
    scales[g] = (uint8_t)sb;                                   // dense [rows, K/16]
}

// K-step-major output: the code and scale bytes of one 64-wide K step are contiguous over rows.
// A workgroup covers ROWS rows x 16 K steps.  Reading: each wave takes ROWS / 4 of the rows, 2 KB
// contiguous per row (lane l: K step l/4, block l%4).  The codes and scale bytes go through LDS so that
// writing is contiguous too: per K step ROWS x 32 code bytes and ROWS x 4 scale bytes.
// HBM-bound for large tensors, bound by one trip to memory for small ones.  ROWS = 4, one row per wave: every
// wave waits for memory once and there are four times as many of them.  ROWS = 16: 512 instead of 128
// contiguous bytes per K step; the waves' rows are then loaded Src::kBatch at a time (all four of
// silu_mul's cost more in registers than they hide).  Which: ktile_rows.
constexpr int kt_stride(int rows) { return rows * 4 + 4; }  // uint2 units per K step in LDS, padded against bank conflicts

// Second half of the transposition: thread `u` < 16 ROWS (K step u / ROWS, row u % ROWS) writes one unit of 32 + 4 bytes.
template <int ROWS>
__device__ __forceinline__ void write_ktile_unit(const uint2 *lc, const uint8_t (*ls)[ROWS][4], int u, int t0, int64_t r0,
                                                 int ksteps, int64_t rows, uint8_t *codes, uint8_t *scales)
{
    const int ot = u / ROWS, orow = u % ROWS;
    if (t0 + ot < ksteps && r0 + orow < rows) {
        const int64_t slot = (int64_t)(t0 + ot) * rows + r0 + orow;
        const uint2 *p = &lc[ot * kt_stride(ROWS) + orow * 4];
        reinterpret_cast<uint4 *>(codes)[slot * 2] = make_uint4(p[0].x, p[0].y, p[1].x, p[1].y);
        reinterpret_cast<uint4 *>(codes)[slot * 2 + 1] = make_uint4(p[2].x, p[2].y, p[3].x, p[3].y);
        reinterpret_cast<uint32_t *>(scales)[slot] = *reinterpret_cast<const uint32_t *>(&ls[ot][orow][0]);
    }
}

template <int ROWS, class Src>
__global__ __launch_bounds__(kThreads) void quantize_ktile_kernel(Src src, int64_t rows, int64_t row_base,
                                                                  int ksteps, const float *__restrict__ alpha_p,
                                                                  uint8_t *__restrict__ codes,
                                                                  uint8_t *__restrict__ scales)
{
    constexpr int RPW = ROWS / 4;                    // rows per wave
    __shared__ uint2 lc[16 * kt_stride(ROWS)];       // [K step][row][block]
    __shared__ uint8_t ls[16][ROWS][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t0 = blockIdx.x * 16;
    const int64_t r0 = row_base + (int64_t)blockIdx.y * ROWS;
    const int tl = lane >> 2, blk = lane & 3;
    const int t = t0 + tl < ksteps ? t0 + tl : ksteps - 1;  // clamped: loaded, not stored
    const int64_t col = (int64_t)t * 64 + blk * kBlock;
    const float alpha = *alpha_p;
    const float d6 = 6.0f * alpha;
    constexpr int BATCH = RPW < Src::kBatch ? RPW : Src::kBatch;
#pragma unroll
    for (int it0 = 0; it0 < RPW; it0 += BATCH) {
        typename Src::Raw raw[BATCH];
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const int64_t row = r0 + wave * RPW + it0 + it;
            raw[it] = src.fetch(row < rows ? row : rows - 1, col);
        }
#pragma unroll
        for (int it = 0; it < BATCH; ++it) {
            const int rl = wave * RPW + it0 + it;
            const int64_t row = r0 + rl;
            if (row < rows && t0 + tl < ksteps) {
                uint4 v0, v1;
                src.values(raw[it], row, col, v0, v1);
                uint32_t c0, c1;
                int sb;
                quantize_block16(v0, v1, alpha, d6, c0, c1, sb);
                lc[tl * kt_stride(ROWS) + rl * 4 + blk] = make_uint2(c0, c1);
                ls[tl][rl][blk] = (uint8_t)sb;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < 16 * ROWS)
        write_ktile_unit<ROWS>(lc, ls, threadIdx.x, t0, r0, ksteps, rows, codes, scales);
}

// ---- RMS normalisation fused with the quantizer ----------------------------------------------

// y[r, k] = x[r, k] / sqrt(mean_k x[r, :]^2 + eps) * w[k] in binary32 (sum of squares: each lane
// adds its elements in ascending k, then a butterfly over the wave), rounded once to BF16, then
// quantized as above.  A workgroup of ROWS waves owns ROWS rows and all of K, one wave per row, so a
// row's sum is a reduction over one wave.  Lane l takes K step c*16 + l/4, block l%4 of chunk c
// (16 K steps = 1024 columns), as in the K-step-major quantizer.
// NC > 0: the row (NC chunks: 8 registers each) stays in registers between the two passes, so x
// is read once; NC == 0: any K, x is read again in the second pass (from cache).
// y_out, when not null, receives the BF16 values (checking aid).
template <int ROWS, int NC, bool KTILE_OUT>
__global__ __launch_bounds__(64 * ROWS) void rmsnorm_quantize_kernel(const uint16_t *__restrict__ x, int64_t rows,
                                                                       int ksteps, int64_t ldx,
                                                                       const uint16_t *__restrict__ w, float eps,
                                                                       float inv_k,
                                                                       const float *__restrict__ alpha_p,
                                                                       uint8_t *__restrict__ codes,
                                                                       uint8_t *__restrict__ scales,
                                                                       uint16_t *__restrict__ y_out, int64_t ldy)
{
    constexpr int NCR = NC > 0 ? NC : 1;
    // K-step-major output: NC > 0 stages all chunks and synchronises once, NC == 0 chunk by chunk
    __shared__ uint2 lc[KTILE_OUT ? NCR : 1][16 * kt_stride(ROWS)];
    __shared__ uint8_t ls[KTILE_OUT ? NCR : 1][16][ROWS][4];
    constexpr int UNITS = 16 * ROWS;  // units of 32 + 4 bytes per chunk
    const int lane = threadIdx.x & 63, rl = threadIdx.x >> 6;  // rl: row within the group = wave
    const int64_t r0 = (int64_t)blockIdx.x * ROWS, row = r0 + rl;
    const bool row_ok = row < rows;
    const float alpha = *alpha_p;
    const float d6 = 6.0f * alpha;
    const int tl = lane >> 2, blk = lane & 3;
    const int chunks = (ksteps + 15) / 16;
    const PlainSrc src{x, ldx};

    auto sumsq = [](uint4 v0, uint4 v1) {
        const uint32_t d[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = __uint_as_float(d[i] << 16), b = __uint_as_float(d[i] & 0xFFFF0000u);
            s += a * a;
            s += b * b;
        }
        return s;
    };
    uint4 keep[NCR][2];
    float ss = 0.0f;
    if constexpr (NC > 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int t = c * 16 + tl;
            uint4 v0 = make_uint4(0, 0, 0, 0), v1 = v0;
            if (row_ok && t < ksteps) {
                const PlainSrc::Raw raw = src.fetch(row, (int64_t)t * 64 + blk * kBlock);
                v0 = raw.v[0], v1 = raw.v[1];
            }
            keep[c][0] = v0;
            keep[c][1] = v1;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) ss += sumsq(keep[c][0], keep[c][1]);
    } else {
        for (int c = 0; c < chunks; ++c) {
            const int t = c * 16 + tl;
            if (row_ok && t < ksteps) {
                const PlainSrc::Raw raw = src.fetch(row, (int64_t)t * 64 + blk * kBlock);
                ss += sumsq(raw.v[0], raw.v[1]);
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    // IEEE square root and division, once per row (the approximate reciprocal square root moved
    // two orders of magnitude more elements across a BF16 rounding boundary than these do)
    const float iv = 1.0f / __fsqrt_rn(ss * inv_k + eps);

    auto norm_pair = [](uint32_t xv, uint32_t wv, float inv) {
        const float a = __uint_as_float(xv << 16) * inv, b = __uint_as_float(xv & 0xFFFF0000u) * inv;
        return pack_bf16(a * __uint_as_float(wv << 16), b * __uint_as_float(wv & 0xFFFF0000u));
    };
    auto chunk = [&](int c, uint4 x0, uint4 x1) {
        const int t = c * 16 + tl;
        if (row_ok && t < ksteps) {
            const uint4 *ws = reinterpret_cast<const uint4 *>(w + (int64_t)t * 64 + blk * kBlock);
            const uint4 w0 = ws[0], w1 = ws[1];
            const uint4 v0 = make_uint4(norm_pair(x0.x, w0.x, iv), norm_pair(x0.y, w0.y, iv),
                                        norm_pair(x0.z, w0.z, iv), norm_pair(x0.w, w0.w, iv));
            const uint4 v1 = make_uint4(norm_pair(x1.x, w1.x, iv), norm_pair(x1.y, w1.y, iv),
                                        norm_pair(x1.z, w1.z, iv), norm_pair(x1.w, w1.w, iv));
            if (y_out) {
                uint4 *dst = reinterpret_cast<uint4 *>(y_out + row * ldy + (int64_t)t * 64 + blk * kBlock);
                dst[0] = v0;
                dst[1] = v1;
            }
            uint32_t c0, c1;
            int sb;
            quantize_block16(v0, v1, alpha, d6, c0, c1, sb);
            if constexpr (KTILE_OUT) {
                const int slot = NC > 0 ? c : 0;
                lc[slot][tl * kt_stride(ROWS) + rl * 4 + blk] = make_uint2(c0, c1);
                ls[slot][tl][rl][blk] = (uint8_t)sb;
            } else {
                const int64_t g = row * ((int64_t)ksteps * 4) + (int64_t)t * 4 + blk;
                reinterpret_cast<uint2 *>(codes)[g] = make_uint2(c0, c1);
                scales[g] = (uint8_t)sb;
            }
        }
        if constexpr (KTILE_OUT && NC == 0) {
            __syncthreads();
            if (threadIdx.x < UNITS)
                write_ktile_unit<ROWS>(lc[0], ls[0], threadIdx.x, c * 16, r0, ksteps, rows, codes, scales);
            __syncthreads();
        }
    };
    if constexpr (NC > 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c < chunks) chunk(c, keep[c][0], keep[c][1]);  // uniform
        if constexpr (KTILE_OUT) {
            __syncthreads();
#pragma unroll
            for (int c = (int)(threadIdx.x / UNITS); c < NC; c += 64 * ROWS / UNITS)
                if (c < chunks)
                    write_ktile_unit<ROWS>(lc[c], ls[c], threadIdx.x % UNITS, c * 16, r0, ksteps, rows, codes, scales);
        }
    } else {
        for (int c = 0; c < chunks; ++c) {
            const int t = c * 16 + tl;
            uint4 x0 = make_uint4(0, 0, 0, 0), x1 = x0;
            if (row_ok && t < ksteps) {
                const PlainSrc::Raw raw = src.fetch(row, (int64_t)t * 64 + blk * kBlock);
                x0 = raw.v[0], x1 = raw.v[1];
            }
            chunk(c, x0, x1);
        }
    }
}

// Byte permutation between the two layouts of an NVFP4 tensor (offline weight pre-pack), HBM-bound: reads
// and writes 0.5625 bytes per element.  A workgroup moves 32 rows x 16 K steps through LDS, so that both
// sides see whole cache lines: 512 contiguous code bytes per row in the row-major order, 1 KB per K step
// in the K-step-major one: [28672, 4096] 32 us (4.2 TB/s) in either direction, against 40 us to the K-step-major
// order and 54 us from it with one thread per 32-byte unit, which touched a line per lane on one side.
// STREAM_OUT: codes are written past the last-level cache, which leaves its room to what is read again, wherever every line of the
// destination is written whole, by one workgroup: 0.70 to 1.0 of the time, cached or not (of quantize and convert together 0.91 to 0.95;
// [6144, 4096] in the same two buffers 5.4 -> 4.4 us).  Lines written in parts cost up to 1.08 ([5121, 12864] 15.3 -> 16.6 us).
// STREAM_IN: they are read past it too where no line is shared by two workgroups, which would fetch it twice ([5120, 3200], rows of 12.5
// lines, behind the quantizer 14.0 -> 14.7 us), and only from kStreamIn units on: smaller tensors may be waiting in the L2 caches,
// the same two buffers of 11 to 18 MB then take 1.05 to 1.19 of the time; from 19.7 MB on 0.80 to 0.93, from HBM 0.69 to 0.76, quantize and
// convert 0.88 ([28672, 4096] 80 -> 70 us).  (At 63 and 70 MB the same two buffers again and again, and nothing else, 0.97 to 1.06.)
// LDS rows hold 32 chunks of 16 bytes plus two: the reads of 8 rows x 2 halves of a K step then fall on
// different banks.
constexpr int R_ROWS = 32, R_STEPS = 16, R_CHUNKS = 2 * R_STEPS, R_STRIDE = R_CHUNKS + 2;
constexpr int64_t kStreamIn = 17 << 15;  // of 36 bytes: 19.1 MB

template <bool TO_KTILE, bool STREAM_IN, bool STREAM_OUT>
__global__ __launch_bounds__(kThreads) void relayout_kernel(const uint8_t *__restrict__ src_c,
                                                            const uint8_t *__restrict__ src_s,
                                                            uint8_t *__restrict__ dst_c, uint8_t *__restrict__ dst_s,
                                                            int64_t rows, int64_t row_base, int64_t row_stride,
                                                            int ksteps, int groups)
{
    __shared__ uint4 lc[R_ROWS * R_STRIDE];
    __shared__ uint32_t ls[R_ROWS * (R_STEPS + 1)];
    const int64_t r0 = row_base + (int64_t)(blockIdx.x / groups) * R_ROWS;
    const int t0 = (int)(blockIdx.x % groups) * R_STEPS;
    // item i of a side: row-major order (row, chunk of 16 bytes); K-step-major order (K step, row, half)
    auto lin = [](int i, int &row, int &chunk) { row = i / R_CHUNKS, chunk = i % R_CHUNKS; };
    auto kt = [](int i, int &row, int &chunk) {
        row = (i / 2) % R_ROWS, chunk = i / (2 * R_ROWS) * 2 + i % 2;
    };
    auto inside = [&](int row, int t) { return r0 + row < rows && t0 + t < ksteps; };
    auto lin_at = [&](int row, int t) { return (r0 + row) * row_stride + t0 + t; };   // unit (row, K step)
    auto kt_at = [&](int row, int t) { return (int64_t)(t0 + t) * rows + r0 + row; };
    auto get = [](const uint4 *p) { return STREAM_IN ? load_stream(p) : *p; };
    auto put = [](uint4 *p, uint4 v) { STREAM_OUT ? store_stream(p, v) : (void)(*p = v); };
#pragma unroll
    for (int j = 0; j < R_ROWS * R_CHUNKS / kThreads; ++j) {
        int row, chunk;
        TO_KTILE ? lin(j * kThreads + threadIdx.x, row, chunk) : kt(j * kThreads + threadIdx.x, row, chunk);
        if (inside(row, chunk / 2))
            lc[row * R_STRIDE + chunk] = get(reinterpret_cast<const uint4 *>(src_c) +
                                             (TO_KTILE ? lin_at(row, chunk / 2) : kt_at(row, chunk / 2)) * 2 + chunk % 2);
    }
#pragma unroll
    for (int j = 0; j < R_ROWS * R_STEPS / kThreads; ++j) {
        const int i = j * kThreads + threadIdx.x;
        const int row = TO_KTILE ? i / R_STEPS : i % R_ROWS, t = TO_KTILE ? i % R_STEPS : i / R_ROWS;
        if (inside(row, t))
            ls[row * (R_STEPS + 1) + t] =
                reinterpret_cast<const uint32_t *>(src_s)[TO_KTILE ? lin_at(row, t) : kt_at(row, t)];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < R_ROWS * R_CHUNKS / kThreads; ++j) {
        int row, chunk;
        TO_KTILE ? kt(j * kThreads + threadIdx.x, row, chunk) : lin(j * kThreads + threadIdx.x, row, chunk);
        if (inside(row, chunk / 2))
            put(reinterpret_cast<uint4 *>(dst_c) + (TO_KTILE ? kt_at(row, chunk / 2) : lin_at(row, chunk / 2)) * 2 + chunk % 2,
                lc[row * R_STRIDE + chunk]);
    }
#pragma unroll
    for (int j = 0; j < R_ROWS * R_STEPS / kThreads; ++j) {
        const int i = j * kThreads + threadIdx.x;
        const int row = TO_KTILE ? i % R_ROWS : i / R_STEPS, t = TO_KTILE ? i / R_ROWS : i % R_STEPS;
        if (inside(row, t))
            reinterpret_cast<uint32_t *>(dst_s)[TO_KTILE ? kt_at(row, t) : lin_at(row, t)] = ls[row * (R_STEPS + 1) + t];
    }
}

// The same permutation, one thread per (row, K step) unit of 32 + 4 bytes, for tensors that the tiles above serve
// badly: fewer than four K steps leave most of a tile empty ([262144, 64] 6.2 us here, 11.6 and 14.2 in tiles;
// [262144, 128] 14.0 / 10.9 against 15.0 / 21.1), and small ones are over before a tile has been through LDS
// ([4096, 1024] 4.1 against 5.0, [8192, 512] 4.0 against 5.1; to the K-step-major order also [16384, 512] 4.9
// against 5.7, but [16384, 1024] 7.0 against 6.6; from it [16384, 512] 5.3 against 4.9).
template <bool TO_KTILE>
__global__ __launch_bounds__(kThreads) void relayout_units_kernel(const uint8_t *__restrict__ src_c,
                                                                  const uint8_t *__restrict__ src_s,
                                                                  uint8_t *__restrict__ dst_c,
                                                                  uint8_t *__restrict__ dst_s, uint32_t rows,
                                                                  uint32_t ksteps, uint32_t units)
{
    const uint32_t u = blockIdx.x * kThreads + threadIdx.x;  // K-step-major unit
    if (u >= units) return;
    const uint32_t t = u / rows, r = u - t * rows;
    const size_t lin = r * ksteps + t, from = TO_KTILE ? lin : u, to = TO_KTILE ? u : lin;
    const uint4 c0 = reinterpret_cast<const uint4 *>(src_c)[from * 2], c1 = reinterpret_cast<const uint4 *>(src_c)[from * 2 + 1];
    const uint32_t sc = reinterpret_cast<const uint32_t *>(src_s)[from];
    reinterpret_cast<uint4 *>(dst_c)[to * 2] = c0;
    reinterpret_cast<uint4 *>(dst_c)[to * 2 + 1] = c1;
    reinterpret_cast<uint32_t *>(dst_s)[to] = sc;
}

// ---- tensor-level scale ------------------------------------------------------------------

__global__ void amax_init_kernel(uint32_t *acc) { *acc = 0u; }

__device__ __forceinline__ uint32_t amax8_bits(uint4 v)
{
    const uint32_t k = 0x7FFF7FFFu;
    u16x2 a = __builtin_bit_cast(u16x2, v.x & k);
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v.y & k));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v.z & k));
    a = __builtin_elementwise_max(a, __builtin_bit_cast(u16x2, v.w & k));
    uint32_t lo = a[0], hi = a[1];
    return lo > hi ? lo : hi;
}

__device__ __forceinline__ float alpha_of(uint32_t amax_bits)  // from the largest |x| as BF16 bits
{
    const float amax = __uint_as_float(amax_bits << 16);
    return amax == 0.0f ? 1.0f : amax / 2688.0f;
}

// Largest |x| of the tensor, into the caller's word `acc`, which is all the memory there is.  At
// most one workgroup of 1024 threads per compute unit, each reading one contiguous share of the
// tensor with four 16-byte loads in flight per thread: atomics on a single address serialise in
// L2, and with 2048 workgroups they cost more than the read itself (measured on [8192, 4096]:
// 30.7 us with 2048 atomics, 13.4 us for the same reads without any, 14.5 us with 256).
// One workgroup (COUNT) writes alpha itself.  Several start from a word that amax_init_kernel has cleared.  COUNT: the word holds the
// largest |x| as BF16 bits in its high half and the number of workgroups accounted for in the low half: a workgroup first
// raises the maximum to its own, which wipes the count it gets back where its own is larger, then adds itself and what it wiped.
// No workgroup is counted before its maximum is in and none is lost, so the one that completes the count holds the
// maximum of all of them and overwrites the word with alpha.  Without COUNT the word holds the BF16 bits, and
// amax_final_kernel does that in a launch of its own.  Counting is two trips to the word in a row behind the last load, and
// they queue with those of the other workgroups; the launch is worth about a hundred of them.  us per call replayed from a
// graph, counted / own launch: 64 KB (one workgroup) 2.5 / 5.5, 256 KB (one) 4.2 / 6.2, 1 MB 5.4 / 6.1, 4 MB 6.2 / 6.7, 6 MB
// (96 workgroups) 7.3 / 7.4; 8 MB 8.1 / 7.8, 12 MB 10.2 / 9.2, 16 MB 12.1 / 10.3.  (A look at the word in front of the first trip,
// which spares the workgroups with a smaller maximum that trip, took 0.4 us more at every size.)
// CONTIG: ldx == K.
constexpr int kAmaxThreads = 1024;
constexpr int64_t kAmaxOne = 4, kAmaxCounted = 96;  // most workgroups of 64 KB served by one, and that count themselves

template <bool CONTIG, bool COUNT>
__global__ __launch_bounds__(kAmaxThreads) void amax_kernel(const uint16_t *__restrict__ x, int64_t total_chunks,
                                                            int chunks_per_row, int64_t ldx, uint32_t *acc)
{
    const int64_t per = (total_chunks + gridDim.x - 1) / gridDim.x;
    const int64_t b0 = (int64_t)blockIdx.x * per, b1 = b0 + per < total_chunks ? b0 + per : total_chunks;
    uint32_t m = 0;
    auto addr = [&](int64_t c) -> const uint4 * {
        if (CONTIG) return reinterpret_cast<const uint4 *>(x) + c;
        const int64_t row = c / chunks_per_row;
        return reinterpret_cast<const uint4 *>(x + row * ldx) + (c - row * chunks_per_row);
    };
    constexpr int64_t T = kAmaxThreads;
    int64_t c = b0 + threadIdx.x;
    for (; c + 3 * T < b1; c += 4 * T) {
        const uint4 v0 = *addr(c), v1 = *addr(c + T), v2 = *addr(c + 2 * T), v3 = *addr(c + 3 * T);
        uint32_t t0 = amax8_bits(v0), t1 = amax8_bits(v1), t2 = amax8_bits(v2), t3 = amax8_bits(v3);
        t0 = t0 > t1 ? t0 : t1;
        t2 = t2 > t3 ? t2 : t3;
        t0 = t0 > t2 ? t0 : t2;
        m = m > t0 ? m : t0;
    }
    for (; c < b1; c += T) {
        const uint32_t t = amax8_bits(*addr(c));
        m = m > t ? m : t;
    }
    for (int off = 32; off > 0; off >>= 1) {
        uint32_t o = __shfl_xor(m, off);
        m = o > m ? o : m;
    }
    __shared__ uint32_t wave_max[kAmaxThreads / 64];
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kAmaxThreads / 64; ++w) m = wave_max[w] > m ? wave_max[w] : m;
        if constexpr (!COUNT) {
            if (m != 0) atomicMax(acc, m);
            return;
        }
        if (gridDim.x == 1) {
            *acc = __float_as_uint(alpha_of(m));
            return;
        }
        const uint32_t old = __hip_atomic_fetch_max(acc, m << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t add = 1 + (m > old >> 16 ? old & 0xFFFFu : 0u);
        const uint32_t now = __hip_atomic_fetch_add(acc, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
        if ((now & 0xFFFFu) == gridDim.x)
            __hip_atomic_store(acc, __float_as_uint(alpha_of(now >> 16)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void amax_final_kernel(uint32_t *acc) { *acc = __float_as_uint(alpha_of(*acc)); }

}  // namespace

namespace {

// Rows per workgroup of quantize_ktile_kernel, by the number of workgroups of sixteen.  us with four rows against
// sixteen, inputs from HBM:
//   plain, K = 4096: [64] 3.8 / 4.5, [2048] 6.3 / 7.7, [3584] 8.4 / 9.5, [4096] 10.0 / 10.4, [5120] 12.9 / 12.6, [8192]
//     18.7 / 17.7, [65536] 138 / 127; K = 5120: ragged [2861] 9.4 / 9.9, [3261] 11.4 / 10.9, [4096] 14.1 / 13.0: sixteen from a
//     thousand workgroups, which fill the chip's wave slots.  A long K with whole lines written by four rows
//     (rows % 4 == 0): [1456, 14336] 12.3 / 13.4, [2336, 14336] 17.4 / 17.9, [4672, 14336] 31.8 / 32.7, [2608, 25600] 31.8 / 32.5,
//     [6848, 14336] 46.2 / 46.1, [8192, 14336] 54.1 / 56.0, [10480, 25600] 138 / 135; ragged [3421, 14336] 25.9 / 24.9.
//   silu_mul, K = 14336: [64] 4.3 / 7.6, [1024] 15.6 / 19.0, [8000] 108 / 113, [18720] 247 / 254; rows % 4 != 0 (the 128 bytes
//     of four rows are then no whole line): [9133] 134.0 / 134.7, [18269] 270 / 261; K = 25600: [7677] 204 / 199.
template <class Src>
int ktile_rows(int64_t rows, int64_t K)
{
    const int64_t groups = (K / 64 + 15) / 16 * ((rows + 15) / 16);
    return groups < Src::few_groups(rows, K) ? 4 : 16;
}

template <class Src>
int launch_quantize_from(const Src &src, int64_t rows, int64_t K, const float *alpha, uint8_t *codes,
                         uint8_t *scales, int layout, hipStream_t s)
{
    const int64_t bpr = K / kBlock;
    const int64_t total = rows * bpr;
    if (total == 0) return MQ_OK;
    if (layout == MQ_LAYOUT_KTILE) {
        const int64_t ksteps = K / 64, gx = (ksteps + 15) / 16;
        const int per = ktile_rows<Src>(rows, K);
        const int64_t gy = (rows + per - 1) / per;
        // grid.y is limited to 65535: fold the excess row groups into extra launches
        for (int64_t y0 = 0; y0 < gy; y0 += 65535) {
            const int64_t ny = gy - y0 < 65535 ? gy - y0 : 65535;
            const dim3 grid((unsigned)gx, (unsigned)ny);
            const int rc = enqueue(per == 16 ? quantize_ktile_kernel<16, Src> : quantize_ktile_kernel<4, Src>, grid, dim3(kThreads), 0, s,
                                   src, rows, y0 * per, (int)ksteps, alpha, codes, scales);
            if (rc != MQ_OK) return rc;
        }
        return MQ_OK;
    }
    const int64_t grid = (total + kThreads - 1) / kThreads;
    if (grid > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    return enqueue(quantize_kernel<Src>, dim3((unsigned)grid), dim3(kThreads), 0, s, src, total, (int)bpr, alpha, codes, scales);
}

}  // namespace

// Row-major quantizer of more than the 256 MB that the last-level cache holds: no whole such tensor can be waiting there, and
// what the pass reads would only displace the codes that the next one wants.  Streamed / through the cache, 266 to 500 MB: alone 0.96 to
// 0.99 of the time, behind the scale pass of the same tensor 0.96, with the conversion behind it 0.95 to 0.97, of a tensor just written 0.89 to
// 0.93.  (Scale and quantizer again and again on one unchanged tensor and nothing else between: 1.02 to 1.12.)  Below, the tensor may
// have just been written: [8192, 4096] then takes 13.5 us, streamed 15.3.
static constexpr int64_t kStreamBytes = 256ll << 20;

int launch_quantize(const uint16_t *x, int64_t rows, int64_t K, int64_t ldx, const float *alpha,
                    uint8_t *codes, uint8_t *scales, int layout, hipStream_t s)
{
    if (layout == MQ_LAYOUT_LINEAR && rows > kStreamBytes / 2 / K)
        return launch_quantize_from(TensorSrc<true>{x, ldx}, rows, K, alpha, codes, scales, layout, s);
    return launch_quantize_from(PlainSrc{x, ldx}, rows, K, alpha, codes, scales, layout, s);
}

int launch_quantize_silu_mul(const uint16_t *gate_up, int64_t rows, int64_t K, int64_t ld, const float *alpha,
                             uint8_t *codes, uint8_t *scales, int layout, uint16_t *p, int64_t ldp, hipStream_t s)
{
    return launch_quantize_from(SiluMulSrc{gate_up, ld, K, p, ldp}, rows, K, alpha, codes, scales, layout, s);
}

// Rows per workgroup of rmsnorm_quantize_kernel.  Four: more workgroups (63 of 16 rows left three quarters of the
// chip idle at 1000 tokens), and registers for longer rows.  us, four rows against sixteen: K = 4096 (the row in 32
// registers per lane either way) [64] 4.5 / 7.4, [1000] 6.0 / 8.6, [4096] 13.6 / 13.5, [65536] 147 / 162; K = 5120
// (64 registers against reading x twice) [1000] 7.4 / 12.3, row-major [8192] 28.2 / 32.4, [65536] 18 % faster, but
// K-step-major, where four rows write 128 bytes per K step and sixteen 512: [6000] 26.9 / 29.1, [8192] 34.1 / 33.1,
// [12000] 1.5 % slower, [65536] 5 % slower, and K = 4160 [8192] 32.2 / 29.1; K = 6144 and 8192 6 to 25 % faster up to
// 32768 rows; K = 14336 (128 registers) [1000] 17.5 / 31.7, [4096] 66 / 47.
static int rmsnorm_rows(int64_t rows, int ksteps, bool ktile)
{
    if (ksteps > 128) return ksteps <= 256 && rows <= 1024 ? 4 : 16;
    return ktile && ksteps > 64 && ksteps < 96 && rows > 6144 ? 16 : 4;
}

int describe_quantize(int source, int64_t rows, int64_t K)
{
    return source == 0   ? ktile_rows<PlainSrc>(rows, K)
           : source == 1 ? ktile_rows<SiluMulSrc>(rows, K)
                         : rmsnorm_rows(rows, (int)(K / 64), true);
}

int launch_quantize_rmsnorm(const uint16_t *x, int64_t rows, int64_t K, int64_t ldx, const uint16_t *w, float eps,
                            const float *alpha, uint8_t *codes, uint8_t *scales, int layout, uint16_t *y,
                            int64_t ldy, hipStream_t s)
{
    if (rows == 0) return MQ_OK;
    const int ksteps = (int)(K / 64);
    const float inv_k = 1.0f / (float)K;
    const bool kt = layout == MQ_LAYOUT_KTILE;
    const int per = rmsnorm_rows(rows, ksteps, kt);
    const bool few = per == 4;
    const int64_t groups = (rows + per - 1) / per;
    if (groups > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    const dim3 grid((unsigned)groups), block(64 * per);
#define MQ_RMS(ROWS_, NC_) \
    enqueue(kt ? rmsnorm_quantize_kernel<ROWS_, NC_, true> : rmsnorm_quantize_kernel<ROWS_, NC_, false>, grid, block, 0, s, \
            x, rows, ksteps, ldx, w, eps, inv_k, alpha, codes, scales, y, ldy)
    if (few && ksteps <= 64) return MQ_RMS(4, 4);
    if (few && ksteps <= 128) return MQ_RMS(4, 8);
    if (few) return MQ_RMS(4, 16);
    return MQ_RMS(16, 0);
#undef MQ_RMS
}

int launch_relayout(const uint8_t *src_c, const uint8_t *src_s, uint8_t *dst_c, uint8_t *dst_s, int64_t rows,
                    int64_t K, bool to_ktile, hipStream_t s)
{
    const int64_t ksteps = K / 64;
    if (rows == 0 || ksteps == 0) return MQ_OK;
    if (rows * ksteps > (int64_t)0x7FFFFFFF * kThreads) return MQ_ERR_SHAPE;
    const int64_t units = rows * ksteps;
    if ((ksteps < 4 && units < (1ll << 31)) || units < (to_ktile ? 3 << 16 : 1 << 17)) {
        auto kern = to_ktile ? relayout_units_kernel<true> : relayout_units_kernel<false>;
        return enqueue(kern, dim3((unsigned)((units + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, src_c, src_s, dst_c, dst_s,
                       (uint32_t)rows, (uint32_t)ksteps, (uint32_t)units);
    }
    const bool whole_lin = K % 256 == 0, whole_kt = rows % 4 == 0;  // every row's or K step's codes are whole lines
    const bool out = (to_ktile ? whole_kt : whole_lin) && reinterpret_cast<uintptr_t>(dst_c) % 128 == 0;
    const bool in = out && units >= kStreamIn && whole_lin && whole_kt && reinterpret_cast<uintptr_t>(src_c) % 128 == 0;
    const int64_t groups = (ksteps + R_STEPS - 1) / R_STEPS, panels = (rows + R_ROWS - 1) / R_ROWS;
    // a launch holds fewer than 2^32 threads: what is more goes into further launches, by rows and, where one panel
    // of rows has more workgroups than that (K beyond 1.7e10), by K steps
    constexpr int64_t max_wgs = (1ll << 24) - 1;
    const int64_t max_groups = groups < max_wgs ? groups : max_wgs, max_panels = max_wgs / max_groups;
    for (int64_t p0 = 0; p0 < panels; p0 += max_panels)
        for (int64_t g0 = 0; g0 < groups; g0 += max_groups) {
            const int64_t n = panels - p0 < max_panels ? panels - p0 : max_panels;
            const int64_t ng = groups - g0 < max_groups ? groups - g0 : max_groups;
            // (a launch sees its K steps as the first ones: the arrays from there on, with the whole row's stride)
            const int64_t t = g0 * R_STEPS, left = ksteps - t < ng * R_STEPS ? ksteps - t : ng * R_STEPS;
            const int64_t from = to_ktile ? t : t * rows, to = to_ktile ? t * rows : t;
            auto kern = to_ktile ? (in ? relayout_kernel<true, true, true> : out ? relayout_kernel<true, false, true> : relayout_kernel<true, false, false>)
                                 : (in ? relayout_kernel<false, true, true> : out ? relayout_kernel<false, false, true> : relayout_kernel<false, false, false>);
            const int rc = enqueue(kern, dim3((unsigned)(n * ng)), dim3(kThreads), 0, s, src_c + from * 32, src_s + from * 4,
                                   dst_c + to * 32, dst_s + to * 4, rows, p0 * R_ROWS, ksteps, (int)left, (int)ng);
            if (rc != MQ_OK) return rc;
        }
    return MQ_OK;
}

int launch_global_scale(const uint16_t *x, int64_t rows, int64_t K, int64_t ldx, float *alpha,
                        hipStream_t s)
{
    uint32_t *acc = reinterpret_cast<uint32_t *>(alpha);
    const int64_t total = rows * (K / 8);
    int64_t grid = (total + kAmaxThreads * 4 - 1) / (kAmaxThreads * 4);
    grid = grid <= kAmaxOne ? 1 : grid > 256 ? 256 : grid;  // one workgroup per compute unit at most
    const bool count = grid <= kAmaxCounted;                // both lines: see amax_kernel
    if (grid > 1)
        if (int rc = enqueue(amax_init_kernel, dim3(1), dim3(1), 0, s, acc)) return rc;
    auto *const kern = ldx == K ? (count ? amax_kernel<true, true> : amax_kernel<true, false>)
                                : (count ? amax_kernel<false, true> : amax_kernel<false, false>);
    if (int rc = enqueue(kern, dim3((unsigned)grid), dim3(kAmaxThreads), 0, s, x, total, (int)(K / 8), ldx, acc)) return rc;
    return count ? MQ_OK : enqueue(amax_final_kernel, dim3(1), dim3(1), 0, s, acc);
}

}  // namespace mq
