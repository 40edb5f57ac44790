// GEMM kernels for gfx950 (CDNA4): the block-scaled NVFP4 W4A4 product of Section 3.3 and the
// BF16 baseline, Y[M,N] = A[M,K] . B[N,K]^T with FP32 accumulation.
//
// Why the NVFP4 product runs on the 16-bit MFMA: an NVFP4 element is sigma*q with sigma an
// E4M3 value (4 significant bits) and q an E2M1 value (2 significant bits), and sigma changes
// every 16 elements along K with a non-power-of-two mantissa.  CDNA4's scaled FP4/FP8 MFMA
// applies one power-of-two (E8M0) scale per 32 elements, and FP8 operands hold only 4
// significant bits, so neither can carry sigma*q exactly.  sigma*q needs 6 significant bits
// and lies in [2^-10, 2688]: it is exactly representable as a normal FP16 number.  The kernel
// therefore expands the codes to FP16 (v_cvt_scalef32_pk_f16_fp4 gives q*2^8, one packed FP16
// multiply by sigma*2^-8 gives sigma*q, both exact) and runs v_mfma_f32_32x32x16_f16 on them:
// every product is exact and the only rounding is the FP32 accumulation.  alpha_a*alpha_b is
// applied once in the epilogue.
//
// Kernels in this file
//   gemm_fp4_direct     NVFP4 from a few hundred tokens on (K % 64 == 0).  Four waves of 128x128 per
//                       workgroup, persistent workgroups, no LDS and no barriers in the K loop:
//                       each wave loads its own operand rows in MFMA order and expands them in
//                       registers (described at the kernel).  A 256x256 tile, a 256x128 tile
//                       with K split over wave pairs, or a 128x128 tile with K split over all
//                       four waves.
//   gemm_fp4_small      NVFP4 problems of up to a thousand tokens or so, and what whole rounds of the tiles
//                       above leave over: 32x32 to 128x64 tiles, one workgroup per tile, K split over
//                       its waves; for a long K with very few tiles also over workgroups
//                       (splitk_reduce_kernel then adds the slabs).
//   gemm_bf16_d2l       the BF16 baseline on large problems: 256x256, 256x192 and 256x128 tiles, four waves of 128x128
//                       to 128x64, tiles loaded from global memory straight into LDS.
//   bf16_ring_kernel    BF16 decode batches: narrow tiles, the waves of a workgroup split K, each with a
//                       ring of its own in LDS; K slabs across workgroups with a workspace.
//   bf16_short_kernel   BF16, up to 16 tokens and K <= 1024: 16x16 tiles, fragments straight into registers.
//   bf16_stage_kernel   BF16 in between: 96x64 to 256x192 tiles, two to six stages in LDS; for a long K with few
//                       tiles K slabs across workgroups with a workspace.
//   gemm_simple_kernel  any K % 16 == 0 / K % 8 == 0 that the tiled kernels do not take.
//
// The LDS pipeline of gemm_bf16_d2l: block tile 256 x 256 x 64, three LDS stages of A and two of B, and the
// latencies covered inside each wave:
//   * a K step of 64 is four MFMA phases of 16; the fragments of phase p+1 are read from LDS
//     into a second register set while the MFMAs of phase p run;
//   * tiles are fetched two K steps ahead straight into the free LDS stages;
//   * one barrier per K step, at the start of phase 3: before it every wave has finished writing
//     tile t+1 and reading tile t; after it tile t's stages are free: B's receives tile t+2 at once, A's
//     tile t+3 in the next K step.
// (An NVFP4 kernel of the same structure, operands expanded once per workgroup on their way
// into LDS, measured 6 % slower than the register-direct kernel on large problems and 1.4-1.8x
// slower on small ones, and is gone.)
// LDS rows are 128 bytes with a bank swizzle (below); tiles are walked in an XCD-aware grouped
// order.  Rows beyond M or N are clamped to the last valid row instead of being zero-filled:
// they only feed outputs that the epilogue does not store.
#include <atomic>
#include <type_traits>

#include "mq_common.h"

namespace mq {

namespace {

constexpr int BK = 64;       // K elements per LDS stage: 64 * 2 bytes = one 128-byte LDS row
constexpr int NUM_XCD = 8;

// LDS rows are 128 bytes = 8 chunks of 16 bytes.  The LDS serves 128-bit reads 16 lanes at a
// time over 64 four-byte banks (256 bytes per clock), i.e. over two consecutive rows, so the
// chunk index is XOR-ed with bits 1..3 of the row: 16 consecutive rows reading the same logical
// chunk then touch 16 different bank groups (measured: XOR with bits 0..2 gives 2-way conflicts).
__device__ __forceinline__ int swz_key(int row) { return (row >> 1) & 7; }

template <int BM_, int BN_, int WAVES_M_, int WAVES_N_>
struct PCfg {
    static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int THREADS = 64 * WAVES_M * WAVES_N;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // per-wave tile
    static constexpr int TM = WM / 32, TN = WN / 32;      // 32x32 MFMA tiles per wave
    // LDS map in bytes: three A stages, two B stages (whose stride fits the 16-bit immediate offset
    // of the LDS instructions)
    static constexpr int A_STAGE = BM * 128, B_STAGE = BN * 128, B_BASE = 3 * A_STAGE;
    static constexpr size_t LDS_BYTES = 3ull * A_STAGE + 2ull * B_STAGE;
    static_assert(TM >= 1 && TN >= 1, "tile too small for this wave grid");
};

// ---- tile order -----------------------------------------------------------------------------

// Workgroup ids are dealt round-robin to the 8 XCDs.  Give each XCD a contiguous range of
// logical tile ids, then walk tiles in groups of GROUP_M tile rows, column by column, so that
// the tiles resident on one XCD at a time share A row-panels and B column-panels in its L2.
__device__ __forceinline__ int logical_id(int wg, int total)
{
    const int xcd = wg % NUM_XCD, idx = wg / NUM_XCD;
    const int per = total / NUM_XCD, rem = total % NUM_XCD;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}

__device__ __forceinline__ void tile_of_logical(int t, int tiles_m, int tiles_n, int &tm, int &tn)
{
    constexpr int GROUP_M = 8;
    const int group_size = GROUP_M * tiles_n;
    const int g = t / group_size;
    const int first_m = g * GROUP_M;
    const int gm = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
    const int in_g = t - g * group_size;
    tm = first_m + in_g % gm;
    tn = in_g / gm;
}

__device__ __forceinline__ void tile_of(int wg, int tiles_m, int tiles_n, int &tm, int &tn)
{
    tile_of_logical(logical_id(wg, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

// Scheduling hint for one phase: per MFMA a few VALU instructions, and now and then a global load.  Nothing moves across a phase
// boundary: in particular no consumer of a global load is hoisted towards the load, which would
// turn the prefetch distance into a stall.
template <int MFMAS, int VALU_PER, int VMEMS = 0>
__device__ __forceinline__ void sched_phase()
{
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                     // MFMA
        if (VALU_PER > 0) __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER, 0);
        if (VMEMS > 0 && i < VMEMS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // VMEM read
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Accumulator register r of a 32x32 tile holds row 8*(r/4) + 4*(lane/32) + r%4, column lane%32.
// A wave tile that lies wholly inside the output takes the first path: one uniform row pointer
// per output row (scalar arithmetic) plus a constant 32-bit lane offset, no guards.  Tiles that
// cross the M or N edge take the guarded element-by-element path.
// I0, NI: the wave stores only its 32-row tiles I0 .. I0+NI-1.
template <class C, bool OUT_BF16, int I0 = 0, int NI = C::TM>
__device__ __forceinline__ void epilogue(const GemmArgs &g, f32x16 (&acc)[C::TM][C::TN], float scale,
                                         int64_t m0, int64_t n0, int wm0, int wn0, int frow, int fhalf)
{
    using T = std::conditional_t<OUT_BF16, __bf16, float>;
    const int64_t mw = m0 + wm0, nw = n0 + wn0;  // uniform over the wave
    if (mw + (I0 + NI) * 32 <= g.M && nw + C::WN <= g.N && g.ldy * (int64_t)(4 * sizeof(T)) < (1ll << 31)) {
        char *const base = static_cast<char *>(g.y) + (mw * g.ldy + nw) * (int64_t)sizeof(T);
        const uint32_t lane_off = (uint32_t)((4 * fhalf) * g.ldy + frow) * (uint32_t)sizeof(T);
        const int64_t row_bytes = g.ldy * (int64_t)sizeof(T);
        // A wave alone on its SIMD executes a chain of dependent instructions at about 8 cycles
        // each, so the values of two output rows go through scaling, rounding and the stores
        // stage by stage (the empty asm statements keep the stages apart), not value by value:
        // measured 5.1 us per 128x128 tile for the value-by-value order.  BF16: one conversion
        // packs the values of rows r and r + 1, stored as the low and the high half.
#pragma unroll
        for (int i = I0; i < I0 + NI; ++i)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                char *const rowp = base + (int64_t)(i * 32 + 8 * (r / 4) + (r % 4)) * row_bytes;
                float v[2][C::TN];
                // (read as AGPRs where they are: copies made through plain assignments let the
                // compiler move the whole accumulator set to VGPRs and scratch at the loop exit)
#pragma unroll
                for (int j = 0; j < C::TN; ++j) {
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[0][j]) : "a"(acc[i][j][r]));
                    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[1][j]) : "a"(acc[i][j][r + 1]));
                }
#pragma unroll
                for (int j = 0; j < C::TN; ++j) v[0][j] *= scale, v[1][j] *= scale;
#pragma unroll
                for (int j = 0; j < C::TN; ++j) asm volatile("" : "+v"(v[0][j]), "+v"(v[1][j]));
                if constexpr (OUT_BF16) {
                    typedef float f32x2 __attribute__((ext_vector_type(2)));
                    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                    uint32_t ob[C::TN];
#pragma unroll
                    for (int j = 0; j < C::TN; ++j)
                        ob[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[0][j], v[1][j]}, bf16x2));
#pragma unroll
                    for (int j = 0; j < C::TN; ++j) asm volatile("" : "+v"(ob[j]));
#pragma unroll
                    for (int j = 0; j < C::TN; ++j) {
                        char *const pj = rowp + (uint64_t)lane_off + j * 32 * sizeof(T);
                        *reinterpret_cast<uint16_t *>(pj) = (uint16_t)ob[j];
                        *reinterpret_cast<uint16_t *>(pj + row_bytes) = (uint16_t)(ob[j] >> 16);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < C::TN; ++j) {
                        char *const pj = rowp + (uint64_t)lane_off + j * 32 * sizeof(T);
                        *reinterpret_cast<float *>(pj) = v[0][j];
                        *reinterpret_cast<float *>(pj + row_bytes) = v[1][j];
                    }
                }
            }
        return;
    }
#pragma unroll
    for (int i = I0; i < I0 + NI; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
            const int64_t n = nw + j * 32 + frow;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t m = mw + i * 32 + 8 * (r / 4) + 4 * fhalf + (r % 4);
                float v;
                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[i][j][r]));
                if (m < g.M && n < g.N) static_cast<T *>(g.y)[m * g.ldy + n] = (T)(v * scale);
            }
        }
}

// ---- NVFP4, register-direct ------------------------------------------------------------------

// The same product without LDS and without barriers.  A wave owns a 128x128 output tile (four
// waves, one per SIMD, cover 256x256) and loads the packed codes of its own 128 A rows and 128 B
// rows straight from global memory in MFMA operand order: lane (r = lane%32, h = lane/32) takes
// the 16 bytes h of row r's 32-byte K step, dword p of which feeds phase p.  Within a K step the
// K index a lane supplies to the MFMA is therefore 32h + 8p + j instead of 16p + 8h + j; A and B
// use the same map, so each MFMA still sums 16 matching products and a K step covers all 64.
// Codes are expanded to FP16 in registers, one phase ahead of the MFMAs that use them; every
// operand row is expanded by the two waves that share it (twice the conversion work of the LDS
// pipeline, but no LDS traffic at all: measured 6 % faster on the 8192-token shapes).  Global
// loads run two K steps ahead, and the first loads of a workgroup's next tile are issued before
// the stores of the finished one.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
struct RawTile {
    uint4 c[8];      // 4 A tiles, 4 B tiles: this lane's 32 codes of each
    uint32_t s[8];   // the rows' four E4M3 scale bytes
};

// SPLIT = 2 (problems that fill the chip only with finer tiles): the workgroup tile is 256x128,
// its four waves are two 128x128 wave tiles times two halves of K; after the K loop each wave
// hands the half of its accumulators that its partner will store to the partner through LDS.
// SPLIT = 4: the workgroup tile is one 128x128 wave tile, its four waves take a quarter of K
// each, and two such exchanges leave every wave with 32 fully summed rows to store.
template <bool OUT_BF16, int SPLIT>
__global__ __launch_bounds__(256) void gemm_fp4_direct(GemmArgs g, int tiles_m, int tiles_n)
{
    using C = PCfg<256, 256, 2, 2>;  // wave-level constants: 128x128 wave tile, 4x4 MFMA tiles
    static_assert(SPLIT == 1 || SPLIT == 2 || SPLIT == 4, "K is split over 1, 2 or 4 waves");
    constexpr int BM = SPLIT == 4 ? 128 : 256, BN = SPLIT == 1 ? 256 : 128;
    constexpr int NSETS = 2;  // register sets of prefetched codes (3, i.e. two K steps of lookahead: no faster)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: the K range depends on it
    const int wm0 = SPLIT == 1 ? (wave >> 1) * 128 : SPLIT == 2 ? (wave & 1) * 128 : 0;
    const int wn0 = SPLIT == 1 ? (wave & 1) * 128 : 0;
    const int kpart = SPLIT == 1 ? 0 : SPLIT == 2 ? wave >> 1 : wave;  // which part of K this wave sums
    // SPLIT > 1: a wave holds its 32-row A tiles in the order i ^ aswap.  The tiles it will store
    // then sit in accumulator rows 0.. and the ones it hands to its partner(s) behind them, the
    // same in every wave (no divergent code): SPLIT = 2 keeps rows 0..1; SPLIT = 4 sends rows
    // 2..3 to wave w^2 first, then row 1 to wave w^1, and keeps row 0 = output tile w.
    const int aswap = SPLIT == 2 ? kpart << 1 : kpart;
    const int frow = lane & 31, fhalf = lane >> 5;
    const int KT = (int)(g.K / BK);
    // this wave's K steps [k0, k1); every part but the last is a whole number of NSETS groups
    const int parts = SPLIT;
    const int KH = SPLIT == 1 ? KT : ((KT + parts - 1) / parts + NSETS - 1) / NSETS * NSETS;
    int k0 = kpart * KH, k1 = (k0 + KH < KT) ? k0 + KH : KT;
    const int total_tiles = tiles_m * tiles_n;
    auto item_of = [&](int item, int &tm, int &tn) { tile_of(item, tiles_m, tiles_n, tm, tn); };

    // Buffer loads: per K step a uniform resource whose 64-bit base is the start of that K step
    // (scalar arithmetic only), plus the lane's row and half as a 32-bit vector offset.  Rows
    // are clamped below, so every access is in bounds by construction and the resources carry
    // the maximal size.
    // The lane offsets are relative to the first row of the wave tile (whose 64-bit address is
    // scalar), so they fit 32 bits for any operand size.
    uint32_t vc[8], vs[8];
    // Running pointers to the K step that the next loads read, for the first A / B row of
    // this wave's tile (codes, scales); advance() moves them on by one K step and stops at the
    // last step of K, so the loads issued past the end of a tile re-read that step.  (Advancing
    // costs some twenty scalar instructions per K step, placed under the MFMAs of the phase in
    // front of the loads; recomputing base + t * step cost thirty, in one block at the loads.)
    const char *pa_c, *pb_c, *pa_s, *pb_s;
    int t_next;
    auto set_tile = [&](int64_t m0, int64_t n0) {
        int64_t ra = m0 + wm0, rb = n0 + wn0;
        ra = ra < g.M ? ra : g.M - 1;
        rb = rb < g.N ? rb : g.N - 1;
        t_next = k0 < KT ? k0 : KT - 1;
        pa_c = static_cast<const char *>(g.a) + ra * g.a_c_row + t_next * g.a_c_step;
        pb_c = static_cast<const char *>(g.b) + rb * g.b_c_row + t_next * g.b_c_step;
        pa_s = reinterpret_cast<const char *>(g.a_scales) + ra * g.a_s_row + t_next * g.a_s_step;
        pb_s = reinterpret_cast<const char *>(g.b_scales) + rb * g.b_s_row + t_next * g.b_s_step;
        // (32-bit arithmetic per lane: offsets within 128 rows fit)
        const int last_a = (int)(g.M - 1 - ra < 127 ? g.M - 1 - ra : 127), last_b = (int)(g.N - 1 - rb < 127 ? g.N - 1 - rb : 127);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool isA = q < 4;
            const int row = (isA ? (q ^ aswap) : q - 4) * 32 + frow, last = isA ? last_a : last_b;
            const uint32_t rel = (uint32_t)(row < last ? row : last);
            vc[q] = rel * (uint32_t)(isA ? g.a_c_row : g.b_c_row) + fhalf * 16;
            vs[q] = rel * (uint32_t)(isA ? g.a_s_row : g.b_s_row);
        }
    };
    RawTile st[NSETS];
    // load u of a K step: codes (u even) or scales of operand tile u / 2
    auto load_one = [&](RawTile &r, int u) {
        auto rsrc = [](const char *p) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, -1, 0x00020000);
        };
        const int q = u / 2;
        if (u % 2 == 0) {
            const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(rsrc(q < 4 ? pa_c : pb_c), (int)vc[q], 0, 0);
            r.c[q] = make_uint4(c[0], c[1], c[2], c[3]);
        } else {
            r.s[q] = __builtin_amdgcn_raw_buffer_load_b32(rsrc(q < 4 ? pa_s : pb_s), (int)vs[q], 0, 0);
        }
    };
    // The K steps in front of the loop, set by set: left to itself the compiler put loads of the second set before some of the first,
    // and the first MFMAs then waited for both (row-major, 4096 tokens on K = 512, N = 4096 28.1 us, in order 27.6; 2500 tokens 28.7 and 28.1).
    // Not where four waves share K: 488 tokens on K = 960, N = 5120 15.4 us, set by set 16.0.
    auto load_tile = [&](RawTile &r) {
#pragma unroll
        for (int u = 0; u < 16; ++u) load_one(r, u);
        if constexpr (SPLIT < 4) __builtin_amdgcn_sched_barrier(0);
    };
    auto advance = [&]() {
        const int64_t adv = -(int64_t)(t_next + 1 < KT);  // all ones while a next K step exists (no branch)
        t_next -= (int)adv;
        pa_c += g.a_c_step & adv;
        pb_c += g.b_c_step & adv;
        pa_s += g.a_s_step & adv;
        pb_s += g.b_s_step & adv;
    };
    // Scale register of the K step being expanded: sigma*2^-8 as FP16 for block 2h in the low
    // half and for block 2h+1 in the high half (an E4M3 byte shifted left by 7 is that number).
    // One byte permute picks the lane's two scale bytes, or zeros for a K step past the end.
    uint32_t sg[8];
    const uint32_t sel_valid = 0x0C000C00u | (uint32_t)(2 * fhalf) | ((uint32_t)(2 * fhalf + 1) << 16);
    auto prep_scale = [&](const RawTile &r, uint32_t sel, int q) {
        uint32_t sc = r.s[q];
        asm("" : "+v"(sc));  // first use of the prefetched register stays here
        sg[q] = __builtin_amdgcn_perm(0u, sc, sel) << 7;
    };
    auto prep_scales = [&](const RawTile &r, bool valid) {
        const uint32_t sel = valid ? sel_valid : 0x0C0C0C0Cu;
#pragma unroll
        for (int q = 0; q < 8; ++q) prep_scale(r, sel, q);
    };
    uint4 fr[2][8];
    // In front of the loop: the first phase's tiles (0..3 = A row tiles, 4..7 = B row tiles) but for the two that kstep expands.
    auto expand_first = [&](const RawTile &r) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q == 2 || q == 3) continue;
            uint32_t w = r.c[q].x;
            asm("" : "+v"(w));
            const _Float16 sig = __builtin_bit_cast(_Float16, (uint16_t)sg[q]);
            const f16x2 s = {sig, sig};
            // (The empty asm statements order through their operands only; they must not be
            // volatile: a volatile asm counts as a side effect that no memory operation may
            // cross.)
            f16x2 c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0);
            f16x2 c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1);
            f16x2 c2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2);
            f16x2 c3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3);
            asm("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
            c0 *= s, c1 *= s, c2 *= s, c3 *= s;
            fr[0][q] = make_uint4(__builtin_bit_cast(uint32_t, c0), __builtin_bit_cast(uint32_t, c1),
                                  __builtin_bit_cast(uint32_t, c2), __builtin_bit_cast(uint32_t, c3));
        }
    };
    f32x16 acc[4][4];
    // The two halves of expanding one operand tile of a phase: four conversions, and, behind the next MFMA, their four multiplies
    // (a multiply right behind the conversion that it consumes stalls the wave).
    f16x2 half[4];
    auto convert = [&](const RawTile &r, int p, int q) {
        uint32_t w = p == 0 ? r.c[q].x : p == 1 ? r.c[q].y : p == 2 ? r.c[q].z : r.c[q].w;
        asm("" : "+v"(w));
        half[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0);
        half[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1);
        half[2] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2);
        half[3] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3);
    };
    auto multiply = [&](int p, int q, uint4(&f)[8]) {
        const _Float16 sig = __builtin_bit_cast(_Float16, (uint16_t)(p < 2 ? sg[q] : sg[q] >> 16));
        const f16x2 s = {sig, sig};
        f[q] = make_uint4(__builtin_bit_cast(uint32_t, half[0] * s), __builtin_bit_cast(uint32_t, half[1] * s),
                          __builtin_bit_cast(uint32_t, half[2] * s), __builtin_bit_cast(uint32_t, half[3] * s));
    };
    // The 16 MFMAs of a phase on fragments f, slot(n) behind MFMA n: four VALU instructions and a load or a few scalar ones fit
    // under an MFMA's 32 cycles.  Nothing moves from one slot to another: left to the compiler within a phase, with only the number of
    // instructions per MFMA asked for, the fours got out of step with the MFMAs, and conversions met their multiplies
    // without one in between.  us, asked for / slot by slot: 8192 tokens on K = 4096, N = 28672 1290 / 1262, on K = 14336,
    // N = 4096 610 / 603; 16384 on N = 4096 371 / 365; 1000 on N = 28672 183 / 181; 4096 on N = 6144 149.3 / 147.2.
    auto phase = [&](const uint4(&f)[8], auto &&slot) {
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            acc[n / 4][n % 4] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                __builtin_bit_cast(f16x8, f[n / 4]), __builtin_bit_cast(f16x8, f[4 + n % 4]), acc[n / 4][n % 4], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            slot(n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int64_t adv = 0;
    // one K step; R = kt % NSETS is the register set that holds tile kt
    auto kstep = [&](int kt, auto rr) {
        constexpr int R = decltype(rr)::value;
        RawTile &cur = st[R], &nxt = st[(R + 1) % NSETS];
        // The last two A row tiles of this step's first phase are expanded here, right before
        // the MFMAs that use them (the ninth onwards), not in the load phase of the previous K
        // step, which is the one phase that fills the wave's issue slots (+0.5-1 %; three tiles
        // deferred: no better).  Ten tiles in sixteen slots: five in eight, two of them sharing a slot with the multiplies
        // of the one before.
        phase(fr[0], [&](int n) {
            const int h = n / 8, e = n % 8;  // c m|c m c m|c m c m
            auto tile = [&](int x, bool c) {  // the x-th of the ten
                const int q = x < 2 ? 2 + x : x - 2;
                if (c)
                    convert(cur, x < 2 ? 0 : 1, q);
                else
                    multiply(x < 2 ? 0 : 1, q, x < 2 ? fr[0] : fr[1]);
            };
            const int t = 5 * h;
            if (e == 0) tile(t, true);
            if (e == 1) tile(t, false), tile(t + 1, true);
            if (e == 2) tile(t + 1, false);
            if (e == 3) tile(t + 2, true);
            if (e == 4) tile(t + 2, false), tile(t + 3, true);
            if (e == 5) tile(t + 3, false);
            if (e == 6) tile(t + 4, true);
            if (e == 7) tile(t + 4, false);
        });
        phase(fr[1], [&](int n) {
            if (n % 2 == 0)
                convert(cur, 2, n / 2);
            else
                multiply(2, n / 2, fr[0]);
        });
        phase(fr[0], [&](int n) {
            if (n % 2 == 0)
                convert(cur, 3, n / 2);
            else
                multiply(3, n / 2, fr[1]);
            // the scalar pointer arithmetic of the loads below, spread under this phase's MFMAs
            if (n == 1) adv = -(int64_t)(t_next + 1 < KT), t_next -= (int)adv;
            if (n == 4) pa_c += g.a_c_step & adv;
            if (n == 7) pb_c += g.b_c_step & adv;
            if (n == 10) pa_s += g.a_s_step & adv;
            if (n == 13) pb_s += g.b_s_step & adv;
        });
        // The only loads in flight here are the 16 of the next K step, a whole step old: one wait
        // for all of them instead of one in front of each first use (this phase is the one that
        // fills the wave's issue slots, and a wait is an instruction like any other: +0.5-0.8 %).
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        // The scales' loads first, then the codes': row-major operands, whose loads touch a line per row, take 1 to 3 % less than with
        // codes and scales in turn, which had made them slower with the slots than without (8192 tokens on K = 14336, N = 4096 988 us
        // before the slots, 997 in turn, 958 now; 3500 tokens 444, 450, 432); K-step-major the same within 0.3 %.
        const uint32_t sel = kt + 1 < k1 ? sel_valid : 0x0C0C0C0Cu;
        phase(fr[1], [&](int n) {
            if (n < 4) {
                prep_scale(nxt, sel, 2 * n);
                prep_scale(nxt, sel, 2 * n + 1);
            } else {
                const int x = (n - 4) / 2, q = x < 2 ? x : x + 2;
                if (n % 2 == 0)
                    convert(nxt, 0, q);
                else
                    multiply(0, q, fr[0]);
            }
            load_one(cur, n < 8 ? 2 * n + 1 : 2 * (n - 8));
        });
    };

    // Persistent workgroups: tile ids blockIdx.x, blockIdx.x + gridDim.x, ...  The first loads of
    // the next tile are issued before the stores of the finished one.
    const float scale = (*g.a_alpha) * (*g.b_alpha);
    int tile = blockIdx.x;
    int tm, tn;
    item_of(tile, tm, tn);
    set_tile((int64_t)tm * BM, (int64_t)tn * BN);
#pragma unroll
    for (int u = 0; u < NSETS; ++u) {
        if (u) advance();
        load_tile(st[u]);
    }
    while (true) {
        const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
        prep_scales(st[0], k0 < k1);
        expand_first(st[0]);
        // No separate tail: the loop runs whole groups of NSETS K steps, and a step past the end
        // multiplies by zero scales.  (Peeled tail steps make the compiler shuffle all 256
        // accumulator registers at the control-flow joins.)
        for (int kt = k0; kt < k1; kt += NSETS) {
            kstep(kt, std::integral_constant<int, 0>{});
            if constexpr (NSETS > 1) kstep(kt + 1, std::integral_constant<int, 1>{});
            if constexpr (NSETS > 2) kstep(kt + 2, std::integral_constant<int, 2>{});
        }
        tile += gridDim.x;
        const bool more = tile < total_tiles;
        if (more) {
            item_of(tile, tm, tn);
            set_tile((int64_t)tm * BM, (int64_t)tn * BN);
#pragma unroll
            for (int u = 0; u < NSETS; ++u) {
                if (u) advance();
                load_tile(st[u]);
            }
        }
        if constexpr (SPLIT == 1) {
            epilogue<C, OUT_BF16>(g, acc, scale, m0, n0, wm0, wn0, frow, fhalf);
        } else {
            // Waves that hold different parts of K for the same 128x128 tile exchange through LDS:
            // a wave sends the accumulator rows [first, first + count) to `partner` and adds what
            // the partner sent to its rows [0, count) (a + b in both, so the result does not
            // depend on which wave adds).  1 KB per (32x32 tile, register quad) and wave.
            extern __shared__ uint4 lds[];
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            f32x4 *const X = reinterpret_cast<f32x4 *>(lds);
            auto exchange = [&](auto firstc, auto countc, int partner) {
                constexpr int first = decltype(firstc)::value, count = decltype(countc)::value;
#pragma unroll
                for (int i = 0; i < count; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const f32x16 &t = acc[first + i][j];
                            X[((wave * 8 + i * 4 + j) * 4 + c) * 64 + lane] =
                                f32x4{t[4 * c], t[4 * c + 1], t[4 * c + 2], t[4 * c + 3]};
                        }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < count; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const f32x4 v = X[((partner * 8 + i * 4 + j) * 4 + c) * 64 + lane];
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[i][j][4 * c + e] += v[e];
                        }
                __syncthreads();  // the next sends must not overtake these reads
            };
            exchange(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, wave ^ 2);
            if constexpr (SPLIT == 2) {
                epilogue<C, OUT_BF16, 0, 2>(g, acc, scale, m0, n0, wm0 + kpart * 64, wn0, frow, fhalf);
            } else {
                exchange(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, wave ^ 1);
                epilogue<C, OUT_BF16, 0, 1>(g, acc, scale, m0, n0, wm0 + wave * 32, wn0, frow, fhalf);
            }
        }
        if (!more) break;
    }
}

// ---- NVFP4, register-direct, small tiles: prefill chunks up to a thousand tokens or so ---------------

// With a few hundred tokens the 128x128 wave tiles above are too few to occupy the chip, and the
// time of a layer is launch latency plus one trip of the weights from HBM.  Here a workgroup owns
// one (32 TM) x (32 TN) output tile; its S waves (8, 4 or, for a short K, 1) take consecutive parts of K and each runs
// the same register-direct K loop as above (operands loaded in MFMA order, expanded in registers, no
// LDS and no barrier in the loop) with NSETS K steps of codes in flight per wave.  The S partial tiles
// are then added through LDS in a fixed order (wave 0, 1, ...: bit-identical from run to run), each
// wave summing, scaling, rounding and storing 1/S of the tile.  One launch per layer, no workspace;
// with one, a long K may also be cut into g.ksplit slabs across workgroups: a work item is then (slab,
// tile), its workgroup writes unscaled FP32 partial sums to g.ws[slab][M][N], and
// splitk_reduce_kernel adds the slabs in ascending order.
// What bounds it: the expansion (16 vector instructions per MFMA for 32x32, 8 for 64x64, 6 for 128x64; at two
// waves per SIMD 8 take 40 to 44 cycles and 6 take 34 to 37 per MFMA, of 32); but a 32x32 tile gives every compute unit work where a
// 64x64 tile leaves three quarters of them idle (64 tokens, K = N = 4096, weights from HBM: 8.0 us against 12.3; K =
// 14336: 15.6 against 17.3 with K slabs), and 64x128 tiles, two workgroups of four waves to a compute unit,
// hide each other's sums and stores, which the one-workgroup kernel above cannot (576 tokens on N =
// 28672: 108 us against 165 in 256x256 tiles; 105 with 512 of them in those).  Two waves per SIMD throughout (at most 256 registers).
template <int TM_, int TN_>
struct SmallCfg {
    static constexpr int TM = TM_, TN = TN_, WN = 32 * TN_;
};

// End of the small-tile kernels: the S waves of a workgroup hold partial sums of one
// (32 TM) x (32 TN) tile over their parts of K.  The partial
// tiles are added through LDS, four 32x32 tiles (16 KB per wave) per pass.  A pass holds 16 chunks
// of four accumulator registers per wave; wave w adds the S copies of chunks w, w + S, ... in
// wave order (bit-identical from run to run), scales, rounds and stores them: chunk c of a tile =
// rows 8c + 4 (lane / 32) .. + 3, column lane % 32.
template <int TM, int TN, int S, bool OUT_BF16>
__device__ __forceinline__ void small_tile_finish(const GemmArgs &g, f32x16 (&acc)[TM][TN], float scale, int64_t m0,
                                                  int64_t n0, int wave, int lane)
{
    constexpr int NM = TM * TN;
    const int frow = lane & 31, fhalf = lane >> 5;
    if constexpr (S == 1) {  // nothing to add
        epilogue<SmallCfg<TM, TN>, OUT_BF16>(g, acc, scale, m0, n0, 0, 0, frow, fhalf);
        return;
    }
    extern __shared__ uint4 lds[];
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    f32x4 *const X = reinterpret_cast<f32x4 *>(lds);
    using T = std::conditional_t<OUT_BF16, __bf16, float>;
    constexpr int PASS = NM < 4 ? NM : 4;  // tiles per pass
#pragma unroll
    for (int p0 = 0; p0 < NM; p0 += PASS) {
        if (p0 > 0) __syncthreads();  // the previous pass has been read
#pragma unroll
        for (int u = 0; u < PASS; ++u) {
            const f32x16 &tl = acc[(p0 + u) / TN][(p0 + u) % TN];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                X[((wave * PASS + u) * 4 + c) * 64 + lane] = f32x4{tl[4 * c], tl[4 * c + 1], tl[4 * c + 2], tl[4 * c + 3]};
        }
        __syncthreads();
#pragma unroll
        for (int ch0 = 0; ch0 < PASS * 4; ch0 += S) {
            const int ch = ch0 + wave;
            if (PASS * 4 % S != 0 && ch >= PASS * 4) break;  // uniform
            f32x4 part[S];  // all reads in flight, then the additions in wave order
#pragma unroll
            for (int w = 0; w < S; ++w) part[w] = X[(w * PASS * 4 + ch) * 64 + lane];
            f32x4 sum = part[0];
#pragma unroll
            for (int w = 1; w < S; ++w) sum += part[w];
            const int tile = p0 + (ch >> 2), c = ch & 3;
            const int64_t n = n0 + (tile % TN) * 32 + frow;
            const int64_t mrow = m0 + (tile / TN) * 32 + 8 * c + 4 * fhalf;
            if (n < g.N) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (mrow + e < g.M) static_cast<T *>(g.y)[(mrow + e) * g.ldy + n] = (T)(sum[e] * scale);
            }
        }
    }
}

// LINE (row-major operands, K % 256 == 0): the unit of work is four K steps, whose codes of a row are one 128-byte line.  In K
// order a load takes 32 bytes of each of 32 lines, and by the time the next K step asks for the next 32 bytes the other waves
// have pushed the lines out of the 32 KB of L1: every line was fetched four times, and a line per row for four scale bytes
// besides.  Those fetches, 64 bytes per clock and compute unit from L2, bound the kernel.  Here lane (r, h) takes the half line
// h of row r in four loads that stand together (chunk t of 16 bytes holds elements 128 h + 32 t ..: A and B permute K alike) and
// the eight scale bytes of the half line in one load, every four K steps.  Tiles of up to three operand rows hold two groups,
// the next one under way while this one is multiplied; 64x64 reloads the registers under the group's last K step, holds all of 256
// registers and spills 8 to 10 of them, in the lines behind the loop, where a short K spends all its time (one or two lines to a
// wave: K = 2048 to 4096 in eight waves), and is faster there than in K order all the same.  us, in K order
// and by lines: 64 tokens on K = N = 4096 in 32x32 tiles 11.6 and 8.9; 128 on K = 14336, N = 4096 in 64x32 51 and 32; 256 on
// K = N = 4096 in 64x64 20.3 and 14.8; 512 28.9 and 24.9; 32 on K = 2048, N = 4096 6.5 and 5.7.
template <int TM, int TN, int S>
constexpr bool may_be_even()
{
    return TM == 2 && TN == 2 && S == 4;
}

template <int TM, int TN, int S, int NSETS, bool OUT_BF16, bool LINE>
__global__ __launch_bounds__(64 * S) __attribute__((amdgpu_waves_per_eu(2))) void gemm_fp4_small(GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int NT = TM + TN;
    constexpr int UNIT = LINE ? 4 : 1;                     // K steps of a unit
    constexpr bool TWO = LINE && NT <= 3;                  // two groups in registers
    constexpr int SETS = TWO ? 8 : NSETS;                  // K steps in registers
    constexpr bool EVEN = LINE && may_be_even<TM, TN, S>();
    static_assert(!LINE || NSETS == 4, "a line is four K steps");
    static_assert((TM * TN) % 4 == 0 || TM * TN < 4, "the LDS reduction moves four 32x32 tiles per pass");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int frow = lane & 31, fhalf = lane >> 5;
    const int KT = (int)(g.K / (BK * UNIT));  // units: K steps, or lines
    // work item = (K slab, tile), slab-major; tiles that share a column panel of B are neighbours
    // in that order and run on one XCD.  g.ksplit == 1: the tile's whole K.
    const int tiles = tiles_m * tiles_n;
    const int item = logical_id(blockIdx.x, tiles * g.ksplit);
    const int slab = item / tiles, t = item - slab * tiles;
    const int tm = t % tiles_m, tn = t / tiles_m;
    const int64_t m0 = (int64_t)tm * (32 * TM), n0 = (int64_t)tn * (32 * TN);  // m0 < M, n0 < N
    // K steps of the slab, then of this wave within it
    const int SL = (KT + g.ksplit - 1) / g.ksplit;
    const int s0 = slab * SL < KT ? slab * SL : KT, s1 = s0 + SL < KT ? s0 + SL : KT;
    const int KH = (s1 - s0 + S - 1) / S;
    const int k0 = s0 + wave * KH < s1 ? s0 + wave * KH : s1;
    const int k1 = k0 + KH < s1 ? k0 + KH : s1;

    // operand q: A row tile q (q < TM), else B row tile q - TM.  Lane offsets relative to the row a0 (b0) of the operand, the tile's
    // first.  Lanes past the operand's last row read that row again: fewer lines, so a last tile of few rows is done early.
    // g.even: they read the rows in front of the tile instead, so that it takes as long as the others (see fp4_even).
    auto first_row = [&](int64_t tile0, int64_t rows, int size) {
        return EVEN && g.even && rows > size && tile0 > rows - size ? rows - size : tile0;
    };
    const int64_t a0 = first_row(m0, g.M, 32 * TM), b0 = first_row(n0, g.N, 32 * TN);
    const char *const ta_c = static_cast<const char *>(g.a) + a0 * g.a_c_row;
    const char *const tb_c = static_cast<const char *>(g.b) + b0 * g.b_c_row;
    const char *const ta_s = reinterpret_cast<const char *>(g.a_scales) + a0 * g.a_s_row;
    const char *const tb_s = reinterpret_cast<const char *>(g.b_scales) + b0 * g.b_s_row;
    uint32_t vc[NT], vs[NT];
    const int last_a = (int)(g.M - a0 < 32 * TM ? g.M - a0 : 32 * TM) - 1, last_b = (int)(g.N - b0 < 32 * TN ? g.N - b0 : 32 * TN) - 1;
    const int skip_a = (int)(m0 - a0), skip_b = (int)(n0 - b0);  // (0 unless g.even and the last tile; `last` is the tile's size - 1 then)
#pragma unroll
    for (int q = 0; q < NT; ++q) {
        const bool isA = q < TM;
        const int row = (isA ? q : q - TM) * 32 + frow, last = isA ? last_a : last_b, skip = isA ? skip_a : skip_b;
        const uint32_t rel = (uint32_t)(row + skip <= last ? row + skip : skip > 0 ? row : last);
        vc[q] = rel * (uint32_t)(isA ? g.a_c_row : g.b_c_row) + fhalf * (16 * UNIT);
        vs[q] = rel * (uint32_t)(isA ? g.a_s_row : g.b_s_row) + (LINE ? fhalf * 8 : 0);
    }
    uint4 rc[SETS][NT];                  // this lane's 32 codes of each operand tile, SETS K steps
    uint32_t rs[LINE ? 1 : SETS][NT];    // the rows' four E4M3 scale bytes of a K step
    uint2 rl[LINE ? SETS / 4 : 1][NT];   // or this lane's eight of a line
    // Resources that start at the wave's first K step (or at a later one, where offsets from there would reach 2 GiB: below); the
    // K step goes into the loads' scalar offset, one multiplication each.  Loads past the wave's last step re-read
    // that step (from L1; its products are multiplied by zero scales).  With running 64-bit pointers and a resource built
    // per load and K step there were 38 scalar instructions per K step instead of 8, and at two waves per SIMD a scalar
    // instruction per MFMA costs about two cycles of the forty.  With the last group below: 64 tokens, K = N = 4096 in 32x32
    // tiles 7.1 -> 6.4 us with W in cache, 256 tokens in 64x64 12.7 -> 11.2, 128 tokens on K = 14336 in 64x32 21.6 -> 20.4.
    const int len = k1 - k0;
    int64_t first = k0 < KT ? k0 : KT - 1;
    auto rsrc = [](const char *base) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, -1, 0x00020000);
    };
    __amdgpu_buffer_rsrc_t rac = rsrc(ta_c + first * UNIT * g.a_c_step), rbc = rsrc(tb_c + first * UNIT * g.b_c_step);
    __amdgpu_buffer_rsrc_t ras = rsrc(ta_s + first * UNIT * g.a_s_step), rbs = rsrc(tb_s + first * UNIT * g.b_s_step);
    // Line l of this wave into register group `buf`: operand tile q, its four chunks one behind the other (apart, the lines have
    // left L1 by the next chunk) and its scales.
    auto load_line = [&](int l, auto bufc, int q) {
        constexpr int buf = decltype(bufc)::value;
        l = l < len - 1 ? l : len - 1;
        const int u = l > 0 ? l : 0;
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(q < TM ? rac : rbc, (int)(vc[q] + 16 * t), u * 128, 0);
            rc[4 * buf + t][q] = make_uint4(c[0], c[1], c[2], c[3]);
        }
        const u32x2 sc = __builtin_amdgcn_raw_buffer_load_b64(q < TM ? ras : rbs, (int)vs[q], u * 16, 0);
        rl[buf][q] = make_uint2(sc[0], sc[1]);
    };
    const uint32_t ca = (uint32_t)g.a_c_step, cb = (uint32_t)g.b_c_step, sa = (uint32_t)g.a_s_step, sb = (uint32_t)g.b_s_step;
    auto load_step = [&](int t, auto setc) {  // K step t from `first`
        constexpr int R = decltype(setc)::value;
        const uint32_t u = (uint32_t)t;
        const int oac = (int)(u * ca), obc = (int)(u * cb), oas = (int)(u * sa), obs = (int)(u * sb);
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(q < TM ? rac : rbc, (int)vc[q], q < TM ? oac : obc, 0);
            rc[R][q] = make_uint4(c[0], c[1], c[2], c[3]);
            rs[R][q] = __builtin_amdgcn_raw_buffer_load_b32(q < TM ? ras : rbs, (int)vs[q], q < TM ? oas : obs, 0);
        }
    };
    // scales, expansion and MFMAs exactly as in gemm_fp4_direct (K index of a lane: 32h + 8p + j)
    uint32_t sg[NT];
    const uint32_t sel_valid = 0x0C000C00u | (uint32_t)(2 * fhalf) | ((uint32_t)(2 * fhalf + 1) << 16);
    auto prep_scales = [&](auto setc, bool valid) {
        constexpr int R = decltype(setc)::value;
        const uint32_t sel = LINE ? (R % 2 ? 0x0C030C02u : 0x0C010C00u) : valid ? sel_valid : 0x0C0C0C0Cu;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            uint32_t sc = LINE ? (R % 4 < 2 ? rl[LINE ? R / 4 : 0][q].x : rl[LINE ? R / 4 : 0][q].y) : rs[LINE ? 0 : R][q];
            asm("" : "+v"(sc));
            sg[q] = __builtin_amdgcn_perm(0u, sc, sel) << 7;
        }
    };
    uint4 fr[2][NT];
    auto expand_phase = [&](auto setc, int p, uint4(&f)[NT]) {
        constexpr int R = decltype(setc)::value;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            uint32_t w = p == 0 ? rc[R][q].x : p == 1 ? rc[R][q].y : p == 2 ? rc[R][q].z : rc[R][q].w;
            asm("" : "+v"(w));
            const _Float16 sig = __builtin_bit_cast(_Float16, (uint16_t)(p < 2 ? sg[q] : sg[q] >> 16));
            const f16x2 sv = {sig, sig};
            f16x2 c0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 0);
            f16x2 c1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 1);
            f16x2 c2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 2);
            f16x2 c3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 256.0f, 3);
            asm("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
            c0 *= sv, c1 *= sv, c2 *= sv, c3 *= sv;
            f[q] = make_uint4(__builtin_bit_cast(uint32_t, c0), __builtin_bit_cast(uint32_t, c1),
                              __builtin_bit_cast(uint32_t, c2), __builtin_bit_cast(uint32_t, c3));
        }
    };
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    auto mfmas = [&](const uint4(&f)[NT]) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                    __builtin_bit_cast(f16x8, f[i]), __builtin_bit_cast(f16x8, f[TM + j]), acc[i][j], 0, 0, 0);
    };
    constexpr int NM = TM * TN, VPER = (NT * 8 + NM - 1) / NM;
    using std::integral_constant;
    auto for_sets = [&](auto &&fn) {  // fn(set index as a constant), sets 0 .. NSETS-1
        fn(integral_constant<int, 0>{});
        if constexpr (NSETS > 1) fn(integral_constant<int, 1>{});
        if constexpr (NSETS > 2) fn(integral_constant<int, 2>{});
        if constexpr (NSETS > 3) fn(integral_constant<int, 3>{});
    };
    static_assert(NSETS >= 2 && NSETS <= 4, "two to four K steps in flight");
    const float scale = (*g.a_alpha) * (*g.b_alpha);
    if constexpr (!LINE) {
        int end = len;  // of this wave's part, as kt counted from `first`
        // K step kt; LAST: of the last group, behind which nothing is loaded
        auto kstep = [&](int kt, auto setc, auto lastc) {
            constexpr int R = decltype(setc)::value;
            constexpr bool LAST = decltype(lastc)::value;
            using Next = integral_constant<int, (R + 1) % NSETS>;
            expand_phase(setc, 1, fr[1]);
            mfmas(fr[0]);
            sched_phase<NM, VPER>();
            expand_phase(setc, 2, fr[0]);
            mfmas(fr[1]);
            sched_phase<NM, VPER>();
            expand_phase(setc, 3, fr[1]);
            mfmas(fr[0]);
            sched_phase<NM, VPER>();
            if constexpr (!LAST || R + 1 < NSETS) {
                prep_scales(Next{}, !LAST || kt + 1 < end);
                expand_phase(Next{}, 0, fr[0]);
            }
            if constexpr (!LAST) load_step(kt + NSETS < end ? kt + NSETS : end - 1, setc);
            mfmas(fr[1]);
            sched_phase<NM, VPER + 2, LAST ? 0 : (2 * NT + NM - 1) / NM>();
        };
        // The first NSETS K steps, issued set by set.  (Left to the scheduler, the B loads of all sets
        // went last, and the counter the compiler waits on in the loop then demanded that nearly
        // everything in flight had landed before each K step: a prefetch distance of one step, not three.)
        for_sets([&](auto u) {
            load_step(decltype(u)::value < len ? decltype(u)::value : len > 0 ? len - 1 : 0, u);
            __builtin_amdgcn_sched_barrier(0);
        });
        prep_scales(integral_constant<int, 0>{}, len > 0);
        expand_phase(integral_constant<int, 0>{}, 0, fr[0]);
        // Whole groups of NSETS K steps, then the last one, which loads nothing and ends at the wave's last step.  (Leaving the
        // loop in the middle of a group made the compiler move all accumulators at the joins: 1.2 to 1.6x slower.  Behind the
        // loop they are moved once.  When the last group was run whole, on zero scales, K = 512 took 5.0 us instead of 3.5, and
        // 100 tokens on K = 6400, N = 5120 17.0 instead of 14.0.)
        // Where the loads of a group would reach further than 2 GiB (g.reach K steps), the resources move up to it: K-step-major
        // operands of 19 GB and more in these tiles (16 tokens on K = 65536, N = 600000 3.7 ms; 7.8 in the direct tiles).
        int kt = 0;
        while (kt + NSETS < end) {
            if (kt + 2 * NSETS - 1 > g.reach) {
                first += kt + NSETS, end -= kt + NSETS, kt = -NSETS;
                rac = rsrc(ta_c + first * g.a_c_step), rbc = rsrc(tb_c + first * g.b_c_step);
                ras = rsrc(ta_s + first * g.a_s_step), rbs = rsrc(tb_s + first * g.b_s_step);
            }
            const int most = end - NSETS < g.reach - 2 * NSETS + 2 ? end - NSETS : g.reach - 2 * NSETS + 2;
            do {
                for_sets([&](auto u) { kstep(kt + decltype(u)::value, u, std::false_type{}); });
                kt += NSETS;
            } while (kt < most);
        }
        auto tail = [&](auto self, auto u) -> void {
            kstep(kt + decltype(u)::value, u, std::true_type{});
            if constexpr (decltype(u)::value + 1 < NSETS)
                if (kt + decltype(u)::value + 1 < end) self(self, integral_constant<int, decltype(u)::value + 1>{});
        };
        tail(tail, integral_constant<int, 0>{});
    } else if (len > 0) {
        // line l of this wave, in register group `buf`; LAST: nothing follows
        auto line = [&](int l, auto bufc, auto lastc) {
            constexpr int buf = decltype(bufc)::value, other = TWO ? buf ^ 1 : buf;
            constexpr bool LAST = decltype(lastc)::value;
            using Other = integral_constant<int, other>;
            for_sets([&](auto tc) {
                constexpr int t = decltype(tc)::value, R = 4 * buf + t;
                using Set = integral_constant<int, R>;
                using Next = integral_constant<int, t < 3 ? R + 1 : 4 * other>;
                constexpr bool LOADS = !LAST && TWO && t == 0;
                if constexpr (LOADS) load_line(l + 1, Other{}, 0);
                expand_phase(Set{}, 1, fr[1]);
                mfmas(fr[0]);
                sched_phase<NM, VPER, LOADS ? NM : 0>();
                if constexpr (LOADS) load_line(l + 1, Other{}, 1);
                expand_phase(Set{}, 2, fr[0]);
                mfmas(fr[1]);
                sched_phase<NM, VPER, LOADS ? NM : 0>();
                if constexpr (LOADS && NT > 2) load_line(l + 1, Other{}, NT - 1);
                expand_phase(Set{}, 3, fr[1]);
                mfmas(fr[0]);
                sched_phase<NM, VPER, (LOADS && (NT > 2)) ? NM : 0>();
                if constexpr (!LAST && !TWO && t == 3) {  // the codes have all been expanded
#pragma unroll
                    for (int q = 0; q < NT; ++q) load_line(l + 1, Other{}, q);
                    mfmas(fr[1]);
                    __builtin_amdgcn_sched_barrier(0);
                    prep_scales(Next{}, true);
                    expand_phase(Next{}, 0, fr[0]);
                    __builtin_amdgcn_sched_barrier(0);
                } else {
                    if constexpr (!LAST || t < 3) {
                        prep_scales(Next{}, true);
                        expand_phase(Next{}, 0, fr[0]);
                    }
                    mfmas(fr[1]);
                    sched_phase<NM, VPER + 2>();
                }
            });
        };
        using Zero = integral_constant<int, 0>;
        using One = integral_constant<int, TWO ? 1 : 0>;
#pragma unroll
        for (int q = 0; q < NT; ++q) load_line(0, Zero{}, q);
        __builtin_amdgcn_sched_barrier(0);
        prep_scales(Zero{}, true);
        expand_phase(Zero{}, 0, fr[0]);
        int l = 0;
        for (; l + 2 < len; l += 2) {
            line(l, Zero{}, std::false_type{});
            line(l + 1, One{}, std::false_type{});
        }
        if (l + 1 < len) {
            line(l, Zero{}, std::false_type{});
            line(l + 1, One{}, std::true_type{});
        } else {
            line(l, Zero{}, std::true_type{});
        }
    }

    if (g.ksplit > 1) {
        GemmArgs part = g;  // the slab's [M, N] FP32 matrix of partial sums; splitk_reduce_kernel scales and rounds
        part.y = g.ws + (int64_t)slab * g.M * g.N;
        part.ldy = g.N;
        small_tile_finish<TM, TN, S, false>(part, acc, 1.0f, m0, n0, wave, lane);
    } else {
        small_tile_finish<TM, TN, S, OUT_BF16>(g, acc, scale, m0, n0, wave, lane);
    }
}

// Second pass of the slab-split product: y[m][n] = round(scale * (ws[0][m][n] + ws[1][m][n] + ...)),
// slabs added in ascending order.  One thread per four consecutive columns (N % 4 == 0 here).
template <bool OUT_BF16>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs g)
{
    const int64_t quads_per_row = g.N / 4, total = g.M * quads_per_row;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int64_t m = i / quads_per_row, n = (i - m * quads_per_row) * 4;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 *p = reinterpret_cast<const f32x4 *>(g.ws + m * g.N + n);
    const int64_t slab_quads = g.M * g.N / 4;
    f32x4 sum = p[0];
    for (int sl = 1; sl < g.ksplit; ++sl) sum += p[sl * slab_quads];
    if (g.a_alpha) sum *= (*g.a_alpha) * (*g.b_alpha);  // NVFP4: the two tensor-level scales; BF16: none
    if constexpr (OUT_BF16) {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        const bf16x4 o = {(__bf16)sum[0], (__bf16)sum[1], (__bf16)sum[2], (__bf16)sum[3]};
        *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(g.y) + m * g.ldy + n) = o;
    } else {
        *reinterpret_cast<f32x4 *>(static_cast<float *>(g.y) + m * g.ldy + n) = sum;
    }
}

// ---- BF16, direct global-to-LDS loads ----------------------------------------------------------

// Loads 8 rows x 128 bytes (one 64-wide K step of eight rows, 1 KB) from global memory straight into
// LDS at `dst`; lane l brings 16 bytes of row l / 8.  In inline assembly because the
// compiler orders every LDS read behind all outstanding LDS-writing loads (s_waitcnt vmcnt(0) right
// after the load), which serialises a pipeline; with it the only waits are the ones written.  m0 is named as clobbered
// so that the compiler never keeps a value of its own in it across the statement (it calls m0 "reserved" and
// warns about any clobber of it: silenced here).  STREAM: non-temporal, for rows of W that no other workgroup reads.
template <bool STREAM>
__device__ __forceinline__ void load_rows_to_lds(uint32_t dst, uint32_t lane_off, const char *base)
{
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(dst), "v"(lane_off), "s"(base)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(dst), "v"(lane_off), "s"(base)
                     : "memory", "m0");
#pragma clang diagnostic pop
}

// The order in which a workgroup takes its K steps: groups of four in turn, each from a step of its own on.  Workgroups of
// one XCD that read the same rows would otherwise all reach a K step together, and all of them wait for its trip from
// memory; so one of them makes the trip and the others, a step or two later, find the lines in L2.  It is the tiles in one column
// (tm), which share rows of W, that have to differ: with a start from tn alone the gain is gone (1.00 of the time without).  So
// the order of a row's FP32 sums depends on its tile.
// K slabs always; else from K = 4096 on.  Staged tiles, weights from HBM, with / without it over 2549 shapes: 0.96 of the time at K = 4096, 0.94
// beyond, where W is less than 16 MB 0.94 and 0.91 (2496 tokens on K = 5120, N = 896 43 us without, 34 with; 671 on N = 1792 32 and 25),
// 0.75 to 1.09; 10 % of the shapes are more than 1.5 % slower, those whose tiles had shared the XCDs' trips well already (2227
// tokens on K = 4096, N = 768 21.3 and 23.2; 769 on N = 1536 19.7 and 20.8, but 762 24.4 and 20.0), which K and N do not tell.  With slabs 0.944.
// A shorter K has the first trip of every line at its start, where four times as many different lines in flight cost more (staged
// tiles, K = 512 to 1800 1.035, 2000 to 4000 0.95 to 1.01).  Where W waits in the last-level cache, there is less of a trip to share: 1.02 to
// 1.03 at K = 4096, 1.01 to 1.02 beyond, 1.015 in gemm_bf16_d2l; the rule cannot see that.  Groups of two or eight: the same within 1 %.
struct KOrder {
    int KT, whole, first;
    __device__ __forceinline__ KOrder(int kt, bool own, int tm, int tn)
        : KT(kt), whole(own ? kt & ~3 : 0), first(__builtin_amdgcn_readfirstlane(tm + 2 * tn))
    {
    }
    __device__ __forceinline__ int at(int k) const
    {
        k = k < KT ? k : KT - 1;  // past the end: a step that was read before, never used
        return k < whole ? (k & ~3) | ((k + first) & 3) : k;
    }
    static constexpr int64_t kFrom = 4096;  // K
};

// Until at most `N` of this wave's loads are in flight (the counter holds 63) and its LDS reads are done.
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N < 63 ? N : 63) : "memory");
}

// 256x256x64 tile with four waves of 128x128 (one per SIMD), 256x192 with 128x96 and 256x128 with 128x64.  The tiles never
// pass through registers: every wave issues 16 global_load_lds_dwordx4 per K step (1 KB each: 8 rows of one
// operand tile), which write LDS at M0 + 16 * lane.  The bank swizzle is applied on the global side: the lane that fills chunk c' of
// row r fetches chunk c' ^ key(r).  The only wait is the one before the
// barrier.
// The loads of tile t+2 are issued one per two MFMAs: B's in the phase behind the barrier that frees their stage, A's in
// the first phase of K step t, into the third stage that the 160 KB of LDS hold for A: four and seven phases before the
// barrier that waits for them.  With two stages of both A's came half a K step later, and their wait was what a K step took
// beyond its MFMAs; K steps in an order of the workgroup's own (KOrder) take another 1 to 6 % off (matrix pipe busy 80 -> 88 % of
// cycles).  us, two stages / three / three and own order: 4096 tokens on K = 4096, N = 6144 187 (in 256x192 staged tiles) / 163 / 160;
// 8192 on K = 14336, N = 4096 725 / 688 / 668; 8192 on K = 4096, N = 28672 1428 / 1422 / 1380; 2048 on N = 4096
// in 256x128 tiles 73 / 63 / 62.  (All 16 loads in one phase: 3 to 8 % slower, the texture path is shared by the four waves and the same
// instants see everybody's loads; 16x16 MFMAs in the same pipeline: no faster, nor the row's MFMAs in alternating order.)
template <class C, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_bf16_d2l(GemmArgs g, int tiles_m, int tiles_n)
{
    static_assert(C::THREADS == 256, "four waves");
    constexpr int GA = C::BM / 32, GB = C::BN / 32, NL = GA + GB;  // 8-row groups per wave and operand
    extern __shared__ uint4 lds[];
    char *const L = reinterpret_cast<char *>(lds);
    int tm, tn;
    tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave / C::WAVES_N) * C::WM, wn0 = (wave % C::WAVES_N) * C::WN;
    const int frow = lane & 31, fhalf = lane >> 5;
    const int KT = (int)(g.K / BK);
    const KOrder order(KT, g.K >= KOrder::kFrom, tm, tn);

    // load u of this wave: rows 8 * (wave * GA + u) .. + 7 of the A tile (u < GA), else of the B tile
    // byte offsets from the tile's first row: 32 bits for any operand size
    uint32_t vo[NL];
    const char *const ta = static_cast<const char *>(g.a) + m0 * g.lda * 2;  // m0 < M, n0 < N
    const char *const tb = static_cast<const char *>(g.b) + n0 * g.ldb * 2;
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const bool isA = u < GA;
        const int r = 8 * (isA ? wave * GA + u : wave * GB + (u - GA)) + (lane >> 3);
        int64_t grow = (isA ? m0 : n0) + r;
        const int64_t total = isA ? g.M : g.N;
        grow = grow < total ? grow : total - 1;
        vo[u] = (uint32_t)((grow - (isA ? m0 : n0)) * (isA ? g.lda : g.ldb) * 2 + (((lane & 7) ^ swz_key(r)) * 16));
    }
    // LDS byte address of the dynamic segment
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)L;
    // load u of the K step that starts `ko` bytes into the rows, into the A stage at byte `sa` (u < GA) or the B stage `sb`
    auto load_group = [&](int64_t ko, uint32_t sa, int sb, int u) {
        const bool isA = u < GA;
        const char *base = (isA ? ta : tb) + ko;
        const uint32_t dst = lds0 + (isA ? sa + (wave * GA + u) * 1024
                                         : C::B_BASE + sb * C::B_STAGE + (wave * GB + (u - GA)) * 1024);
        load_rows_to_lds<false>(dst, vo[u], base);
    };

    int fa[4], fb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        fa[ks] = ((wm0 + frow) * 8 + ((ks * 2 + fhalf) ^ swz_key(frow))) * 16;
        fb[ks] = C::B_BASE + ((wn0 + frow) * 8 + ((ks * 2 + fhalf) ^ swz_key(frow))) * 16;
    }
    uint4 fra[2][C::TM], frb[2][C::TN];
    f32x16 acc[C::TM][C::TN];
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    constexpr int NMFMA = C::TM * C::TN;

#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int u = 0; u < NL; ++u) load_group((int64_t)order.at(d) * (BK * 2), d * C::A_STAGE, d, u);
    wait_loads<NL>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < C::TM; ++i) fra[0][i] = *reinterpret_cast<const uint4 *>(L + fa[0] + i * 4096);
#pragma unroll
    for (int j = 0; j < C::TN; ++j) frb[0][j] = *reinterpret_cast<const uint4 *>(L + fb[0] + j * 4096);

    // One phase: the MFMAs of one 16-wide K sub-step on fragments (ca, cb); meanwhile the
    // fragments of sub-step ks of the stages (ra, rb) are read into (na, nb), one per MFMA while any remain,
    // and loads [U0, U1) of tile t go to the stages (la, lb), spread evenly over the MFMAs.
    auto phase = [&](const uint4(&ca)[C::TM], const uint4(&cb)[C::TN], uint4(&na)[C::TM], uint4(&nb)[C::TN], int ks,
                     uint32_t ra, int rb, int t, uint32_t la, int lb, auto u0c, auto u1c) {
        constexpr int U0 = decltype(u0c)::value, U1 = decltype(u1c)::value;
        const char *const pa = L + fa[ks] + ra;
        const int64_t ko = U0 < U1 ? (int64_t)order.at(t) * (BK * 2) : 0;
#pragma unroll
        for (int n = 0; n < NMFMA; ++n) {
            const int i = n / C::TN, j = n % C::TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, ca[i]), __builtin_bit_cast(bf16x8, cb[j]), acc[i][j], 0, 0, 0);
            if (n < C::TM)
                na[n] = *reinterpret_cast<const uint4 *>(pa + n * 4096);
            else if (n < C::TM + C::TN)
                nb[n - C::TM] = *reinterpret_cast<const uint4 *>(L + fb[ks] + (n - C::TM) * 4096 + rb * C::B_STAGE);
#pragma unroll
            for (int u = U0 + n * (U1 - U0) / NMFMA; u < U0 + (n + 1) * (U1 - U0) / NMFMA; ++u) load_group(ko, la, lb, u);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using U_0 = std::integral_constant<int, 0>;
    using U_A = std::integral_constant<int, GA>;
    using U_N = std::integral_constant<int, NL>;
    // A stages of this K step, the next one and the one after it, in turn
    uint32_t a0 = 0, a1 = C::A_STAGE, a2 = 2 * C::A_STAGE;
    auto kstep = [&](int kt, auto par) {
        constexpr int cur = decltype(par)::value, nxt = cur ^ 1;
        phase(fra[0], frb[0], fra[1], frb[1], 1, a0, cur, kt + 2, a2, 0, U_0{}, U_A{});
        phase(fra[1], frb[1], fra[0], frb[0], 2, a0, cur, 0, 0, 0, U_N{}, U_N{});
        phase(fra[0], frb[0], fra[1], frb[1], 3, a0, cur, 0, 0, 0, U_N{}, U_N{});
        // tile kt+1 has landed in this wave's share of its stages (the A loads of tile kt+2 may still be on their
        // way), after the barrier in everyone's, and nobody reads the stages of tile kt any more (this wave's last
        // fragment reads of them have returned: lgkmcnt, which the MFMAs behind the barrier would wait for
        // anyway): B's receives tile kt+2 now, A's tile kt+3 in the next K step
        wait_loads<GA>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        phase(fra[1], frb[1], fra[0], frb[0], 0, a1, nxt, kt + 2, 0, cur, U_A{}, U_N{});
        const uint32_t t = a0;
        a0 = a1, a1 = a2, a2 = t;
    };
    int kt = 0;
    for (; kt + 1 < KT; kt += 2) {
        kstep(kt, std::integral_constant<int, 0>{});
        kstep(kt + 1, std::integral_constant<int, 1>{});
    }
    if (kt < KT) kstep(kt, std::integral_constant<int, 0>{});
    wait_loads<0>();  // the clamped loads past the end still target LDS

    epilogue<C, OUT_BF16>(g, acc, 1.0f, m0, n0, wm0, wn0, frow, fhalf);
}

// ---- BF16, tiles of 16x16 MFMAs: decode batches and everything up to a few thousand tokens --------

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Lane offset (bytes from the first row of the tile) of load group `rr / 8`: row rr of the tile, clamped to
// the last of `total` rows, with the bank swizzle applied on the global side.
__device__ __forceinline__ uint32_t row_offset(int64_t first, int rr, int64_t total, int64_t ld, int lane)
{
    int64_t row = first + rr;
    row = row < total ? row : total - 1;
    return (uint32_t)((row - first) * ld * 2 + (((lane & 7) ^ swz_key(rr)) * 16));
}

// Accumulator i of a 16x16 tile (W rows as the A operand, tokens as the B operand): W row 4 (lane / 16) + i,
// token lane % 16, i.e. four consecutive columns of one row of Y.
template <bool OUT_BF16>
__device__ __forceinline__ void store_quad(const GemmArgs &g, f32x4 v, int64_t m, int64_t n)
{
    using T = std::conditional_t<OUT_BF16, __bf16, float>;
    if (m >= g.M || n >= g.N) return;
    T *dst = static_cast<T *>(g.y) + m * g.ldy + n;
    if constexpr (!OUT_BF16) {
        // (a copy that the compiler cannot see through: it may store quads straight from accumulation registers,
        // and then kept the accumulators of the staged kernels half in one kind of register and half in the other
        // and moved all of them twice per K step)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = v[i];
            float c;
            asm("v_mov_b32 %0, %1" : "=v"(c) : "v"(a));
            v[i] = c;
        }
    }
    if (n + 3 < g.N) {
        if constexpr (OUT_BF16) {
            typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
            *reinterpret_cast<bf16x4 *>(dst) = bf16x4{(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        } else {
            *reinterpret_cast<f32x4 *>(dst) = v;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (n + i < g.N) dst[i] = (T)v[i];
    }
}

// Decode batches: a narrow tile per workgroup, its S waves take the 64-wide K steps in turn.
//
// What bounds these sizes is the weights' one trip from HBM, and the activations' trips from L2 to
// the compute units (every workgroup reads its 16 MT tokens for 16 NT rows of W).  Tiles are
// therefore narrow (a workgroup for every compute unit even at N = 4096) and every byte is fetched in
// whole 128-byte lines: a lane-per-row load in MFMA operand order touches 64 different lines per
// instruction and moves a quarter of the bytes per clock (the kernels that this one replaced did
// that: 64 tokens, K = N = 4096, 22.5 us against 12.2 here; 16 tokens 11.8 against 8.8).  Each wave owns
// a private ring of two slots in LDS, one K step of X and W rows each, filled by direct-to-LDS loads:
// no barrier in the K loop, and every byte is read back once, into registers, before the MFMAs of
// the previous step, after which its slot is refilled at once, so a wave always has between one and
// two steps of loads in flight (three or four slots: no faster).  The S partial tiles are added through
// LDS in wave order (bit-identical from run to run).  Measured over the four layers of the 8B shapes,
// weights from HBM, in us (this kernel / before / one trip of the weights at 5.3 TB/s): 16 tokens
// 90 / 115 / 82, 48 tokens 112 / 159 / 82, 64 tokens 121 / 170 / 82.
// g.ksplit > 1: a work item is (K slab, tile), its FP32 partial sums go to g.ws[slab][M][N] and
// splitk_reduce_kernel adds the slabs in ascending order.
template <int MT, int NT, int S, bool STREAM, bool OUT_BF16>
__global__ __launch_bounds__(64 * S) void bf16_ring_kernel(GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int D = 2;                      // slots per wave
    constexpr int NL = 2 * (MT + NT);         // loads per K step: eight rows each
    constexpr int SLOT = NL * 1024, NF = MT + NT, T = MT * NT;
    extern __shared__ uint4 lds[];
    char *const L = reinterpret_cast<char *>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = tiles_m * tiles_n;
    const int item = logical_id(blockIdx.x, tiles * g.ksplit);
    const int slab = item / tiles, t = item - slab * tiles;
    const int64_t m0 = (int64_t)(t % tiles_m) * (16 * MT), n0 = (int64_t)(t / tiles_m) * (16 * NT);
    const int KT = (int)(g.K / BK);
    const int SL = (KT + g.ksplit - 1) / g.ksplit;
    const int s0 = slab * SL < KT ? slab * SL : KT, s1 = s0 + SL < KT ? s0 + SL : KT;
    const int steps = s1 - s0 > wave ? (s1 - s0 - wave + S - 1) / S : 0;  // of this wave: s0 + wave, + S, ...

    uint32_t vo[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u)
        vo[u] = u < 2 * MT ? row_offset(m0, u * 8 + (lane >> 3), g.M, g.lda, lane)
                           : row_offset(n0, (u - 2 * MT) * 8 + (lane >> 3), g.N, g.ldb, lane);
    const char *const tx = static_cast<const char *>(g.a) + m0 * g.lda * 2;  // m0 < M, n0 < N
    const char *const tw = static_cast<const char *>(g.b) + n0 * g.ldb * 2;
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)L + wave * (D * SLOT);
    auto load_step = [&](int i, int slot) {
        const int k = s0 + wave + i * S;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            if (u < 2 * MT)
                load_rows_to_lds<false>(ring + slot * SLOT + u * 1024, vo[u], tx + (int64_t)k * (BK * 2));
            else
                load_rows_to_lds<STREAM>(ring + slot * SLOT + u * 1024, vo[u], tw + (int64_t)k * (BK * 2));
        }
    };
    const int row = lane & 15, grp = lane >> 4;
    const int f0 = wave * (D * SLOT) + row * 128 + ((grp ^ swz_key(row)) * 16);
    const int f1 = wave * (D * SLOT) + row * 128 + (((4 + grp) ^ swz_key(row)) * 16);
    uint4 fr[2][2][NF];  // [register set][half of the K step][token tiles, then W tiles]
    auto read_step = [&](int slot, uint4(&f)[2][NF]) {
#pragma unroll
        for (int q = 0; q < NF; ++q) {
            f[0][q] = *reinterpret_cast<const uint4 *>(L + f0 + slot * SLOT + q * 2048);
            f[1][q] = *reinterpret_cast<const uint4 *>(L + f1 + slot * SLOT + q * 2048);
        }
    };
    f32x4 acc[NT][MT];
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // (steps is uniform over the wave; nothing is loaded past the end: with eight waves on K = 4096 two
    // idle steps per wave would be a quarter of all loads)
    if (steps > 0) load_step(0, 0);
    if (steps > 1) {
        load_step(1, 1);
        wait_loads<NL>();
    } else {
        wait_loads<0>();
    }
    if (steps > 0) read_step(0, fr[0]);
    // step i: its fragments are in register set i % 2 (or on their way there), its slot is `slot`
    auto kstep = [&](int i, int slot, auto setc) {
        constexpr int P = decltype(setc)::value;
        if (i + D < steps) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // slot read: refill it
            load_step(i + D, slot);
            wait_loads<NL>();                                   // the other slot (step i + 1) has landed
        } else {
            wait_loads<0>();
        }
        if (i + 1 < steps) read_step(slot ^ 1, fr[P ^ 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int a = 0; a < NT; ++a)
#pragma unroll
                for (int b = 0; b < MT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fr[P][k][MT + a]),
                                                                        __builtin_bit_cast(bf16x8, fr[P][k][b]),
                                                                        acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    int i = 0;
    for (; i + 1 < steps; i += 2) {
        kstep(i, 0, std::integral_constant<int, 0>{});
        kstep(i + 1, 1, std::integral_constant<int, 1>{});
    }
    if (i < steps) kstep(i, 0, std::integral_constant<int, 0>{});
    __syncthreads();  // every wave is done with its ring: the partial tiles go there

    f32x4 *const X = reinterpret_cast<f32x4 *>(lds);
#pragma unroll
    for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) X[(wave * T + a * MT + b) * 64 + lane] = acc[a][b];
    __syncthreads();
    for (int q = wave; q < T; q += S) {
        f32x4 sum = X[q * 64 + lane];
        for (int w = 1; w < S; ++w) sum += X[(w * T + q) * 64 + lane];
        const int64_t m = m0 + (q % MT) * 16 + row, n = n0 + (q / MT) * 16 + 4 * grp;
        if (g.ksplit > 1) {  // unscaled partial sums of this slab (N % 4 == 0 here)
            if (m < g.M && n < g.N) *reinterpret_cast<f32x4 *>(g.ws + ((int64_t)slab * g.M + m) * g.N + n) = sum;
        } else {
            store_quad<OUT_BF16>(g, sum, m, n);
        }
    }
}

// A few tokens against a short K: the same tile, K order and sums as bf16_ring_kernel<1, 1, S>, but every lane
// loads its fragments straight into registers, two K steps per wave in flight.  With one or two steps per
// wave there is no stream to keep up; what counts is the latency of one load, and the trip through the ring
// is added to it.  us, here / in the ring / in the register-streaming kernel before both: one token on K = 256, N = 4096
// 4.4 / 4.8 / 4.4, K = 512 4.8 / 5.1 / 4.8, K = 1024 5.5 / 5.8 / 5.5 (K = 2048 7.2 / 7.3 / 7.1: left to the
// ring); 16 tokens, K = 512 5.2 / 5.2 / 5.1.
template <int S, bool OUT_BF16>
__global__ __launch_bounds__(64 * S) void bf16_short_kernel(GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int D = 2;
    __shared__ f32x4 X[S * 64];
    const int tid = threadIdx.x, lane = tid & 63, row = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = logical_id(blockIdx.x, tiles_m * tiles_n);
    const int64_t m0 = (int64_t)(t % tiles_m) * 16, n0 = (int64_t)(t / tiles_m) * 16;  // m0 < M, n0 < N
    const int KT = (int)(g.K / BK);
    const int64_t mr = m0 + row < g.M ? m0 + row : g.M - 1, nr = n0 + row < g.N ? n0 + row : g.N - 1;
    const uint4 *const px = reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(g.a) + mr * g.lda) + grp;
    const uint4 *const pw = reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(g.b) + nr * g.ldb) + grp;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = wave; k0 < KT; k0 += D * S) {
        uint4 x[D][2], w[D][2];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int64_t k = k0 + d * S;
            if (k < KT) {  // uniform
                w[d][0] = pw[k * 8], w[d][1] = pw[k * 8 + 4];
                x[d][0] = px[k * 8], x[d][1] = px[k * 8 + 4];
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (k0 + d * S < KT)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[d][h]),
                                                                  __builtin_bit_cast(bf16x8, x[d][h]), acc, 0, 0, 0);
    }
    X[wave * 64 + lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    for (int w = 1; w < S; ++w) acc += X[w * 64 + lane];
    store_quad<OUT_BF16>(g, acc, m0 + row, n0 + 4 * grp);
}

// From about a hundred tokens: a (16 TM WM) x (16 TN WN) tile per workgroup of WM x WN waves, NST stages of
// 64-wide K steps in LDS filled by direct-to-LDS loads, one barrier per K step.  Same row layout, swizzle
// and fragment order as above.  A K step is two phases of 32: the fragments of the next phase are
// read while the MFMAs of the current one run, the barrier stands in front of the second phase, and
// the stage it frees receives the K step NST ahead, so NST - 1 steps of loads are in flight at the
// barrier's wait.  That depth is what the two-stage kernels of the same tiles lacked: their K step
// waited for HBM (256x128 tile, 2048 tokens, K = 14336, N = 4096: 251 us with two stages, 186 with
// three; 128x64 tile, 512 tokens: 93 against 211 for a register-staged 128x128 tile with one step of
// look-ahead).  Beyond 96 to 144 KB of stages nothing is gained.  What bounds them then is the
// LDS: a tile's bytes are written once at 64 and its fragments read at 128 bytes per clock, and, with few tiles to a
// long K, what a compute unit loads: 48 to 55 bytes per ns whatever the depth (32 KB of lines in flight).  There K
// slabs across workgroups (SLABS) allow larger tiles, whose operands are fewer bytes per product: 200 tokens on
// K = 14336, N = 4096 3.7 MB per unit and 51 us in 64x64 tiles, 1.8 MB and 41 us in 128x128 with four slabs, second pass included.
template <int TM, int TN, int WM, int WN, int NST, bool SLABS, bool OUT_BF16>
__global__ __launch_bounds__(64 * WM * WN) void bf16_stage_kernel(GemmArgs g, int tiles_m, int tiles_n)
{
    constexpr int W = WM * WN, BM = 16 * TM * WM, BN = 16 * TN * WN, STAGE = (BM + BN) * 128;
    constexpr int NLX = BM / 8 / W, NL = (BM + BN) / 8 / W;  // loads per wave and K step: X, all
    constexpr int NF = TM + TN, NM = TM * TN;
    static_assert(BM / 8 % W == 0 && BN / 8 % W == 0, "whole loads per wave");
    extern __shared__ uint4 lds[];
    char *const L = reinterpret_cast<char *>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = tiles_m * tiles_n, item = logical_id(blockIdx.x, SLABS ? tiles * g.ksplit : tiles);
    const int slab = SLABS ? item / tiles : 0;
    int tm, tn;
    tile_of_logical(item - slab * tiles, tiles_m, tiles_n, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int wm0 = (wave / WN) * (16 * TM), wn0 = (wave % WN) * (16 * TN);
    // this slab's K steps [s0, s0 + KT): the launcher leaves no slab empty
    const int KA = (int)(g.K / BK), SL = SLABS ? (KA + g.ksplit - 1) / g.ksplit : KA;
    const int s0 = slab * SL, KT = s0 + SL < KA ? SL : KA - s0;

    const KOrder order(KT, SLABS || g.K >= KOrder::kFrom, tm, tn);

    uint32_t vo[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u)
        vo[u] = u < NLX ? row_offset(m0, (u * W + wave) * 8 + (lane >> 3), g.M, g.lda, lane)
                        : row_offset(n0, ((u - NLX) * W + wave) * 8 + (lane >> 3), g.N, g.ldb, lane);
    const char *const tx = static_cast<const char *>(g.a) + m0 * g.lda * 2 + (int64_t)s0 * (BK * 2);  // m0 < M, n0 < N
    const char *const tw = static_cast<const char *>(g.b) + n0 * g.ldb * 2 + (int64_t)s0 * (BK * 2);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)L;
    // load u of the K step that starts `ko` bytes into the rows
    auto load_group = [&](int64_t ko, uint32_t stage, int u) {
        if (u < NLX)
            load_rows_to_lds<false>(lds0 + stage + (u * W + wave) * 1024, vo[u], tx + ko);
        else
            load_rows_to_lds<false>(lds0 + stage + BM * 128 + ((u - NLX) * W + wave) * 1024, vo[u], tw + ko);
    };
    const int row = lane & 15, grp = lane >> 4;
    int fx[2], fw[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int c = ((4 * k + grp) ^ swz_key(row)) * 16;
        fx[k] = (wm0 + row) * 128 + c;
        fw[k] = BM * 128 + (wn0 + row) * 128 + c;
    }
    uint4 fr[2][NF];
    auto read_frag = [&](uint32_t stage, int k, int q) {
        return *reinterpret_cast<const uint4 *>(L + stage + (q < TM ? fx[k] + q * 2048 : fw[k] + (q - TM) * 2048));
    };
    f32x4 acc[TN][TM];
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // The MFMAs on fragments f; between them the fragments of half `k` of `stage` into nf, and (LOAD) the
    // loads of K step kl into `lstage`, both spread evenly.
    auto phase = [&](const uint4(&f)[NF], uint4(&nf)[NF], int k, uint32_t stage, int kl, uint32_t lstage, auto loadc) {
        constexpr bool LOAD = decltype(loadc)::value;
        const int64_t ko = LOAD ? (int64_t)order.at(kl) * (BK * 2) : 0;
#pragma unroll
        for (int n = 0; n < NM; ++n) {
#pragma unroll
            for (int q = n * NF / NM; q < (n + 1) * NF / NM; ++q) nf[q] = read_frag(stage, k, q);
            if constexpr (LOAD)
#pragma unroll
                for (int u = n * NL / NM; u < (n + 1) * NL / NM; ++u) load_group(ko, lstage, u);
            acc[n / TM][n % TM] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[TM + n / TM]),
                                                                          __builtin_bit_cast(bf16x8, f[n % TM]),
                                                                          acc[n / TM][n % TM], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int d = 0; d < NST; ++d)
#pragma unroll
        for (int u = 0; u < NL; ++u) load_group((int64_t)order.at(d) * (BK * 2), d * STAGE, u);
    wait_loads<(NST - 1) * NL>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < NF; ++q) fr[0][q] = read_frag(0, 0, q);
    uint32_t cur = 0;
    for (int k = 0; k < KT; ++k) {
        const uint32_t nxt = cur + STAGE < NST * STAGE ? cur + STAGE : 0;
        phase(fr[0], fr[1], 1, cur, 0, 0, std::false_type{});
        // K step k + 1 has landed in this wave's share of stage nxt, after the barrier in everyone's, and
        // nobody reads stage cur any more (the waits cover this wave's last fragment reads of it)
        wait_loads<(NST - 2) * NL>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        phase(fr[1], fr[0], 0, nxt, k + NST, cur, std::true_type{});
        cur = nxt;
    }
    wait_loads<0>();  // the loads past the end still target LDS

    GemmArgs out = g;
    if constexpr (SLABS) {
        // the slab's [M, N] FP32 matrix of partial sums, through store_quad and its copy like any other output: with quads stored straight
        // from the accumulators seven of the eight tiles moved all of them in every K step, us moved / clean: 300 tokens on K = 14336,
        // N = 4096 (160x128, three slabs) 67 / 57; 0.88 of the time in 160x128 on 460 shapes, 0.94 in 96x128, 0.97 in 96x64
        out.y = g.ws + (int64_t)slab * g.M * g.N;
        out.ldy = g.N;
    }
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
            store_quad<OUT_BF16>(out, acc[a][b], m0 + wm0 + b * 16 + row, n0 + wn0 + a * 16 + 4 * grp);
}

// ---- fallback for K not a multiple of 64: one thread per output, exact products ---------------

__device__ __forceinline__ float e2m1_f32(uint32_t c)
{
    const uint32_t m = c & 7u;
    float v = (m >= 2u) ? __uint_as_float((((m >> 1) + 126u) << 23) | ((m & 1u) << 22)) : 0.5f * (float)m;
    return (c & 8u) ? -v : v;
}

template <bool FP4, bool OUT_BF16>
__global__ __launch_bounds__(256) void gemm_simple_kernel(GemmArgs g)
{
    const int64_t n = (int64_t)blockIdx.x * 16 + (threadIdx.x & 15);
    const int64_t m = (int64_t)blockIdx.y * 16 + (threadIdx.x >> 4);
    if (m >= g.M || n >= g.N) return;
    float acc = 0.0f;
    if constexpr (FP4) {
        const uint8_t *ac = static_cast<const uint8_t *>(g.a) + m * g.a_c_row;
        const uint8_t *bc = static_cast<const uint8_t *>(g.b) + n * g.b_c_row;
        const uint8_t *as = g.a_scales + m * g.a_s_row, *bs = g.b_scales + n * g.b_s_row;
        for (int64_t b = 0; b < g.K / 16; ++b) {
            // block b of a row: K step b/4 (stride *_step), 8 code bytes and 1 scale byte at b%4
            const uint8_t *xa = ac + (b >> 2) * g.a_c_step + (b & 3) * 8;
            const uint8_t *xb = bc + (b >> 2) * g.b_c_step + (b & 3) * 8;
            float dot = 0.0f;  // sum of 16 products q*q: multiples of 1/4 up to 576, exact
            for (int i = 0; i < 8; ++i) {
                const uint32_t x = xa[i], w = xb[i];
                dot += e2m1_f32(x & 15u) * e2m1_f32(w & 15u);
                dot += e2m1_f32(x >> 4) * e2m1_f32(w >> 4);
            }
            const float sx = __builtin_amdgcn_cvt_pk_f32_fp8((int)as[(b >> 2) * g.a_s_step + (b & 3)], false)[0];
            const float sw = __builtin_amdgcn_cvt_pk_f32_fp8((int)bs[(b >> 2) * g.b_s_step + (b & 3)], false)[0];
            acc += (sx * sw) * dot;
        }
        acc *= (*g.a_alpha) * (*g.b_alpha);
    } else {
        const uint16_t *a = static_cast<const uint16_t *>(g.a) + m * g.lda;
        const uint16_t *b = static_cast<const uint16_t *>(g.b) + n * g.ldb;
        for (int64_t k = 0; k < g.K; ++k)
            acc += __uint_as_float((uint32_t)a[k] << 16) * __uint_as_float((uint32_t)b[k] << 16);
    }
    if constexpr (OUT_BF16)
        static_cast<__bf16 *>(g.y)[m * g.ldy + n] = (__bf16)acc;
    else
        static_cast<float *>(g.y)[m * g.ldy + n] = acc;
}

// ---- matrix-pipe rate probe -------------------------------------------------------------------

// A loop of independent v_mfma_f32_32x32x16_f16 on pseudo-random operands, one wave per SIMD,
// nothing else: what the matrix pipe sustains on this chip at the clock its power management
// allows for realistic operand toggling.  Used by the benchmark as the measured roof next to the
// published peak.
__global__ __launch_bounds__(256) void mfma_probe_kernel(float *out, int iters)
{
    f16x8 a[4], b[4];
    f32x16 c0, c1, c2, c3;
    unsigned h = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
    for (int q = 0; q < 4; ++q)
        for (int j = 0; j < 8; ++j) {
            h = h * 1664525u + 1013904223u;
            a[q][j] = (_Float16)(((int)(h >> 20) - 2048) * (1.0f / 512.0f));
            h = h * 1664525u + 1013904223u;
            b[q][j] = (_Float16)(((int)(h >> 20) - 2048) * (1.0f / 512.0f));
        }
    for (int r = 0; r < 16; ++r) c0[r] = c1[r] = c2[r] = c3[r] = 0.0f;
    for (int i = 0; i < iters; ++i) {
        c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[0], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[1], c1, 0, 0, 0);
        c2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[2], b[2], c2, 0, 0, 0);
        c3 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[3], b[3], c3, 0, 0, 0);
        c0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[1], b[2], c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[2], b[3], c1, 0, 0, 0);
        c2 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[3], b[0], c2, 0, 0, 0);
        c3 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[0], b[1], c3, 0, 0, 0);
    }
    float s = 0.0f;
    for (int r = 0; r < 16; ++r) s += c0[r] + c1[r] + c2[r] + c3[r];
    if (s == 123.456f) out[0] = s;  // keeps the loop alive; practically never true
}

// ---- launchers ------------------------------------------------------------------------------

template <class Kern>
int launch_tiles(Kern kern, size_t lds_bytes, int bm, int bn, int threads, const GemmArgs &g, hipStream_t s)
{
    const int64_t tiles_m = (g.M + bm - 1) / bm, tiles_n = (g.N + bn - 1) / bn;
    if (tiles_m * tiles_n > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    return enqueue(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(threads), lds_bytes, s, g, (int)tiles_m, (int)tiles_n);
}

// Persistent register-direct kernels: one workgroup per compute unit (a wave of 512 registers
// fills its SIMD), each walking tile ids wg, wg + grid, ...
inline int compute_units(int &n)
{
    static std::atomic<int> cus{0};
    n = cus.load(std::memory_order_acquire);
    if (n == 0) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return note_launch(e);
        n = n >= NUM_XCD ? n / NUM_XCD * NUM_XCD : NUM_XCD;  // a multiple of the XCD count keeps wg % 8 = XCD
        cus.store(n, std::memory_order_release);
    }
    return MQ_OK;
}

template <class Kern>
int launch_persistent(Kern kern, int bm, int bn, size_t lds_bytes, const GemmArgs &g, hipStream_t s, int cus)
{
    const int64_t tiles_m = (g.M + bm - 1) / bm, tiles_n = (g.N + bn - 1) / bn;
    if (tiles_m * tiles_n > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    const int64_t grid = tiles_m * tiles_n < cus ? tiles_m * tiles_n : cus;
    return enqueue(kern, dim3((unsigned)grid), dim3(256), lds_bytes, s, g, (int)tiles_m, (int)tiles_n);
}

template <int TM, int TN, int S>
constexpr size_t small_lds()
{
    return S == 1 ? 0 : (size_t)S * (TM * TN < 4 ? TM * TN : 4) * 4096;
}

// The second pass of a product in K slabs.
template <bool OUT_BF16>
int launch_slab_sum(const GemmArgs &g, hipStream_t s)
{
    const int64_t quads = g.M * (g.N / 4);
    return enqueue(splitk_reduce_kernel<OUT_BF16>, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, g);
}

// Row-major operands are read in whole lines (LINE) where a line is four K steps of one row and each of eight waves has one: at
// K = 1024 and 1536 half or a quarter of the waves would be idle.  Tiles of six operand rows have no registers for a line.
static bool fp4_lines(int layout, int64_t K) { return layout == MQ_LAYOUT_LINEAR && K % (4 * BK) == 0 && K >= 32 * BK; }
template <int TM, int TN, int S>
constexpr bool has_lines()
{
    return TM + TN <= 4 && S > 1;
}

// K steps of `step` bytes that a scalar offset of less than 2 GiB spans.
static int fp4_reach(int64_t step) { return (int)(0x7FFFFFFF / step); }

// By lines, 64x64 tiles of four waves stand two to a compute unit.  Where what is left behind the first 2 * cus tiles has a unit
// each to itself, it has it only if those end together: where a last row of tiles with few rows ends early, pairs form on their
// units while others stand empty.  449 to 479 tokens on K = 4096, N = 6144 (768 tiles, 256 units) took 47 to 43 us, 480 to 512 tokens
// 35; 36 with even tiles; 966 on K = 4096, N = 3072 44 and 36.  The early end is worth more with fewer tiles (65 to 96 tokens on
// N = 51200, 96 us, 105 even; 386 to 415 on N = 5120, 2.19 tiles to a unit, 39 and 41), with more (130 to 158 on N = 28672, 5.25, 65 and
// 68), where the last row is a third of all (129 on N = 14336 33.7 and 36.8), and a long K gains nothing (459 on K = 12800,
// N = 5120 88 and 92).
static bool fp4_even(int64_t tiles_m, int64_t tiles, int64_t K, int cus)
{
    return tiles > 2 * cus + cus / 4 && tiles <= 3 * cus && tiles_m >= 7 && K <= 8192;
}

// One workgroup of S waves per (32 TM) x (32 TN) tile and K slab.
template <int TM, int TN, int S, int NSETS, bool OUT_BF16, bool LINE = false>
int launch_small(const GemmArgs &g0, hipStream_t s, int slabs, int cus)
{
    if constexpr (!LINE && has_lines<TM, TN, S>())
        if (fp4_lines(g0.b_c_row == 32 ? MQ_LAYOUT_KTILE : MQ_LAYOUT_LINEAR, g0.K))
            return launch_small<TM, TN, S, 4, OUT_BF16, true>(g0, s, slabs, cus);
    GemmArgs g = g0;
    g.ksplit = slabs;
    g.reach = fp4_reach(g.a_c_step > g.b_c_step ? g.a_c_step : g.b_c_step);
    const int64_t tiles_m = (g.M + 32 * TM - 1) / (32 * TM), tiles_n = (g.N + 32 * TN - 1) / (32 * TN);
    if (tiles_m * tiles_n * g.ksplit > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    g.even = fp4_even(tiles_m, tiles_m * tiles_n * g.ksplit, g.K, cus);
    const int rc = enqueue(gemm_fp4_small<TM, TN, S, NSETS, OUT_BF16, LINE>, dim3((unsigned)(tiles_m * tiles_n * g.ksplit)),
                           dim3(64 * S), small_lds<TM, TN, S>(), s, g, (int)tiles_m, (int)tiles_n);
    return rc != MQ_OK || g.ksplit == 1 ? rc : launch_slab_sum<OUT_BF16>(g, s);
}

template <bool FP4, bool OUT_BF16>
int launch_simple(const GemmArgs &g, hipStream_t s)
{
    dim3 grid((unsigned)((g.N + 15) / 16), (unsigned)((g.M + 15) / 16));
    if ((g.M + 15) / 16 > 65535) return MQ_ERR_SHAPE;
    return enqueue(gemm_simple_kernel<FP4, OUT_BF16>, grid, dim3(256), 0, s, g);
}

// A launch holds fewer than 2^32 threads: kernels with a workgroup per tile, of up to 512 threads, take no
// more tiles than this (hundreds of millions of rows in narrow tiles), the larger tiles serve what is left.
static constexpr int64_t kMaxSmallTiles = (1ll << 23) - 1;

// ---- what a launch costs, as the choice of a tile sees it -------------------------------------------

// Time of one launch in a given tile: two things hide behind each other for the most part, the operands' one trip
// from memory (`mem` us) and the K steps of the rounds of workgroups (one per compute unit); what is written
// comes on top.  In ns: `start` once, `round` per round (first loads, sums, stores of a workgroup), `step` per K
// step and round, `share` per K step and full round by how full the chip is on average (all
// compute units busy share caches and clock: a round of 224 workgroups of 256 is no eighth cheaper, but cheaper).
// `out`: percent of what writing Y takes at 5 TB/s.
struct TileCost {
    float start, round, step, share, out;
};
static double launch_us(const TileCost &c, int64_t tiles, double kt, double mem, double hidden, double out_bytes, int cus)
{
    const double loop = ((double)((tiles + cus - 1) / cus) * (c.round + kt * c.step) + (double)tiles / cus * kt * c.share) * 1e-3;
    return c.start * 1e-3 + (loop > mem ? loop + hidden * mem : mem + hidden * loop) + c.out * 1e-2 * out_bytes / 5e6;
}

// The plans of the shapes that this thread asked for last (a program comes back with the same few): a plan is a pure
// function of its key, the search for it takes 0.4 (BF16, few tokens) to 0.8 us (NVFP4, hundreds of tokens).
template <class Plan>
struct RecentPlans {
    struct Key {
        int64_t M, N, K, slab_limit;
        int cus, order;
        bool operator==(const Key &o) const
        {
            return M == o.M && N == o.N && K == o.K && slab_limit == o.slab_limit && cus == o.cus && order == o.order;
        }
    };
    static constexpr int kEntries = 32;
    Key keys[kEntries] = {};  // (M == 0: empty; no such product reaches the search)
    Plan plans[kEntries] = {};
    template <class Search>
    const Plan &get(const Key &k, Search &&search)
    {
        const uint64_t h = ((uint64_t)k.M * 0x9E3779B97F4A7C15ull ^ (uint64_t)k.N) * 0xC2B2AE3D27D4EB4Full ^ (uint64_t)k.K;
        const int i = (int)((h * 0x9E3779B97F4A7C15ull) >> 59);
        if (!(keys[i] == k)) plans[i] = search(), keys[i] = k;
        return plans[i];
    }
};

// ---- which BF16 kernel and tile ---------------------------------------------------------------------

// The tiles (tokens x rows of W) that the BF16 kernels are built in, and their costs (above).
struct Bf16Tile {
    mq_kernel kernel;
    int bm, bn, waves;
};
#define MQ_RING(X) /* MT, NT, S */ \
    X(1, 1, 8) X(1, 2, 4) X(1, 4, 4) X(2, 1, 8) X(2, 2, 4) X(2, 4, 4) X(3, 2, 4) X(3, 4, 4) X(4, 2, 4) X(4, 4, 4) X(3, 7, 4)
#define MQ_STAGE(X) /* TM, TN, WM, WN, NST */ \
    X(3, 2, 2, 2, 6) X(4, 2, 2, 2, 4) X(3, 4, 2, 2, 4) X(4, 2, 2, 4, 4) X(5, 4, 2, 2, 4) X(7, 4, 2, 2, 3) X(8, 4, 2, 2, 3) X(8, 6, 2, 2, 2)
static constexpr Bf16Tile kBf16Tiles[] = {
#define MQ_X(MT, NT, S) {MQ_KERNEL_BF16_RING, 16 * MT, 16 * NT, S},
    MQ_RING(MQ_X)
#undef MQ_X
#define MQ_X(TM, TN, WM, WN, NST) {MQ_KERNEL_BF16_STAGE, 16 * TM * WM, 16 * TN * WN, WM * WN},
    MQ_STAGE(MQ_X)
#undef MQ_X
    {MQ_KERNEL_BF16_D2L, 256, 128, 4}, {MQ_KERNEL_BF16_D2L, 256, 192, 4}, {MQ_KERNEL_BF16_D2L, 256, 256, 4}, {MQ_KERNEL_BF16_SHORT, 16, 16, 8}};
static constexpr TileCost kBf16Costs[] = {
    {3990.7, 490.23, 33.944, 0, 215.64}, {4232.3, 285.89, 67.673, 0, 121.71}, {4290.4, 1760.9, 116.09, 0, 101.7},
    {2500, 1917.2, 67.252, 0, 400}, {4165.3, 476.99, 85.889, 0, 152.39}, {3802.9, 1712.7, 145.39, 0, 63.315},
    {4418.7, 542.73, 126.77, 0, 42.119}, {3161.5, 2935.1, 160.67, 0, 139.48}, {3178.4, 1632.6, 142.34, 3.1851, 395.14},
    {3862.2, 2348.2, 178.4, 0, 108.89}, {2134.7, 8581.8, 196.48, 21.579, 10}, {3306.3, 2445.4, 255.17, 0, 25.607},
    {3621.8, 2048.8, 209.56, 109.8, 53.171}, {3817.3, 2209.3, 219.72, 163.53, 116.05},
    {3155.8, 3662.8, 313.3, 93.312, 95.188}, {2998.9, 6086, 430.49, 59.295, 34.702},
    {2467.5, 6351.1, 397.88, 240.48, 97.026}, {2354.8, 6066.9, 636.14, 0, 134.09}, {2523.8, 8830.3, 678.75, 188.09, 35.62},
    {1771, 7053.4, 593.91, 212.65, 75.361}, {3188.5, 4334.3, 740.91, 276.68, 87.327},
    {2283, 7691.4, 903.92, 286.82, 58.652}, {2665.9, 650.8, 106.65, 17.193, 247.09}};
static_assert(sizeof(kBf16Costs) / sizeof(TileCost) == sizeof(kBf16Tiles) / sizeof(Bf16Tile), "one cost per tile");

// us: the second pass of K slabs in the staged tiles, and each MB of partial sums
static constexpr double kBf16SecondPass = 3.08, kBf16PartialSums = 0.212;

// Whether a staged tile of `bn` rows of W exists with K slabs: 256x192 runs below K = 512 only, slabs are for a long K.
constexpr bool stage_slabs(int bn) { return bn != 192; }

struct Bf16Plan {
    int tile;   // index into kBf16Tiles
    int slabs;  // K slabs across workgroups (1: none)
};

// The tile that costs least: the weights, and a third of the activations, make the trip from memory (5.3 TB/s; the other
// two thirds come from caches), of which 55 % of the shorter one of trip and K steps hides.  A tile shape that leaves
// a nearly empty last round loses to one that does not.  The costs are fitted to every tile's time on 4100 shapes
// (1 to 8192 tokens; the 8B and 32B layers, their 2-, 4- and 8-way shards and shorter, narrower and wider ones;
// weights from HBM; both output types), those of gemm_bf16_d2l and of the second pass on 2000 later ones (32 to 8192 tokens), when the
// slabs' loops were slower than they are.  On 1995 shapes outside the fit (65 to 900 tokens, K = 3000 to 25600) the choice is on average
// 1.4 % slower than the fastest tile without slabs up to K = 5120 (95 % of the shapes within 10 %), and 4 % slower than the fastest tile and
// slab count from K = 8256 on (within 20 %); of 428 choices with slabs three were slower than the best tile without, by 6 to 10 %.
// (The output type does not enter: the BF16 output is the rounded FP32 output bit for bit.)  200 tokens on K = 4096, N = 28672: the weights
// alone take 44 us, the 224x128 tile 61 to 66: what a compute unit can load bounds it.
// Slabs, when the caller's workspace allows some, shorten the K loop for a second pass: 33 to 64 tokens in narrow tiles
// (64 on K = 14336, N = 4096: 30.8 us against 36.4 without; 33 to 57 tokens 27 to 30 us); more tokens in staged tiles (100 on the
// same layer 43 -> 34 us, 200 53 -> 42, 300 59 -> 56, 400 70 -> 63, 200 on K = 25600, N = 5120 99 -> 82), where a margin of 5 % keeps
// the rule's error from costing more than slabs bring.
static Bf16Plan bf16_plan(int64_t M, int64_t N, int64_t K, int64_t slab_limit, int cus)
{
    const double kt = (double)(K / BK), mem = 2.0 * ((double)N + 0.3 * (double)M) * (double)K / 5.3e6;
    const double out_bytes = 2.0 * (double)M * (double)N;
    Bf16Plan best{0, 1};
    double best_us = 1e300;
    for (int i = 0; i < (int)(sizeof(kBf16Tiles) / sizeof(kBf16Tiles[0])); ++i) {
        const Bf16Tile &t = kBf16Tiles[i];
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        if (tiles > (t.kernel == MQ_KERNEL_BF16_D2L ? 0x7FFFFFFF : kMaxSmallTiles)) continue;
        if (t.kernel == MQ_KERNEL_BF16_SHORT && (M > 16 || K > 1024)) continue;
        // 112 rows of W: fewer trips of 33 to 48 tokens to the compute units where N is wide (48 on K = 5120, N = 51200 114 us in 48x64
        // tiles, 94 here; 40 on N = 25600 56 and 46; 33 to 48 on K = 4096, N = 28672 1 to 5 % faster) or, with K slabs, K long (48 on
        // K = 25600, N = 5120 51.1 in three slabs of 48x64, 48.9 in five of these; on 38 shapes where the rule takes it 0.68 to
        // 1.00 of the best other plan).  Fewer tokens are left to the narrow tiles, though not all are better off: 17 to 32 on K = 5120, N = 25600
        // and 51200 would take 0.86 to 0.95 of the time in this tile, on N = 28672 and 20480 1.00 to 1.10, on N = 12800 and 14336 1.26 to 1.44.
        if (t.bn == 112 && (M <= 32 || M > 48)) continue;
        // 256x192 exists twice: staged for a few K steps (1424 tokens on K = 192, N = 5384 14.3 us against 14.7), else with X one
        // stage further ahead and 32x32 products (a tenth faster from K = 512 on)
        if (t.bn == 192 && (t.kernel == MQ_KERNEL_BF16_STAGE) != (K < 512)) continue;
        auto us = [&](int64_t slabs) {
            return launch_us(kBf16Costs[i], tiles * slabs, kt / (double)slabs, mem, 0.45, out_bytes, cus);
        };
        auto take = [&](double t, int64_t slabs) {
            if (t < best_us) best_us = t, best = Bf16Plan{i, (int)slabs};
        };
        take(us(1), 1);
        if (t.kernel == MQ_KERNEL_BF16_RING && M <= 64 && 2 * tiles <= cus) {
            const int64_t slabs = cus / tiles < slab_limit ? cus / tiles : slab_limit;
            if (slabs >= 2) take(us(slabs) + 3.0, slabs);
        }
        if (t.kernel == MQ_KERNEL_BF16_STAGE && M > 64 && stage_slabs(t.bn))
            for (int64_t slabs = 2; slabs <= slab_limit && slabs * tiles <= cus; ++slabs) {
                const int64_t part = (K / BK + slabs - 1) / slabs;
                if ((slabs - 1) * part >= K / BK) continue;  // (the last one would be empty)
                take(1.05 * (us(slabs) + kBf16SecondPass + kBf16PartialSums * 4e-6 * (double)M * (double)N * (double)slabs), slabs);
            }
    }
    return best;
}

template <int MT, int NT, int S>
constexpr size_t ring_lds()
{
    constexpr size_t ring = (size_t)S * 2 * (MT + NT) * 2048, sums = (size_t)S * MT * NT * 1024;
    return ring > sums ? ring : sums;
}
template <int TM, int TN, int WM, int WN, int NST>
constexpr size_t stage_lds()
{
    return (size_t)NST * (16 * TM * WM + 16 * TN * WN) * 128;
}

template <int MT, int NT, int S, bool OUT_BF16>
int launch_ring(const GemmArgs &g0, hipStream_t s, int slabs)
{
    GemmArgs g = g0;
    g.ksplit = slabs;
    const int64_t tiles_m = (g.M + 16 * MT - 1) / (16 * MT), tiles_n = (g.N + 16 * NT - 1) / (16 * NT);
    if (tiles_m * tiles_n * slabs > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    const dim3 grid((unsigned)(tiles_m * tiles_n * slabs)), block(64 * S);
    // W rows are read by the workgroups of tiles_m tiles: non-temporal only when that is one (two percent
    // faster then, slower when the second reader finds the lines gone from L2)
    auto *const kern = tiles_m == 1 ? bf16_ring_kernel<MT, NT, S, true, OUT_BF16> : bf16_ring_kernel<MT, NT, S, false, OUT_BF16>;
    const int rc = enqueue(kern, grid, block, ring_lds<MT, NT, S>(), s, g, (int)tiles_m, (int)tiles_n);
    return rc != MQ_OK || slabs == 1 ? rc : launch_slab_sum<OUT_BF16>(g, s);
}

// W through the last-level cache (256 MB) also where one row of tiles reads it.  us of 128 tokens on K = 4096, N = 28672 (224 MB), through it /
// past it: from HBM 56.3 / 54.2, a W that waits there 38.7 / 55.5; over 66 to 256 tokens and W of 96 to 256 MB 0.94 to 1.015 of the
// time from HBM, 1.05 to 1.55 where it waits.  Larger ones: 266 MB 1.3 when read again and again, 288 to 448 MB 0.97 to 1.04
// either way, 500 MB 0.975: no line that gains and costs nothing.
template <int TM, int TN, int WM, int WN, int NST, bool OUT_BF16>
int launch_stage(const GemmArgs &g0, hipStream_t s, int slabs)
{
    constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
    GemmArgs g = g0;
    g.ksplit = slabs;
    const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    if (tiles_m * tiles_n * slabs > 0x7FFFFFFF) return MQ_ERR_SHAPE;
    auto *kern = bf16_stage_kernel<TM, TN, WM, WN, NST, false, OUT_BF16>;
    if (slabs > 1) {
        if constexpr (stage_slabs(BN))
            kern = bf16_stage_kernel<TM, TN, WM, WN, NST, true, false>;  // (the partial sums are FP32 for either output type)
        else
            return MQ_ERR_SHAPE;
    }
    const int rc = enqueue(kern, dim3((unsigned)(tiles_m * tiles_n * slabs)), dim3(64 * WM * WN),
                           stage_lds<TM, TN, WM, WN, NST>(), s, g, (int)tiles_m, (int)tiles_n);
    return rc != MQ_OK || slabs == 1 ? rc : launch_slab_sum<OUT_BF16>(g, s);
}

template <bool OUT_BF16>
int launch_bf16(const GemmArgs &g, hipStream_t s)
{
    int cus = 0;
    if (int rc = compute_units(cus)) return rc;
    static thread_local RecentPlans<Bf16Plan> recent;
    const int64_t slab_limit = gemm_bf16_slab_limit(g.M, g.N, g.K, g.ws ? g.ws_bytes : 0, cus);
    const Bf16Plan plan =
        recent.get({g.M, g.N, g.K, slab_limit, cus, 0}, [&] { return bf16_plan(g.M, g.N, g.K, slab_limit, cus); });
    int i = 0;
#define MQ_X(MT, NT, S) \
    if (plan.tile == i++) return launch_ring<MT, NT, S, OUT_BF16>(g, s, plan.slabs);
    MQ_RING(MQ_X)
#undef MQ_X
#define MQ_X(TM, TN, WM, WN, NST) \
    if (plan.tile == i++) return launch_stage<TM, TN, WM, WN, NST, OUT_BF16>(g, s, plan.slabs);
    MQ_STAGE(MQ_X)
#undef MQ_X
    using Mid = PCfg<256, 128, 2, 2>;
    using Wide = PCfg<256, 192, 2, 2>;
    using Big = PCfg<256, 256, 2, 2>;
    if (plan.tile == i++) return launch_tiles(gemm_bf16_d2l<Mid, OUT_BF16>, Mid::LDS_BYTES, 256, 128, Mid::THREADS, g, s);
    if (plan.tile == i++) return launch_tiles(gemm_bf16_d2l<Wide, OUT_BF16>, Wide::LDS_BYTES, 256, 192, Wide::THREADS, g, s);
    if (plan.tile == i++) return launch_tiles(gemm_bf16_d2l<Big, OUT_BF16>, Big::LDS_BYTES, 256, 256, Big::THREADS, g, s);
    return launch_tiles(bf16_short_kernel<8, OUT_BF16>, 0, 16, 16, 512, g, s);
}

// ---- which NVFP4 kernel and tile --------------------------------------------------------------------

// The workgroup tiles (tokens x rows of W) of the NVFP4 kernels, gemm_fp4_direct with K whole, split over two or
// over four waves, and gemm_fp4_small, and their costs (TileCost) in either byte order.  The row-major one costs about twice
// the step (a load touches a line per row instead of whole lines), most where the tiles are small, but for the tiles that
// read it in lines.
struct Fp4Tile {
    mq_kernel kernel;
    int bm, bn, waves;
};
#define MQ_SMALL(X) /* TM, TN, S, NSETS */                                                                        \
    X(1, 1, 8, 4) X(1, 2, 8, 4) X(2, 1, 8, 4) X(1, 2, 4, 4) X(2, 1, 4, 4) X(2, 2, 8, 4) X(2, 2, 4, 4) X(2, 4, 8, 2) \
    X(2, 4, 4, 2) X(4, 2, 8, 2) X(4, 2, 4, 2) X(2, 2, 1, 4)
static constexpr Fp4Tile kFp4Tiles[] = {
    {MQ_KERNEL_FP4_DIRECT, 256, 256, 4}, {MQ_KERNEL_FP4_DIRECT, 256, 128, 4}, {MQ_KERNEL_FP4_DIRECT, 128, 128, 4},
#define MQ_X(TM, TN, S, NSETS) {MQ_KERNEL_FP4_SMALL, 32 * TM, 32 * TN, S},
    MQ_SMALL(MQ_X)
#undef MQ_X
};
constexpr int kFp4Directs = 3, kFp4TileCount = (int)(sizeof(kFp4Tiles) / sizeof(kFp4Tiles[0]));
enum { ROW_MAJOR, K_STEP_MAJOR, ROW_MAJOR_LINES };  // rows of kFp4Costs
static constexpr TileCost kFp4Costs[3][kFp4TileCount] = {
    {{6271.7, 6184.9, 1209.8, 886.09, 17.221}, {3469.8, 7200.5, 713.71, 346.48, 107.32},
     {6440.7, 4307, 376.79, 172.48, 107.44},
     {4239.8, 2522.9, 115.35, 20.165, 27.543}, {4933.4, 1970.5, 213.73, 28.547, 158.6},
     {5169.4, 417.19, 215.26, 26.575, 374.97}, {4841.2, 1108, 225.34, 0, 19.288},
     {5092, 646.75, 176.73, 18.397, 234.85}, {4109.1, 3679.6, 289.57, 0, 600}, {4943.6, 2717.7, 247.73, 17.939, 10},
     {7478.9, 719.42, 302.3, 186.41, 261.14}, {4944.2, 3294, 386.65, 44.621, 116.6},
     {7500.5, 2876.1, 181.1, 338.58, 107.4}, {6575.9, 100, 394.94, 6.7359, 330.19}, {6876.3, 100, 346.69, 0, 10}},
    {{6938.1, 8606.2, 630.39, 663.88, 10.011}, {6208.2, 8413, 320.75, 329.2, 15.19},
     {3592.6, 8314.6, 175.14, 152.97, 58.696},
     {4868.5, 564.77, 41.643, 0, 594.93}, {5062.1, 1191.6, 60.656, 0, 276}, {4130.7, 2109.2, 62.464, 0, 12.686},
     {5059.1, 1075.9, 64.775, 0, 12.815}, {5511.2, 673.55, 73.031, 0, 85.618},
     {3776.4, 4046.2, 85.976, 11.681, 40.941}, {5723.5, 1305.4, 106.28, 0, 142.13},
     {2750.6, 5815.8, 118.51, 43.59, 175.04}, {6678.2, 1478.8, 126.74, 47.794, 133.13},
     {3251.3, 5072.4, 119.84, 88.484, 25.163}, {6802.3, 1402.1, 109.41, 83.132, 94.333},
     {6680.1, 481.62, 141.96, 0, 10}},
    {{5090.2, 6365.7, 1212.9, 879.81, 18.582}, {3048.2, 7096.8, 715.85, 348.62, 99.27},
     {3607.9, 4317.9, 395.39, 188.46, 158.25},
     {4130.4, 121.9, 71.787, 10.882, 529.24}, {4518.3, 1360.1, 109.45, 8.5061, 125.13},
     {3700.7, 1338.1, 106.56, 3.6642, 562.03}, {6005.3, 100, 106.11, 6.5875, 13.38},
     {5517.3, 298.81, 84.589, 18.184, 190.27}, {4306.1, 2082.3, 160.2, 4.2803, 107.61},
     {7230.4, 625.18, 136.7, 9.0327, 65.049},
     {7478.9, 719.42, 302.3, 186.41, 261.14}, {4944.2, 3294, 386.65, 44.621, 116.6},
     {7500.5, 2876.1, 181.1, 338.58, 107.4}, {6575.9, 100, 394.94, 6.7359, 330.19}, {6876.3, 100, 346.69, 0, 10}}};
// us: the second pass of K slabs, and what two launches overlap by
static constexpr double kSecondPass[3] = {4.02, 3.20, 4.02}, kOverlap[3] = {1.00, 3.64, 0.04};
// By lines, a plan with a small tile has to be cheaper than one of direct tiles alone by this factor (see fp4_plan).
static constexpr double kSmallMargin[3] = {1.0, 1.0, 1.0077};

struct Fp4Plan {
    int tile;                  // index into kFp4Tiles
    int slabs;                 // K slabs across workgroups (1: none)
    int64_t m_first, n_first;  // one of them > 0: these first rows / columns of Y with `tile`, the others with
    int tile_rest;             // tile_rest in a second launch
};

// The plan that costs least (launch_us; the weights' 0.5625 bytes per element at 5.3 TB/s, a fifth of the shorter one of
// trip and K steps does not hide).  The costs are fitted to every tile's time, and to pairs of them: in K order on 3200
// shapes (K-step-major) and 1800 (row-major) of 16 to 16384 tokens, the 8B and 32B layers, their 2-, 4- and 8-way shards and shorter,
// narrower and wider ones, with the K loop that the small tiles had before their loads got fixed resources (they have become
// faster by 1 to 12 %, most with few tokens).  With the K loop as it is the plan is on average 1.3 % slower than the fastest
// one measured, 95 % of the shapes within 6.2 % (3200 drawn shapes); row-major in K order 2.4 % and 11.2 % (3500 shapes, most of
// them of a K below 2048).
// By lines: 7100 shapes of the same kinds, K from 2048, 1 to 16384 tokens, fitted for the distance to the fastest plan and, eight
// times as heavily, for whatever would be slower than the plan that ran there in K order.  31 shapes are held to the plan that
// a test asserts.  The direct tiles, the same kernels in both row-major orders, have costs of their own here: what counts is how
// they compare with the small tiles' model error.  On 2700 shapes outside the fit the plan is 0.8 % slower than the
// fastest on average, 95 % of them within 4.0 %.  On 9800 others, 1 to 6000 tokens, the product takes 0.75 of the time that it took in K order,
// and more than 2.5 % longer on 11 (7 % at most; 5700 to 5820 tokens on K = 25600, N = 5120 1650 us there and 1740 here).  A fit
// without that weight and without the margin of kSmallMargin was slower there by up to 11 % (2100 tokens on K = 25600,
// N = 5120: 64x64 tiles for the last columns, 697 us against 636 in direct tiles).
// (The output type does not enter: the BF16 output is the rounded FP32 output bit for bit.)
// Small tiles occupy more compute units and larger ones expand fewer operand rows per product (8 vector
// instructions per MFMA for 64x64, 16 for 32x32, 4 for 128x128): 64 tokens on K = N = 4096, weights from HBM, take 8.0 us in
// 32x32 tiles and 12.3 in 64x64; 512 tokens on N = 28672 88 us in 256x256 and 96 in 64x128.
// Two launches where the large tiles leave a ragged last round: whole rounds of one of the direct
// tiles on the first rows or columns of Y, the others in whatever tile suits them (5003 tokens on
// K = 14336, N = 4096: one round of 256x256 tiles on 4096 rows and 907 rows in 128x128 tiles; 333 tokens on N = 28672: 256
// rows in 256x128 tiles and 77 in 128x128, 78 us against 79 in 64x128 tiles and 90 in 256x256, which hold 333 rows of 512).
static Fp4Plan fp4_plan(int64_t M, int64_t N, int64_t K, int layout, int64_t slab_limit, int cus)
{
    const int order = layout == MQ_LAYOUT_KTILE || K == BK ? K_STEP_MAJOR  // (the same bytes when K == 64)
                      : fp4_lines(layout, K)               ? ROW_MAJOR_LINES
                                                           : ROW_MAJOR;
    auto tiles_of = [](const Fp4Tile &t, int64_t m, int64_t n) { return ((m + t.bm - 1) / t.bm) * ((n + t.bn - 1) / t.bn); };
    auto cost = [&](int i, int64_t m, int64_t n, int64_t slabs) {
        const int64_t tiles = tiles_of(kFp4Tiles[i], m, n);
        if (tiles > (kFp4Tiles[i].kernel == MQ_KERNEL_FP4_SMALL ? kMaxSmallTiles : 0x7FFFFFFF)) return 1e300;
        // (many rounds of one-wave tiles: 6144 tokens on K = 128, N = 2048 15.4 us against 13.4 in 256x256 tiles, 6342 on K = 64, N = 15304
        // 83 against 66)
        if (kFp4Tiles[i].waves == 1 && tiles > 8 * cus) return 1e300;
        // a wave of the small tiles loads up to four K steps of its part from one base (22 million rows, K-step-major)
        const int64_t part = (K / BK + slabs * kFp4Tiles[i].waves - 1) / (slabs * kFp4Tiles[i].waves), span = part < 4 ? part - 1 : 3;
        if (kFp4Tiles[i].kernel == MQ_KERNEL_FP4_SMALL && layout == MQ_LAYOUT_KTILE && fp4_reach((M > N ? M : N) * 32) < span)
            return 1e300;
        return launch_us(kFp4Costs[order][i], tiles * slabs, (double)(K / BK) / (double)slabs, 0.5625 * (double)n * (double)K / 5.3e6,
                         0.2, 2.0 * (double)m * (double)n, cus) +
               (slabs > 1 ? kSecondPass[order] : 0.0);
    };
    auto margin = [&](int i) { return kFp4Tiles[i].kernel == MQ_KERNEL_FP4_SMALL ? kSmallMargin[order] : 1.0; };
    Fp4Plan best{0, 1, 0, 0, 0};
    double best_us = 1e300;
    for (int i = 0; i < kFp4TileCount; ++i) {
        const Fp4Tile &t = kFp4Tiles[i];
        const double us = cost(i, M, N, 1) * margin(i);
        if (us < best_us) best_us = us, best = Fp4Plan{i, 1, 0, 0, 0};
        if (t.kernel != MQ_KERNEL_FP4_SMALL || slab_limit < 2) continue;
        const int64_t tiles = tiles_of(t, M, N);
        const int64_t slabs = cus / tiles < slab_limit ? cus / tiles : slab_limit;
        if (slabs < 2) continue;
        const double us_slabs = cost(i, M, N, slabs) * margin(i);
        if (us_slabs < best_us) best_us = us_slabs, best = Fp4Plan{i, (int)slabs, 0, 0, 0};
    }
    for (int i = 0; i < kFp4Directs; ++i) {
        const Fp4Tile &t = kFp4Tiles[i];
        const int64_t tiles_m = (M + t.bm - 1) / t.bm, tiles_n = (N + t.bn - 1) / t.bn;
        const int64_t rounds = (tiles_m * tiles_n + cus - 1) / cus;
        for (int64_t r = rounds - 1; r >= 1 && r >= rounds - 2; --r)
            for (int by_m = 0; by_m < 2; ++by_m) {
                const int64_t m = by_m ? r * cus / tiles_n * t.bm : M, n = by_m ? N : r * cus / tiles_m * t.bn;
                if (m == 0 || n == 0 || (by_m ? m >= M : n >= N)) continue;
                const double first = cost(i, m, n, 1) - kOverlap[order];
                for (int j = 0; first < best_us && j < kFp4TileCount; ++j) {
                    const double us = (first + cost(j, by_m ? M - m : M, by_m ? N : N - n, 1)) * margin(j);
                    if (us < best_us) best_us = us, best = Fp4Plan{i, 1, by_m ? m : 0, by_m ? 0 : n, j};
                }
            }
    }
    return best;
}

template <bool OUT_BF16>
int launch_fp4_tile(int tile, int slabs, const GemmArgs &g, hipStream_t s, int cus)
{
    constexpr size_t X = 128 * 1024;  // accumulator exchange of the K-split variants
    int i = 0;
    if (tile == i++) return launch_persistent(gemm_fp4_direct<OUT_BF16, 1>, 256, 256, 0, g, s, cus);
    if (tile == i++) return launch_persistent(gemm_fp4_direct<OUT_BF16, 2>, 256, 128, X, g, s, cus);
    if (tile == i++) return launch_persistent(gemm_fp4_direct<OUT_BF16, 4>, 128, 128, X, g, s, cus);
#define MQ_X(TM, TN, S, NSETS) \
    if (tile == i++) return launch_small<TM, TN, S, NSETS, OUT_BF16>(g, s, slabs, cus);
    MQ_SMALL(MQ_X)
#undef MQ_X
    return MQ_ERR_SHAPE;
}

template <bool OUT_BF16>
int launch_fp4(const GemmArgs &g, hipStream_t s)
{
    int cus = 0;
    if (int rc = compute_units(cus)) return rc;
    const int layout = g.b_c_row == 32 ? MQ_LAYOUT_KTILE : MQ_LAYOUT_LINEAR;
    static thread_local RecentPlans<Fp4Plan> recent;
    const int64_t slab_limit = gemm_fp4_slab_limit(g.M, g.N, g.K, g.ws ? g.ws_bytes : 0, cus);
    const Fp4Plan plan = recent.get({g.M, g.N, g.K, slab_limit, cus, layout},
                                    [&] { return fp4_plan(g.M, g.N, g.K, layout, slab_limit, cus); });
    if (plan.n_first == 0 && plan.m_first == 0) return launch_fp4_tile<OUT_BF16>(plan.tile, plan.slabs, g, s, cus);
    constexpr int64_t T = OUT_BF16 ? 2 : 4;
    GemmArgs ga = g, gb = g;  // (the K step strides keep those of the whole operands)
    if (plan.m_first > 0) {
        ga.M = plan.m_first;
        gb.M = g.M - plan.m_first;
        gb.a = static_cast<const char *>(g.a) + plan.m_first * g.a_c_row;
        gb.a_scales = g.a_scales + plan.m_first * g.a_s_row;
        gb.y = static_cast<char *>(g.y) + plan.m_first * g.ldy * T;
    } else {
        ga.N = plan.n_first;
        gb.N = g.N - plan.n_first;
        gb.b = static_cast<const char *>(g.b) + plan.n_first * g.b_c_row;
        gb.b_scales = g.b_scales + plan.n_first * g.b_s_row;
        gb.y = static_cast<char *>(g.y) + plan.n_first * T;
    }
    if (int rc = launch_fp4_tile<OUT_BF16>(plan.tile, 1, ga, s, cus)) return rc;
    return launch_fp4_tile<OUT_BF16>(plan.tile_rest, 1, gb, s, cus);
}

template <bool FP4, bool OUT_BF16>
int launch_any(const GemmArgs &g, hipStream_t s)
{
    if (g.M == 0 || g.N == 0) return MQ_OK;
    // The tiled kernels step K by 64.
    if (g.K % BK != 0) return launch_simple<FP4, OUT_BF16>(g, s);
    if constexpr (FP4)
        return launch_fp4<OUT_BF16>(g, s);
    else
        return launch_bf16<OUT_BF16>(g, s);
}

}  // namespace

// Raises the dynamic-LDS limit of every kernel that asks for more than the default.  Done once
// per device before the first launch (mq_init, or the first product on a device), so that no
// launch path has one-time work left that a stream capture could trip over.
int configure_gemm_kernels()
{
    auto set = [](auto kern, size_t bytes) {
        if (bytes == 0) return hipSuccess;
        return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bytes);
    };
    using Mid = PCfg<256, 128, 2, 2>;
    using Wide = PCfg<256, 192, 2, 2>;
    using Big = PCfg<256, 256, 2, 2>;
    constexpr size_t X = 128 * 1024;  // accumulator exchange of the K-split variants
    hipError_t e = hipSuccess;
    auto both = [&](auto k_bf16, auto k_fp32, size_t bytes) {
        if (e == hipSuccess) e = set(k_bf16, bytes);
        if (e == hipSuccess) e = set(k_fp32, bytes);
    };
    both(gemm_fp4_direct<true, 2>, gemm_fp4_direct<false, 2>, X);
    both(gemm_fp4_direct<true, 4>, gemm_fp4_direct<false, 4>, X);
#define MQ_X(TM, TN, S, NSETS) \
    both(gemm_fp4_small<TM, TN, S, NSETS, true, false>, gemm_fp4_small<TM, TN, S, NSETS, false, false>, small_lds<TM, TN, S>()); \
    if constexpr (has_lines<TM, TN, S>()) \
        both(gemm_fp4_small<TM, TN, S, 4, true, true>, gemm_fp4_small<TM, TN, S, 4, false, true>, small_lds<TM, TN, S>());
    MQ_SMALL(MQ_X)
#undef MQ_X
    both(gemm_bf16_d2l<Mid, true>, gemm_bf16_d2l<Mid, false>, Mid::LDS_BYTES);
    both(gemm_bf16_d2l<Wide, true>, gemm_bf16_d2l<Wide, false>, Wide::LDS_BYTES);
    both(gemm_bf16_d2l<Big, true>, gemm_bf16_d2l<Big, false>, Big::LDS_BYTES);
#define MQ_X(MT, NT, S) \
    both(bf16_ring_kernel<MT, NT, S, true, true>, bf16_ring_kernel<MT, NT, S, true, false>, ring_lds<MT, NT, S>()); \
    both(bf16_ring_kernel<MT, NT, S, false, true>, bf16_ring_kernel<MT, NT, S, false, false>, ring_lds<MT, NT, S>());
    MQ_RING(MQ_X)
#undef MQ_X
#define MQ_X(TM, TN, WM, WN, NST) \
    both(bf16_stage_kernel<TM, TN, WM, WN, NST, false, true>, bf16_stage_kernel<TM, TN, WM, WN, NST, false, false>, \
         stage_lds<TM, TN, WM, WN, NST>()); \
    if constexpr (stage_slabs(16 * TN * WN))  \
        if (e == hipSuccess) e = set(bf16_stage_kernel<TM, TN, WM, WN, NST, true, false>, stage_lds<TM, TN, WM, WN, NST>());
    MQ_STAGE(MQ_X)
#undef MQ_X
    return note_launch(e);
}

// Most K slabs across workgroups that the NVFP4 product may use, given this much workspace (0 or 1: none); how many it
// does use, if any, is the cost rule's choice (at most one work item per compute unit), and depends on the byte
// order.  A bound in 64x64 tiles for either of them: a long K (below about 7000 the second pass costs more than it saves)
// with at most half as many such tiles as compute units, one round of work items, at least four K steps
// for each of eight waves.
int gemm_fp4_slab_limit(int64_t M, int64_t N, int64_t K, int64_t ws_bytes, int cus)
{
    if (M <= 0 || N <= 0 || K <= 0 || K % BK != 0 || ws_bytes <= 0 || N % 4 != 0) return 0;
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64), kt = K / BK, waves = kt >= 16 ? 8 : kt / 2 > 0 ? kt / 2 : 1;
    if (2 * tiles > cus) return 0;
    int64_t ks = cus / tiles;
    if (ks > kt / (waves * 4)) ks = kt / (waves * 4);
    if (ks > ws_bytes / (M * N * 4)) ks = ws_bytes / (M * N * 4);
    return ks >= 2 && kt * (ks - 1) > 9 * waves * ks ? (int)ks : 0;
}

// Most K slabs across workgroups that the BF16 product may use, given this much workspace (0 or 1: none); the cost
// rule decides how many it does use, at most one work item per compute unit.  33 to 64 tokens (narrow tiles): a long K and a narrow N; every slab keeps 512 of K, and the partial
// sums' traffic (8 bytes per output and slab) stays below half of the weights'.  More tokens (staged tiles): every slab
// keeps 768 of K and the partial sums 16 MiB.  The line at K = 8192 is on the safe side of the rule's error, not where slabs cease to gain:
// the best plan with slabs takes 0.96 of the time of the best one without over K = 5120 to 6144 (and is slower for half of the shapes), 0.93
// to 7168, 0.91 to 8192, 0.73 beyond.  With these costs the rule would gain 5, 9 and 14 % there where it took slabs, but be more than
// 1.5 % slower than without in 14 of 56, 6 of 80 and 2 of 79 such shapes (by 11 % at most), beyond in 3 of 375.
int gemm_bf16_slab_limit(int64_t M, int64_t N, int64_t K, int64_t ws_bytes, int cus)
{
    if (M <= 32 || N <= 0 || ws_bytes <= 0 || N % 4 != 0) return 0;
    if (M > 64) {
        if (K <= 8192 || K % BK != 0) return 0;
        if (ws_bytes > (16 << 20)) ws_bytes = 16 << 20;
        if (M > ws_bytes / 8 || N > ws_bytes / 8) return 0;  // (M * N * 4 does not overflow below)
        const int64_t most = ws_bytes / (M * N * 4), ks = K / BK / 12;
        const int64_t got = ks < most ? ks : most;
        return got >= 2 ? (int)got : 0;
    }
    if (K < 8192 || K % 128 != 0) return 0;
    const int64_t groups = (N + 127) / 128, steps = K / 128;
    if (2 * groups >= cus) return 0;
    int64_t ks = 2 * cus / groups;
    if (ks > steps / 4) ks = steps / 4;
    if (ks > K / (8 * M)) ks = K / (8 * M);
    if (ks > ws_bytes / (M * N * 4)) ks = ws_bytes / (M * N * 4);
    if (ks < 2 || 2 * groups * ks < cus) return 0;  // too few workgroups even so
    return (int)ks;
}

static int describe_simple(int64_t M, int64_t N, mq_launch *out)
{
    out[0] = mq_launch{MQ_KERNEL_SIMPLE, 16, 16, 4, 1, M, N};
    return 1;
}

int describe_gemm_fp4(int64_t M, int64_t N, int64_t K, int layout, int64_t ws_bytes, int cus, mq_launch *out)
{
    if (K % BK != 0) return describe_simple(M, N, out);
    const Fp4Plan p = fp4_plan(M, N, K, layout, gemm_fp4_slab_limit(M, N, K, ws_bytes, cus), cus);
    const Fp4Tile &t = kFp4Tiles[p.tile], &r = kFp4Tiles[p.tile_rest];
    out[0] = mq_launch{t.kernel, t.bm, t.bn, t.waves, p.slabs, p.m_first ? p.m_first : M, p.n_first ? p.n_first : N};
    if (p.m_first == 0 && p.n_first == 0) return 1;
    out[1] = mq_launch{r.kernel, r.bm, r.bn, r.waves, 1, p.m_first ? M - p.m_first : M, p.n_first ? N - p.n_first : N};
    return 2;
}

int describe_gemm_bf16(int64_t M, int64_t N, int64_t K, int64_t ws_bytes, int cus, mq_launch *out)
{
    if (K % BK != 0) return describe_simple(M, N, out);
    const Bf16Plan p = bf16_plan(M, N, K, gemm_bf16_slab_limit(M, N, K, ws_bytes, cus), cus);
    const Bf16Tile &t = kBf16Tiles[p.tile];
    out[0] = mq_launch{t.kernel, t.bm, t.bn, t.waves, p.slabs, M, N};
    return 1;
}

int launch_mfma_probe(float *out, int iters, int blocks, hipStream_t s)
{
    return enqueue(mfma_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, s, out, iters);
}

int launch_gemm_fp4(const GemmArgs &g, hipStream_t s)
{
    return g.out == MQ_OUT_BF16 ? launch_any<true, true>(g, s) : launch_any<true, false>(g, s);
}

int launch_gemm_bf16(const GemmArgs &g, hipStream_t s)
{
    return g.out == MQ_OUT_BF16 ? launch_any<false, true>(g, s) : launch_any<false, false>(g, s);
}

}  // namespace mq
