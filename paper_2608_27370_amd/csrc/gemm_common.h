// Declarations shared by the GEMM's host planner (gemm.hip) and its kernel
// variants (gemm_kernel.hip, compiled once per operand-format pair and scale
// kind so that the instantiations build in parallel).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.h"

namespace puro {
namespace gemm_detail {

constexpr int kBK = 128;                   // k block of the grouped scales (and of split-K ranges)

// Division of x < 2^31 by a positive d fixed on the host: the high word of x
// times m = ceil(2^(32 + s) / d), shifted by s, with 2^s < d <= 2^(s + 1); m d
// exceeds 2^(32 + s) by less than d <= 2^(s + 1), which x < 2^31 keeps from
// reaching the quotient.
struct Divisor {
    uint32_t d, m, s;
    static Divisor of(uint32_t d) {
        Divisor r{d, 0u, 0u};
        if (d < 2) return r;
        while ((2u << r.s) < d) ++r.s;
        r.m = (uint32_t)(((1ull << (32 + r.s)) + d - 1) / d);
        return r;
    }
    __device__ __forceinline__ uint32_t quotient(uint32_t x) const { return d == 1 ? x : __umulhi(x, m) >> s; }
};

struct Params {
    const uint8_t* A;
    const uint8_t* B;
    const float* sa;
    const float* sb;
    void* D;
    float* partial;
    int64_t lda, ldb, ldd;
    int M, N, K;
    int a_mode, b_mode;
    int a_kmajor, b_kmajor;    // grouped scales k-block-major rather than row-major
    int ld_sa, ld_sb;          // scale pitch: K/128 (row-major) or the row (block) count (k-major)
    uint32_t sa_bytes, sb_bytes;  // sizes of the scale arrays (grouped modes)
    int ksteps, ksteps_per_split, splits;
    int gm;                    // tile rows per group within an XCD's range of tiles
    int tiles_m, tiles_n;
    Divisor per_split;         // tiles of a problem's k range,
    Divisor per_problem;       // of a problem (per_split * splits),
    Divisor per_group;         // and of a group of gm tile rows
    int accumulate;
    float alpha;               // host-known factor of the sums (with the per-tensor scales)
    const uint16_t* bias;      // OUT kOutBF16Epi: optional bias [N] and residual [M, N] (pitch ldr)
    const uint16_t* residual;
    int64_t ldr;
    float res_scale;           // factor of the residual
    int upper;                 // only the tiles on or above the diagonal (square tiles, M == N)
    int nt_f32;                // a binary32 D is stored with non-temporal (streaming) stores
    int batch;                 // problems of one launch: A, B, D advance by bsa, bsb, bsd bytes,
    int64_t bsa, bsb, bsd;     // the residual by bsr elements, the split-K partials by
    int64_t bsr;               // splits * M * N floats

    // LM-head output kinds (kOutLseStats, kOutSoftmaxGrad; 128-column wave tiles)
    const int32_t* targets;    // target vocabulary id per row
    int col0;                  // vocabulary column of this GEMM's column 0
    float2* stats;             // [M][stats_ld]: (max, sum exp(z - max)) per 128-column block
    int64_t stats_ld;
    float* zt;                 // [M]: the target's logit
    const float* lse;          // [M]
    float grad_scale;
    uint8_t* q8;               // kOutSoftmaxGradQ: dz's FP8 copies (the GemmProblem fields)
    float* q8_scale;
    uint8_t* q8t;
    float* q8t_scale;
};

struct TileCfg {
    int bm, bn;          // workgroup tile
    int wm, wn;          // wave grid (wave tile bm/wm x bn/wn)
    int sl, nst;         // k bytes per pipeline slice, ring stages
    int xa;              // spare 64-row units of the A ring (fewer where LDS lacks room for them)
    int prod;            // producer waves issue the global->LDS loads
    float fixed_us;      // time model: per wave of work units ...
    float slice_us;      // ... plus per k slice of a unit (MI355X, all CUs busy),
    float grouped;       // times this with block scales
};
// Four MFMA waves (one per SIMD) in a 2x2 grid. The large wave tiles need
// the least LDS traffic per MFMA (128x128: 16 MFMAs per 16 KB of fragment
// reads); the 128x128 tiles give more work units on narrow problems, with a
// deep ring (one workgroup per CU) or a short one (two per CU). A 128x128
// tile moves as many bytes global->LDS per k slice as the texture unit
// passes (about 64 B per clock per CU) while its MFMAs run, so its loads
// often wait for queue space: the deep-ring variant adds four producer waves
// that issue them (the tile's registers leave room for two waves per SIMD),
// 15-20% faster on long-K Wgrad than issuing them from the MFMA waves. The
// 64x64 tiles are for problems of few rows, which leave most of the chip idle
// and are bound by latency: four times the work units of 128x128, and an
// 8-deep ring that has most of a K 1536 reduction in flight at once
// (77x2048x1536 8.8 -> 6.0 us, 256x1536x1536 7.5 -> 6.1 us, both unsplit;
// split over k the 128x128 tiles took 8.6 and 12.4 us with their reduction).
// 256x128 fits the grids that the larger tiles leave half empty: 3968x2048x8192
// is 256 of its tiles, one per CU (64.6 -> 57.1 us block-scaled, the LM head's
// dX at that size; 128 tiles of 256x256 take 75 us).
// The time constants are fits to measured kernel times (graph replays) of 44
// shapes, per-tensor and block-scaled, from 16 to 16384 rows, at six splits
// (1, 2, 3, 4, 6, 8), under the condition that the plans the tests name and
// those of four optimiser batches stay as they were.
// Checked on 57 other random shapes of that range with rotating operands (so
// that none is in an L2 from the call before), every configuration at 13
// splits: the choice takes 3.4% longer than the best of them on average and
// 27% at most (1322x616x1920, 11.5 us; 64x64 tiles, which small_tiles in
// gemm.hip leaves out there and in four of the next five, take 9.1).
// Block scales lengthen a slice by what the scales' loads and conversion add
// beside its MFMAs: 1.02 - 1.07 (256x256, measured from K 4096 to 8192 on grids
// of 16 to 256 tiles), 1.06 - 1.14 (256x192), 1.2 - 1.5 and 1.0 - 1.25 (128x128,
// 4- and 2-deep), 1.0 - 1.15 (64x64), 1.1 - 1.35 (256x128), more where both
// operands have a scale per row. Without the factor long reductions stayed
// unsplit that are faster split: 973x1240x4736 24.3 us against 19.1, the QKV
// Wgrad 2048x1536x16384 70.0 against 60.2. On 220 random block-scaled shapes
// with rotating operands the choice is 1.1% from the best plan (1.9% without),
// and two of them are slower by it (7 and 14%).
#define PURO_TILE_LIST(X)                                         \
    X(0, 256, 256, 2, 2, 128, 2, 4, 0, 9.276f, 1.343f, 1.05f)     \
    X(1, 256, 192, 2, 2, 128, 2, 4, 0, 9.429f, 0.990f, 1.10f)     \
    X(2, 128, 128, 2, 2, 128, 4, 0, 1, 6.424f, 0.3645f, 1.38f)    \
    X(3, 128, 128, 2, 2, 128, 2, 0, 0, 4.071f, 0.8992f, 1.30f)    \
    X(4, 64, 64, 2, 2, 128, 8, 0, 0, 3.031f, 0.2984f, 1.10f)      \
    X(5, 256, 128, 2, 2, 128, 2, 3, 0, 6.577f, 0.7372f, 1.20f)
#define PURO_TILE_ROW(i, bm, bn, wm, wn, sl, nst, xa, prod, f, s, g) {bm, bn, wm, wn, sl, nst, xa, prod, f, s, g},

constexpr int kLdsBytes = 160 * 1024;
// LDS bytes of a configuration with xa spare A units, and the spare units
// that fit (block-scaled operands keep their scales in LDS too).
constexpr int tile_lds(int bm, int bn, int sl, int nst, int xa, bool grouped) {
    return (bm + bn) * sl * nst + xa * 64 * sl + (grouped ? (bm + bn) * 4 * nst : 0);
}
constexpr int spare_units(int bm, int bn, int sl, int nst, int xa, bool grouped) {
    return xa > 0 && tile_lds(bm, bn, sl, nst, xa, grouped) > kLdsBytes ? spare_units(bm, bn, sl, nst, xa - 1, grouped)
                                                                        : xa;
}

// The bias / residual epilogue: the BF16 bias of columns n..n+3 and the BF16
// residual of row m at those columns added to four binary32 results (the
// sum stays binary32 until the output's one rounding).
// The residual is multiplied by rs in the same fused step as its addition
// (rs = 1 adds it exactly as a plain sum).
__device__ __forceinline__ void add_epilogue4(float4& v, const uint16_t* bias, const uint16_t* residual,
                                              int64_t ldr, int64_t m, int64_t n, float rs) {
    if (bias) {
        const uint2 b = *reinterpret_cast<const uint2*>(bias + n);
        v.x += bf16lo(b.x); v.y += bf16hi(b.x); v.z += bf16lo(b.y); v.w += bf16hi(b.y);
    }
    if (residual) {
        const uint2 r = *reinterpret_cast<const uint2*>(residual + m * ldr + n);
        v.x = fmaf(rs, bf16lo(r.x), v.x); v.y = fmaf(rs, bf16hi(r.x), v.y);
        v.z = fmaf(rs, bf16lo(r.y), v.z); v.w = fmaf(rs, bf16hi(r.y), v.w);
    }
}
__device__ __forceinline__ float add_epilogue1(float v, const uint16_t* bias, const uint16_t* residual, int64_t ldr,
                                               int64_t m, int64_t n, float rs) {
    if (bias) v += __uint_as_float((uint32_t)bias[n] << 16);
    if (residual) v = fmaf(rs, __uint_as_float((uint32_t)residual[m * ldr + n] << 16), v);
    return v;
}

// Enqueue the kernel of tile configuration `cfg` (index into the list above)
// for output kind `out` (kOutBF16, kOutF32, kOutBF16Epi, or 2: split-K
// partial sums) over `grid` workgroups; defined in gemm_kernel.hip for each
// (FA, FB, GROUPED).
template <int FA, int FB, bool GROUPED>
void launch_variant(const Params& prm, int cfg, int out, int grid, hipStream_t stream);

}  // namespace gemm_detail
}  // namespace puro
