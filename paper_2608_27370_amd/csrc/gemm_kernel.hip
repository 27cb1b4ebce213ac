// Scaled FP8 GEMM kernel for gfx950: D[m, n] = sum_k A[m, k] * B[n, k].
//
// Section 3.2 of the paper runs the Fprop, Dgrad and Wgrad GEMMs of every
// linear layer on FP8 operands with higher-precision accumulation; operands
// carry a per-tensor scale or power-of-two scales per 128 values along k
// (per row, or per 128x128 block).
//
// Design (CDNA4):
//  * Both operands reduction-contiguous ("TN"); Dgrad and Wgrad are posed
//    this way by feeding the transposed FP8 copies the quantiser writes.
//  * Four waves per workgroup, one per SIMD, in a 2x2 grid; workgroup tiles
//    up to 256x256 (wave tiles up to 128x128, accumulators in AGPRs).
//  * Operand tiles move global -> LDS by buffer_load ... lds (16 bytes per
//    lane, no VGPR staging) in k slices of SL = 128 bytes: one 1 KB DMA load
//    covers 8 rows x 128 bytes, whole cache lines. A ring of NST slices
//    keeps the next ones in flight while one is multiplied.
//  * Within a slice the wave works in 64-byte k steps; the fragments of
//    the next step are read from LDS into a second register set while the
//    MFMAs of the current one run, and the DMA loads are spread between
//    the MFMAs of both steps: A's ring has spare units of 64 rows that take
//    the next slice's first rows early. The loop body has no branches and
//    waits on constant counts; one barrier per slice.
//  * What bounds it: the long reductions run at 2.6 - 2.9 PFLOP/s, the clock
//    held down by the matrix cores' power (gate/up Dgrad 16384x1536x17920 410
//    -> 336 us over these steps: the spread loads 410 -> 385, the loop's
//    arithmetic between the MFMAs 385 -> 338); at K 1536 a 256x256 tile spends
//    a third of its time in prologue and epilogue (gate/up Fprop 471 -> 432).
//  * LDS rows are XOR-swizzled in 16-byte chunks (conflict-free reads; the
//    swizzle is applied on the global side because the DMA writes lane l at
//    base + 16 l).
//  * v_mfma_scale_f32_32x32x64_f8f6f4: 32x32 outputs per 64-long k step.
//    Grouped scales become the instruction's E8M0 operands (exact powers of
//    two, applied inside the MFMA); per-tensor scales multiply the FP32
//    result once in the epilogue. The instruction is issued with the B tile
//    as its first operand, so each lane's accumulators hold four consecutive
//    output columns of one row.
//  * Out-of-range rows and the k tail are zero-filled by the buffer
//    descriptor's range check (num_records) rather than by branches.
//  * Tiles are remapped so the eight XCDs (workgroups are dealt round-robin
//    to them) each own a contiguous range of tiles, grouped by row panels to
//    share operand panels in that XCD's L2.
//  * The epilogue stages each wave's FP32 tile in the idle ring and stores
//    whole rows; tiles inside the matrix, and edge tiles of whole 4-column
//    vectors, take a branch-free path that issues all LDS reads of a group
//    before its stores (before, edge tiles went element by element: quantise +
//    GEMM with residual 3001x2056x2064 40 -> 35 us).
//  * Small grids split K into ranges whose FP32 partial sums a second kernel
//    adds in a fixed order (deterministic).

// This file is compiled once per operand-format pair and scale kind
// (PURO_FA, PURO_FB, PURO_GROUPED), each object holding that variant's tile
// configurations and output kinds.

#include <climits>
#include <type_traits>

#include "device_common.h"
#include "gemm_common.h"
#include "kernels.h"

#if !defined(PURO_FA) || !defined(PURO_FB) || !defined(PURO_GROUPED)
#error "gemm_kernel.hip is compiled with -DPURO_FA=<0|1> -DPURO_FB=<0|1> -DPURO_GROUPED=<0|1>"
#endif

namespace puro {
namespace gemm_detail {

namespace {


typedef int v8i __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void_t;

constexpr uint32_t kRsrcWord3 = 0x00020000u;  // raw buffer, 32-bit data format
constexpr uint32_t kOOB = 0x80000000u;     // offset that fails the range check


// f(std::integral_constant<int, i>) for i = 0 .. N-1, each call with its own
// compile-time index (no loop left for the unroller to decide on).
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// BF16 outputs of FP8 operands are a linear layer's: far larger than the L2
// and next read by another kernel, they are stored past the caches
// (non-temporal). Those of BF16 operands, MuonH's, are read back at once.
// (Binary32 outputs of FP8 operands are both a Wgrad's, read later, and the
// LM head's dX accumulator, read back by the next chunk: Params::nt_f32.)
template <int FA> constexpr bool kStreamOut = FA != kBF16;

constexpr int cgcd(int a, int b) { return b == 0 ? a : cgcd(b, a % b); }



typedef int v4i __attribute__((ext_vector_type(4)));

// Raw buffer descriptor (base, num_records bytes; 32-bit data format); every
// field is made wave-uniform so that it lives in SGPRs.
__device__ __forceinline__ v4i make_rsrc(const void* base, uint32_t bytes) {
    const uint64_t a = (uint64_t)base;
    v4i r;
    r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xFFFFu));
    r.z = __builtin_amdgcn_readfirstlane((int)bytes);
    r.w = (int)kRsrcWord3;
    return r;
}

// Arithmetic on the wave-uniform x stays behind this point (the empty asm
// takes and gives x; the compiler moves neither it nor what uses x after it).
__device__ __forceinline__ void pin(int& x) {
    x = __builtin_amdgcn_readfirstlane(x);
    asm volatile("" : "+s"(x));
}

// LDS byte address of a __shared__ object (the value M0 takes for a DMA).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p;
}

// Global -> LDS DMA of BYTES (16 or 4) per lane: lane l's data lands at
// LDS address lds + BYTES * l; soff (wave-uniform) adds to every lane's
// offset, and offsets at or beyond the descriptor's num_records read as zero
// (soff must not exceed num_records: the range check compares voff with
// num_records - soff). Issued from inline assembly so that the compiler,
// which cannot tell which LDS bytes a DMA writes, does not make every later
// LDS read wait for it: the kernel waits explicitly (s_waitcnt vmcnt +
// barrier) before reading a stage. One wait state separates the M0 write
// from the DMA that reads it. M0 is written without being saved and named as
// a clobber, so that a value the compiler keeps there itself (an indexed
// register move, an LDS builtin) is made again after it; saving it here would
// cost two scalar moves per load.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"     // (M0 is a reserved register)
template <int BYTES>
__device__ __forceinline__ void dma_to_lds(v4i rsrc, uint32_t lds, uint32_t voff, uint32_t soff) {
    lds = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds);   // wave-uniform by construction
    soff = (uint32_t)__builtin_amdgcn_readfirstlane((int)soff);
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "buffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                     "buffer_load_dword %1, %2, %3 offen lds"
                     :: "s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
#pragma clang diagnostic pop

// dz's E4M3 copies from a wave's staged 128 x 128 BF16 tile (row r at
// ep + 256 r, its 16-byte chunk c at position c ^ (r & 15)), for the LM
// head's backward: the same codes and power-of-two scales as the 1x128 +
// 128x1 quantiser gives for that BF16 dz (its groups are 128-aligned, so
// each lies in one wave tile), written where the dX and dW GEMMs read them.
//  * rows: lane l quantises staged rows l and l + 64, each one 1x128 group;
//  * columns: lane l takes 8 columns (chunk c = l & 15) over the row blocks
//    of 8 rows b = (l >> 4) + 4 k; the 4 lanes of a chunk share the column
//    maxima through two shuffles, each 8 x 8 block is transposed in
//    registers and its 8 columns' codes go to the transposed copy.
template <class P>
__device__ __forceinline__ void quantize_staged_dz(const P& p, const uint8_t* ep, int64_t mrow0, int64_t ncol0,
                                                   int lane) {
    typedef unsigned int v4u __attribute__((ext_vector_type(4)));
    constexpr int F = kE4M3;
    const int64_t M = p.M, N = p.N;
    auto chunk = [&](int r, int c) __attribute__((always_inline)) {
        return *reinterpret_cast<const v4u*>(ep + r * 256 + ((c ^ (r & 15)) << 4));
    };
    // ---- rows
    const __amdgpu_buffer_rsrc_t rq =
        __builtin_amdgcn_make_buffer_rsrc(p.q8 + mrow0 * N + ncol0, 0, (int)(127 * N + 128), 0x00020000);
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
        const int r = lane + 64 * rr;
        uint32_t w[16][4];
        uint32_t m = 0;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const v4u v = chunk(r, c);
            w[c][0] = v.x; w[c][1] = v.y; w[c][2] = v.z; w[c][3] = v.w;
            m = max(m, absmax_bits8(w[c]));
        }
        float s;
        uint2 q[16];
        if (m <= 0x7F7Fu) {
            const int e = pow2_exponent_bf16<F>(m);
            s = exp2i(e);
            if (e > -127) {
#pragma unroll
                for (int c = 0; c < 16; ++c) q[c] = encode8_pow2<F>(w[c], s);
            } else {
#pragma unroll
                for (int c = 0; c < 16; ++c) q[c] = encode8<F, false>(w[c], exp2i(-e));
            }
        } else {
            // an infinity: the largest scale, saturated codes; a NaN: NaN scale and codes
            const bool inf = m == 0x7F80u;
            s = inf ? exp2i(127) : __uint_as_float(0x7FC00000u);
            const float rinv = inf ? exp2i(-127) : s;
#pragma unroll
            for (int c = 0; c < 16; ++c) q[c] = encode8<F, true>(w[c], rinv);
        }
#pragma unroll
        for (int c = 0; c < 16; c += 2)
            __builtin_amdgcn_raw_buffer_store_b128(v4u{q[c].x, q[c].y, q[c + 1].x, q[c + 1].y}, rq,
                                                   (int)(r * N + c * 8), 0, 0);
        p.q8_scale[(ncol0 / 128) * M + mrow0 + r] = s;
    }
    // ---- columns
    const int cb = lane & 15, b0 = lane >> 4;
    uint32_t cm[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const v4u v = chunk((b0 + 4 * k) * 8 + i, cb);
            cm[0] = pk_max_u16(cm[0], mag2(v.x)); cm[1] = pk_max_u16(cm[1], mag2(v.y));
            cm[2] = pk_max_u16(cm[2], mag2(v.z)); cm[3] = pk_max_u16(cm[3], mag2(v.w));
        }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        cm[j] = pk_max_u16(cm[j], (uint32_t)__shfl_xor((int)cm[j], 16, 64));
        cm[j] = pk_max_u16(cm[j], (uint32_t)__shfl_xor((int)cm[j], 32, 64));
    }
    float scol[8], rcol[8];
    bool finite = true, normal = true;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t m = (j & 1) ? (cm[j >> 1] >> 16) : (cm[j >> 1] & 0xFFFFu);
        if (m <= 0x7F7Fu) {
            const int e = pow2_exponent_bf16<F>(m);
            scol[j] = exp2i(e);
            rcol[j] = exp2i(-e);
            normal = normal && e > -127;
        } else if (m == 0x7F80u) {
            scol[j] = exp2i(127);
            rcol[j] = exp2i(-127);
            finite = false;
        } else {
            scol[j] = rcol[j] = __uint_as_float(0x7FC00000u);
            finite = false;
        }
    }
    // the transposed copy's rows ncol0 + 8 cb + j hold columns mrow0 + 8 b + (0..7)
    const __amdgpu_buffer_rsrc_t rt =
        __builtin_amdgcn_make_buffer_rsrc(p.q8t + ncol0 * M + mrow0, 0, (int)(127 * M + 128), 0x00020000);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int b = b0 + 4 * k;
        uint32_t w[8][4];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const v4u v = chunk(b * 8 + i, cb);
            w[i][0] = v.x; w[i][1] = v.y; w[i][2] = v.z; w[i][3] = v.w;
        }
        uint2 ct[8];
        if (finite && normal) {
            uint32_t wt[8][4];
            transpose8x8_b16(w, wt);
#pragma unroll
            for (int j = 0; j < 8; ++j) ct[j] = encode8_pow2<F>(wt[j], scol[j]);
        } else {
            uint2 c[8];
            if (finite) {
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = encode8_cols<F, false>(w[i], rcol);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = encode8_cols<F, true>(w[i], rcol);
            }
            transpose8x8(c, ct);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(unsigned int __attribute__((ext_vector_type(2))), ct[j]),
                                                  rt, (int)((cb * 8 + j) * M + b * 8), 0, 0);
    }
    if (b0 == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) p.q8t_scale[(mrow0 / 128) * N + ncol0 + cb * 8 + j] = scol[j];
    }
}

// PROD: the workgroup has NW more waves that only issue the global->LDS
// loads (producers); the NW MFMA waves (consumers) then only read LDS and
// multiply, so a load that cannot issue (the texture unit's queue full)
// does not hold up their matrix instructions. Both kinds meet at the one
// barrier per slice.
template <int BM, int BN, int WM, int WN, int FA, int FB, int OUT, bool GROUPED, int SL, int NST, int XA, bool PROD>
__global__ __launch_bounds__(WM * WN * 64 * (PROD ? 2 : 1)) void gemm_fp8_kernel(Params p) {
    constexpr int NW = WM * WN;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int FM = WTM / 32, FN = WTN / 32;
    constexpr int KH = SL / 64;                     // 64-byte MFMA k steps per slice
    constexpr int A_BYTES = BM * SL, B_BYTES = BN * SL;   // of a slice
    constexpr int STAGE = A_BYTES + B_BYTES;        // one SL-byte k slice of both tiles
    // 1 KB DMA loads (RPL rows of SL bytes) per wave and slice: load q of a
    // wave brings row block q * NW + wave of its operand
    constexpr int RPL = 1024 / SL;                  // rows per DMA load
    constexpr int CPR = SL / 16;                    // 16-byte chunks per LDS row
    constexpr int A_BLK = BM / RPL, B_BLK = BN / RPL;
    constexpr int A_PER = A_BLK / NW, B_PER = B_BLK / NW;
    constexpr int SC_BLK = (BM + BN) / 64;          // 64 scales per 4-byte DMA load
    constexpr int SC_PER = GROUPED ? (SC_BLK + NW - 1) / NW : 0;
    constexpr int LOADS = A_PER + B_PER + SC_PER;
    // A's ring is counted in units of 64 rows (AU per slice): NST slices and
    // XA spare units. The spare units take the first XA units of slice
    // sl + NST while slices sl .. sl + NST - 1 are all still in use, so a
    // slice's DMA loads spread over both of its k steps (LOADS0 of them in
    // the first) instead of crowding the second, whose MFMAs they held up.
    constexpr int AU = BM / 64;
    constexpr int UNIT = 64 * SL;
    constexpr int RA = NST * AU + XA;
    constexpr int LPU = 64 / RPL / NW;              // loads per wave and A unit
    constexpr int LOADS0 = XA * LPU;
    constexpr int A_RING = RA * UNIT;
    constexpr int SMEM = A_RING + NST * B_BYTES;
    static_assert(SL == kBK, "a slice is one k block");
    static_assert(BM % 64 == 0 && BN % 32 == 0 && (BM + BN) % 64 == 0, "tile shape");
    static_assert(A_BLK % NW == 0 && B_BLK % NW == 0 && LPU * NW * RPL == 64 && NW % 2 == 0, "whole loads per wave");
    static_assert(XA == 0 || (KH == 2 && !PROD && XA <= AU), "spare units");
    static_assert(NST >= 2 && (NST - 1) * LOADS + LOADS0 <= 63, "pipeline depth");
    static_assert(XA == 0 || WTM % 64 == 0, "a wave's rows are whole A units of a wrapping ring");

    // A's ring, B's stages, and the grouped scales of a slice's rows (A then
    // B), float, DMA'd like the operands
    __shared__ __attribute__((aligned(1024))) uint8_t smem[SMEM + (GROUPED ? NST * (BM + BN) * 4 : 0)];
    float* const ssc = reinterpret_cast<float*>(smem + SMEM);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = PROD && wave_id >= NW;
    // consumer waves 0..NW-1; a producer takes the DMA share of consumer wave_id - NW
    const int wave = producer ? wave_id - NW : wave_id;
    const int wm = wave / WN, wn = wave % WN;

    // ---- tile index: contiguous ranges per XCD, grouped by p.gm row panels
    const int T = gridDim.x;
    const int b = blockIdx.x;
    int lt = (T % 8 == 0) ? (b % 8) * (T / 8) + b / 8 : b;
    // (divisions by host-made multipliers, skipped where the quotient is
    // zero: integer division is a long dependent chain, and a tile's first
    // loads wait for this index; a symmetric product has only the tiles on or
    // above the diagonal)
    const int per_split = (int)p.per_split.d;
    if (p.batch > 1) {
        // problem bi of a batched launch: its operands, output and partials
        const int bi = (int)p.per_problem.quotient((uint32_t)lt);
        lt -= bi * (int)p.per_problem.d;
        p.A += bi * p.bsa;
        p.B += bi * p.bsb;
        p.D = reinterpret_cast<uint8_t*>(p.D) + bi * p.bsd;
        if (p.residual) p.residual += bi * p.bsr;
        p.partial += (int64_t)bi * p.splits * p.M * p.N;
    }
    const int ks = p.splits > 1 ? (int)p.per_split.quotient((uint32_t)lt) : 0;
    const int rem = lt - ks * per_split;
    int tm, tn;
    if (p.upper) {
        // row tm of the upper triangle holds tiles_n - tm tiles (a uniform scalar walk)
        int r = rem;
        tm = 0;
        while (r >= p.tiles_n - tm) {
            r -= p.tiles_n - tm;
            ++tm;
        }
        tn = tm + r;
    } else {
        const int group = (int)p.per_group.quotient((uint32_t)rem);
        const int first_m = group * p.gm;
        const int gsz = min(p.gm, p.tiles_m - first_m);
        const int r2 = rem - group * p.gm * p.tiles_n;
        // r2 / gsz, gsz <= 4 (2^32 / 3 rounded up: exact below 2^31)
        tn = gsz == 4 ? r2 >> 2 : gsz == 3 ? (int)__umulhi((uint32_t)r2, 0x55555556u) : gsz == 2 ? r2 >> 1 : r2;
        tm = first_m + r2 - tn * gsz;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    // k slices [s0, s1): this split's 128-byte k blocks
    const int s0 = ks * p.ksteps_per_split;
    const int s1 = min((ks + 1) * p.ksteps_per_split, p.ksteps);

    const int valid_m = min(BM, p.M - m0), valid_n = min(BN, p.N - n0);
    const v4i ra = make_rsrc(p.A + (int64_t)m0 * p.lda, (uint32_t)(valid_m * p.lda));
    const v4i rb = make_rsrc(p.B + (int64_t)n0 * p.ldb, (uint32_t)(valid_n * p.ldb));

    // LDS layout of a slice: row r of a tile is SL bytes (CPR 16-byte chunks)
    // and its logical chunk c sits at position c ^ key(r), key(r) = (r & 7) ^
    // ((r >> 3) & 1). The 16 (or 8) lanes of a ds_read_b128 phase read 16 (8)
    // consecutive rows at the same logical chunk: of 16 rows the 8 even (odd)
    // ones, which share the lower (upper) half of a 256-byte bank line, get
    // distinct keys, and 8 rows in a 128-byte line get the keys 0..7.
    // Lane l of a DMA load fills row RPL * blk + l / CPR at position l % CPR,
    // so it fetches the logical chunk (l % CPR) ^ key(row) of that row.
    auto row_key = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
    // logical k byte a lane fetches (a wave's row blocks all have its parity)
    const int kch = ((lane % CPR) ^ row_key((wave & 1) * RPL + lane / CPR)) * 16;
    const uint32_t blkA = (uint32_t)(RPL * p.lda), blkB = (uint32_t)(RPL * p.ldb);
    const uint32_t voffA = (uint32_t)((lane / CPR) * p.lda) + wave * blkA + kch;
    const uint32_t voffB = (uint32_t)((lane / CPR) * p.ldb) + wave * blkB + kch;
    const uint32_t smem_lds = lds_addr(smem);
    const uint32_t ssc_lds = smem_lds + SMEM;

    v4i rsa{}, rsb{};
    // Scale load j of this wave brings entries 64 t .. 64 t + 63 (t = its
    // chunk) of a slice's scale vector: BM entries for A, then BN for B. A
    // row-scaled operand has one entry per tile row, a block-scaled one one
    // per 128-row block (entries past that are unused). Lane l loads the
    // element at byte sc_base[j] + kb * sc_kstride[j] for k block kb
    // (row-major scales: a stride of one element; k-major: the array's row
    // pitch), or nothing when sc_base[j] is kOOB; all of it is fixed before
    // the main loop.
    uint32_t sc_base[SC_PER > 0 ? SC_PER : 1], sc_kstride[SC_PER > 0 ? SC_PER : 1];
    bool sc_is_a[SC_PER > 0 ? SC_PER : 1];
    auto scale_setup = [&](int lane) __attribute__((always_inline)) {
        rsa = make_rsrc(p.sa, p.a_mode == kSTensor ? 0u : p.sa_bytes);
        rsb = make_rsrc(p.sb, p.b_mode == kSTensor ? 0u : p.sb_bytes);
#pragma unroll
        for (int j = 0; j < SC_PER; ++j) {
            const int t = (wave * SC_PER + j) % SC_BLK;
            const bool is_a = t * 64 < BM;
            const int r = t * 64 + lane - (is_a ? 0 : BM);
            const int mode = is_a ? p.a_mode : p.b_mode;
            const bool km = is_a ? p.a_kmajor : p.b_kmajor;
            const int ld = is_a ? p.ld_sa : p.ld_sb;
            const int row0 = is_a ? m0 : n0;
            const int rows = is_a ? p.M : p.N;
            // row (row scales) or 128-row block (block scales) of this lane's
            // entry, and the number of them that exist or the tile touches
            const bool blocks = mode == kSBlock;
            const int unit = (blocks ? row0 >> 7 : row0) + r;
            const int tile_end = ((row0 + (is_a ? BM : BN) - 1) >> 7) + 1;
            const int end = mode == kSTensor ? 0 : blocks ? min(tile_end, (rows + 127) >> 7) : rows;
            sc_is_a[j] = is_a;
            sc_base[j] = unit < end ? (uint32_t)(unit * (km ? 1 : ld)) * 4u : kOOB;
            // (no stride without scales: an empty descriptor takes no offset)
            sc_kstride[j] = mode == kSTensor ? 0u : (km ? (uint32_t)ld : 1u) * 4u;
        }
    };
    (void)sc_base; (void)sc_kstride; (void)sc_is_a;

    // positions in A's ring, bytes
    auto wrap = [](int u) __attribute__((always_inline)) { return u >= A_RING ? u - A_RING : u; };
    // What the DMA loads of slice `sl` share: the lane offsets into A and B
    // (out of range in the k tail, K % SL != 0, which reads as zeros on
    // purpose), the k offset, and where the slice starts in A's ring. Past
    // the last slice (!valid) the loads still issue, so that every wave
    // always has the same number in flight and waits on constant counts, but
    // read out of range: no memory traffic, zeros into a place no later slice
    // uses.
    struct Slice {
        uint32_t va, vb, soff;
        int ua;
        bool valid;
    };
    auto slice_loads = [&](int ua, int sl, bool valid) __attribute__((always_inline)) {
        const int k0 = sl * SL;
        const bool in = k0 + kch < (valid ? p.K : 0);
        return Slice{in ? voffA : kOOB, in ? voffB : kOOB, valid ? (uint32_t)k0 : 0u, ua, valid};
    };
    // DMA load q (0 <= q < LOADS) of this wave: A's into the ring, the rest
    // into stage `st`.
    auto dma_one = [&](const Slice& s, int st, int q) __attribute__((always_inline)) {
        if (q < A_PER) {
            dma_to_lds<16>(ra, smem_lds + wrap(s.ua + q / LPU * UNIT) + (q % LPU) * (NW * 1024) + wave * 1024,
                           s.va + q * (NW * blkA), s.soff);
        } else if (q < A_PER + B_PER) {
            dma_to_lds<16>(rb, smem_lds + A_RING + st * B_BYTES + (q - A_PER) * (NW * 1024) + wave * 1024,
                           s.vb + (q - A_PER) * (NW * blkB), s.soff);
        } else if constexpr (GROUPED) {
            const int j = q - A_PER - B_PER;
            const int t = (wave * SC_PER + j) % SC_BLK;
            const uint32_t dst = ssc_lds + (st * (BM + BN) + t * 64) * 4;
            dma_to_lds<4>(sc_is_a[j] ? rsa : rsb, dst, s.valid ? sc_base[j] : kOOB, (s.soff / kBK) * sc_kstride[j]);
        }
    };

    v16f acc[FM][FN];

    const int fr = lane & 31;                 // fragment row of this lane
    const int c0 = (lane >> 5) * 2;           // first of this lane's two chunks in a 64-byte k step
    // key of the lane's fragment rows (fragments start at multiples of 32)
    const int key = row_key(fr);

    // The operand fragments of one 64-byte k step as this wave holds them:
    // for each 32-row fragment (A fragments first) 32 bytes of k per lane,
    // bytes 32 (l >> 5) .. + 31 of the step in row l & 31, from two 16-byte
    // LDS reads; and the E8M0 scale of each fragment row.
    struct Frags {
        v8i f[FM + FN];
        uint32_t sc[FM + FN];
    };
    // the LDS entry of each fragment row's scale within a stage's scale
    // vector (block scales: the row's 128-row block counted from the block
    // of the tile's first row, which need not start a block when the tile
    // is 192 rows)
    int sc_off[FM + FN];
#pragma unroll
    for (int fi = 0; fi < FM + FN; ++fi) {
        const bool is_a = fi < FM;
        const int r = is_a ? wm * WTM + fi * 32 + fr : wn * WTN + (fi - FM) * 32 + fr;   // tile row
        const int row0 = is_a ? m0 : n0;
        const int mode = is_a ? p.a_mode : p.b_mode;
        sc_off[fi] = (is_a ? 0 : BM) + (mode == kSBlock ? ((row0 + r) >> 7) - (row0 >> 7) : r);
    }
    // read piece t of k step h of the slice in stage st: t < FM + FN are
    // the operand fragments, the rest the scales (their raw binary32 bits:
    // scale_e8m0 turns them into the instruction's operands once they have
    // landed, so that no read waits on its own result)
    // (LDS addresses: `at` holds a lane's two 16-byte chunks of the k step in
    // each of its A units' first fragment row, then in B's)
    constexpr int NPIECE = (FM + FN) * (GROUPED ? 2 : 1);
    // a wave's A units (without spare units a slice does not wrap: one run)
    constexpr int UW = XA ? WTM / 64 : 1;
    struct Addr {
        uint32_t lo[UW + 1], hi[UW + 1];
    };
    typedef const __attribute__((address_space(3))) v4i* lds_v4i;
    uint32_t lane_at[KH][2];
#pragma unroll
    for (int h = 0; h < KH; ++h)
#pragma unroll
        for (int c = 0; c < 2; ++c) lane_at[h][c] = smem_lds + fr * SL + (((4 * h + c0 + c) ^ key) << 4);
    auto address = [&](int ua, int st, int h) __attribute__((always_inline)) {
        Addr at;
#pragma unroll
        for (int u = 0; u <= UW; ++u) {
            const uint32_t off = u < UW ? wrap(ua + wm * WTM * SL + u * UNIT) : A_RING + st * B_BYTES + wn * WTN * SL;
            at.lo[u] = lane_at[h][0] + off;
            at.hi[u] = lane_at[h][1] + off;
        }
        return at;
    };
    auto read_piece = [&](Frags& f, const Addr& at, int st, int t) __attribute__((always_inline)) {
        if (t < FM + FN) {
            const int u = t < FM ? (XA ? t / 2 : 0) : UW, off = (t < FM ? (XA ? t % 2 : t) : t - FM) * (32 * SL);
            const v4i lo = *(lds_v4i)(uintptr_t)(at.lo[u] + off);
            const v4i hi = *(lds_v4i)(uintptr_t)(at.hi[u] + off);
            f.f[t] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            const int fi = t - (FM + FN);
            f.sc[fi] = __float_as_uint(ssc[st * (BM + BN) + sc_off[fi]]);
        }
    };
    // The matrix instruction's scale operand of fragment fi: the E8M0
    // exponent in the top byte (the instruction takes byte 3; the bits below
    // it are ignored), 127 (a factor of 1) for a per-tensor scaled operand,
    // whose LDS entries are zeros and whose factor the epilogue applies. The
    // empty asm keeps the shift here: the compiler would otherwise place it
    // at the LDS read and wait for that read at once.
    const uint32_t unit_a = p.a_mode == kSTensor ? 127u << 24 : 0u;
    const uint32_t unit_b = p.b_mode == kSTensor ? 127u << 24 : 0u;
    auto scale_e8m0 = [&](Frags& f, int fi) __attribute__((always_inline)) {
        if constexpr (GROUPED) {
            asm volatile("" : "+v"(f.sc[fi]));
            f.sc[fi] = (f.sc[fi] << 1) | (fi < FM ? unit_a : unit_b);
        }
    };
    auto mfma_one = [&](const Frags& f, int t) __attribute__((always_inline)) {
        const int i = t / FN, j = t % FN;
        if constexpr (FA == kBF16) {
            // BF16: the lane's 32 bytes are 16 k values; each half feeds one
            // 32x32x16 instruction. A and B split k the same way, so the two
            // instructions together add every product of the 64-byte step.
            const v4i blo = __builtin_shufflevector(f.f[FM + j], f.f[FM + j], 0, 1, 2, 3);
            const v4i bhi = __builtin_shufflevector(f.f[FM + j], f.f[FM + j], 4, 5, 6, 7);
            const v4i alo = __builtin_shufflevector(f.f[i], f.f[i], 0, 1, 2, 3);
            const v4i ahi = __builtin_shufflevector(f.f[i], f.f[i], 4, 5, 6, 7);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, blo),
                                                                __builtin_bit_cast(v8bf, alo), acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, bhi),
                                                                __builtin_bit_cast(v8bf, ahi), acc[i][j], 0, 0, 0);
        } else if constexpr (GROUPED)
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                f.f[FM + j], f.f[i], acc[i][j], FB, FA, 3, (int)f.sc[FM + j], 3, (int)f.sc[i]);
        else
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                f.f[FM + j], f.f[i], acc[i][j], FB, FA, 0, 127, 0, 127);
    };

    // One pipeline step: the MFMAs of k step h of slice sl (fragments in
    // `cur`, read during the previous step) with the LDS reads of the next
    // k step (into `nxt`, from `at`) and DMA loads of slice sl + NST
    // interleaved between them, so that LDS and memory latency hide behind
    // the MFMAs: the loads into A's spare units in the first k step, the rest
    // in the last.
    // Before the reads of the next slice (in its last k step) a wave waits
    // until its loads of slice sl + 1 have landed (the NST - 2 slices after
    // it and the LOADS0 loads just issued may still be in flight) and until
    // its reads of slice sl are complete (lgkmcnt(0)). After the barrier
    // every wave is at that point: slice sl + 1 is in LDS and the places of
    // slice sl are free for the DMA of slice sl + NST. The loop body has no
    // branches: reads past the last slice fetch stale LDS data that is never
    // used, and DMA loads past it read nothing.
    // Everything but the MFMAs has to fit into the 16 issue slots an MFMA
    // leaves its wave: the wait and the barrier come after the step's first
    // MFMA (which needs only registers), the DMA loads' shared state after
    // the second, the next step's read addresses three before the last. Empty
    // asm statements keep the compiler from moving that arithmetic (pin) or
    // the MFMAs themselves ("+a").
    constexpr int NMFMA = FM * FN;
    constexpr int SC0 = NMFMA / 2, SCD = NMFMA / 4;
    constexpr int TAT = NMFMA > 4 ? NMFMA - 3 : NMFMA / 2, TLD = NMFMA > 1 ? 1 : 0;
    // (a step of one MFMA takes everything after it)
    auto load_at = [](int q, int n) { return TLD + q * (NMFMA - TLD) / (n > 0 ? n : 1); };
    int ua = 0, st = 0;                        // where slice sl starts in A's ring, its stage
    int un = 0, stn = 0;                       // the same of slice sl + 1
    Slice ld{};
    auto step = [&](int sl, int h, Frags& cur, Frags& nxt, const Addr& at, Addr& at_next) __attribute__((always_inline)) {
        const bool last = h == KH - 1;
        // fragment read u goes after MFMA u * NMFMA / NPIECE in the last k
        // step, and spread over three quarters of the first; DMA load q
        // after MFMA load_at(q, the step's loads) (constant loop
        // bounds, so that everything unrolls and the fragments stay in
        // registers). A slice's k steps share its scales (one 128-wide k
        // block): the last step reads the next slice's, two after each MFMA
        // from the middle on, and makes them operands a quarter step later;
        // the first passes them on.
        if constexpr (GROUPED) {
            if (!last) {
#pragma unroll
                for (int fi = 0; fi < FM + FN; ++fi) nxt.sc[fi] = cur.sc[fi];
            }
        }
        auto sc_at = [](int fi) { return SC0 + fi / 2 + SCD < NMFMA - 1 ? SC0 + fi / 2 + SCD : NMFMA - 1; };
#pragma unroll
        for (int t = 0; t < NMFMA; ++t) {
            mfma_one(cur, t);
            asm volatile("" : "+a"(acc[t / FN][t % FN]));
            if (t == 0 && last) {
                if constexpr (PROD)
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                else
                    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((NST - 2) * LOADS + LOADS0) : "memory");
                __syncthreads();
            }
            if (t == TLD && !last) {
                pin(ua); pin(st); pin(sl);
                un = wrap(ua + AU * UNIT);
                stn = st + 1 == NST ? 0 : st + 1;
                // slice sl + NST starts XA units before slice sl's first
                // (NST AU = RA - XA units on)
                if (!PROD)
                    ld = slice_loads(XA ? (ua >= XA * UNIT ? ua - XA * UNIT : ua - XA * UNIT + A_RING) : ua, sl + NST,
                                     sl + NST < s1);
            }
            if (t == TAT) {
                pin(un); pin(stn);
                at_next = address(un, stn, last ? 1 : 0);
            }
#pragma unroll
            for (int u = 0; u < FM + FN; ++u)
                if (last ? u * NMFMA / NPIECE == t : u * (NMFMA * 3 / 4) / (FM + FN) == t) read_piece(nxt, at, stn, u);
            if (last) {
#pragma unroll
                for (int u = FM + FN; u < NPIECE; ++u)
                    if (SC0 + (u - FM - FN) / 2 == t) read_piece(nxt, at, stn, u);
#pragma unroll
                for (int fi = 0; fi < FM + FN; ++fi)
                    if (sc_at(fi) == t) scale_e8m0(nxt, fi);
            }
            if (!PROD) {
                constexpr int L1 = LOADS - LOADS0;
#pragma unroll
                for (int q = 0; q < (last ? L1 : LOADS0); ++q)
                    if ((NMFMA == 1 ? 0 : load_at(q, last ? L1 : LOADS0)) == t)
                        dma_one(ld, st, last ? LOADS0 + q : q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // prologue: slices s0 .. s0 + NST - 1 in flight, then k step 0 of slice
    // s0 read. The operands' loads issue as soon as their offsets are known,
    // no faster than the texture unit takes them (64 bytes per clock): the
    // scales' set-up follows slice s0's, and the accumulators are cleared
    // between the loads (not in a deep ring's prologue, which is a loop: its
    // addresses would not fit into the scalar registers unrolled).
    constexpr bool kRolled = PROD || NST > 4;
    auto clear = [&](int n, int of) __attribute__((always_inline)) {
        constexpr int R = FM * FN;
#pragma unroll
        for (int e = R * n / of; e < R * (n + 1) / of; ++e) {
            // 0 x 0 + 0: one instruction for a fragment's 16 registers
            acc[e / FN][e % FN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v8bf{}, v8bf{}, v16f{}, 0, 0, 0);
            asm volatile("" : "+a"(acc[e / FN][e % FN]));      // here, not earlier
        }
    };
    if (!PROD || producer) {
        if constexpr (kRolled && GROUPED) scale_setup(lane);
        auto issue = [&](int t) __attribute__((always_inline)) {
            const Slice first = slice_loads(t * AU * UNIT, s0 + t, s0 + t < s1);
#pragma unroll
            for (int q = 0; q < LOADS; ++q) {
                if constexpr (!kRolled && GROUPED) {
                    if (t == 0 && q == A_PER + B_PER) {
                        int l = lane;
                        asm volatile("" : "+v"(l));
                        scale_setup(l);
                    }
                }
                dma_one(first, t, q);
                if constexpr (!kRolled) clear(t * LOADS + q, NST * LOADS);
            }
        };
        if constexpr (kRolled) {
#pragma unroll 1
            for (int t = 0; t < NST; ++t) issue(t);
        } else {
#pragma unroll
            for (int t = 0; t < NST; ++t) issue(t);
        }
    }
    if constexpr (kRolled) clear(0, 1);
    // per-tensor scales, applied to the FP32 sums in the epilogue (loaded
    // here so that their latency hides behind the main loop)
    float alpha = p.alpha;
    if (OUT != 2) {
        if (p.a_mode == kSTensor) alpha *= p.sa[0];
        if (p.b_mode == kSTensor) alpha *= p.sb[0];
    }
    if (!PROD || producer) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 1) * LOADS) : "memory");
    __syncthreads();
    if constexpr (PROD) {
        if (producer) {
            // per slice: slice sl + 1 landed, then (after the barrier at which
            // the consumers have read all of slice sl) its stage refilled with
            // slice sl + NST; the same barriers as the consumers' loop and
            // epilogue
            for (int sl = s0; sl < s1; ++sl) {
                asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 2) * LOADS) : "memory");
                __syncthreads();
                const int st = (sl - s0) % NST;
#pragma unroll
                for (int q = 0; q < LOADS; ++q) dma_one(slice_loads(st * AU * UNIT, sl + NST, sl + NST < s1), st, q);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();   // the epilogue's barrier: the ring is idle
            return;
        }
    }
    Frags F0, F1;
    Addr at0 = address(0, 0, 0), at1;
#pragma unroll
    for (int t = 0; t < NPIECE; ++t) read_piece(F0, at0, 0, t);
#pragma unroll
    for (int fi = 0; fi < FM + FN; ++fi) scale_e8m0(F0, fi);
    at0 = address(0, 0, 1);
    for (int sl = s0; sl < s1; ++sl) {
        step(sl, 0, F0, F1, at0, at1);
        step(sl, 1, F1, F0, at1, at0);
        ua = un;
        st = stn;
    }
    // the loads issued for slices past the end write zeros into the ring,
    // which the epilogue reuses: let them land first. And the last MFMA's
    // results: a 16-pass matrix instruction's take 20 wait states to reach a
    // VALU read, which the compiler does not insert before the reads in
    // inline assembly below.
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 3" ::: "memory");

    // An accumulator read at its point of use (a copy the compiler may not
    // hoist): otherwise it moves accumulators to VGPRs ahead of the epilogue's
    // branches, and spills. (Volatile, so it stays behind the wait above, as
    // that stays behind the MFMAs, each followed by a volatile statement on
    // its result.)
    auto acc_at = [&](int i, int j, int e) __attribute__((always_inline)) {
        float v;
        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[i][j][e]));
        return v;
    };

    // ---- The LM head's forward statistics, straight from the accumulators.
    // Of each of its rows i*32 + (l & 31), lane l holds the 64 columns
    // j*32 + 8g + 4(l >> 5) + {0..3} of the wave tile; lane l ^ 32 holds the
    // other 64. A row's maximum and its sum of e^(z - max) over the 128
    // columns are the lane's over its 64 sums, combined with the partner's by
    // one exchange each: no staging, every logit read once. The exponent is
    // one FMA, z log2(e) - max log2(e), fed to the exp2 instruction. Its
    // rounding errs by a relative 2^-24 of |z| on each term and of |max| on
    // all of them alike, far inside the error of a binary32 log-sum-exp.
    if constexpr (OUT == kOutLseStats) {
        static_assert(!PROD && FN == 4 && WTN == 128, "LM-head statistics: 128-column wave tiles");
        const int mrow0 = m0 + wm * WTM, ncol0 = n0 + wn * WTN;
        if (ncol0 >= p.N) return;      // a wave tile wholly past N (the ragged last tile) has no block
        const int hl = lane >> 5;
        // each row's target column, relative to the lane's first column of
        // the wave tile (4 hl), or out of range
        int tcol[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int64_t m = (int64_t)mrow0 + i * 32 + (lane & 31);
            tcol[i] = m < p.M ? p.targets[m] - p.col0 - ncol0 - 4 * hl : INT_MIN;
        }
        constexpr float kLog2e = 1.44269504088896340736f;
        static_for<FM>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            float v[FN * 16];
#pragma unroll
            for (int e = 0; e < FN * 16; ++e) v[e] = acc_at(i, e / 16, e % 16);
            if (alpha != 1.0f) {
#pragma unroll
                for (int e = 0; e < FN * 16; ++e) v[e] *= alpha;
            }
            float mq[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
            for (int e = 4; e < FN * 16; ++e) mq[e % 4] = fmaxf(mq[e % 4], v[e]);
            float mx = fmaxf(fmaxf(mq[0], mq[1]), fmaxf(mq[2], mq[3]));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float m2 = mx * kLog2e;
            float sq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < FN * 16; ++e) sq[e % 4] += __builtin_amdgcn_exp2f(fmaf(v[e], kLog2e, -m2));
            float sum = (sq[0] + sq[1]) + (sq[2] + sq[3]);
            sum += __shfl_xor(sum, 32, 64);
            const int64_t m = (int64_t)mrow0 + i * 32 + (lane & 31);
            if (hl == 0 && m < p.M) p.stats[m * p.stats_ld + ncol0 / 128] = make_float2(mx, sum);
            // the target's logit, where this wave tile holds it: entry
            // (j, g, t) of fragment row i is column j*32 + 8g + t past the
            // lane's first (rare: a branch taken by the whole wave or not)
            const int tc = tcol[i];
            const bool mine = tc >= 0 && tc < WTN && ((tc >> 2) & 1) == 0;
            if (__builtin_amdgcn_ballot_w64(mine)) {
                float zt = 0.0f;
#pragma unroll
                for (int e = 0; e < FN * 16; ++e) {
                    const int j = e / 16, g = (e % 16) / 4, t = e % 4;
                    zt = tc == j * 32 + 8 * g + t ? v[e] : zt;
                }
                if (mine) p.zt[m] = zt;
            }
        });
        return;
    }

    // ---- epilogue. Lane l holds, for fragment (i, j), wave-tile row
    // i*32 + (l & 31) and columns j*32 + 8g + 4(l >> 5) + {0..3}, g = 0..3.
    // Written straight to memory that would scatter 16-byte pieces over 32
    // rows per store; instead each wave stages its FP32 tile in its own part
    // of the (now idle) stage buffers, 16-byte chunks XOR-swizzled by row so
    // that both the writes and the row reads are free of bank conflicts, and
    // then stores whole rows: consecutive lanes on consecutive 16-byte chunks
    // (4 FP32 values), converted and scaled on the way out.
    constexpr int ROWB = WTN * 4;                 // bytes of one staged wave-tile row (FP32)
    constexpr int ECPR = ROWB / 16;               // 16-byte chunks per staged row
    constexpr int REGION = NST * STAGE / NW;      // LDS bytes per wave
    constexpr int RFIT = REGION / ROWB;          // rows that fit in the region
    // rows per pass: WTM halved until it fits
    constexpr int RPP = WTM <= RFIT ? WTM : (WTM / 2 <= RFIT ? WTM / 2 : WTM / 4);
    // XOR key of the chunk swizzle: 16 distinct keys when rows have 16*k chunks, else 8
    constexpr int SWZ = (ECPR % 16 == 0) ? 15 : 7;
    static_assert(RPP >= 32 && WTM % RPP == 0 && (RPP * ECPR) % 64 == 0, "epilogue tiling");
    static_assert(ECPR % 8 == 0, "row swizzle needs 8k chunks per row");
    uint8_t* ep = smem + wave * REGION;
    const int mrow0 = m0 + wm * WTM;
    const int ncol0 = n0 + wn * WTN;
    float* const part = p.partial + (int64_t)ks * p.M * p.N;
    // a tile inside the matrix whose sums overwrite the output (or, binary32,
    // add to it) stores whole 4-column vectors everywhere: a branch-free path
    // that issues all of a pass's LDS reads before its stores
    constexpr int ES = (OUT == kOutF32 || OUT == 2) ? 4 : 2;    // bytes per output element
    const int64_t ldo = OUT == 2 ? (int64_t)p.N : p.ldd;          // output pitch (elements)
    // (and whose rows, and residual rows, lie within 2^31 bytes of its first:
    // the fast path addresses them with 32-bit buffer offsets)
    const bool fast = m0 + BM <= p.M && n0 + BN <= p.N && (OUT == 2 || OUT == kOutF32 || !p.accumulate) &&
                      (int64_t)WTM * ldo * ES <= INT32_MAX &&
                      (OUT != kOutBF16Epi || (int64_t)WTM * p.ldr * 2 <= INT32_MAX);
    // the bias of the lane's columns in the fast path below: lane chunk
    // (it * 64 + lane) % ECPR repeats with period ECPR / gcd(64, ECPR) in it
    constexpr int EP = ECPR / ((ECPR & -ECPR) < 64 ? (ECPR & -ECPR) : 64);
    uint2 eb[OUT == kOutBF16Epi ? EP : 1];
    if constexpr (OUT == kOutBF16Epi) {
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(p.bias), 0, p.bias ? p.N * 2 : 0, 0x00020000);
#pragma unroll
        for (int it = 0; it < EP; ++it)
            eb[it] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(
                rb, (uint32_t)((ncol0 + ((it * 64 + lane) % ECPR) * 4) * 2), 0, 0));
    }
    __syncthreads();   // every wave is done with the last stage
    // A plain BF16 output of a tile inside the matrix, 128-column wave tiles:
    // the lane rounds its sums to BF16 first and stages those, half the LDS
    // bytes of the binary32 staging below, and the whole wave tile fits its
    // region in one pass. Staged row r is 256 bytes, 32 units of 8 bytes
    // (four columns), and unit u sits at position u ^ 2 (r & 15): the two
    // units of each 16-byte chunk stay side by side and in order, so a chunk
    // reads back with one 16-byte load and leaves with one 16-byte store (a
    // store covers four whole rows); a chunk's position in its row depends
    // on r & 15, so the 16 lanes of a read phase, one row's 16 chunks, hit
    // distinct banks.
    // The LM head's backward output (dz of the logits) takes the same path:
    // each lane forms dz = g (exp(z - lse) - [column == target]) from its
    // sums directly, with the lse and target column of its FM rows loaded
    // first, and rounds it to BF16. The exponential is 2^t (1 + c): with
    // lse log2(e) split per row into its binary32 rounding P and the rest,
    // t = z log2(e)_hi - P is one FMA, which rounds once as z - lse would,
    // and 1 + c, the rest of the exponent times ln 2, is another.
    // Its dz kinds take every wave tile this way (M and N are multiples of
    // 128, so a wave tile lies wholly inside the output or wholly outside):
    // kOutSoftmaxGradQ quantises the staged tile (below).
    constexpr bool kDz = OUT == kOutSoftmaxGrad || OUT == kOutSoftmaxGradQ;
    static_assert(!kDz || (ECPR == 32 && WTM == 128 && WTM * 256 <= REGION), "dz kinds: 128 x 128 wave tiles");
    if constexpr ((OUT == kOutBF16 || OUT == kOutBF16Epi || kDz) && ECPR == 32 && WTM * 256 <= REGION) {
        if constexpr (kDz) {
            if (mrow0 + WTM > p.M || ncol0 + WTN > p.N) return;
        }
        if (kDz || fast) {
            // per row: P = lse log2(e)_hi rounded, K = 1 - (the rest of
            // lse log2(e)) ln 2 (rounded once), and the target's column
            // relative to the lane's first column of the wave tile
            constexpr float kL2eHi = 1.44269502162933349609375f;     // log2(e) rounded to binary32
            constexpr float kL2eLo = 1.925962989e-8f;                // log2(e) - kL2eHi
            constexpr float kLn2 = 0.693147180559945309f;
            constexpr float kL2eLoLn2 = kL2eLo * kLn2;
            float row_p[kDz ? FM : 1], row_k[kDz ? FM : 1];
            int row_tgt[kDz ? FM : 1];
            if constexpr (kDz) {
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    const int64_t m = (int64_t)mrow0 + i * 32 + (lane & 31);
                    row_tgt[i] = p.targets[m] - p.col0 - ncol0 - 4 * (lane >> 5);
                    const float l = p.lse[m];
                    row_p[i] = l * kL2eHi;
                    row_k[i] = 1.0f - (fmaf(l, kL2eHi, -row_p[i]) + l * kL2eLo) * kLn2;
                }
            }
            (void)row_p; (void)row_k; (void)row_tgt;
            // The bias / residual epilogue in the same one pass: the wave's
            // residual block arrives in its LDS region by DMA, each 16-byte
            // chunk already where the staged output chunk will sit (the lane
            // that lands chunk position q of row r loads the residual's chunk
            // q ^ (r & 15)); the lane then reads the four residual values of
            // each of its output units there, forms alpha acc + bias + rs
            // residual in binary32 with one rounding to BF16, and writes the
            // result over them. The bias of the lane's 64 columns is loaded
            // into registers once.
            uint2 bq[OUT == kOutBF16Epi ? FN * 4 : 1];
            if constexpr (OUT == kOutBF16Epi) {
                if (p.bias) {
                    const __amdgpu_buffer_rsrc_t rbq = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<uint16_t*>(p.bias), 0, p.N * 2, 0x00020000);
#pragma unroll
                    for (int e = 0; e < FN * 4; ++e)
                        bq[e] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(
                            rbq, (uint32_t)((ncol0 + (e / 4) * 32 + 8 * (e % 4) + 4 * (lane >> 5)) * 2), 0, 0));
                }
                if (p.residual) {
                    const v4i rr = make_rsrc(p.residual + (int64_t)mrow0 * p.ldr + ncol0,
                                             (uint32_t)((WTM - 1) * p.ldr * 2 + WTN * 2));
                    const uint32_t ep_lds = smem_lds + wave * REGION;
#pragma unroll
                    for (int q = 0; q < WTM / 4; ++q) {          // 1 KB: four rows of 256 bytes
                        const int r = q * 4 + (lane >> 4), c = (lane & 15) ^ (r & 15);
                        dma_to_lds<16>(rr, ep_lds + q * 1024, (uint32_t)((r * p.ldr + c * 8) * 2), 0u);
                    }
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            (void)bq;
            // Stores: chunk l & 15 of staged row 4 it + (l >> 4) in iteration
            // it; (r & 15) repeats every 4 iterations, so four lane addresses
            // serve all of them with compile-time offsets.
            typedef unsigned int v4u __attribute__((ext_vector_type(4)));
            const int rl = lane >> 4, cl = lane & 15;
            uint32_t la[4];
#pragma unroll
            for (int ph = 0; ph < 4; ++ph) {
                const int r = 4 * ph + rl;
                la[ph] = r * 256 + ((cl ^ (r & 15)) << 4);
            }
            const uint32_t row_bytes = (uint32_t)(p.ldd * 2);
            const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
                reinterpret_cast<uint8_t*>(p.D) + ((int64_t)mrow0 * p.ldd + ncol0) * 2, 0,
                (int)((WTM - 1) * row_bytes + WTN * 2), 0x00020000);
            const int voff = (int)(rl * row_bytes + cl * 16);
            (void)la; (void)rd; (void)voff;
            // one fragment (i, j) of the wave tile; `onehot` when some lane's
            // row has its target among the lane's columns of this wave tile
            // (a few rows in a hundred), else dz is g e throughout
            auto stage_one = [&](auto scaled, auto onehot, auto epi, int i, int j) __attribute__((always_inline)) {
                const int r = i * 32 + (lane & 31);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v0 = acc_at(i, j, 4 * g), v1 = acc_at(i, j, 4 * g + 1);
                    float v2 = acc_at(i, j, 4 * g + 2), v3 = acc_at(i, j, 4 * g + 3);
                    if constexpr (decltype(scaled)::value) {
                        v0 *= alpha; v1 *= alpha; v2 *= alpha; v3 *= alpha;
                    }
                    if constexpr (kDz) {
                        // the four sums are columns j*32 + 8g + {0..3} past the
                        // lane's first: tr is the target's position among them
                        const int tr = row_tgt[i] - (j * 32 + 8 * g);
                        const float P = row_p[i], K = row_k[i], gs = p.grad_scale;
                        auto dz = [&](float z, int c) __attribute__((always_inline)) {
                            // 2^(z log2 e - lse log2 e) = 2^t (1 + c)
                            const float e = __builtin_amdgcn_exp2f(fmaf(z, kL2eHi, -P)) * fmaf(z, kL2eLoLn2, K);
                            if constexpr (decltype(onehot)::value) return fmaf(gs, e, c == tr ? -gs : 0.0f);
                            else return gs * e;
                        };
                        v0 = dz(v0, 0); v1 = dz(v1, 1); v2 = dz(v2, 2); v3 = dz(v3, 3);
                    }
                    const int u = j * 8 + 2 * g + (lane >> 5);
                    uint2* const pos = reinterpret_cast<uint2*>(ep + r * 256 + ((u ^ (2 * (r & 15))) << 3));
                    if constexpr (OUT == kOutBF16Epi) {
                        // each term only when given: adding +0 would turn a -0 sum into +0
                        if constexpr ((decltype(epi)::value & 1) != 0) {
                            const uint2 b = bq[j * 4 + g];
                            v0 += bf16lo(b.x); v1 += bf16hi(b.x); v2 += bf16lo(b.y); v3 += bf16hi(b.y);
                        }
                        if constexpr ((decltype(epi)::value & 2) != 0) {
                            const uint2 rv = *pos;
                            const float rs = p.res_scale;
                            v0 = fmaf(rs, bf16lo(rv.x), v0); v1 = fmaf(rs, bf16hi(rv.x), v1);
                            v2 = fmaf(rs, bf16lo(rv.y), v2); v3 = fmaf(rs, bf16hi(rv.y), v3);
                        }
                    }
                    *pos = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
                }
            };
            // Fragment row i is staged while row i - 1 leaves: after each
            // fragment, two of the eight 16-byte chunks of row i - 1 that the
            // lane stores, whose LDS reads were issued before it. (The region
            // belongs to this wave alone, and LDS takes a wave's accesses in
            // their order: no wait between writing a row and reading it.)
            constexpr bool kStore = OUT != kOutSoftmaxGradQ;
            constexpr int AUX = OUT != kOutSoftmaxGrad && kStreamOut<FA> ? 2 : 0;   // 2: the non-temporal bit
            auto stage_row = [&](auto scaled, auto onehot, auto epi, auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value;
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    v4u d[2];
                    if constexpr (kStore && i > 0) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int it = (i - 1) * 8 + 2 * j + e, ph = it % 4;
                            d[e] = *reinterpret_cast<const v4u*>(ep + la[ph] + (it - ph) * 4 * 256);
                        }
                    }
                    if constexpr (i < FM) stage_one(scaled, onehot, epi, i, j);
                    if constexpr (kStore && i > 0) {
#pragma unroll
                        for (int e = 0; e < 2; ++e)
                            __builtin_amdgcn_raw_buffer_store_b128(d[e], rd, voff,
                                                                   (int)(((i - 1) * 8 + 2 * j + e) * 4 * row_bytes), AUX);
                    }
                    (void)d;
                    // one fragment at a time: otherwise every accumulator
                    // is read into VGPRs before the first write
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            auto stage = [&](auto scaled, auto epi) __attribute__((always_inline)) {
                static_for<FM + 1>([&](auto i_c) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_c)::value;
                    if constexpr (kDz && i < FM) {
                        // set for the lane that holds its row's target (and
                        // maybe for its partner lane): a wave-uniform branch
                        if (__builtin_amdgcn_ballot_w64((unsigned)row_tgt[i] < (unsigned)WTN))
                            stage_row(scaled, std::true_type{}, epi, i_c);
                        else
                            stage_row(scaled, std::false_type{}, epi, i_c);
                    } else {
                        stage_row(scaled, std::false_type{}, epi, i_c);
                    }
                });
            };
            // epi: bit 0 a bias, bit 1 a residual (bias / residual epilogue only)
            auto stage_epi = [&](auto epi) __attribute__((always_inline)) {
                if (alpha == 1.0f) stage(std::false_type{}, epi);
                else stage(std::true_type{}, epi);
            };
            if constexpr (OUT == kOutBF16Epi) {
                const int which = (p.bias ? 1 : 0) | (p.residual ? 2 : 0);
                if (which == 3) stage_epi(std::integral_constant<int, 3>{});
                else if (which == 2) stage_epi(std::integral_constant<int, 2>{});
                else if (which == 1) stage_epi(std::integral_constant<int, 1>{});
                else stage_epi(std::integral_constant<int, 0>{});
            } else {
                stage_epi(std::integral_constant<int, 0>{});
            }
            if constexpr (OUT == kOutSoftmaxGradQ) {
                // the region belongs to this wave alone
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                // its arguments are read here: scalar registers that would
                // hold them through the main loop are short
                const __attribute__((address_space(4))) Params* kp =
                    (const __attribute__((address_space(4))) Params*)__builtin_amdgcn_kernarg_segment_ptr();
                asm volatile("" : "+s"(kp));
                quantize_staged_dz(*kp, ep, mrow0, ncol0, lane);
            }
            return;
        }
    }
    // A tile that ends inside the matrix's last rows or columns (edge) stores
    // the same way where its lanes' 4-column vectors lie wholly in or out
    // (N % 4 == 0): its buffers end with its last valid row, lanes whose
    // columns lie outside get an offset out of range, and the row offsets go
    // into the lane offsets (as scalar operands they could exceed a buffer's
    // size, which the range check must not see).
    const int vrows = min(WTM, p.M - mrow0), vcols = min(WTN, p.N - ncol0);
    if (vrows <= 0 || vcols <= 0) return;
    const bool edge = !fast && p.N % 4 == 0 && (OUT == 2 || OUT == kOutF32 || !p.accumulate) &&
                      (int64_t)WTM * ldo * ES <= INT32_MAX &&
                      (OUT != kOutBF16Epi || (int64_t)WTM * p.ldr * 2 <= INT32_MAX);
    const bool sized = fast || edge;
    // Fast-path addressing. Iteration it of a pass covers staged row r and
    // chunk c with it * 64 + lane = r * ECPR + c. That map repeats every FP
    // iterations, FR rows further on, and the rows' chunk swizzle every NPH
    // such periods. So the lane parts of the LDS addresses (NPH x FP) and of
    // the output and residual offsets (FP) are computed here, once per tile;
    // an iteration adds a compile-time LDS offset and a wave-uniform row
    // offset (the buffer access's scalar operand). No store then computes a
    // 64-bit address.
    constexpr int FP = EP;
    constexpr int FR = 64 * FP / ECPR;
    constexpr int NPH = (SWZ + 1) / cgcd(FR, SWZ + 1);
    const uint32_t row_bytes = (uint32_t)(ldo * ES);
    const uint32_t rrow_bytes = OUT == kOutBF16Epi ? (uint32_t)(p.ldr * 2) : 0u;
    uint32_t laddr[NPH][FP], goff[FP], roff[FP];
#pragma unroll
    for (int vv = 0; vv < FP; ++vv) {
        const int q = vv * 64 + lane;
        const int rv = q / ECPR, cv = q % ECPR;
        goff[vv] = cv * 4 < vcols ? rv * row_bytes + cv * 4 * ES : kOOB;
        roff[vv] = cv * 4 < vcols ? rv * rrow_bytes + cv * 8 : kOOB;
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph) {
            const int r = ph * FR + rv;
            laddr[ph][vv] = r * ROWB + ((cv ^ (r & SWZ)) << 4);
        }
    }
    // the wave tile's output (and residual) rows as buffers: base at its
    // first element, range to its last valid row's last valid element
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
        OUT == 2 ? (void*)(part + (int64_t)mrow0 * p.N + ncol0)
                 : (void*)(reinterpret_cast<uint8_t*>(p.D) + ((int64_t)mrow0 * p.ldd + ncol0) * ES),
        0, sized ? (int)((vrows - 1) * row_bytes + vcols * ES) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
        OUT == kOutBF16Epi && p.residual ? const_cast<uint16_t*>(p.residual + (int64_t)mrow0 * p.ldr + ncol0) : nullptr,
        0, OUT == kOutBF16Epi && p.residual && sized ? (int)((vrows - 1) * rrow_bytes + vcols * 2) : 0, 0x00020000);
    (void)laddr; (void)goff; (void)roff; (void)rd; (void)rres;
    // one pass per constant: the accumulators are indexed by the pass, and a
    // loop the unroller leaves rolled would move them to scratch memory
    static_for<WTM / RPP>([&](auto pass_c) __attribute__((always_inline)) {
        constexpr int pass = decltype(pass_c)::value;
#pragma unroll
        for (int ii = 0; ii < RPP / 32; ++ii) {
            const int i = pass * (RPP / 32) + ii;
            const int r = ii * 32 + (lane & 31);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int chunk = j * 8 + g * 2 + (lane >> 5);
                    const float4 v = make_float4(acc_at(i, j, 4 * g), acc_at(i, j, 4 * g + 1),
                                                 acc_at(i, j, 4 * g + 2), acc_at(i, j, 4 * g + 3));
                    *reinterpret_cast<float4*>(ep + r * ROWB + ((chunk ^ (r & SWZ)) << 4)) = v;
                }
        }
        // the region belongs to this wave alone: once its own writes are
        // done other lanes of the wave may read them (and the next pass
        // writes only after this pass's reads have returned their data)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        constexpr int IT = RPP * ECPR / 64;
        if (sized) {
            // the residual is loaded before the LDS reads of its group of
            // iterations, so that its latency overlaps those reads and the
            // group's stores wait once (a load issued after stores waits for
            // them); an absent residual is a zero-range buffer (no branch, no
            // traffic). Groups of at most 16 iterations keep the residual and
            // the staged values in registers beside the accumulators of the
            // passes still to come.
            // With ACC (binary32 output added to what D holds) each group
            // first loads the outputs it replaces, with the stores' own
            // addressing, in the same place as the residual.
            auto run_groups = [&](auto acc_c, auto edge_c) __attribute__((always_inline)) {
                constexpr bool ACC = decltype(acc_c)::value;
                // where an iteration's row offset goes: the scalar operand,
                // or (edge) the lane offset
                auto lane_off = [](uint32_t off, uint32_t row) __attribute__((always_inline)) {
                    return (int)(decltype(edge_c)::value ? off + row : off);
                };
                auto row_off = [](uint32_t row) __attribute__((always_inline)) {
                    return (int)(decltype(edge_c)::value ? 0u : row);
                };
                constexpr int EG = ((OUT == kOutBF16Epi || ACC) && IT > 16) ? IT / 2 : IT;
                static_assert(IT % EG == 0 && EG % FP == 0, "epilogue groups");
                typedef unsigned int v4a __attribute__((ext_vector_type(4)));
#pragma unroll
                for (int g0 = 0; g0 < IT; g0 += EG) {
                    v4a ea[ACC ? EG : 1];
                    if constexpr (ACC) {
#pragma unroll
                        for (int e = 0; e < EG; ++e) {
                            const int u = (g0 + e) / FP, vv = (g0 + e) % FP;
                            const uint32_t row = (pass * RPP + u * FR) * row_bytes;
                            ea[e] = __builtin_bit_cast(v4a, __builtin_amdgcn_raw_buffer_load_b128(
                                rd, lane_off(goff[vv], row), row_off(row), 0));
                        }
                    }
                    (void)ea;
                    uint2 er[OUT == kOutBF16Epi ? EG : 1];
                    if constexpr (OUT == kOutBF16Epi) {
#pragma unroll
                        for (int e = 0; e < EG; ++e) {
                            const int u = (g0 + e) / FP, vv = (g0 + e) % FP;
                            const uint32_t row = (pass * RPP + u * FR) * rrow_bytes;
                            er[e] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(
                                rres, lane_off(roff[vv], row), row_off(row), 0));
                        }
                    }
                    float4 v[EG];
#pragma unroll
                    for (int e = 0; e < EG; ++e) {
                        const int u = (g0 + e) / FP, vv = (g0 + e) % FP, ph = u % NPH;
                        v[e] = *reinterpret_cast<const float4*>(ep + laddr[ph][vv] + (u - ph) * FR * ROWB);
                    }
                    if constexpr (OUT != 2) {
                        if (alpha != 1.0f) {
#pragma unroll
                            for (int e = 0; e < EG; ++e) {
                                v[e].x *= alpha; v[e].y *= alpha; v[e].z *= alpha; v[e].w *= alpha;
                            }
                        }
                    }
                    // AUX 2 is the buffer store's non-temporal bit
                    auto store_group = [&](auto nt_c) __attribute__((always_inline)) {
                        constexpr int AUX = decltype(nt_c)::value ? 2 : 0;
#pragma unroll
                        for (int e = 0; e < EG; ++e) {
                            const int u = (g0 + e) / FP, vv = (g0 + e) % FP;
                            const uint32_t row = (pass * RPP + u * FR) * row_bytes;
                            const int voff = lane_off(goff[vv], row), soff = row_off(row);
                            float4 w = v[e];
                            if constexpr (OUT == kOutBF16Epi) {
                                // each term only when given: adding +0 would turn a -0 sum into +0
                                if (p.bias) {
                                    const uint2 b = eb[vv];
                                    w.x += bf16lo(b.x); w.y += bf16hi(b.x); w.z += bf16lo(b.y); w.w += bf16hi(b.y);
                                }
                                if (p.residual) {
                                    const uint2 rv = er[e];
                                    const float rs = p.res_scale;
                                    w.x = fmaf(rs, bf16lo(rv.x), w.x); w.y = fmaf(rs, bf16hi(rv.x), w.y);
                                    w.z = fmaf(rs, bf16lo(rv.y), w.z); w.w = fmaf(rs, bf16hi(rv.y), w.w);
                                }
                            }
                            if constexpr (ES == 4) {
                                if constexpr (ACC) {
                                    const float4 o = __builtin_bit_cast(float4, ea[e]);
                                    w.x += o.x; w.y += o.y; w.z += o.z; w.w += o.w;
                                }
                                typedef unsigned int v4u __attribute__((ext_vector_type(4)));
                                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, w), rd, voff, soff, AUX);
                            } else {
                                typedef unsigned int v2u __attribute__((ext_vector_type(2)));
                                __builtin_amdgcn_raw_buffer_store_b64(v2u{pack_bf16x2(w.x, w.y), pack_bf16x2(w.z, w.w)}, rd,
                                                                      voff, soff, AUX);
                            }
                        }
                    };
                    if constexpr (ES == 2) {
                        store_group(std::bool_constant<kStreamOut<FA>>{});
                    } else {
                        if (OUT != 2 && p.nt_f32) store_group(std::true_type{});
                        else store_group(std::false_type{});
                    }
                }
            };
            auto run = [&](auto edge_c) __attribute__((always_inline)) {
                if constexpr (OUT == kOutF32) {
                    if (p.accumulate) run_groups(std::true_type{}, edge_c);
                    else run_groups(std::false_type{}, edge_c);
                } else {
                    run_groups(std::false_type{}, edge_c);
                }
            };
            if (fast) run(std::false_type{});
            else run(std::true_type{});
            return;
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int q = it * 64 + lane;
            const int r = q / ECPR, c = q % ECPR;
            float4 v = *reinterpret_cast<const float4*>(ep + r * ROWB + ((c ^ (r & SWZ)) << 4));
            const int m = mrow0 + pass * RPP + r;
            const int n = ncol0 + c * 4;
            if (m >= p.M || n >= p.N) continue;
            if constexpr (OUT == 2) {
                // split-K partial sums, dense [splits][M][N] FP32 (N % 4 == 0)
                *reinterpret_cast<float4*>(part + (int64_t)m * p.N + n) = v;
                continue;
            }
            v.x *= alpha; v.y *= alpha; v.z *= alpha; v.w *= alpha;
            if (n + 3 < p.N) {
                if constexpr (OUT == kOutBF16Epi) add_epilogue4(v, p.bias, p.residual, p.ldr, m, n, p.res_scale);
                if constexpr (OUT == kOutF32) {
                    float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float*>(p.D) + (int64_t)m * p.ldd + n);
                    if (p.accumulate) {
                        const float4 o = *dst;
                        v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
                    }
                    *dst = v;
                } else {
                    uint2* dst = reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(p.D) + (int64_t)m * p.ldd + n);
                    if (p.accumulate) {
                        const uint2 o = *dst;
                        v.x += bf16lo(o.x); v.y += bf16hi(o.x); v.z += bf16lo(o.y); v.w += bf16hi(o.y);
                    }
                    *dst = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
                }
            } else {
                // ragged right edge: element by element
                const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (n + t >= p.N) continue;
                    if constexpr (OUT == kOutF32) {
                        float* dst = reinterpret_cast<float*>(p.D) + (int64_t)m * p.ldd + n + t;
                        *dst = p.accumulate ? *dst + vv[t] : vv[t];
                    } else {
                        uint16_t* dst = reinterpret_cast<uint16_t*>(p.D) + (int64_t)m * p.ldd + n + t;
                        float o = p.accumulate ? vv[t] + __uint_as_float((uint32_t)*dst << 16) : vv[t];
                        if constexpr (OUT == kOutBF16Epi) o = add_epilogue1(o, p.bias, p.residual, p.ldr, m, n + t, p.res_scale);
                        *dst = to_bf16(o);
                    }
                }
            }
        }
    });
}

template <int BM, int BN, int WM, int WN, int SL, int NST, int XA, int PROD, int FA, int FB, bool GROUPED, int OUT>
void launch_cfg(const Params& prm, int grid, hipStream_t stream) {
    constexpr int threads = WM * WN * 64 * (PROD ? 2 : 1);
    gemm_fp8_kernel<BM, BN, WM, WN, FA, FB, OUT, GROUPED, SL, NST, spare_units(BM, BN, SL, NST, XA, GROUPED), PROD != 0><<<grid, threads, 0, stream>>>(prm);
}

template <int BM, int BN, int WM, int WN, int SL, int NST, int XA, int PROD, int FA, int FB, bool GROUPED>
void launch_tile(const Params& prm, int out, int grid, hipStream_t stream) {
    // the LM-head kinds exist for BF16 operands and blockwise E4M3 operands,
    // on 128-column wave tiles
    constexpr bool lm = (FA == kBF16 && FB == kBF16 && !GROUPED) || (FA == kE4M3 && FB == kE4M3 && GROUPED);
    if (out == 2) launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, 2>(prm, grid, stream);
    else if (out == kOutF32) launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutF32>(prm, grid, stream);
    else if (out == kOutBF16Epi)
        launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutBF16Epi>(prm, grid, stream);
    else if (out == kOutLseStats || out == kOutSoftmaxGrad) {
        if constexpr (lm && BN / WN == 128) {
            if (out == kOutLseStats) launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutLseStats>(prm, grid, stream);
            else launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutSoftmaxGrad>(prm, grid, stream);
        }
    } else if (out == kOutSoftmaxGradQ) {
        // the blockwise E4M3 recipe's backward, 128 x 128 wave tiles
        if constexpr (FA == kE4M3 && FB == kE4M3 && GROUPED && BM / WM == 128 && BN / WN == 128)
            launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutSoftmaxGradQ>(prm, grid, stream);
    } else launch_cfg<BM, BN, WM, WN, SL, NST, XA, PROD, FA, FB, GROUPED, kOutBF16>(prm, grid, stream);
}

}  // namespace

template <int FA, int FB, bool GROUPED>
void launch_variant(const Params& prm, int cfg, int out, int grid, hipStream_t stream) {
#define PURO_TILE_CASE(i, bm, bn, wm, wn, sl, nst, xa, prod, f, s, g) \
    case i: launch_tile<bm, bn, wm, wn, sl, nst, xa, prod, FA, FB, GROUPED>(prm, out, grid, stream); break;
    switch (cfg) { PURO_TILE_LIST(PURO_TILE_CASE) }
#undef PURO_TILE_CASE
}

template void launch_variant<PURO_FA, PURO_FB, (PURO_GROUPED != 0)>(const Params&, int, int, int, hipStream_t);

}  // namespace gemm_detail
}  // namespace puro
