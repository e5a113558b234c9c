// Eq. 3 (Sec. 2.2) from the 2:4 compressed Down-Proj: out = y Wdown^T on the sparse matrix cores
// (v_smfmac_f32_32x32x32_bf16), the hardware use of N:M sparsity that Sec. 2.2 points to.
//
// The sparse operand of that instruction is its first one, so Wdown's output features are the
// MFMA "M" index and tokens the "N" index: a workgroup owns 256 features x 256 tokens, its four
// wavefronts 128 x 128 each (16 accumulator blocks = all 256 accumulation registers).
// Operand layout (checked on the GPU against a host product): a lane (row, half c) takes 8
// consecutive stored values of its row = the dense K range 16 c .. 16 c + 15 of the instruction's
// 32, the 16 bits of those four groups' position codes as its index operand, and from the dense
// side K 8 c .. 8 c + 7 and 16 + 8 c .. 16 + 8 c + 7.  The compressed form of dass_compress_24
// (groups along the columns) is exactly that: no shuffling, only addresses.
//
// K slabs of 64 dense columns go from global memory straight into a ring of three LDS stages
// (buffer_load ... lds): 256 rows x 64 B of values and 256 tokens x 128 B of y = 48 KB a stage;
// the codes come eight slabs at a time (64 bytes of a row; four where the ring leaves 16 KB), a part of them with
// every second or fourth slab.  The tiles that do not fill the chip are bound by the number of row pieces they request:
// with codes of two slabs (16 bytes of a row) these were 128 of 512 requests a slab of the 256 x 128 tile, and the
// loads alone took 0.66 of the slab's 0.76 us (the rest alone: 0.47).  That tile takes the values two slabs at a time
// as well, 128 bytes of a row: 320 requests, 0.64 us.  Back to back, 2048 tokens of 4096 x 11008 132 -> 118 us by the
// codes, 114 by the values; 1024 of 8192 x 28672 384 -> 328, 310.  The 128 x 128 tile by the codes alone (by the values
// within 2 % either way): 1024 of 4096 x 11008 87 -> 75, 300 of 2048 x 5632 39 -> 34.  A grid of few such tiles, each
// compute unit with one wavefront per SIMD, is bound by the number of instructions a slab, so its loop is unrolled by the
// four slabs between two parts of the codes: what a part is and where a chunk lies then costs next to nothing (with a
// part every second slab, half of them rows past the last feature, and places computed for each slab, 128 tokens of 1024
// x 4096 took 24.0 us, now 22.8; codes of two slabs 22.7).
// The largest tile is within 1 % of before.  (A ring of four or six stages, more bytes in flight, gave nothing: 0 to 4
// us slower.)  Rows are XOR-swizzled in 16-byte chunks so that the fragment reads spread over the banks.  One barrier
// per slab; the loads of slab s + 3 are issued right after it.
#include "dass_internal.h"
#include "tile_order.h"

#include <type_traits>

namespace dass {
namespace sp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) __bf16 bf16x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kFM = 256, kTN = 256, kBK = 64;          // features, tokens of the largest tile; dense K per slab
constexpr int kStages = 3;
// The tile of a workgroup is FB x NB blocks of 32 x 32 per wavefront (4 x 4: the one described above).
template <int FB, int NB>
struct Tile {
    static constexpr int kFM = 64 * FB, kTN = 64 * NB;
    static constexpr int kABytes = kFM * (kBK / 2) * 2;           // 16 KB of values
    static constexpr int kBBytes = kTN * kBK * 2;                 // 32 KB of y
    static constexpr int kStage = kABytes + kBBytes;              // 48 KB
    // The middle tile takes the values two slabs at a time, whole 128-byte lines of a row: three units of those,
    // behind three of y.
    static constexpr bool kWide = FB * NB == 8;
    // codes of kMSlabs slabs, 8 B a row each: a block of kMParts parts, one wave-load (1 KB) a wavefront each, fetched
    // a part every kMEvery slabs.
    static constexpr int kMSlabs = FB * NB >= 8 ? 4 : 8;
    static constexpr int kMRow = 8 * kMSlabs, kMChunks = kMRow / 16;   // bytes and 16-byte chunks of a row of codes
    static constexpr int kMBlock = kFM * kMRow, kMParts = kMBlock / 4096, kMEvery = kMSlabs / kMParts;
    static constexpr int kMBase = kWide ? 3 * kBBytes + 6 * kABytes : kStages * kStage;   // two such blocks behind the ring
    static constexpr int kLds = kMBase + 2 * kMBlock;
    static_assert(kLds == (FB * NB >= 8 ? 160 : 88) * 1024, "160 KB is what a compute unit has");
    // wave-loads a wavefront issues for slab s: FB of values, 2 NB of y, and with slabs 2, 2 + kMEvery, .. a part of the
    // codes of a later block
    static constexpr int kLoads = FB + 2 * NB;
};

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}
// The same, and no LDS access.
template <int N>
__device__ __forceinline__ void wait_loads()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}
// One wave-load of 16 bytes a lane from a buffer straight into LDS.  (Not a template: with arguments that
// depend on one, the compiler's host pass rejects the builtin and drops the kernel's stub without a word.)
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, char *dst, uint32_t lane_off, int off)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, lane_off, off, 0, 0);
}
__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// Two f32 rounded to bf16 (nearest even), `lo` in the low half of the word: one v_cvt_pk_bf16_f32.
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

template <int FB, int NB>
__global__ __launch_bounds__(256) void down_sparse24_kernel(
    const uint16_t *__restrict__ Y, int64_t T, int64_t ldy, const uint16_t *__restrict__ values, int64_t ldv,
    const uint8_t *__restrict__ meta, int64_t ldm, int64_t d, int64_t d_int, uint16_t *__restrict__ out,
    int64_t ldo, const TileOrder order)
{
    using P = Tile<FB, NB>;
    constexpr int kFM = P::kFM, kTN = P::kTN, kABytes = P::kABytes, kStage = P::kStage, kMBlock = P::kMBlock,
                  kMBase = P::kMBase, kMSlabs = P::kMSlabs, kMRow = P::kMRow, kMParts = P::kMParts, kMEvery = P::kMEvery,
                  kLoads = P::kLoads;
    extern __shared__ __attribute__((aligned(1024))) char lds[];   // P::kLds bytes

    uint32_t tile_t, tile_f;   // tile_order.h
    if (!tile_of_block(order, blockIdx.x, tile_t, tile_f))
        return;
    const int64_t t0 = (int64_t)tile_t * kTN, f0 = (int64_t)tile_f * kFM;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;   // feature half, token half of the tile
    const int fr = lane & 31, fc = lane >> 5;

    // ---- global -> LDS.  Rows past the end of a matrix lie beyond the end of its buffer
    // descriptor and read as zeros.  (A raw buffer's lane is out of range if its offset is not below the buffer's
    // length less the scalar offset.  That is never negative here: the last block of codes asked for begins at 8 S + 40
    // bytes of a row at most, the values end with their row, and there are 8 features or more, 64 S bytes of codes.)
    const int64_t rows_f = d - f0 < kFM ? d - f0 : kFM, rows_t = T - t0 < kTN ? T - t0 : kTN;
    constexpr int kRawBuffer = 0x00020000;
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(values + f0 * ldv), 0, (int)((rows_f - 1) * ldv * 2 + d_int), kRawBuffer);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t *>(meta + f0 * ldm), 0, (int)((rows_f - 1) * ldm + d_int / 8), kRawBuffer);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(Y + t0 * ldy), 0, (int)((rows_t - 1) * ldy * 2 + d_int * 2), kRawBuffer);
    // values: a wave-load is 16 rows x 64 B; lane l fills slot l % 4 of row l / 4 with chunk slot ^ (row / 4 & 3).
    // Two slabs at a time: 8 rows x 128 B, as y below.
    constexpr bool kWide = P::kWide;
    uint32_t a_off[kWide ? 2 * FB : FB], m_off, m_row_bytes, b_off[2 * NB];
#pragma unroll
    for (int q = 0; q < (kWide ? 2 * FB : FB); ++q) {
        if constexpr (kWide) {
            const int r = (wave * 2 * FB + q) * 8 + (lane >> 3);
            a_off[q] = (uint32_t)((int64_t)r * ldv * 2 + (((lane & 7) ^ ((r >> 1) & 7)) * 16));
        } else {
            const int r = (wave * FB + q) * 16 + (lane >> 2);
            a_off[q] = (uint32_t)((int64_t)r * ldv * 2 + (((lane & 3) ^ ((r >> 2) & 3)) * 16));
        }
    }
    // codes: a wave-load is 1024 / kMRow rows; lane l fills slot l % kMChunks of row l / kMChunks with a chunk of
    // that row that changes every 256 bytes of rows.  Part i of a block is the rows from i x 4 wave-loads on.
    constexpr int kMRows = 1024 / kMRow;
    auto m_swizzle = [](int r) { return (r / (256 / P::kMRow)) & (P::kMChunks - 1); };
    {
        const int r = wave * kMRows + lane / P::kMChunks;
        m_off = (uint32_t)((int64_t)r * ldm + ((lane % P::kMChunks) ^ m_swizzle(r)) * 16);
        m_row_bytes = (uint32_t)(4 * kMRows * ldm);
    }
    static_assert((4 * kMRows / (256 / P::kMRow)) % P::kMChunks == 0, "every part of a block has the same swizzle");
    // y: a wave-load is 8 rows x 128 B; lane l fills slot l % 8 of row l / 8 with chunk slot ^ (row / 2 & 7)
#pragma unroll
    for (int q = 0; q < 2 * NB; ++q) {
        const int r = (wave * 2 * NB + q) * 8 + (lane >> 3);
        b_off[q] = (uint32_t)((int64_t)r * ldy * 2 + (((lane & 7) ^ ((r >> 1) & 7)) * 16));
    }
    // Part i of block b of the codes.  Rows past the last feature lie past the buffer's end.
    auto load_codes = [&](int b, int i) {
        load_to_lds(rm, lds + kMBase + (b & 1) * kMBlock + (i * 4 + wave) * 1024, m_off + (uint32_t)i * m_row_bytes, b * kMRow);
    };
    // q-th wave-load of slab s: FB of values, 2 NB of y, the last (slabs 2, 2 + kMEvery, ..) a part of the codes.  The
    // block after the one of slab s' = s - 2: its place is free when slab s' - 1, the last that reads the codes there, has
    // read them, and its last part lands with the first slab that needs it or before.
    auto load_one = [&](int s, int q) {
        char *st = lds + (s % kStages) * kStage;
        if (q < FB)
            load_to_lds(rv, st + (wave * FB + q) * 1024, a_off[q], s * kBK);
        else if (q < kLoads)
            load_to_lds(ry, st + kABytes + (wave * 2 * NB + q - FB) * 1024, b_off[q - FB], s * kBK * 2);
        else
            load_codes((s - 2) / kMSlabs + 1, (s - 2) % kMSlabs / kMEvery);
    };
    auto issue_slab = [&](int s) {   // prologue only; slab by slab, the waits count
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kLoads; ++q)
            load_one(s, q);
        if (s == 2)
            load_one(s, kLoads);
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- LDS -> registers
    int a_row[FB], b_row[NB];
#pragma unroll
    for (int i = 0; i < FB; ++i)
        a_row[i] = wm * (kFM / 2) + i * 32 + fr;
#pragma unroll
    for (int j = 0; j < NB; ++j)
        b_row[j] = wn * (kTN / 2) + j * 32 + fr;
    constexpr int kReads = FB + 2 * NB;   // fragment reads of a K step: FB sparse, 2 NB dense halves
    struct Frags {
        bf16x8 a[FB], lo[NB], hi[NB];   // the dense operand of block j is lo[j] followed by hi[j]
    };
    // q-th of the fragment reads of K step kk of the slab in stage st
    auto read_one = [&](Frags &f, const char *st, int kk, int q) {
        if (q < FB) {
            const int r = a_row[q];
            f.a[q] = *reinterpret_cast<const bf16x8 *>(st + (r * 4 + ((2 * kk + fc) ^ ((r >> 2) & 3))) * 16);
        } else {
            const int j = (q - FB) >> 1, r = b_row[j];
            const char *row = st + kABytes + r * 128;
            const int sw = (r >> 1) & 7;
            if (((q - FB) & 1) == 0)
                f.lo[j] = *reinterpret_cast<const bf16x8 *>(row + (((4 * kk + fc) ^ sw) * 16));
            else
                f.hi[j] = *reinterpret_cast<const bf16x8 *>(row + (((4 * kk + 2 + fc) ^ sw) * 16));
        }
    };
    u32x2 codes[FB], codes_next[FB];   // the 16 nibbles of a slab of each of this lane's FB rows
    int code_row[FB];   // a row of codes and its first chunk; the chunk's other places differ in bits that are 0 in the row's
#pragma unroll
    for (int i = 0; i < FB; ++i)
        code_row[i] = a_row[i] * kMRow + m_swizzle(a_row[i]) * 16;
    auto read_codes = [&](u32x2 *c, int s, int i) {   // slab s: half s % 2 of a 16-byte chunk of the row
        c[i] = *reinterpret_cast<const u32x2 *>(lds + (kMBase + ((s / kMSlabs) & 1) * kMBlock + (s & 1) * 8) +
                                              (code_row[i] ^ (s % kMSlabs / 2 * 16)));
    };

    f32x16 acc[FB][NB];
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;
    auto mfma = [&](const Frags &f, const u32x2 *c, int kk, int q) {
        const int i = q / NB, j = q % NB;
        const bf16x16 b = __builtin_shufflevector(f.lo[j], f.hi[j], 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
        acc[i][j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(f.a[i], b, acc[i][j], (int)(c[i][kk] >> (16 * fc)), 0, 0);
    };

    constexpr int kMfmas = FB * NB;
    const int S = (int)(d_int / kBK);   // the host guarantees d_int % 64 == 0

    if constexpr (kWide) {
        // ---- main loop of the middle tile.  Step s, the time from the barrier of slab s to that of the next one,
        // requests a part of the codes (odd s), the y of slab s + 3 and half of the rows of a unit of values: of
        // unit (s + 5) / 2 with s odd, whose place is free since slab s is read, the other half in the step after.
        // Only slabs and units that exist are requested, so the last slabs have bodies of their own.  (With requests
        // from an empty buffer instead, which keep the load path as busy as real ones, 2048 tokens of 4096 x 256 took
        // 8.5 us, now 8.1, 8200 of 512 x 256 7.7, now 7.3, 2048 of 4096 x 1024 15.5, now 15.2.)
        constexpr int kUnit = 2 * kABytes, kUnits = 3 * P::kBBytes;   // values of two slabs; where the units begin
        auto load_y = [&](int s, int q) {
            load_to_lds(ry, lds + s % 3 * P::kBBytes + (wave * 2 * NB + q) * 1024, b_off[q], s * kBK * 2);
        };
        auto load_values = [&](int unit, int q) {   // q-th of 2 FB
            load_to_lds(rv, lds + kUnits + unit % 3 * kUnit + (wave * 2 * FB + q) * 1024, a_off[q], unit * 128);
        };
        auto step_load = [&](int s, bool odd, int q) {   // q-th of a step's loads: the codes first
            if (odd) {
                if (q == 0) {
                    load_codes((s + 1) / kMSlabs + 1, (s + 1) % kMSlabs / kMEvery);
                    return;
                }
                --q;
            }
            if (q < 2 * NB)
                load_y(s + 3, q);
            else
                load_values(odd ? (s + 5) / 2 : (s + 4) / 2, q - 2 * NB + (odd ? 0 : FB));
        };
        auto read_wide = [&](Frags &f, int s, int kk, int q) {
            const char *ys = lds + s % 3 * P::kBBytes, *vs = lds + kUnits + s / 2 % 3 * kUnit;
            if (q < FB) {
                const int r = a_row[q];
                f.a[q] = *reinterpret_cast<const bf16x8 *>(vs + r * 128 + (((4 * (s & 1) + 2 * kk + fc) ^ ((r >> 1) & 7)) * 16));
            } else {
                const int j = (q - FB) >> 1, r = b_row[j], c = 4 * kk + fc + ((q - FB) & 1 ? 2 : 0);
                const bf16x8 v = *reinterpret_cast<const bf16x8 *>(ys + r * 128 + ((c ^ ((r >> 1) & 7)) * 16));
                if (((q - FB) & 1) == 0)
                    f.lo[j] = v;
                else
                    f.hi[j] = v;
            }
        };
        // Steps -5 to -1, as far as there is something in them; in this order, the waits count.
#pragma unroll
        for (int i = 0; i < kMParts; ++i)
            load_codes(0, i);
#pragma unroll
        for (int q = 0; q < 2 * FB; ++q)
            load_values(0, q);
        auto y_and_values = [&](int slab, int unit, int half) {
            __builtin_amdgcn_sched_barrier(0);
            if (slab < S) {
#pragma unroll
                for (int q = 0; q < 2 * NB; ++q)
                    load_y(slab, q);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (2 * unit < S) {
#pragma unroll
                for (int q = 0; q < FB; ++q)
                    load_values(unit, q + half * FB);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        y_and_values(0, 1, 0);
        y_and_values(1, 1, 1);
        if (S > kMSlabs)
            load_codes(1, 0);
        y_and_values(2, 2, 0);
        // the codes, unit 0 and the y of slab 0 have landed
        if (S > 4)
            wait_loads<FB + 2 * (2 * NB + FB) + 1>();
        else if (S > 2)
            wait_loads<2 * (2 * NB + FB)>();
        else if (S == 2)
            wait_loads<2 * NB>();
        else
            wait_loads<0>();
        static_assert(kMSlabs == 4, "the first of these waits counts a part of the codes");
        block_barrier();
        Frags fa, fb;
#pragma unroll
        for (int q = 0; q < kReads; ++q)
            read_wide(fa, 0, 0, q);
#pragma unroll
        for (int i = 0; i < FB; ++i)
            read_codes(codes, 0, i);
        // LEFT: how many slabs follow, 5 for all that request a half unit of values (an even slab does that with four
        // left too).  Below 4 the slab may be an even or an odd one.
        auto body = [&](int s, auto odd_tag, auto left_tag) {
            constexpr bool ODD = decltype(odd_tag)::value;
            constexpr int LEFT = decltype(left_tag)::value;
            constexpr int kCodes = LEFT >= 4 && ODD ? 1 : 0;
            constexpr int kLoads = LEFT >= 5 ? 2 * NB + FB + kCodes : LEFT >= 3 ? 2 * NB + kCodes : 0;
#pragma unroll
            for (int q = 0; q < kMfmas; ++q) {   // K step 0
#pragma unroll
                for (int x = q; x < kReads; x += kMfmas)
                    read_wide(fb, s, 1, x);
                mfma(fa, codes, 0, q);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (LEFT > 0) {
                // The y of slab s + 1, requested in step s - 2 behind the codes, has landed, and the values, which are
                // requested earlier; the values of step s - 2 and what step s - 1 requested may be in flight: both
                // halves of a unit and the y of slab s + 2, or as much of that as is there whatever slab this is.
                wait_loads<LEFT >= 4 ? FB + 2 * NB + FB : LEFT == 3 ? FB + 2 * NB : LEFT == 2 ? 2 * NB : 0>();
                block_barrier();
            }
            if constexpr (LEFT == 3) {
                if (s & 1)
                    step_load(s, true, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < kMfmas; ++q) {   // K step 1
#pragma unroll
                for (int x = q * kLoads / kMfmas; x < (q + 1) * kLoads / kMfmas; ++x) {   // in this order
                    step_load(s, kCodes != 0, x);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (LEFT > 0) {
#pragma unroll
                    for (int x = q; x < kReads + FB; x += kMfmas) {
                        if (x < kReads)
                            read_wide(fa, s + 1, 0, x);
                        else
                            read_codes(codes_next, s + 1, x - kReads);
                    }
                }
                mfma(fb, codes, 1, q);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (LEFT > 0) {
#pragma unroll
                for (int i = 0; i < FB; ++i)
                    codes[i] = codes_next[i];
            }
        };
        using Even = std::false_type;
        using Odd = std::true_type;
        using Steady = std::integral_constant<int, 5>;
        int s = 0;
        for (; s + 6 < S; s += 2) {
            body(s, Even{}, Steady{});
            body(s + 1, Odd{}, Steady{});
        }
        if (s + 4 < S)
            body(s++, Even{}, Steady{});
        if (s + 4 < S)
            body(s++, Odd{}, std::integral_constant<int, 4>{});
        if (s + 3 < S)
            body(s++, Even{}, std::integral_constant<int, 3>{});
        if (s + 2 < S)
            body(s++, Even{}, std::integral_constant<int, 2>{});
        if (s + 1 < S)
            body(s++, Even{}, std::integral_constant<int, 1>{});
        body(s, Even{}, std::integral_constant<int, 0>{});
    } else {
    // ---- main loop.  A slab is two K steps of FB NB sparse MFMAs (16).  Under the MFMAs of K step 0 go
    // the fragment reads of K step 1; then one barrier - slab s + 1 has landed, nobody reads slab
    // s from LDS any more, so its stage takes slab s + 3 - and under the MFMAs of K step 1 go those
    // loads and the fragment reads of K step 0 of slab s + 1.
#pragma unroll
    for (int i = 0; i < kMParts; ++i)
        load_codes(0, i);
    issue_slab(0);
    if (S > 1)
        issue_slab(1);
    if (S > 2)
        issue_slab(2);
    if (S > 2)
        wait_vmcnt<2 * kLoads + 1>();   // slabs 1 and 2 may be in flight
    else if (S > 1)
        wait_vmcnt<kLoads>();
    else
        wait_vmcnt<0>();
    block_barrier();
    Frags fa, fb;
#pragma unroll
    for (int q = 0; q < kReads; ++q)
        read_one(fa, lds, 0, q);
#pragma unroll
    for (int i = 0; i < FB; ++i)
        read_codes(codes, 0, i);
    // read_codes of slab s + 1; a chunk holds an even slab and the next, whose place is then known.
    int code_at[FB];
    auto next_codes = [&](int s, int i, auto phase_tag) {
        constexpr int PHASE = decltype(phase_tag)::value;
        if (PHASE % 2 == 1 || PHASE == kMEvery)
            code_at[i] = ((s + 1) / kMSlabs & 1) * kMBlock + (code_row[i] ^ ((s + 1) % kMSlabs / 2 * 16));
        codes_next[i] = *reinterpret_cast<const u32x2 *>(
            lds + (kMBase + (PHASE == kMEvery ? ((s + 1) & 1) : 1 - PHASE % 2) * 8) + code_at[i]);
    };
#pragma unroll
    for (int i = 0; i < FB; ++i)
        code_at[i] = code_row[i];
    // MORE: a slab follows; LOAD: slab s + 3 exists; AHEAD: slab s + 2 exists (it may be in flight
    // at the barrier).  All three are compile-time: the steady state has no branch between MFMAs.
    // PHASE: s modulo kMEvery, which says whether slabs s + 2 and s + 3 bring a part of the codes, or kMEvery when
    // it is only known at run time (the last slabs): then the barrier waits as if slab s + 2 brought none (one
    // load more has to land, harmless).
    auto slab_body = [&](int s, auto more_tag, auto load_tag, auto ahead_tag, auto phase_tag) {
        constexpr bool MORE = decltype(more_tag)::value, LOAD = decltype(load_tag)::value,
                       AHEAD = decltype(ahead_tag)::value;
        constexpr int PHASE = decltype(phase_tag)::value;
        constexpr int kAhead = kLoads + (PHASE == 0 ? 1 : 0);                        // loads of slab s + 2
        constexpr int kIssue = kLoads + (PHASE == kMEvery - 1 ? 1 : 0);              // loads of slab s + 3
        static_assert(kAhead < 16, "the low four bits of the wait's counter hold it");
        const char *st = lds + (s % kStages) * kStage, *st_next = lds + ((s + 1) % kStages) * kStage;
#pragma unroll
        for (int q = 0; q < kMfmas; ++q) {   // K step 0
#pragma unroll
            for (int x = q; x < kReads; x += kMfmas)
                read_one(fb, st, 1, x);
            mfma(fa, codes, 0, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        // slab s + 1 has landed (only slab s + 2, kAhead loads, may be in flight) and this wavefront holds
        // its last fragments of slab s: vmcnt(kAhead or 0), lgkmcnt(0)
        if (AHEAD)
            __builtin_amdgcn_s_waitcnt(0x0070 | kAhead);
        else
            __builtin_amdgcn_s_waitcnt(0x0070);
        block_barrier();
#pragma unroll
        for (int q = 0; q < kMfmas; ++q) {   // K step 1
            if (LOAD) {
#pragma unroll
                for (int x = q; x < kIssue; x += kMfmas)
                    load_one(s + 3, x);
            }
            if (MORE) {
#pragma unroll
                for (int x = q; x < kReads + FB; x += kMfmas) {
                    if (x < kReads)
                        read_one(fa, st_next, 0, x);
                    else
                        next_codes(s, x - kReads, phase_tag);
                }
            }
            mfma(fb, codes, 1, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (MORE) {
#pragma unroll
            for (int i = 0; i < FB; ++i)
                codes[i] = codes_next[i];
        }
    };
    using Yes = std::true_type;
    using No = std::false_type;
    using Any = std::integral_constant<int, kMEvery>;
    auto at_phase = [&](int s, auto phase_tag) { slab_body(s, Yes{}, Yes{}, Yes{}, phase_tag); };
    static_assert(kMEvery == 2 || kMEvery == 4 || kWide, "the loop below");
    int s = 0;
    for (; s + kMEvery + 2 < S; s += kMEvery) {   // s is a multiple of kMEvery here
        at_phase(s, std::integral_constant<int, 0>{});
        at_phase(s + 1, std::integral_constant<int, 1>{});
        if constexpr (kMEvery == 4) {
            at_phase(s + 2, std::integral_constant<int, 2>{});
            at_phase(s + 3, std::integral_constant<int, 3>{});
        }
    }
    if (s + 3 < S)   // the slabs before S - 3 that the loop left
        at_phase(s++, std::integral_constant<int, 0>{});
    if constexpr (kMEvery == 4) {
        if (s + 3 < S)
            at_phase(s++, std::integral_constant<int, 1>{});
        if (s + 3 < S)
            at_phase(s++, std::integral_constant<int, 2>{});
    }
    if (s + 2 < S)
        slab_body(s++, Yes{}, No{}, Yes{}, Any{});    // slab S - 3
    if (s + 1 < S)
        slab_body(s++, Yes{}, No{}, No{}, Any{});     // slab S - 2
    slab_body(s, No{}, No{}, No{}, Any{});            // slab S - 1

    }

    // ---- epilogue: the tile goes to LDS as bf16 [token][feature] (row stride 528 B) and leaves it
    // in whole 16-byte chunks of output rows.  A lane holds, per block, 4 x 4 consecutive features
    // of one token: 8-byte writes.
    block_barrier();   // every wavefront is done with the last slab
    constexpr int SROW = kFM * 2 + 16;
    static_assert(kTN * SROW <= P::kLds, "the tile fits in the ring");
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int token = wn * (kTN / 2) + j * 32 + fr, feature = wm * (kFM / 2) + i * 32 + 8 * g + 4 * fc;
                u32x2 w;
                w[0] = bf16_pair(acc[i][j][4 * g], acc[i][j][4 * g + 1]);
                w[1] = bf16_pair(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
                *reinterpret_cast<u32x2 *>(lds + token * SROW + feature * 2) = w;
            }
    __syncthreads();
    constexpr int CPR = kFM / 8;   // 16-byte chunks per tile row
    for (int c = tid; c < kTN * CPR; c += 256) {
        const int row = c / CPR, cc = c % CPR;
        const int64_t t = t0 + row, f = f0 + cc * 8;
        if (t < T && f < d)   // d is a multiple of 8: a chunk is inside or outside
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(lds + row * SROW + cc * 16),
                                        reinterpret_cast<u32x4 *>(out + t * ldo + f));   // streamed: not read again from L2
    }
}

template <int FB, int NB>
static hipError_t launch_tile(hipStream_t stream, const uint16_t *Y, int64_t T, int64_t ldy, const uint16_t *values,
                              int64_t ldv, const uint8_t *meta, int64_t ldm, int64_t d, int64_t d_int, uint16_t *out,
                              int64_t ldo, const TileOrder &order)
{
    constexpr int kLds = Tile<FB, NB>::kLds;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(down_sparse24_kernel<FB, NB>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((down_sparse24_kernel<FB, NB>), dim3(order.blocks), dim3(256), kLds, stream, Y, T, ldy, values, ldv,
                       meta, ldm, d, d_int, out, ldo, order);
    return hipSuccess;
}

}  // namespace sp
}  // namespace dass

extern "C" dass_status dass_down_proj_sparse24(const void *Y, int64_t T, int64_t ldy, const void *values, int64_t ldv,
                                               const uint8_t *meta, int64_t ldm, int64_t d, int64_t d_int,
                                               dass_dtype dt, void *out, int64_t ldo, void *hip_stream)
{
    using namespace dass;
    const char *fn = "dass_down_proj_sparse24";
    if (!Y || !values || !meta || !out)
        return fail(DASS_ERR_NULL, "%s: Y, values, meta and out must not be NULL", fn);
    if (!valid_dtype(dt))
        return fail(DASS_ERR_DTYPE, "%s: unknown dtype %d", fn, (int)dt);
    if (dt != DASS_BF16)
        return fail(DASS_ERR_DTYPE, "%s: only bf16 is implemented", fn);
    if (T <= 0 || d <= 0 || d_int <= 0)
        return fail(DASS_ERR_SHAPE, "%s: T=%lld d=%lld d_int=%lld must be positive", fn, (long long)T, (long long)d,
                    (long long)d_int);
    if (d_int % 64 != 0 || d % 8 != 0)
        return fail(DASS_ERR_SHAPE, "%s: d_int=%lld must be a multiple of 64 and d=%lld of 8", fn, (long long)d_int,
                    (long long)d);
    if (ldy < d_int || ldv < d_int / 2 || ldm < d_int / 8 || ldo < d)
        return fail(DASS_ERR_SHAPE, "%s: a leading dimension is shorter than its row", fn);
    if (!aligned16(Y) || !aligned16(values) || !aligned16(out) || (reinterpret_cast<uintptr_t>(meta) & 3u))
        return fail(DASS_ERR_ALIGN, "%s: Y, values and out must be 16-byte aligned, meta 4-byte", fn);
    if (ldy % 8 != 0 || ldv % 8 != 0 || ldo % 8 != 0 || ldm % 4 != 0)
        return fail(DASS_ERR_ALIGN, "%s: ldy, ldv, ldo must be multiples of 8 elements, ldm of 4 bytes", fn);
    // 32-bit byte offsets inside a tile's rows
    if ((int64_t)sp::kTN * ldy * 2 >= 0x7fffffffLL || (int64_t)sp::kFM * ldv * 2 >= 0x7fffffffLL ||
        (int64_t)sp::kFM * ldm >= 0x7fffffffLL)
        return fail(DASS_ERR_SHAPE, "%s: rows too long for the tile addressing", fn);
    const TileShape shape = sparse_tile_shape(T, d);
    // Patches from 1024 tiles on, us, taken in turn with runs: 64 and 128 x 16 tiles (4096 x 14336) 1052 1095, 2118
    // 2173; 64 and 96 x 20 (5120 x 13824) 1274 1304, 1972 2033; 4096 x 11008 and 8192 x 8192 within 0.7 %.
    const TileOrder order = make_tile_order(shape.tiles_t, shape.tiles_n, true, shape.which == 1 ? 8 : kPatchT, 1023);
    if (order.blocks == 0)
        return fail(DASS_ERR_SHAPE, "%s: too many tiles for one launch; split the tokens", fn);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const auto launch = shape.which == 0   ? sp::launch_tile<4, 4>
                        : shape.which == 1 ? sp::launch_tile<4, 2>
                                           : sp::launch_tile<2, 2>;
    const hipError_t e = launch(stream, static_cast<const uint16_t *>(Y), T, ldy, static_cast<const uint16_t *>(values), ldv,
                                meta, ldm, d, d_int, static_cast<uint16_t *>(out), ldo, order);
    if (e != hipSuccess)
        return fail(DASS_ERR_HIP, "%s: cannot reserve the ring's LDS: %s", fn, hipGetErrorString(e));
    return check_launch("sparse down-projection kernel");
}
