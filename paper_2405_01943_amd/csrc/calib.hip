// Stage 1: calibration statistics.  For every intermediate neuron i
//     sumsq[i] (+)= sum_t ( act(x_t . Wgate_i) * (x_t . Wup_i) )^2
// i.e. the GLU product of Sec. 2.2 Eq. 2 reduced to the squared L2 norm that
// Sec. 3 uses as the group-importance indicator, over all calibration tokens.
// The two projections are dense contractions; y lives only in accumulators.
//
// bf16: MFMA kernels.  A workgroup owns a 256-token x 128-neuron tile and keeps
// a gate and an up accumulator for it (all 256 accumulator registers of its four
// wavefronts); X, Wgate and Wup slabs of BK columns are staged through LDS in
// 16-byte chunks, XOR-swizzled so that the 16-byte fragment reads of a wavefront
// spread over all banks.  Tokens are the MFMA "M" index and neurons the "N"
// index, so the 16 accumulator registers a lane holds for one 32x32 block belong
// to ONE neuron and 16 tokens: the sum over tokens starts as plain register
// adds, then one cross-lane add, then one f32 atomic per neuron and wavefront.
//   calib_pipe64_kernel  d a multiple of 64 (every model shape): slabs of 64
//                      columns go from global memory straight into a ring of
//                      five 32 KB LDS units (no register staging), whole
//                      128-byte lines per request; loads, fragment reads and
//                      MFMAs of consecutive slabs are interleaved by hand.  The
//                      same main loop also serves Eq. 2 + Eq. 3 themselves
//                      (dass_mlp_forward) through two storing epilogues.
//   calib_mfma_kernel  any other d (a multiple of 8): register-staged,
//                      double-buffered; the K tail is masked.
//
// f32: calib_f32_kernel, the f32 matrix instruction on fragments straight from global memory.
#include "dass_internal.h"
#include "tile_order.h"

#include <type_traits>

namespace dass {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;  // one 16-byte chunk = 8 bf16

// ------------------------------------------------------------- activations --
template <int ACT>
__device__ __forceinline__ float glu_act_fast(float g)
{
    // exp2 and the reciprocal are the hardware's 1-ulp instructions; a true division costs a
    // dozen instructions per element and the bf16 path is good to 1e-6 without it.
    if constexpr (ACT == DASS_ACT_SILU) {
        return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
    } else if constexpr (ACT == DASS_ACT_GELU_TANH) {
        // 0.5 g (1 + tanh z) = g / (1 + exp(-2 z)),  z = sqrt(2/pi) (g + 0.044715 g^3)
        // exp(-2 z) = exp2(g (c0 + c1 g^2)),  c0 = -2 sqrt(2/pi) log2(e),  c1 = 0.044715 c0
        const float e = g * fmaf(-0.10294324f, g * g, -2.3022082f);
        return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(e));
    } else if constexpr (ACT == DASS_ACT_GELU_ERF) {
        // erf by the classical five-term rational form in t = 1 / (1 + p z) times exp(-z^2)
        // (Abramowitz & Stegun 7.1.26, absolute error of erf below 1.5e-7), written on z = |g| / sqrt(2)
        // so that neither branch cancels: with h = (1 - erf z) / 2 = P(t) exp(-g^2 / 2) / 2,
        // GELU(g) = g (1 - h) for g >= 0 and g h for g < 0.  The library's erff is several times the
        // instructions; the norms are good to 1e-6 either way.
        const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(g), 0.3275911f * 0.70710678f, 1.0f));
        float P = fmaf(t, 1.061405429f, -1.453152027f);
        P = fmaf(t, P, 1.421413741f);
        P = fmaf(t, P, -0.284496736f);
        P = fmaf(t, P, 0.254829592f);
        const float h = 0.5f * t * P * __builtin_amdgcn_exp2f(g * g * -0.72134752f);   // exp(-g^2 / 2)
        return g * (g >= 0.0f ? 1.0f - h : h);
    } else {
        return fmaxf(g, 0.0f);
    }
}

__device__ __forceinline__ float glu_act_precise(float g, int act)
{
    switch (act) {
    case DASS_ACT_SILU:
        return g / (1.0f + expf(-g));
    case DASS_ACT_GELU_TANH: {
        const float z2 = 1.5957691216057308f * g * (1.0f + 0.044715f * g * g);
        return g / (1.0f + expf(-z2));
    }
    case DASS_ACT_GELU_ERF:
        return 0.5f * g * (1.0f + erff(g * 0.7071067811865476f));
    default:
        return fmaxf(g, 0.0f);
    }
}

// ------------------------------------------------------- small helper kernels --
__global__ void fill_zero_kernel(float *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = 0.0f;
}

__global__ void sqrt_kernel(const float *__restrict__ sumsq, float *__restrict__ norms, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        norms[i] = (float)sqrt((double)sumsq[i]);
}

// ------------------------------------------------------------------ bf16 MFMA --
// Slot (in 16-byte units) of K-chunk c of tile row r inside the row's CHUNKS
// slots.  A 16-byte fragment read is served for 16 lanes = 16 consecutive rows
// at a time; 16 / CHUNKS rows share one 256-byte line of the 64 banks, so the
// XOR term changes every 16 / CHUNKS rows and the 16 reads land on 16 distinct
// (line half, slot) places.
template <int CHUNKS>
__device__ __forceinline__ int swizzle(int r, int c)
{
    return c ^ ((r / (16 / CHUNKS)) & (CHUNKS - 1));
}

template <int BM, int BN, int BK, int WM, int WN, int MINB, int ACT>
__global__ __launch_bounds__(64 * WM * WN, MINB) void calib_mfma_kernel(
    const uint16_t *__restrict__ X, int64_t T, int64_t ldx, const uint16_t *__restrict__ Wg,
    const uint16_t *__restrict__ Wu, int64_t ldw, int64_t d, int64_t d_int,
    float *__restrict__ sumsq, int64_t tiles_t, int64_t tiles_n)
{
    constexpr int NT = 64 * WM * WN;       // threads
    constexpr int CH = BK / 8;             // 16-byte chunks per tile row
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int MI = TM / 32, NI = TN / 32;
    constexpr int A_CHUNKS = BM * CH / NT;  // chunks per thread per slab
    constexpr int B_CHUNKS = BN * CH / NT;  // per matrix
    constexpr int ROWS_PER_PASS = NT / CH;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    constexpr int STAGE = A_BYTES + 2 * B_BYTES;
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0 && BK % 16 == 0, "tile shape");
    static_assert((BM * CH) % NT == 0 && (BN * CH) % NT == 0, "staging split");
    static_assert(CH == 4 || CH == 8, "swizzle assumes 4 or 8 chunks per row");

    __shared__ __attribute__((aligned(16))) char lds[2 * STAGE];

    // ---- tile assignment: consecutive workgroup ids go to different XCDs (8 of
    // them, each with its own L2); give each XCD a contiguous run of a tile order
    // in which any 32 consecutive tiles form a 4-token-tile x 8-neuron-tile patch.
    const int64_t n_tiles = tiles_t * tiles_n;
    const int64_t per_xcd = (n_tiles + 7) / 8;
    const int64_t lin = (int64_t)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (lin >= n_tiles)
        return;
    constexpr int BAND = 8;
    const int64_t full_bands = tiles_n / BAND;
    int64_t tile_t, tile_n;
    if (lin < full_bands * BAND * tiles_t) {
        const int64_t band = lin / (BAND * tiles_t), rem = lin % (BAND * tiles_t);
        tile_t = rem / BAND;
        tile_n = band * BAND + rem % BAND;
    } else {
        const int64_t rem = lin - full_bands * BAND * tiles_t;
        const int64_t bw = tiles_n - full_bands * BAND;
        tile_t = rem / bw;
        tile_n = full_bands * BAND + rem % bw;
    }
    const int64_t t0 = tile_t * BM, n0 = tile_n * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;

    // ---- global -> register staging: thread owns chunk column (tid % CH) of rows
    // tid / CH + p * ROWS_PER_PASS.  Out-of-range rows are clamped to the last
    // valid row: their products are discarded in the epilogue.
    const int ld_c = tid % CH, ld_r = tid / CH;
    const uint16_t *a_ptr[A_CHUNKS];
    const uint16_t *g_ptr[B_CHUNKS];
    const uint16_t *u_ptr[B_CHUNKS];
#pragma unroll
    for (int p = 0; p < A_CHUNKS; ++p) {
        int64_t r = t0 + ld_r + p * ROWS_PER_PASS;
        r = r < T ? r : T - 1;
        a_ptr[p] = X + r * ldx + ld_c * 8;
    }
#pragma unroll
    for (int p = 0; p < B_CHUNKS; ++p) {
        int64_t r = n0 + ld_r + p * ROWS_PER_PASS;
        r = r < d_int ? r : d_int - 1;
        g_ptr[p] = Wg + r * ldw + ld_c * 8;
        u_ptr[p] = Wu + r * ldw + ld_c * 8;
    }
    u32x4 a_st[A_CHUNKS], g_st[B_CHUNKS], u_st[B_CHUNKS];

    auto load_slab = [&](int64_t k0) {
#pragma unroll
        for (int p = 0; p < A_CHUNKS; ++p)
            a_st[p] = *reinterpret_cast<const u32x4 *>(a_ptr[p] + k0);
#pragma unroll
        for (int p = 0; p < B_CHUNKS; ++p) {
            g_st[p] = *reinterpret_cast<const u32x4 *>(g_ptr[p] + k0);
            u_st[p] = *reinterpret_cast<const u32x4 *>(u_ptr[p] + k0);
        }
    };
    // Last slab when d is not a multiple of BK: chunks past d are read from the
    // row's first chunk instead (always in range) and cleared.
    auto load_slab_tail = [&](int64_t k0) {
        const bool k_ok = k0 + ld_c * 8 < d;
        const int64_t off = k_ok ? k0 : -(int64_t)(ld_c * 8);
        const uint32_t keep = k_ok ? 0xffffffffu : 0u;
#pragma unroll
        for (int p = 0; p < A_CHUNKS; ++p)
            a_st[p] = *reinterpret_cast<const u32x4 *>(a_ptr[p] + off) & keep;
#pragma unroll
        for (int p = 0; p < B_CHUNKS; ++p) {
            g_st[p] = *reinterpret_cast<const u32x4 *>(g_ptr[p] + off) & keep;
            u_st[p] = *reinterpret_cast<const u32x4 *>(u_ptr[p] + off) & keep;
        }
    };
    auto store_slab = [&](int buf) {
        char *base = lds + buf * STAGE;
#pragma unroll
        for (int p = 0; p < A_CHUNKS; ++p) {
            const int r = ld_r + p * ROWS_PER_PASS;
            *reinterpret_cast<u32x4 *>(base + (r * CH + swizzle<CH>(r, ld_c)) * 16) = a_st[p];
        }
#pragma unroll
        for (int p = 0; p < B_CHUNKS; ++p) {
            const int r = ld_r + p * ROWS_PER_PASS;
            const int off = (r * CH + swizzle<CH>(r, ld_c)) * 16;
            *reinterpret_cast<u32x4 *>(base + A_BYTES + off) = g_st[p];
            *reinterpret_cast<u32x4 *>(base + A_BYTES + B_BYTES + off) = u_st[p];
        }
    };

    f32x16 acc_g[MI][NI], acc_u[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc_g[i][j][r] = 0.0f;
                acc_u[i][j][r] = 0.0f;
            }

    // fragment read positions: lane holds tile row (lane % 32) and the
    // (lane / 32)-th 8-element K chunk of each 16-wide K step
    const int fr = lane & 31, fc = lane >> 5;

    const int64_t n_slabs = (d + BK - 1) / BK;
    const bool ragged_k = d % BK != 0;
    auto fetch = [&](int64_t slab) {
        if (ragged_k && slab == n_slabs - 1)
            load_slab_tail(slab * BK);
        else
            load_slab(slab * BK);
    };
    fetch(0);
    store_slab(0);
    __syncthreads();

    for (int64_t ks = 0; ks < n_slabs; ++ks) {
        const int cur = (int)(ks & 1);
        const bool more = ks + 1 < n_slabs;
        if (more)
            fetch(ks + 1);

        const char *base = lds + cur * STAGE;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 af[MI], gf[NI], uf[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int r = wm * TM + i * 32 + fr;
                af[i] = *reinterpret_cast<const bf16x8 *>(
                    base + (r * CH + swizzle<CH>(r, kk * 2 + fc)) * 16);
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int r = wn * TN + j * 32 + fr;
                const int off = (r * CH + swizzle<CH>(r, kk * 2 + fc)) * 16;
                gf[j] = *reinterpret_cast<const bf16x8 *>(base + A_BYTES + off);
                uf[j] = *reinterpret_cast<const bf16x8 *>(base + A_BYTES + B_BYTES + off);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    acc_g[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], gf[j],
                                                                          acc_g[i][j], 0, 0, 0);
                    acc_u[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], uf[j],
                                                                          acc_u[i][j], 0, 0, 0);
                }
        }
        if (more)
            store_slab(cur ^ 1);
        __syncthreads();
    }

    // ---- epilogue: y = act(g) * u, squared and summed over the tile's tokens.
    // Accumulator register r of lane l in a 32x32 block is token row
    // 8 * (r / 4) + 4 * (l / 32) + r % 4 and neuron column l % 32.
    const bool full_t = t0 + BM <= T;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        float part = 0.0f;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float y = glu_act_fast<ACT>(acc_g[i][j][r]) * acc_u[i][j][r];
                const int64_t t = t0 + wm * TM + i * 32 + 8 * (r / 4) + 4 * fc + (r % 4);
                part += (full_t || t < T) ? y * y : 0.0f;
            }
        }
        part += __shfl_xor(part, 32, 64);
        const int64_t n = n0 + wn * TN + j * 32 + fr;
        if (fc == 0 && n < d_int)
            atomicAdd(sumsq + n, part);
    }
}

// ------------------------------------------------------- bf16 MFMA, pipelined --
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// s_waitcnt that only constrains the vector-memory counter (6 bits, split field).
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}

// One wave-load of 16 bytes a lane from a buffer straight into LDS.  (Not a template: with arguments that
// depend on one, the compiler's host pass rejects the builtin and drops the kernel's stub without a word.)
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, char *dst, uint32_t lane_off, int off)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)dst, 16, lane_off, off, 0, 0);
}

// Workgroup barrier that the compiler may not move LDS traffic across (the
// direct-to-LDS loads are invisible to its alias analysis).
__device__ __forceinline__ void block_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Largest workgroup tile of calib_pipe64_kernel, shared with the host-side checks.
constexpr int P_BM = 256, P_BN = 128;

// ------------------------------------------------- bf16 MFMA, 128-byte rows --
// The workgroup tile and wavefront tiles of calib_mfma_kernel (256 tokens x 128 neurons x {gate,
// up}; a wavefront 128 x 64 x 2), fed by direct global -> LDS loads instead of register staging.
// K slabs are 64 columns: a wave-load covers 8 tile rows x 128 bytes, so every request to L2 is a
// whole 128-byte line (half as many requests as with 64-byte row pieces, measured +9 % at the
// same board power), and there is one barrier per 64 columns.
//
// 64 KB per slab leaves room for 2.5 slabs in the 160 KB of LDS, so the A part (X: 256 rows x
// 128 B) and the B part (Wgate and Wup: 2 x 128 rows x 128 B) of a slab are ring units of their
// own, five units of 32 KB: slab s keeps its A part in unit 2 s mod 5 and its B part in unit
// (2 s + 1) mod 5.  Both are free once every wavefront holds its last fragments of slab s, i.e.
// after the barrier that follows K step 2 of 4; what goes into them is the B part of slab s + 2
// (due one slab later) and the A part of slab s + 3 (due two slabs later), one wave-load every
// second MFMA pair, the B part first.
//
// What happens to the finished tile is a template parameter:
//   kEpiNorms  the calibration statistic: y = act(g) u squared and summed over the tokens
//   kEpiGlu    Eq. 2 itself: y rounded to bf16 and stored, [T, d_int] row-major
//   kEpiGemm   no activation: a plain product X W^T stored as bf16 (Eq. 3 with X = y, W = Wdown).
//              The "gate" rows of a tile are W rows n0 .. n0 + 127, its "up" rows the next 128,
//              so a tile is 256 x 256 outputs and Wu is not used.
// The two storing forms go through LDS (free after the last barrier of the main loop): lanes
// pair neighbouring columns into 32-bit words, the workgroup then writes whole 16-byte chunks
// of output rows.
//
// The tile is MI x NI blocks of 16 x 16 per wavefront and {gate, up}: 8 x 4 is the one described above;
// 4 x 4 (128 tokens) and 4 x 2 (128 tokens x 64 neurons) are for grids that leave compute units idle,
// where a slab's time is that of its loads on one compute unit (tile_order.h chooses).  A slab's MFMAs
// (0.2 to 0.4 us) are then shorter than its loads are on their way (0.8 us out of the memory-side cache, 2.5 us
// out of HBM), so these tiles keep a ring of whole parts for each operand and request a part as soon as
// its place is free, two to four slabs ahead, instead of the half to one slab of the schedule above.  Whole
// dass_mlp_forward calls, that schedule with its units partly filled against this one: 2048 tokens of 4096 x 11008
// 451-465 -> 428-436 us, 512 of it 203-207 -> 178-181, 1500 of 3072 x 24576 695-718 -> 636-640, 128 of 2048 x 8192
// 85-87 -> 76, 128 of 1024 x 4096 46-47 -> 40; dass_calib_norms of 512 tokens of 11008 x 2048 90 -> 68.
constexpr int P64_LDS = 5 * 32768;
enum { kEpiNorms = 0, kEpiGlu = 1, kEpiGemm = 2 };

// Two f32 rounded to bf16 (nearest even), `lo` in the low half of the word: one v_cvt_pk_bf16_f32.
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

template <int ACT, int EPI, int MI, int NI>
__global__ __launch_bounds__(256) void calib_pipe64_kernel(
    const uint16_t *__restrict__ X, int64_t T, int64_t ldx, const uint16_t *__restrict__ Wg,
    const uint16_t *__restrict__ Wu, int64_t ldw, int64_t d, int64_t d_int,
    float *__restrict__ sumsq, uint16_t *__restrict__ out, int64_t ldo, const TileOrder order)
{
    constexpr int BM = 32 * MI, BN = 32 * NI, BK = 64, WN = 2;
    static_assert(BM <= P_BM && BN <= P_BN && MI % 2 == 0, "the tile fits the ring's units");
    constexpr int BN_TILE = EPI == kEpiGemm ? 2 * BN : BN;   // rows of W (output columns) per tile
    constexpr int TM = 16 * MI, TN = 16 * NI;   // wavefront tile
    constexpr int CH = BK / 8;               // 16-byte chunks per tile row
    constexpr int B_HALF = BN * BK * 2;      // 16 KB at most
    constexpr bool DEEP = MI < 8;
    constexpr int NA = !DEEP ? 5 : NI == 4 ? 4 : 5, NB = !DEEP ? 5 : NI == 4 ? 3 : 5;   // ring units
    constexpr int A_UNIT = DEEP ? BM * BK * 2 : 32768, B_UNIT = DEEP ? 2 * B_HALF : 32768;
    constexpr int B_BASE = DEEP ? NA * A_UNIT : 0;   // 8 x 4: one ring for both parts
    static_assert(!DEEP || NA * A_UNIT + NB * B_UNIT <= P64_LDS, "the rings fit");
    constexpr int A_WL = MI, B_WL = NI;      // wave-loads (8 rows x 128 B) per wavefront per slab: MI + NI + NI

    extern __shared__ __attribute__((aligned(1024))) char lds64[];   // P64_LDS bytes

    uint32_t tile_t, tile_n;   // tile_order.h
    if (!tile_of_block(order, blockIdx.x, tile_t, tile_n))
        return;
    const int64_t t0 = (int64_t)tile_t * BM, n0 = (int64_t)tile_n * BN_TILE;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // ---- global -> LDS.  Lane l of a wave-load fills slot (l % 8) of row (l / 8) of an 8-row
    // block, i.e. it fetches K chunk (l % 8) ^ swizzle of that row.  Rows past the end of the
    // matrix are clamped.  Each operand is addressed as a raw buffer that starts at the tile's
    // first row and ends with its last valid element: the per-lane byte offset is a 32-bit
    // register, the K offset a scalar, and a read outside the buffer returns 0 instead of faulting.
    const int wl_row = lane >> 3, wl_slot = lane & 7;
    const int64_t rows_x = T - t0 < BM ? T - t0 : BM, rows_w = d_int - n0 < BN ? d_int - n0 : BN;
    // kEpiGemm: the second half of the tile's rows may be fewer, or none (then an empty buffer:
    // its reads fetch nothing and return 0; clamped rows beyond its end do the same)
    const int64_t left_u = d_int - n0 - BN;
    const int64_t rows_u = EPI != kEpiGemm ? rows_w : left_u < 0 ? 0 : left_u < BN ? left_u : BN;
    uint32_t a_off[A_WL], b_off[B_WL];
#pragma unroll
    for (int p = 0; p < A_WL; ++p) {
        // rows past T are not clamped: they lie beyond the end of the buffer and read as 0, which
        // the epilogues rely on (act(0) * 0 adds nothing to a norm; stores are bounded by T)
        const int r = (wave * A_WL + p) * 8 + wl_row;
        a_off[p] = (uint32_t)((int64_t)r * ldx * 2 + (wl_slot ^ swizzle<CH>(r, 0)) * 16);
    }
#pragma unroll
    for (int p = 0; p < B_WL; ++p) {
        const int r = (wave * B_WL + p) * 8 + wl_row;
        const int64_t rr = r < rows_w ? r : rows_w - 1;
        b_off[p] = (uint32_t)(rr * ldw * 2 + (wl_slot ^ swizzle<CH>(r, 0)) * 16);
    }
    constexpr int kRawBuffer = 0x00020000;
    const int span_x = (int)((rows_x - 1) * ldx * 2 + d * 2), span_w = (int)((rows_w - 1) * ldw * 2 + d * 2);
    const int span_u = rows_u > 0 ? (int)((rows_u - 1) * ldw * 2 + d * 2) : 0;
    const uint16_t *up_rows = EPI == kEpiGemm ? Wg + (n0 + BN) * ldw : Wu + n0 * ldw;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(X + t0 * ldx), 0, span_x, kRawBuffer);
    const __amdgpu_buffer_rsrc_t rg =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(Wg + n0 * ldw), 0, span_w, kRawBuffer);
    const __amdgpu_buffer_rsrc_t ru =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(up_rows), 0, span_u, kRawBuffer);

    // q-th of this wavefront's A_WL loads of an A part (slab at byte offset kb) into ring unit `unit`
    auto issue_a = [&](int unit, int kb, int q) {
        load_to_lds(rx, lds64 + unit * A_UNIT + (wave * A_WL + q) * 1024, a_off[q], kb);
    };
    // q-th of its 2 B_WL loads of a B part: B_WL of Wgate, then B_WL of Wup
    auto issue_b = [&](int unit, int kb, int q) {
        if (q < B_WL)
            load_to_lds(rg, lds64 + B_BASE + unit * B_UNIT + (wave * B_WL + q) * 1024, b_off[q], kb);
        else
            load_to_lds(ru, lds64 + B_BASE + unit * B_UNIT + B_HALF + (wave * B_WL + q - B_WL) * 1024, b_off[q - B_WL], kb);
    };

    f32x4 acc_g[MI][NI], acc_u[MI][NI];

    // ---- LDS -> registers.  The MFMA is v_mfma_f32_16x16x32_bf16: a lane holds tile row
    // (lane % 16) of a 16-row block and K chunk kk * 4 + lane / 16 of K step kk (0, 1: 32 columns
    // each); kk * 4 and lane / 16 occupy different bits, so the byte offset inside a unit is that
    // of K step 0 XOR kk * 64.  Blocks of 16 rows are 2048 bytes apart and swizzled alike.
    int a_frag0, b_frag0;
    {
        const int fr = lane & 15, fc = lane >> 4;
        const int ra = wm * TM + fr, rb = wn * TN + fr;
        a_frag0 = (ra * CH + swizzle<CH>(ra, fc)) * 16;
        b_frag0 = (rb * CH + swizzle<CH>(rb, fc)) * 16;
    }
    struct Frags {
        bf16x8 a[MI], g[NI], u[NI];
    };
    constexpr int N_READS = MI + 2 * NI;   // fragment reads per K step (16)
    // q-th fragment of K step kk of the slab in units (ua, ub), in the order the MFMAs need them:
    // a0 a1 g0 u0 g1 u1 .. a2 a3 ..
    auto read_one = [&](Frags &f, int ua, int ub, int kk, int q) {
        const char *pa = lds64 + ua * A_UNIT + (a_frag0 ^ (kk * 64)), *pb = lds64 + B_BASE + ub * B_UNIT + (b_frag0 ^ (kk * 64));
        if (q < 2) {
            f.a[q] = *reinterpret_cast<const bf16x8 *>(pa + q * 2048);
        } else if (q < 2 + 2 * NI) {
            const int j = (q - 2) >> 1;
            if ((q - 2) & 1)
                f.u[j] = *reinterpret_cast<const bf16x8 *>(pb + B_HALF + j * 2048);
            else
                f.g[j] = *reinterpret_cast<const bf16x8 *>(pb + j * 2048);
        } else {
            const int i = q - 2 * NI;
            f.a[i] = *reinterpret_cast<const bf16x8 *>(pa + i * 2048);
        }
    };
    constexpr int N_PAIRS = MI * NI, N_HALF = N_PAIRS / 2;   // pairs of MFMAs per K step (32)
    // Pair q of a K step.  The order is a Gray code over the operands: every MFMA shares one operand
    // with the one before, (a0, g) (a1, g) (a1, u) (a0, u) for g = g_0 .. g_3 with its u, then the next
    // two A blocks.  Measured against A-block-major order (a_i with g_0 u_0 g_1 u_1 ..): +1.5 %.
    auto mfma_pair = [&](const Frags &f, int q) {
        const int ip = q / (2 * NI), r = q % (2 * NI), j = r / 2;
        const int i0 = 2 * ip, i1 = 2 * ip + 1;
        if (r % 2 == 0) {
            acc_g[i0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i0], f.g[j], acc_g[i0][j], 0, 0, 0);
            acc_g[i1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i1], f.g[j], acc_g[i1][j], 0, 0, 0);
        } else {
            acc_u[i1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i1], f.u[j], acc_u[i1][j], 0, 0, 0);
            acc_u[i0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i0], f.u[j], acc_u[i0][j], 0, 0, 0);
        }
    };

    const int S = (int)(d / BK);   // slabs; the host guarantees d % 64 == 0
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc_g[i][j][r] = 0.0f;
                acc_u[i][j][r] = 0.0f;
            }
    if constexpr (DEEP) {
    // ---- small tiles.  Under the MFMAs of K step 0 go the fragment reads of K step 1; the second half of K step
    // 1, after the slab's one barrier, carries those of K step 0 of the next slab.  The B part of slab s + NB goes into
    // the unit of slab s from that barrier on, one load a pair, and the A part of slab s + NA under K step 0 of slab
    // s + 1 (all in the second half, 1 to 3 us more of every figure above).  Only slabs that exist are requested: the
    // last NB slabs have bodies of their own with fewer loads to wait for, and so have the first of a K of 3 to NB.
    // (Requests from an empty buffer instead, with one count for every wait, keep the load path as busy as real ones.  A
    // launch with those and now: one slab of 64 5.5 -> 5.0 us, two 6.1 -> 5.6, twelve 8.9 -> 8.5, 32 15.3 -> 14.9.)
    constexpr int N_LOADS = A_WL + 2 * B_WL, A_LEAD = NA - NB;   // the A parts run A_LEAD slabs further ahead
    static_assert(N_HALF == 2 * B_WL && N_PAIRS >= A_WL && (A_LEAD == 0 || A_LEAD == 1), "every load has its place");
    auto request_a = [&](int slab, int unit, int q) {
        issue_a(unit, slab * BK * 2, q);
        __builtin_amdgcn_sched_barrier(0);   // in this order: the waits count
    };
    auto request_b = [&](int slab, int unit, int q) {
        issue_b(unit, slab * BK * 2, q);
        __builtin_amdgcn_sched_barrier(0);
    };
    // A0 first where the A parts lead, then B0, A0 or A1, B1, ..: two of each before the first wait and the others of
    // the rings under the MFMAs of slab 0 (all five of K = 320 before the first wait, 0.4 us more).
    auto request_b_of = [&](int p) {
#pragma unroll
        for (int q = 0; q < 2 * B_WL; ++q)
            request_b(p, p, q);
    };
    auto request_a_of = [&](int p) {
#pragma unroll
        for (int q = 0; q < A_WL; ++q)
            request_a(p, p, q);
    };
    if (A_LEAD > 0)
        request_a_of(0);
    Frags f0, f1;
    auto begin = [&]() __attribute__((always_inline)) {   // slab 0 has landed
        block_barrier();
#pragma unroll
        for (int q = 0; q < N_READS; ++q)
            read_one(f0, 0, 0, 0, q);
    };
    int ua = 0, ub = 0, pa = 0;   // ring units of slab s, of the A part of slab s - 1
    // LEFT: how many slabs follow; NB stands for NB and more.
    auto slab_body = [&](int s, auto first_tag, auto left_tag) {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr int LEFT = decltype(left_tag)::value;
        constexpr bool LATE_A = !FIRST && LEFT >= NA - 1, NEXT_B = LEFT >= NB;
        constexpr int N_REST = !FIRST ? 0 : LEFT < NB ? (LEFT - 1) * N_LOADS - A_LEAD * A_WL : (NB - 2) * N_LOADS;
        constexpr int N_FREE = N_PAIRS + N_HALF;
        auto rest = [&](int q) {   // the prologue's other loads, spread over the pairs before the barrier
#pragma unroll
            for (int x = q * N_REST / N_FREE; x < (q + 1) * N_REST / N_FREE; ++x) {
                const int p = 2 + x / N_LOADS, y = x % N_LOADS;
                __builtin_amdgcn_sched_barrier(0);
                if (y < 2 * B_WL)
                    request_b(p, p, y);
                else
                    request_a(p + A_LEAD, p + A_LEAD, y - 2 * B_WL);
            }
        };
        const int ua1 = ua + 1 == NA ? 0 : ua + 1, ub1 = ub + 1 == NB ? 0 : ub + 1;
#pragma unroll
        for (int q = 0; q < N_PAIRS; ++q) {   // K step 0
            rest(q);
            if constexpr (LATE_A) {
#pragma unroll
                for (int x = q * A_WL / N_PAIRS; x < (q + 1) * A_WL / N_PAIRS; ++x)
                    issue_a(pa, (s - 1 + NA) * BK * 2, x);
            }
#pragma unroll
            for (int x = (q * N_READS + N_PAIRS - 1) / N_PAIRS; x < ((q + 1) * N_READS + N_PAIRS - 1) / N_PAIRS; ++x)
                read_one(f1, ua, ub, 1, x);
            mfma_pair(f0, q);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < N_HALF; ++q) {   // K step 1, first half
            rest(N_PAIRS + q);
            mfma_pair(f1, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (LEFT > 0) {
            // slab s + 1 has landed and this wavefront holds its last fragments of slab s: lgkmcnt(0) and vmcnt of
            // what was requested after both parts of slab s + 1
            constexpr int B_AHEAD = LEFT < NB - 1 ? LEFT : NB - 1, A_AHEAD = LEFT < NA - 1 ? LEFT : NA - 1;
            constexpr int AHEAD = (B_AHEAD - 1) * 2 * B_WL + (A_AHEAD - 1) * A_WL;
            static_assert(AHEAD < 64, "vmcnt is a 6-bit counter");
            __builtin_amdgcn_s_waitcnt(0x0070 | (AHEAD & 15) | ((AHEAD >> 4) << 14));
            block_barrier();
        }
#pragma unroll
        for (int q = 0; q < N_HALF; ++q) {   // K step 1, second half
            if constexpr (NEXT_B)
                issue_b(ub, (s + NB) * BK * 2, q);
            if constexpr (LEFT > 0) {
#pragma unroll
                for (int x = (q * N_READS + N_HALF - 1) / N_HALF; x < ((q + 1) * N_READS + N_HALF - 1) / N_HALF; ++x)
                    read_one(f0, ua1, ub1, 0, x);
            }
            mfma_pair(f1, N_HALF + q);
            __builtin_amdgcn_sched_barrier(0);
        }
        pa = ua;
        ua = ua1;
        ub = ub1;
    };
    int s = 0;
    if (S > 2) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            request_b_of(p);
            request_a_of(p + A_LEAD);
        }
        wait_vmcnt<N_LOADS + A_LEAD * A_WL>();
        begin();
        // (the first slab on its own: with one loop the compiler gave the accumulators other registers in every slab
        // and moved them back)
        if (S > NB) {
            slab_body(s++, std::true_type{}, std::integral_constant<int, NB>{});
            for (; s + NB < S; ++s)
                slab_body(s, std::false_type{}, std::integral_constant<int, NB>{});
        } else if (S == 3) {
            slab_body(s++, std::true_type{}, std::integral_constant<int, 2>{});
        } else if constexpr (NB == 5) {
            if (S == 4)
                slab_body(s++, std::true_type{}, std::integral_constant<int, 3>{});
            else
                slab_body(s++, std::true_type{}, std::integral_constant<int, 4>{});
        }
        static_assert(NB == 3 || NB == 5, "every S has its first slab");
    } else {
        request_b_of(0);
        if (A_LEAD == 0)
            request_a_of(0);
        if (S == 2) {
            if (A_LEAD > 0)
                request_a_of(1);
            request_b_of(1);
            if (A_LEAD == 0)
                request_a_of(1);
        }
        // The sums are cleared while the loads are on their way; left to itself the compiler does it behind the wait.
        // (Slab 0 above begins with constant ones.)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                asm volatile("" : "+a"(acc_g[i][j]), "+a"(acc_u[i][j]));
        if (S == 2)
            wait_vmcnt<N_LOADS>();
        else
            wait_vmcnt<0>();
        begin();
    }
    auto last = [&](auto left_tag) {
        constexpr int LEFT = decltype(left_tag)::value;
        if constexpr (LEFT < NB) {
            if (s + LEFT < S)
                slab_body(s++, std::false_type{}, left_tag);
        }
    };
    last(std::integral_constant<int, 4>{});
    last(std::integral_constant<int, 3>{});
    last(std::integral_constant<int, 2>{});
    last(std::integral_constant<int, 1>{});
    last(std::integral_constant<int, 0>{});
    block_barrier();   // the rings are about to be used again
    } else {
    // ---- prologue: A0 B0 A1 B1 A2 fill the five units, in this order: the waits count
#pragma unroll
    for (int q = 0; q < A_WL; ++q)
        issue_a(0, 0, q);
#pragma unroll
    for (int q = 0; q < 2 * B_WL; ++q)
        issue_b(1, 0, q);
    __builtin_amdgcn_sched_barrier(0);
    if (S > 1) {
#pragma unroll
        for (int q = 0; q < A_WL; ++q)
            issue_a(2, BK * 2, q);
#pragma unroll
        for (int q = 0; q < 2 * B_WL; ++q)
            issue_b(3, BK * 2, q);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (S > 2) {
#pragma unroll
        for (int q = 0; q < A_WL; ++q)
            issue_a(4, 2 * BK * 2, q);
    }
    if (S > 2)
        wait_vmcnt<2 * A_WL + 2 * B_WL>();   // slab 0 has landed
    else if (S > 1)
        wait_vmcnt<A_WL + 2 * B_WL>();
    else
        wait_vmcnt<0>();
    block_barrier();
    Frags f0, f1;
#pragma unroll
    for (int q = 0; q < N_READS; ++q)
        read_one(f0, 0, 1, 0, q);

    // ---- main loop.  One slab = 2 K steps of N_PAIRS gate/up MFMA pairs, the first on f0, the second
    // on f1.  During K step 0 a wavefront reads the fragments of K step 1, evenly between the pairs (8 x 4
    // tile: one read every second pair); during the second half of K step 1, after the slab's one barrier,
    // those of K step 0 of the next slab (one read a pair).  One global->LDS wave-load goes out every
    // A_GAP or B_GAP pairs (fourth pair): the rest of the B part of slab s + 1 (first half of K step 0),
    // then the A part of slab s + 2 (up to the barrier), then the first half of the B part of slab s + 2
    // into the A unit of slab s, which is free once every wavefront holds its last fragments of slab s.
    // B1, A2, B2:
    // whether these parts exist and were not issued by the prologue; NEXT: whether a slab follows.
    // All four are compile-time, so the steady state has no branch between its MFMAs.
    int ua = 0, ub = 1;   // ring units of slab s
    constexpr int A_GAP = N_HALF / (A_WL / 2), B_GAP = N_HALF / B_WL;   // MFMA pairs per wave-load (4)
    static_assert(N_HALF % (A_WL / 2) == 0 && N_HALF % B_WL == 0 && A_WL < 16, "every load has its place");
    auto slab_body = [&](int s, auto b1_tag, auto a2_tag, auto b2_tag, auto next_tag) {
        constexpr bool B1 = decltype(b1_tag)::value, A2 = decltype(a2_tag)::value, B2 = decltype(b2_tag)::value,
                       NEXT = decltype(next_tag)::value;
        const int ua1 = ua + 2 >= 5 ? ua - 3 : ua + 2, ub1 = ub + 2 >= 5 ? ub - 3 : ub + 2;   // units of slab s + 1
        const int uam = ua >= 2 ? ua - 2 : ua + 3, ubm = ub >= 2 ? ub - 2 : ub + 3;           // units of slab s - 1
        const int k1 = (s + 1) * BK * 2, k2 = (s + 2) * BK * 2;
#pragma unroll
        for (int q = 0; q < N_PAIRS; ++q) {   // K step 0
            if (B1 && q < N_HALF && q % B_GAP == 0)
                issue_b(uam, k1, B_WL + q / B_GAP);
            if (A2 && q >= N_HALF && (q - N_HALF) % A_GAP == 0)
                issue_a(ubm, k2, (q - N_HALF) / A_GAP);
#pragma unroll
            for (int x = (q * N_READS + N_PAIRS - 1) / N_PAIRS; x < ((q + 1) * N_READS + N_PAIRS - 1) / N_PAIRS; ++x)
                read_one(f1, ua, ub, 1, x);
            mfma_pair(f0, q);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < N_HALF; ++q) {   // K step 1, first half
            if (A2 && q % A_GAP == 0)
                issue_a(ubm, k2, A_WL / 2 + q / A_GAP);
            mfma_pair(f1, q);
            __builtin_amdgcn_sched_barrier(0);
        }
        // Slab s + 1 has landed (only the A part of slab s + 2, the last A_WL loads, may be in
        // flight) and this wavefront holds its last fragments of slab s: vmcnt(A_WL or 0), lgkmcnt(0).
        if (A2)
            __builtin_amdgcn_s_waitcnt(0x0070 | A_WL);
        else
            __builtin_amdgcn_s_waitcnt(0x0070);
        block_barrier();
#pragma unroll
        for (int q = 0; q < N_HALF; ++q) {   // K step 1, second half; the units of slab s are free
            if (B2 && q % B_GAP == 0)
                issue_b(ua, k2, q / B_GAP);
            if (NEXT) {
#pragma unroll
                for (int x = (q * N_READS + N_HALF - 1) / N_HALF; x < ((q + 1) * N_READS + N_HALF - 1) / N_HALF; ++x)
                    read_one(f0, ua1, ub1, 0, x);
            }
            mfma_pair(f1, N_HALF + q);
            __builtin_amdgcn_sched_barrier(0);
        }
        ua = ua1;
        ub = ub1;
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (S >= 3) {
        slab_body(0, No{}, No{}, Yes{}, Yes{});   // B1 and A2 went out in the prologue
        int s = 1;
        for (; s + 2 < S; ++s)
            slab_body(s, Yes{}, Yes{}, Yes{}, Yes{});
        slab_body(s, Yes{}, No{}, No{}, Yes{});       // slab S - 2
        slab_body(s + 1, No{}, No{}, No{}, No{});     // slab S - 1
    } else if (S == 2) {
        slab_body(0, No{}, No{}, No{}, Yes{});
        slab_body(1, No{}, No{}, No{}, No{});
    } else {
        slab_body(0, No{}, No{}, No{}, No{});
    }
    }

    if constexpr (EPI == kEpiNorms) {
        // ---- epilogue: y = act(g) * u, squared and summed over the tile's tokens (tokens are the
        // MFMA's M index: the 4 registers a lane holds of a 16 x 16 block are rows 4 (lane / 16) ..
        // + 3 of column lane % 16, i.e. 4 tokens of one neuron).  Tokens past T were read as zeros, so
        // their y is 0 and no test is needed.  The lane's neuron index is derived here from the lane
        // number afresh: nothing per-lane has to survive the main loop for it (a spill would give
        // the kernel a scratch segment).
        uint32_t lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(lane_e));
        const int fr_e = lane_e & 15, fc_e = lane_e >> 4;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            float part = 0.0f;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float y = glu_act_fast<ACT>(acc_g[i][j][r]) * acc_u[i][j][r];
                    part = fmaf(y, y, part);
                }
            }
            part += __shfl_xor(part, 16, 64);
            part += __shfl_xor(part, 32, 64);
            const int64_t n = n0 + wn * TN + j * 16 + fr_e;
            if (fc_e == 0 && n < d_int)
                atomicAdd(sumsq + n, part);
        }
    } else {
        // ---- storing epilogues.  Every wavefront is past the last barrier and the last LDS read
        // of the main loop, so the ring is free: the tile goes there as bf16, row stride SROW (16
        // bytes of padding), and leaves it in whole 16-byte chunks of output rows.
        constexpr int COLS = BN_TILE;                // output columns of the tile
        constexpr int SROW = COLS * 2 + 16;
        static_assert(BM * SROW <= P64_LDS, "the tile fits in the ring");
        // A lane holds rows r and r + 1 (registers 2 k, 2 k + 1) of column fr; with its neighbour
        // fr ^ 1 it trades one of them, so that even lanes own row 2 k and odd lanes row 2 k + 1
        // of the column pair: one 32-bit LDS write each.
        uint32_t lane_s = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));   // afresh, as above
        asm volatile("" : "+v"(lane_s));
        const int fr = lane_s & 15, fc = lane_s >> 4;
        auto put_pair = [&](float v0, float v1, int row_even, int col_base) {
            const bool odd = fr & 1;
            const float mine = odd ? v1 : v0, send = odd ? v0 : v1;
            const float got = __shfl_xor(send, 1, 64);
            const uint32_t word = odd ? bf16_pair(got, mine) : bf16_pair(mine, got);
            const int row = row_even + (odd ? 1 : 0), col = col_base + (fr & ~1);
            *reinterpret_cast<uint32_t *>(lds64 + row * SROW + col * 2) = word;
        };
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int row_even = wm * TM + i * 16 + 4 * fc + 2 * k;
                    const int col_base = wn * TN + j * 16;
                    if constexpr (EPI == kEpiGlu) {
                        put_pair(glu_act_fast<ACT>(acc_g[i][j][2 * k]) * acc_u[i][j][2 * k],
                                 glu_act_fast<ACT>(acc_g[i][j][2 * k + 1]) * acc_u[i][j][2 * k + 1], row_even, col_base);
                    } else {
                        put_pair(acc_g[i][j][2 * k], acc_g[i][j][2 * k + 1], row_even, col_base);
                        put_pair(acc_u[i][j][2 * k], acc_u[i][j][2 * k + 1], row_even, BN + col_base);
                    }
                }
        __syncthreads();
        constexpr int CPR = COLS / 8;   // 16-byte chunks per tile row
        for (int c = tid; c < BM * CPR; c += 256) {
            const int row = c / CPR, cc = c % CPR;
            const int64_t t = t0 + row, n = n0 + cc * 8;
            if (t < T && n < d_int)   // d_int is a multiple of 8: a chunk is inside or outside
                __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(lds64 + row * SROW + cc * 16),
                                            reinterpret_cast<u32x4 *>(out + t * ldo + n));   // streamed: not read again from L2
        }
    }
}

// ------------------------------------------------------------------- f32 MFMA --
// v_mfma_f32_16x16x4_f32 on fragments that come straight from global memory.  A wavefront owns 32
// tokens x 32 neurons x {gate, up}: 8 accumulator blocks, and per 16 columns of K 6 fragments of 16
// rows x 64 bytes.  Lane l holds columns 4 (l / 16) .. + 3 of row l % 16 of a fragment as one 16-byte
// load, and the i-th of its four floats goes into the i-th MFMA of the chunk: that MFMA then covers
// columns i, 4 + i, 8 + i, 12 + i, the same ones of both operands.  The f32 matrix rate is 256 flop
// a clock and CU, so 6 KB for 1024 clocks of a SIMD is within what L1 and L2 deliver; there is no LDS
// and no barrier in the loop, and kDepth - 1 chunks per wavefront are in flight.  (An LDS-tiled kernel
// of vector FMAs took 823 us for 4096 tokens of 1024 x 4096 and 32 us for 512 of 256 x 688; this one
// 688 and 19, launches included.)
//   KSPLIT = 1   a workgroup is 2 x 2 wavefront tiles (64 tokens x 64 neurons) that share rows in L1.
//   KSPLIT = 4   a workgroup is one wavefront tile; its four wavefronts take every fourth chunk and
//                add up through LDS.  Four times the workgroups, each a quarter as long.
constexpr int F_WT = 32;      // tokens and neurons of a wavefront tile
constexpr int F_KC = 16;      // columns of a chunk

template <int KSPLIT>
__global__ __launch_bounds__(256) void calib_f32_kernel(
    const float *__restrict__ X, int64_t T, int64_t ldx, const float *__restrict__ Wg,
    const float *__restrict__ Wu, int64_t ldw, int64_t d, int64_t d_int, int act,
    float *__restrict__ sumsq, const TileOrder order)
{
    constexpr int kDepth = 4;
    constexpr int WGT = KSPLIT == 1 ? 2 * F_WT : F_WT;   // tokens and neurons of a workgroup

    uint32_t tile_t, tile_n;   // tile_order.h
    if (!tile_of_block(order, blockIdx.x, tile_t, tile_n))
        return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fc = lane >> 4;
    const int64_t t0 = (int64_t)tile_t * WGT + (KSPLIT == 1 ? wave / 2 * F_WT : 0);
    const int64_t n0 = (int64_t)tile_n * WGT + (KSPLIT == 1 ? wave % 2 * F_WT : 0);

    // Rows past the end are clamped to the last one; the epilogue drops what they give.
    const float *row[6];   // X, X + 16 rows, Wgate, + 16, Wup, + 16
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t t = t0 + 16 * h + fr, n = n0 + 16 * h + fr;
        row[h] = X + (t < T ? t : T - 1) * ldx;
        row[2 + h] = Wg + (n < d_int ? n : d_int - 1) * ldw;
        row[4 + h] = Wu + (n < d_int ? n : d_int - 1) * ldw;
    }
    f32x4 frag[kDepth][6];
    auto load_chunk = [&](int buf, int64_t chunk) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            frag[buf][q] = *reinterpret_cast<const f32x4 *>(row[q] + chunk * F_KC + 4 * fc);
    };

    f32x4 acc_g[2][2], acc_u[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc_g[i][j][r] = acc_u[i][j][r] = 0.0f;

    auto multiply = [&](int buf) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc_g[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(frag[buf][i][k], frag[buf][2 + j][k], acc_g[i][j], 0, 0, 0);
                    acc_u[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(frag[buf][i][k], frag[buf][4 + j][k], acc_u[i][j], 0, 0, 0);
                }
    };
    const int64_t chunks = d / F_KC;   // whole ones
    const int64_t first = KSPLIT == 1 ? 0 : wave;
#pragma unroll
    for (int b = 0; b < kDepth - 1; ++b)
        if (first + b * KSPLIT < chunks)
            load_chunk(b, first + b * KSPLIT);
    int64_t c = first;
    for (; c + (2 * kDepth - 2) * KSPLIT < chunks; c += kDepth * KSPLIT) {
#pragma unroll
        for (int b = 0; b < kDepth; ++b) {
            load_chunk((b + kDepth - 1) % kDepth, c + (b + kDepth - 1) * KSPLIT);
            multiply(b);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of these MFMAs
        }
    }
    for (; c < chunks; c += kDepth * KSPLIT) {   // the last one or two rounds
#pragma unroll
        for (int b = 0; b < kDepth; ++b) {
            if (c + (b + kDepth - 1) * KSPLIT < chunks)
                load_chunk((b + kDepth - 1) % kDepth, c + (b + kDepth - 1) * KSPLIT);
            if (c + b * KSPLIT < chunks)
                multiply(b);
        }
    }
    if (d % F_KC != 0 && (KSPLIT == 1 || chunks % KSPLIT == wave)) {
        // Columns past d (a multiple of 4) read column 0 and become 0.
        const int64_t k = chunks * F_KC + 4 * fc;
        const bool in = k < d;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(row[q] + (in ? k : 0));
#pragma unroll
            for (int i = 0; i < 4; ++i)
                frag[0][q][i] = in ? v[i] : 0.0f;
        }
        multiply(0);
    }

    // Register r of lane l of a block is token 4 (l / 16) + r and neuron l % 16.
    auto column_sum = [&](const f32x4 &g, const f32x4 &u, int64_t t_block) {
        float part = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // a row past the end is a copy of the last token: its y may be infinite, and 0 times that a NaN
            const float y = t_block + 4 * fc + r < T ? glu_act_precise(g[r], act) * u[r] : 0.0f;
            part = fmaf(y, y, part);
        }
        return part;
    };
    // All tokens of the workgroup are added up before the one atomic per neuron.
    __shared__ float halves[2][WGT];   // [token half][neuron of the workgroup]
    auto column_total = [&](float part, int half, int col) {
        part += __shfl_xor(part, 16, 64);
        part += __shfl_xor(part, 32, 64);
        if (fc == 0)
            halves[half][col + fr] = part;
    };
    if constexpr (KSPLIT == 1) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            column_total(column_sum(acc_g[0][j], acc_u[0][j], t0) + column_sum(acc_g[1][j], acc_u[1][j], t0 + 16), wave / 2,
                         wave % 2 * F_WT + 16 * j);
    } else {
        __shared__ __attribute__((aligned(16))) f32x4 sums[KSPLIT][2][4][64];   // [wavefront][gate, up][block][lane]
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sums[wave][0][q][lane] = acc_g[q / 2][q % 2];
            sums[wave][1][q][lane] = acc_u[q / 2][q % 2];
        }
        __syncthreads();
        f32x4 g = sums[0][0][wave][lane], u = sums[0][1][wave][lane];   // each wavefront finishes one block
#pragma unroll
        for (int w = 1; w < KSPLIT; ++w) {
            g += sums[w][0][wave][lane];
            u += sums[w][1][wave][lane];
        }
        column_total(column_sum(g, u, t0 + 16 * (wave / 2)), wave / 2, 16 * (wave % 2));
    }
    __syncthreads();
    const int64_t n = (int64_t)tile_n * WGT + threadIdx.x;
    if (threadIdx.x < WGT && n < d_int)
        atomicAdd(sumsq + n, halves[0][threadIdx.x] + halves[1][threadIdx.x]);
}

// ------------------------------------------------------------------ host side --
template <int BM, int BN, int BK, int WM, int WN, int MINB>
static void launch_mfma(int act, dim3 grid, hipStream_t stream, const uint16_t *X, int64_t T,
                        int64_t ldx, const uint16_t *Wg, const uint16_t *Wu, int64_t ldw, int64_t d,
                        int64_t d_int, float *sumsq, int64_t tiles_t, int64_t tiles_n)
{
    const dim3 block(64 * WM * WN);
    switch (act) {
    case DASS_ACT_SILU:
        hipLaunchKernelGGL((calib_mfma_kernel<BM, BN, BK, WM, WN, MINB, DASS_ACT_SILU>), grid, block, 0,
                           stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, tiles_t, tiles_n);
        break;
    case DASS_ACT_GELU_TANH:
        hipLaunchKernelGGL((calib_mfma_kernel<BM, BN, BK, WM, WN, MINB, DASS_ACT_GELU_TANH>), grid, block,
                           0, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, tiles_t, tiles_n);
        break;
    case DASS_ACT_GELU_ERF:
        hipLaunchKernelGGL((calib_mfma_kernel<BM, BN, BK, WM, WN, MINB, DASS_ACT_GELU_ERF>), grid, block,
                           0, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, tiles_t, tiles_n);
        break;
    default:
        hipLaunchKernelGGL((calib_mfma_kernel<BM, BN, BK, WM, WN, MINB, DASS_ACT_RELU>), grid, block, 0,
                           stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, tiles_t, tiles_n);
        break;
    }
}

template <int ACT, int EPI, int MI, int NI>
static hipError_t launch_pipe64_tile(hipStream_t stream, const uint16_t *X, int64_t T, int64_t ldx,
                                     const uint16_t *Wg, const uint16_t *Wu, int64_t ldw, int64_t d, int64_t d_int,
                                     float *sumsq, uint16_t *out, int64_t ldo, const TileOrder &order)
{
    // the kernel's ring takes all 160 KB of LDS, more than a launch gets without asking
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(calib_pipe64_kernel<ACT, EPI, MI, NI>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, P64_LDS);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL((calib_pipe64_kernel<ACT, EPI, MI, NI>), dim3(order.blocks), dim3(256), P64_LDS, stream, X, T, ldx,
                       Wg, Wu, ldw, d, d_int, sumsq, out, ldo, order);
    return hipSuccess;
}

template <int ACT, int EPI>
static hipError_t launch_pipe64_act(const TileShape &shape, hipStream_t stream, const uint16_t *X, int64_t T, int64_t ldx,
                                    const uint16_t *Wg, const uint16_t *Wu, int64_t ldw, int64_t d, int64_t d_int,
                                    float *sumsq, uint16_t *out, int64_t ldo, const TileOrder &order)
{
    if (shape.which == 0)
        return launch_pipe64_tile<ACT, EPI, 8, 4>(stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo, order);
    if (shape.which == 1)
        return launch_pipe64_tile<ACT, EPI, 4, 4>(stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo, order);
    return launch_pipe64_tile<ACT, EPI, 4, 2>(stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo, order);
}

template <int EPI>
static hipError_t launch_pipe64(int act, const TileShape &shape, hipStream_t stream, const uint16_t *X, int64_t T, int64_t ldx,
                                const uint16_t *Wg, const uint16_t *Wu, int64_t ldw, int64_t d, int64_t d_int,
                                float *sumsq, uint16_t *out, int64_t ldo, const TileOrder &order)
{
    switch (act) {
    case DASS_ACT_SILU:
        return launch_pipe64_act<DASS_ACT_SILU, EPI>(shape, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo,
                                                         order);
    case DASS_ACT_GELU_TANH:
        return launch_pipe64_act<DASS_ACT_GELU_TANH, EPI>(shape, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo,
                                                         order);
    case DASS_ACT_GELU_ERF:
        return launch_pipe64_act<DASS_ACT_GELU_ERF, EPI>(shape, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo,
                                                         order);
    default:
        return launch_pipe64_act<DASS_ACT_RELU, EPI>(shape, stream, X, T, ldx, Wg, Wu, ldw, d, d_int, sumsq, out, ldo,
                                                         order);
    }
}

// Whether a wavefront tile gets a workgroup of its own (calib_f32_kernel, KSPLIT = 4): when the 64 x 64
// tiles are no more than the 256 compute units.  Whole calls, split and not: 512 tokens, 256 x 688 (88
// tiles) 18.9 and 21.2 us, 128 tokens, 1024 x 4096 (128) 34 and 54 us; 1024 tokens, 512 x 2048 (512) 66 and
// 58 us, 4096 tokens, 1024 x 4096 738 and 688 us (100 TFLOP/s).
static bool split_f32(int64_t T, int64_t d_int)
{
    return ((T + 2 * F_WT - 1) / (2 * F_WT)) * ((d_int + 2 * F_WT - 1) / (2 * F_WT)) <= 256;
}

// Whether `matrices` matrices of this size stay in the 256 MB memory-side cache.
static bool fits_memory_cache(int64_t matrices, int64_t rows, int64_t cols, int dt)
{
    return matrices * rows * cols * elem_bytes(dt) <= (256LL << 20);
}

}  // namespace dass

extern "C" size_t dass_calib_workspace_bytes(int64_t T, int64_t d, int64_t d_int, dass_dtype dt)
{
    (void)T; (void)d; (void)d_int; (void)dt;
    return 0;  // the accumulation goes straight into sumsq
}

extern "C" dass_status dass_calib_norms(const void *X, int64_t T, int64_t ldx, const void *Wgate,
                                        const void *Wup, int64_t ldw, int64_t d, int64_t d_int,
                                        dass_dtype dt, dass_act act, float *sumsq, int accumulate,
                                        float *norms_out, void *workspace, size_t workspace_bytes,
                                        void *hip_stream)
{
    using namespace dass;
    const char *fn = "dass_calib_norms";
    (void)workspace;
    (void)workspace_bytes;
    if (!X || !Wgate || !Wup || !sumsq)
        return fail(DASS_ERR_NULL, "%s: X, Wgate, Wup and sumsq must not be NULL", fn);
    if (!valid_dtype(dt))
        return fail(DASS_ERR_DTYPE, "%s: unknown dtype %d", fn, (int)dt);
    if ((int)act < DASS_ACT_SILU || (int)act > DASS_ACT_RELU)
        return fail(DASS_ERR_DTYPE, "%s: unknown activation %d", fn, (int)act);
    if (T <= 0 || d <= 0 || d_int <= 0)
        return fail(DASS_ERR_SHAPE, "%s: T=%lld d=%lld d_int=%lld must be positive", fn,
                    (long long)T, (long long)d, (long long)d_int);
    if (ldx < d || ldw < d)
        return fail(DASS_ERR_SHAPE, "%s: ldx=%lld, ldw=%lld must be >= d=%lld", fn, (long long)ldx,
                    (long long)ldw, (long long)d);
    const int vec = vec_elems(dt);
    if (d % vec != 0)
        return fail(DASS_ERR_SHAPE, "%s: d=%lld must be a multiple of %d", fn, (long long)d, vec);
    if (!aligned16(X) || !aligned16(Wgate) || !aligned16(Wup) ||
        (reinterpret_cast<uintptr_t>(sumsq) & 3u) ||
        (norms_out && (reinterpret_cast<uintptr_t>(norms_out) & 3u)))
        return fail(DASS_ERR_ALIGN, "%s: X, Wgate, Wup must be 16-byte aligned", fn);
    if (ldx % vec != 0 || ldw % vec != 0)
        return fail(DASS_ERR_ALIGN, "%s: ldx, ldw must be multiples of %d elements", fn, vec);

    // ---- launch plan; every size check comes before the first launch
    constexpr int BM = P_BM, BN = P_BN, BK = 64;
    const bool bf16 = dt == DASS_BF16;
    const bool f32_split = !bf16 && split_f32(T, d_int);
    const int f_tile = f32_split ? F_WT : 2 * F_WT;
    // calib_pipe64_kernel: d a multiple of its 64-column slab, and 32-bit byte offsets inside a
    // tile's rows.
    const bool pipe64 = bf16 && d % 64 == 0 && (int64_t)BM * ldx * 2 < 0x7fffffffLL &&
                        (int64_t)BN * ldw * 2 < 0x7fffffffLL;
    const TileShape shape = pipe64 ? dense_tile_shape(T, d_int, true) : TileShape{};
    const int64_t tiles_t = pipe64 ? shape.tiles_t : bf16 ? (T + BM - 1) / BM : (T + f_tile - 1) / f_tile;
    const int64_t tiles_n = pipe64 ? shape.tiles_n : bf16 ? (d_int + BN - 1) / BN : (d_int + f_tile - 1) / f_tile;
    const TileOrder order = make_tile_order(tiles_t, tiles_n, fits_memory_cache(2, d_int, d, dt),
                                            pipe64 && shape.which == 1 ? 8 : kPatchT);
    const int64_t blocks = pipe64 || !bf16 ? order.blocks : (tiles_t * tiles_n + 7) / 8 * 8;
    if (blocks <= 0 || blocks > 0x7fffffffLL)
        return fail(DASS_ERR_SHAPE, "%s: too many tiles for one launch; split the tokens", fn);

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const unsigned vgrid = (unsigned)((d_int + 255) / 256);
    if (!accumulate) {
        hipLaunchKernelGGL(fill_zero_kernel, dim3(vgrid), dim3(256), 0, stream, sumsq, d_int);
        dass_status s = check_launch("fill kernel");
        if (s != DASS_OK)
            return s;
    }
    if (pipe64) {
        const hipError_t e = launch_pipe64<kEpiNorms>((int)act, shape, stream, static_cast<const uint16_t *>(X), T, ldx,
                                                      static_cast<const uint16_t *>(Wgate),
                                                      static_cast<const uint16_t *>(Wup), ldw, d, d_int, sumsq,
                                                      nullptr, 0, order);
        if (e != hipSuccess)
            return fail(DASS_ERR_HIP, "%s: cannot reserve %d bytes of LDS: %s", fn, P64_LDS, hipGetErrorString(e));
    } else if (bf16) {
        launch_mfma<BM, BN, BK, 4, 2, 1>((int)act, dim3((unsigned)blocks), stream, static_cast<const uint16_t *>(X),
                                         T, ldx, static_cast<const uint16_t *>(Wgate),
                                         static_cast<const uint16_t *>(Wup), ldw, d, d_int, sumsq, tiles_t, tiles_n);
    } else {
        const auto kernel = f32_split ? calib_f32_kernel<4> : calib_f32_kernel<1>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                           static_cast<const float *>(X), T, ldx, static_cast<const float *>(Wgate),
                           static_cast<const float *>(Wup), ldw, d, d_int, (int)act, sumsq, order);
    }
    dass_status s = check_launch("calibration kernel");
    if (s != DASS_OK)
        return s;
    if (norms_out) {
        hipLaunchKernelGGL(sqrt_kernel, dim3(vgrid), dim3(256), 0, stream, (const float *)sumsq,
                           norms_out, d_int);
        s = check_launch("sqrt kernel");
    }
    return s;
}

// ------------------------------------------------------------- MLP output --
extern "C" size_t dass_mlp_forward_workspace_bytes(int64_t T, int64_t d, int64_t d_int, dass_dtype dt)
{
    (void)d;
    if (T <= 0 || d_int <= 0 || dt != DASS_BF16)
        return 0;
    return (size_t)T * (size_t)d_int * 2;   // y of Eq. 2 as bf16, [T, d_int]
}

extern "C" dass_status dass_mlp_forward(const void *X, int64_t T, int64_t ldx, const void *Wgate, const void *Wup,
                                        int64_t ldw, const void *Wdown, int64_t ldd, int64_t d, int64_t d_int,
                                        dass_dtype dt, dass_act act, void *out, int64_t ldo, void *workspace,
                                        size_t workspace_bytes, void *hip_stream)
{
    using namespace dass;
    const char *fn = "dass_mlp_forward";
    const bool eq2_only = Wdown == nullptr;   // y stays in the workspace; out and ldd, ldo are not used
    if (!X || !Wgate || !Wup || !workspace || (!eq2_only && !out))
        return fail(DASS_ERR_NULL, "%s: X, Wgate, Wup, workspace (and out, unless Wdown is NULL) must not be NULL", fn);
    if (!valid_dtype(dt))
        return fail(DASS_ERR_DTYPE, "%s: unknown dtype %d", fn, (int)dt);
    if (dt != DASS_BF16)
        return fail(DASS_ERR_DTYPE, "%s: only bf16 is implemented", fn);
    if ((int)act < DASS_ACT_SILU || (int)act > DASS_ACT_RELU)
        return fail(DASS_ERR_DTYPE, "%s: unknown activation %d", fn, (int)act);
    if (T <= 0 || d <= 0 || d_int <= 0)
        return fail(DASS_ERR_SHAPE, "%s: T=%lld d=%lld d_int=%lld must be positive", fn, (long long)T,
                    (long long)d, (long long)d_int);
    if (d % 64 != 0 || d_int % 64 != 0)
        return fail(DASS_ERR_SHAPE, "%s: d=%lld and d_int=%lld must be multiples of 64", fn, (long long)d,
                    (long long)d_int);
    if (ldx < d || ldw < d || (!eq2_only && (ldd < d_int || ldo < d)))
        return fail(DASS_ERR_SHAPE, "%s: a leading dimension is shorter than its row", fn);
    if (!aligned16(X) || !aligned16(Wgate) || !aligned16(Wup) || !aligned16(workspace) ||
        (!eq2_only && (!aligned16(Wdown) || !aligned16(out))))
        return fail(DASS_ERR_ALIGN, "%s: every pointer must be 16-byte aligned", fn);
    if (ldx % 8 != 0 || ldw % 8 != 0 || (!eq2_only && (ldd % 8 != 0 || ldo % 8 != 0)))
        return fail(DASS_ERR_ALIGN, "%s: leading dimensions must be multiples of 8 elements", fn);
    if (workspace_bytes < dass_mlp_forward_workspace_bytes(T, d, d_int, dt))
        return fail(DASS_ERR_WORKSPACE, "%s: workspace of %zu bytes, %zu needed", fn, workspace_bytes,
                    dass_mlp_forward_workspace_bytes(T, d, d_int, dt));
    // 32-bit byte offsets inside a tile's rows, as in dass_calib_norms
    if ((int64_t)P_BM * ldx * 2 >= 0x7fffffffLL || (int64_t)P_BN * ldw * 2 >= 0x7fffffffLL ||
        (int64_t)P_BM * d_int * 2 >= 0x7fffffffLL || (!eq2_only && (int64_t)P_BN * ldd * 2 >= 0x7fffffffLL))
        return fail(DASS_ERR_SHAPE, "%s: rows too long for the tile addressing", fn);

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint16_t *Y = static_cast<uint16_t *>(workspace);
    // Eq. 2: y = act(X Wgate^T) * (X Wup^T), tiles of up to 256 tokens x 128 neurons
    {
        const TileShape shape = dense_tile_shape(T, d_int, true);
        const TileOrder order = make_tile_order(shape.tiles_t, shape.tiles_n, fits_memory_cache(2, d_int, d, dt),
                                                shape.which == 1 ? 8 : kPatchT);
        if (order.blocks == 0)
            return fail(DASS_ERR_SHAPE, "%s: too many tiles for one launch; split the tokens", fn);
        const hipError_t e = launch_pipe64<kEpiGlu>((int)act, shape, stream, static_cast<const uint16_t *>(X), T, ldx,
                                                    static_cast<const uint16_t *>(Wgate),
                                                    static_cast<const uint16_t *>(Wup), ldw, d, d_int, nullptr, Y,
                                                    d_int, order);
        if (e != hipSuccess)
            return fail(DASS_ERR_HIP, "%s: cannot reserve %d bytes of LDS: %s", fn, P64_LDS, hipGetErrorString(e));
        const dass_status s = check_launch("GLU kernel");
        if (s != DASS_OK || eq2_only)
            return s;
    }
    // Eq. 3: out = y Wdown^T, tiles of up to 256 tokens x 256 output features, K = d_int
    {
        const TileShape shape = dense_tile_shape(T, d, false);
        const TileOrder order = make_tile_order(shape.tiles_t, shape.tiles_n, fits_memory_cache(1, d_int, d, dt),
                                                shape.which == 1 ? 8 : kPatchT);
        if (order.blocks == 0)
            return fail(DASS_ERR_SHAPE, "%s: too many tiles for one launch; split the tokens", fn);
        const hipError_t e = launch_pipe64_act<DASS_ACT_RELU, kEpiGemm>(
            shape, stream, Y, T, d_int, static_cast<const uint16_t *>(Wdown), nullptr, ldd, d_int, d,
            nullptr, static_cast<uint16_t *>(out), ldo, order);
        if (e != hipSuccess)
            return fail(DASS_ERR_HIP, "%s: cannot reserve %d bytes of LDS: %s", fn, P64_LDS, hipGetErrorString(e));
        return check_launch("down-projection kernel");
    }
}
