// The input-feature norms of the Wanda metric (Sec. 2.1 Eq. 1): ||X_j||_2 over all tokens, the
// quantity that the Down-Proj score of Eq. 5 is built like and the paper's main comparison
// system scores every layer with.  sumsq[j] (+)= sum_t X[t, j]^2, norms = sqrt(sumsq).
//
// The pass is bound by reading X once (HBM).  No atomics, so the result does not depend on the
// order in which workgroups finish.
//   input_strip_kernel    few tokens: one launch.  A workgroup owns the 64-byte strip of 32 bf16 / 16
//                         f32 columns and all rows, so nothing has to be added up across workgroups.
//   input_partial_kernel  many tokens: a thread owns the 16 bytes of one column slot (8 bf16 / 4 f32
//                         columns) and the rows of one row block; it adds the squares in f32
//                         and writes its sums to partial[row block][column].
//   input_reduce_kernel   adds the row blocks' partial sums of a column in f64, in a fixed order,
//                         and writes sumsq (optionally added to what is there) and the norm.
#include "select.h"

namespace dass {

constexpr int kInBlock = 256;     // threads = column slots per workgroup
constexpr int kInUnroll = 8;      // rows in flight per thread
constexpr int kInMaxRows = 512;   // rows per row block, at most (a multiple of kInUnroll)
constexpr int64_t kReduceCols = 1 << 27;   // columns of one reduction launch, at most: a grid has fewer than 2^32 threads

// The last step of either path: sumsq (+)= total, norm = sqrt(sumsq).
__device__ __forceinline__ void finish_column(double total, int64_t j, float *__restrict__ sumsq, int accumulate,
                                              float *__restrict__ norms)
{
    if (accumulate)
        total += (double)sumsq[j];
    const float s32 = (float)total;
    sumsq[j] = s32;
    if (norms)
        norms[j] = (float)sqrt((double)s32);
}

constexpr int kStripThreads = 1024;
constexpr int kStripSlots = 4;                                // 16-byte slots of a strip: half a memory line
constexpr int kStripRows = kStripThreads / kStripSlots;       // rows read at once

template <int DT>
__global__ __launch_bounds__(kStripThreads) void input_strip_kernel(
    const void *__restrict__ Xv, int64_t T, int64_t ldx, int64_t d, float *__restrict__ sumsq, int accumulate,
    float *__restrict__ norms)
{
    constexpr int EPV = DT == DASS_BF16 ? 8 : 4;
    constexpr int EB = DT == DASS_BF16 ? 2 : 4;
    constexpr int COLS = kStripSlots * EPV;
    __shared__ float part[kStripThreads / 64][COLS];
    // workgroup b runs on XCD b % 8: the two strips of a 128-byte line go to one XCD, whose L2
    // then fetches the line once
    const int64_t xcd = blockIdx.x % 8, i = blockIdx.x / 8;
    const int64_t strip = (i / 2 * 8 + xcd) * 2 + i % 2;
    const int64_t c0 = strip * COLS;
    if (c0 >= d)
        return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int slot = tid % kStripSlots;
    const int64_t c = c0 + slot * EPV;
    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e)
        acc[e] = 0.0f;
    if (c < d) {
        const char *X = static_cast<const char *>(Xv) + c * EB;
        int64_t r = tid / kStripSlots;
        for (; r + (kInUnroll - 1) * kStripRows < T; r += kInUnroll * kStripRows) {
            u32x4 v[kInUnroll];
#pragma unroll
            for (int k = 0; k < kInUnroll; ++k)
                v[k] = *reinterpret_cast<const u32x4 *>(X + (r + k * kStripRows) * ldx * EB);
#pragma unroll
            for (int k = 0; k < kInUnroll; ++k)
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float x = elem_of<DT>(v[k], e);
                    acc[e] = fmaf(x, x, acc[e]);
                }
        }
        // up to kInUnroll - 1 rows left: all loads first; a row past the end is neither loaded nor added
        u32x4 v[kInUnroll - 1];
#pragma unroll
        for (int k = 0; k < kInUnroll - 1; ++k)
            if (r + k * kStripRows < T)
                v[k] = *reinterpret_cast<const u32x4 *>(X + (r + k * kStripRows) * ldx * EB);
#pragma unroll
        for (int k = 0; k < kInUnroll - 1; ++k)
            if (r + k * kStripRows < T) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float x = elem_of<DT>(v[k], e);
                    acc[e] = fmaf(x, x, acc[e]);
                }
            }
    }
    // 16 lanes of a wavefront hold rows of the same slot
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
#pragma unroll
        for (int s = kStripSlots; s < 64; s *= 2)
            acc[e] += __shfl_xor(acc[e], s, 64);
    }
    if (lane < kStripSlots) {
#pragma unroll
        for (int e = 0; e < EPV; ++e)
            part[wave][lane * EPV + e] = acc[e];
    }
    __syncthreads();
    if (tid < COLS && c0 + tid < d) {
        double total = 0.0;
#pragma unroll
        for (int w = 0; w < kStripThreads / 64; ++w)
            total += (double)part[w][tid];
        finish_column(total, c0 + tid, sumsq, accumulate, norms);
    }
}

template <int DT>
__global__ __launch_bounds__(kInBlock) void input_partial_kernel(
    const void *__restrict__ Xv, int64_t T, int64_t ldx, int64_t d, int64_t rows_per_block,
    float *__restrict__ partial)
{
    constexpr int EPV = DT == DASS_BF16 ? 8 : 4;
    constexpr int EB = DT == DASS_BF16 ? 2 : 4;
    const int64_t slots = d / EPV;
    const uint32_t nbx = (uint32_t)((slots + kInBlock - 1) / kInBlock);
    const uint32_t bx = blockIdx.x % nbx, rb = blockIdx.x / nbx;
    const int64_t slot = (int64_t)bx * kInBlock + threadIdx.x;
    if (slot >= slots)
        return;
    const int64_t r0 = (int64_t)rb * rows_per_block;
    const int64_t r1 = r0 + rows_per_block < T ? r0 + rows_per_block : T;
    const char *X = static_cast<const char *>(Xv) + slot * 16;

    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e)
        acc[e] = 0.0f;
    int64_t r = r0;
    for (; r + kInUnroll <= r1; r += kInUnroll) {
        u32x4 v[kInUnroll];
#pragma unroll
        for (int k = 0; k < kInUnroll; ++k)
            v[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(X + (r + k) * ldx * EB));
#pragma unroll
        for (int k = 0; k < kInUnroll; ++k)
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                const float x = elem_of<DT>(v[k], e);
                acc[e] = fmaf(x, x, acc[e]);
            }
    }
    for (; r < r1; ++r) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(X + r * ldx * EB));
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float x = elem_of<DT>(v, e);
            acc[e] = fmaf(x, x, acc[e]);
        }
    }
    float *out = partial + (int64_t)rb * d + slot * EPV;
#pragma unroll
    for (int q = 0; q < EPV / 4; ++q) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = __float_as_uint(acc[4 * q + i]);
        *reinterpret_cast<u32x4 *>(out + 4 * q) = w;
    }
}

// A workgroup owns 64 columns; wavefront w adds the partial sums of every kReduceWaves-th row block
// (w, w + kReduceWaves, ...) in f64, then the wavefronts' sums are added in a fixed order.
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(64 * kReduceWaves) void input_reduce_kernel(
    const float *__restrict__ partial, int64_t n_row_blocks, int64_t d, int64_t j0, float *__restrict__ sumsq,
    int accumulate, float *__restrict__ norms)
{
    __shared__ double part[kReduceWaves][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t j = j0 + (int64_t)blockIdx.x * 64 + lane;
    double s = 0.0;
    if (j < d) {
        int64_t b = w;
        for (; b + 3 * kReduceWaves < n_row_blocks; b += 4 * kReduceWaves) {   // four loads in flight
            const float x0 = partial[b * d + j], x1 = partial[(b + kReduceWaves) * d + j],
                        x2 = partial[(b + 2 * kReduceWaves) * d + j], x3 = partial[(b + 3 * kReduceWaves) * d + j];
            s += (double)x0;
            s += (double)x1;
            s += (double)x2;
            s += (double)x3;
        }
        for (; b < n_row_blocks; b += kReduceWaves)
            s += (double)partial[b * d + j];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && j < d) {
        double total = 0.0;
#pragma unroll
        for (int i = 0; i < kReduceWaves; ++i)
            total += part[i][lane];
        finish_column(total, j, sumsq, accumulate, norms);
    }
}

// Rows per row block of input_partial_kernel: about 1024 wavefronts (one per SIMD) whatever the
// shape, each with as long a run of rows as that leaves, between 32 (below, the reduction of the
// partial sums is the longer part) and 512 (f32 sums).  With 512 rows always, a batch of a few thousand
// tokens ran on 8 workgroups: bf16, d = 4096, 2048 / 8192 / 16384 / 65536 tokens took 50 / 51 / 52 / 78 us;
// 12 / 15 / 24 / 78 us with this rule (4.4, 5.7 and 6.9 TB/s for the last three).
// A workspace with room for fewer than that rule's blocks, but at least `blocks_fit` >= T / 512 of them, gets
// longer ones.
static int64_t input_rows_per_block(int64_t T, int64_t d, int64_t blocks_fit)
{
    const int64_t waves = (d / 8 + 63) / 64;   // of a row, bf16
    const int64_t rule = (T * waves + 1023) / 1024, room = (T + blocks_fit - 1) / blocks_fit;
    const int64_t rows = ((rule > room ? rule : room) + kInUnroll - 1) / kInUnroll * kInUnroll;
    return rows < 32 ? 32 : rows > kInMaxRows ? kInMaxRows : rows;
}

// The most row blocks that input_rows_per_block() makes of T or fewer tokens when it has the room:
// blocks of 32 rows up to 1024 wavefronts, then 1024 wavefronts, then blocks of 512 rows.  It does not
// decrease in T, so that a workspace for the longest chunk of a stream serves the shorter ones.
static int64_t input_most_blocks(int64_t T, int64_t d)
{
    const int64_t waves = (d / 8 + 63) / 64;
    const int64_t small = (T + 31) / 32, full = (1024 + waves - 1) / (waves > 0 ? waves : 1), large = (T + kInMaxRows - 1) / kInMaxRows;
    const int64_t blocks = small < full ? small : full;
    return blocks > large ? blocks : large;
}

// Few tokens take input_strip_kernel: its workgroups read 64 bytes of every row, so there is no second
// launch to wait for, but its time grows with T whatever d is, and with the rounds of workgroups that a long
// row takes.  us a call, strips against row blocks: bf16, 4096 tokens 6.8 and 9.8 (d = 1024), 7.3 and 10.6
// (2048), 17.6 and 11.3 (4096); 2048 tokens 6.6 and 10.3 (4096), 11.8 and 10.8 (8192); f32, 2048 tokens 10.8
// and 10.5 (4096), 63.6 and 42.2 (28672), 1024 tokens 6.7 and 10.1 (5120), 11.1 and 11.2 (8192).  The two
// meet at 24 to 32 MB of X.
static bool input_by_strips(int64_t T, int64_t row_bytes)
{
    return (T <= 2048 || (T <= 4096 && row_bytes <= 4096)) && row_bytes <= (24LL << 20) / T;
}

}  // namespace dass

extern "C" size_t dass_input_norms_workspace_bytes(int64_t T, int64_t d)
{
    if (T <= 0 || d <= 0)
        return 0;
    return dass::round_up((size_t)dass::input_most_blocks(T, d) * (size_t)d * sizeof(float), 256);
}

extern "C" dass_status dass_input_norms(const void *X, int64_t T, int64_t ldx, int64_t d, dass_dtype dt,
                                        float *sumsq, int accumulate, float *norms_out, void *workspace,
                                        size_t workspace_bytes, void *hip_stream)
{
    using namespace dass;
    const char *fn = "dass_input_norms";
    if (!X || !sumsq)
        return fail(DASS_ERR_NULL, "%s: X and sumsq must not be NULL", fn);
    if (!valid_dtype(dt))
        return fail(DASS_ERR_DTYPE, "%s: unknown dtype %d", fn, (int)dt);
    if (T <= 0 || d <= 0)
        return fail(DASS_ERR_SHAPE, "%s: T=%lld d=%lld must be positive", fn, (long long)T, (long long)d);
    if (ldx < d)
        return fail(DASS_ERR_SHAPE, "%s: ldx=%lld smaller than d=%lld", fn, (long long)ldx, (long long)d);
    if (d % 8 != 0)
        return fail(DASS_ERR_SHAPE, "%s: d=%lld must be a multiple of 8", fn, (long long)d);
    if (!aligned16(X) || !aligned16(sumsq) || (norms_out && !aligned16(norms_out)))
        return fail(DASS_ERR_ALIGN, "%s: X, sumsq and norms_out must be 16-byte aligned", fn);
    if (ldx % vec_elems(dt) != 0)
        return fail(DASS_ERR_ALIGN, "%s: ldx=%lld must be a multiple of %d elements", fn, (long long)ldx,
                    vec_elems(dt));
    // partial sums of blocks of 512 rows have to fit; room for more of them only makes the call faster
    const size_t need = round_up((size_t)((T + kInMaxRows - 1) / kInMaxRows) * (size_t)d * sizeof(float), 256);
    if (!workspace || workspace_bytes < need)
        return fail(DASS_ERR_WORKSPACE, "%s: workspace of %zu bytes needed, %zu given", fn, need,
                    workspace ? workspace_bytes : (size_t)0);
    if (!aligned16(workspace))
        return fail(DASS_ERR_ALIGN, "%s: workspace must be 16-byte aligned", fn);

    const int64_t rows = input_rows_per_block(T, d, (int64_t)(workspace_bytes / ((size_t)d * sizeof(float))));
    const int64_t n_row_blocks = (T + rows - 1) / rows;
    const int64_t slots = d / vec_elems(dt);
    const int64_t nbx = (slots + kInBlock - 1) / kInBlock;
    if (nbx * n_row_blocks > 0x7fffffffLL)
        return fail(DASS_ERR_SHAPE, "%s: too many tokens for one launch; split them", fn);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (input_by_strips(T, d * elem_bytes(dt))) {
        const int64_t n_strips = (slots + kStripSlots - 1) / kStripSlots;
        const unsigned grid = (unsigned)((n_strips + 15) / 16 * 16);
        if (dt == DASS_BF16)
            hipLaunchKernelGGL(input_strip_kernel<DASS_BF16>, dim3(grid), dim3(kStripThreads), 0, stream, X, T, ldx, d,
                               sumsq, accumulate, norms_out);
        else
            hipLaunchKernelGGL(input_strip_kernel<DASS_F32>, dim3(grid), dim3(kStripThreads), 0, stream, X, T, ldx, d,
                               sumsq, accumulate, norms_out);
        return check_launch("input-norm kernel");
    }
    float *partial = static_cast<float *>(workspace);
    if (dt == DASS_BF16)
        hipLaunchKernelGGL(input_partial_kernel<DASS_BF16>, dim3((unsigned)(nbx * n_row_blocks)), dim3(kInBlock), 0,
                           stream, X, T, ldx, d, rows, partial);
    else
        hipLaunchKernelGGL(input_partial_kernel<DASS_F32>, dim3((unsigned)(nbx * n_row_blocks)), dim3(kInBlock), 0,
                           stream, X, T, ldx, d, rows, partial);
    dass_status s = check_launch("input-norm kernel");
    if (s != DASS_OK)
        return s;
    for (int64_t j0 = 0; j0 < d; j0 += kReduceCols) {
        const int64_t n = d - j0 < kReduceCols ? d - j0 : kReduceCols;
        hipLaunchKernelGGL(input_reduce_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64 * kReduceWaves), 0, stream,
                           (const float *)partial, n_row_blocks, d, j0, sumsq, accumulate, norms_out);
        s = check_launch("input-norm reduction");
        if (s != DASS_OK)
            return s;
    }
    return DASS_OK;
}
