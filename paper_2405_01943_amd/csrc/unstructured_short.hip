// Unstructured selection on short lines, of at most 2048 weights (Sec. 3 "Pruning Granularity"): one wavefront
// per line, the whole line's scores in its registers.
//
// What bounds such calls is not memory (a 688 x 256 matrix is 0.7 MB) but the chain of dependent steps.
// The workgroup-wide radix select of unstructured.hip clears, fills and scans 64 KB of histograms twice
// behind a dozen barriers; here the threshold is found bit by bit, most significant first, and a bit costs
// a compare and an add per 64 scores and one cross-lane sum: no histogram, no atomics, no barrier, and the
// search ends at the first bit at which the count is the wanted one (about 20 of 31 bits).  Ties at the
// threshold go on with the error terms and then the indexes in the same way.
// Three matrices a call each, copies of the dense weights and the host's calls included, against the
// workgroup-wide kernel: f32 256 x 688 with mask 63 -> 34 us; bf16 8192 x 1000 261 -> 125 (before the loads of
// short_cols_kernel went out at once).  A bit's cost grows
// with the line: at 4096 the other kernels are ahead (256 x 4096 112 -> 144, 4096 x 4096 161 -> 425).  Which
// lines come here is decided in unstructured.hip.
//
// Order of positions: (A, B, 0xFFFF - index) as in unstructured.hip, A and B the two-term f32 score or, in a
// line with a factor or product outside its range, the two words of the f64 product.
#include "select.h"
#include "unstructured_tiled.h"

#include <type_traits>

namespace dass {
namespace shortl {

constexpr int kMaxLine = 2048, kWords = kMaxLine / 64;

__device__ __forceinline__ uint32_t mono(float q)   // unsigned integer that grows with q
{
    const uint32_t b = __float_as_uint(q);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}

// Sum over the 64 lanes, on every lane: an inclusive scan inside the rows of 16 lanes, then across them.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// How many of the wavefront's x[k] are >= t.  Counted per lane and then added up: a population count of
// the compare's lane mask per score makes the scalar unit wait for every compare (4096 weights: 3 x slower).
template <int E>
__device__ __forceinline__ uint32_t count_from(const uint32_t (&x)[E], uint32_t t)
{
    uint32_t c[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < E; ++k)
        c[k % 4] += x[k] >= t ? 1u : 0u;
    return wave_sum((c[0] + c[1]) + (c[2] + c[3]));
}

// Largest t of `bits` bits with at least `need` of the wavefront's x[k] >= t, and how many those are;
// stops at the first t with exactly `need` (then x >= t is the wanted set).  need >= 1.
template <int E>
__device__ __forceinline__ uint32_t search(const uint32_t (&x)[E], uint32_t need, int bits, uint32_t &at_or_above)
{
    uint32_t t = 0;
    at_or_above = 64 * E;
    for (int b = bits - 1; b >= 0 && at_or_above != need; --b) {   // uniform
        const uint32_t trial = t | (1u << b);
        const uint32_t c = count_from(x, trial);
        if (c >= need) {
            t = trial;
            at_or_above = c;
        }
    }
    return t;
}

// Bit k of the result: the lane's k-th position is kept.  weight(k) is |w|, factor(k) the unscaled factor,
// index(k) the position in the line, valid(k) whether there is one.  0 < n_keep < the line's length.
template <int E, typename Weight, typename Factor, typename Index, typename Valid>
__device__ __forceinline__ uint32_t keep_bits(uint32_t n_keep, Weight weight, Factor factor, Index index, Valid valid)
{
    // positions beyond the line hold 0 in every field: no trial threshold (>= 1) counts them
    uint32_t a[E];
    bool fast = true;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const float f = factor(k);
        const uint32_t p = __float_as_uint(weight(k) * (f * kFactorScale));
        a[k] = valid(k) ? p : 0u;
        fast &= !valid(k) | (factor_in_fast_range(f) & (p < 0x7f800000u));
    }
    const bool exact = __ballot(!fast) != 0;
    if (exact) {   // f64 products (uniform)
#pragma unroll
        for (int k = 0; k < E; ++k)
            a[k] = valid(k) ? (uint32_t)((uint64_t)__double_as_longlong((double)weight(k) * (double)factor(k)) >> 32) : 0u;
    }
    uint32_t n;
    const uint32_t ta = search<E>(a, n_keep, 32, n);
    uint32_t kept = 0;
    if (n == n_keep) {
#pragma unroll
        for (int k = 0; k < E; ++k)
            kept |= (uint32_t)(a[k] >= ta) << k;
        return kept;
    }
    // equal leading terms at the threshold: the error terms decide, then the lower index
    uint32_t need = n_keep - count_from(a, ta + 1);   // ta < 0xffffffff: a finite score's word
    uint32_t b[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        uint32_t v;
        if (exact) {
            v = (uint32_t)(uint64_t)__double_as_longlong((double)weight(k) * (double)factor(k));
        } else {
            const float w = weight(k), fs = factor(k) * kFactorScale;
            v = mono(fmaf(w, fs, -(w * fs)));
        }
        b[k] = valid(k) && a[k] == ta ? v : 0u;
    }
    const uint32_t tb = search<E>(b, need, 32, n);
    if (tb != 0xffffffffu)   // a low word may be all ones
        need -= count_from(b, tb + 1);
    uint32_t c[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        c[k] = valid(k) && a[k] == ta && b[k] == tb ? 0xFFFFu - index(k) : 0u;
    }
    const uint32_t tc = search<E>(c, need, 16, n);   // n == need: indexes differ
#pragma unroll
    for (int k = 0; k < E; ++k)
        kept |= (uint32_t)((a[k] > ta) | ((a[k] == ta) & ((b[k] > tb) | ((b[k] == tb) & (c[k] >= tc))))) << k;
    return kept;
}

// Lines are rows: a workgroup is one wavefront, lane l holds vectors l, l + 64, ... of its row.
template <int DT, int E>
__global__ __launch_bounds__(64) void short_rows_kernel(void *__restrict__ Wv, int64_t cols, int64_t ld,
                                                        const float *__restrict__ norms, int fmode, int along,
                                                        uint32_t n_keep, uint8_t *__restrict__ mask)
{
    constexpr int EPV = DT == DASS_BF16 ? 8 : 4, EB = DT == DASS_BF16 ? 2 : 4, V = E / EPV;
    const int64_t row = blockIdx.x;
    const int lane = threadIdx.x;
    const int n_vec = (int)(cols / EPV);
    char *W = static_cast<char *>(Wv) + row * ld * EB;
    u32x4 x[V];
    float f[E];   // dead once the scores are there, unless the line ties or leaves the two-term range
    const float f_row = along ? 0.0f : factor_of(norms[row], fmode);
#pragma unroll
    for (int j = 0; j < V; ++j) {
        // beyond the line its last vector: a load behind a branch would be waited for on its own
        const int v = lane + 64 * j < n_vec ? lane + 64 * j : n_vec - 1;
        x[j] = *reinterpret_cast<const u32x4 *>(W + (int64_t)v * 16);
#pragma unroll
        for (int q = 0; q < EPV / 4; ++q) {
            u32x4 n = {0, 0, 0, 0};
            if (along)   // uniform
                n = *reinterpret_cast<const u32x4 *>(norms + v * EPV + 4 * q);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                f[j * EPV + 4 * q + i] = along ? factor_of(__uint_as_float(n[i]), fmode) : f_row;
        }
    }
    const uint32_t kept = keep_bits<E>(
        n_keep, [&](int k) { return fabsf(elem_of<DT>(x[k / EPV], k % EPV)); }, [&](int k) { return f[k]; },
        [&](int k) { return (uint32_t)((lane + 64 * (k / EPV)) * EPV + k % EPV); },
        [&](int k) { return lane + 64 * (k / EPV) < n_vec; });
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int v = lane + 64 * j;
        const uint32_t bits = (kept >> (j * EPV)) & ((1u << EPV) - 1);
        const uint32_t next = EPV == 4 ? __shfl_xor(bits, 1, 64) : 0u;   // n_vec is even with f32: cols is a multiple of 8
        if (v < n_vec) {
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                zero_lane_if<DT>(x[j], e, !((bits >> e) & 1));
            *reinterpret_cast<u32x4 *>(W + (int64_t)v * 16) = x[j];
            if (mask) {
                if constexpr (EPV == 8)
                    mask[row * n_vec + v] = (uint8_t)bits;
                else if ((lane & 1) == 0)
                    mask[row * (cols / 8) + v / 2] = (uint8_t)(bits | next << 4);
            }
        }
    }
}

// Lines are columns: a workgroup of eight wavefronts takes 8 neighbouring columns through LDS, column by
// column there, so that a wavefront reads its own without bank conflicts and the global accesses stay
// 16 bytes a lane.  The 8 workgroups that share 64 columns run on one XCD, as in unstructured.hip.
// ALONG: a factor a position; else one a line, in one register.  Calls with one factor a line, from the norm behind the
// barrier, a copy of it a position, one register, us: f32 2048 x 8192 97 101 89, 1000 x 8192 37 38 31, 1000 x 1024 16 17
// 15; bf16 1000 x 8192 71 72 63.
template <int DT, int E, bool ALONG>
__global__ __launch_bounds__(512) void short_cols_kernel(void *__restrict__ Wv, int64_t rows, int64_t cols, int64_t ld,
                                                         const float *__restrict__ norms, int fmode, uint32_t n_keep,
                                                         uint8_t *__restrict__ mask)
{
    constexpr int EPV = DT == DASS_BF16 ? 8 : 4, EB = DT == DASS_BF16 ? 2 : 4, VR = 8 / EPV;
    using elem_t = std::conditional_t<DT == DASS_BF16, uint16_t, uint32_t>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint64_t *keepw = reinterpret_cast<uint64_t *>(smem);            // [8][kWords]: bit l of word k: row 64 k + l is kept
    elem_t *tile = reinterpret_cast<elem_t *>(smem + 8 * kWords * 8);   // [8][stride]
    const uint32_t slot = blockIdx.x / 8;
    const int64_t octet = (int64_t)((slot / 8) * 8 + blockIdx.x % 8) * 8 + slot % 8;
    if (octet >= cols / 8)
        return;   // uniform
    const int len = (int)rows, stride = (len + 15) / 16 * 16 + 8;
    char *W = static_cast<char *>(Wv) + octet * 8 * EB;
    const int tid = threadIdx.x, lane = tid & 63, col = tid >> 6;

    auto valid = [&](int k) { return lane + 64 * k < len; };
    // positions beyond the line read its last one: a load behind a branch would be waited for on its own
    auto place = [&](int k) { return valid(k) ? lane + 64 * k : len - 1; };
    // Norms and weights are all requested before anything is waited for: a matrix this small costs trips to memory, not
    // bytes.  Against a loop of loads and the norms behind the barrier, a call with mask: f32 688 x 256 21 -> 13 us, 1500 x
    // 512 24 -> 20.5, bf16 1000 x 8192 44 -> 37, 512 x 2048 17.6 -> 16.
    float f[ALONG ? E : 1];
#pragma unroll
    for (int k = 0; k < (ALONG ? E : 1); ++k)
        f[k] = norms[ALONG ? place(k) : octet * 8 + col];
    constexpr int NV = (64 * E * VR + 511) / 512;   // vectors of a thread
    u32x4 in[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int v = tid + 512 * q < len * VR ? tid + 512 * q : len * VR - 1;
        in[q] = *reinterpret_cast<const u32x4 *>(W + (int64_t)(v / VR) * ld * EB + (v % VR) * 16);
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int v = tid + 512 * q, r = v / VR, c = (v % VR) * EPV;
        if (v < len * VR) {
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                tile[(c + e) * stride + r] = DT == DASS_BF16 ? (elem_t)(in[q][e / 2] >> (16 * (e % 2))) : (elem_t)in[q][e % 4];
        }
    }
#pragma unroll
    for (int k = 0; k < (ALONG ? E : 1); ++k)
        f[k] = factor_of(f[k], fmode);
    __syncthreads();
    elem_t *mine = tile + col * stride;
    const uint32_t kept = keep_bits<E>(
        n_keep,
        [&](int k) {
            const uint32_t w = mine[place(k)];
            return fabsf(__uint_as_float(DT == DASS_BF16 ? w << 16 : w));
        },
        [&](int k) { return f[ALONG ? k : 0]; },
        [&](int k) { return (uint32_t)(lane + 64 * k); }, valid);
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const bool keep = (kept >> k) & 1;
        if (valid(k) && !keep)
            mine[lane + 64 * k] = 0;
        const uint64_t word = __ballot(keep);
        if (lane == 0)
            keepw[col * kWords + k] = word;
    }
    __syncthreads();
    for (int v = tid; v < len * VR; v += 512) {
        const int r = v / VR, c = (v % VR) * EPV;
        u32x4 x;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x[i] = DT == DASS_BF16 ? (uint32_t)tile[(c + 2 * i) * stride + r] | (uint32_t)tile[(c + 2 * i + 1) * stride + r] << 16
                                   : (uint32_t)tile[(c + i) * stride + r];
        *reinterpret_cast<u32x4 *>(W + (int64_t)r * ld * EB + c * EB) = x;
    }
    if (mask)
        for (int r = tid; r < len; r += 512) {
            uint32_t bits = 0;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                bits |= (uint32_t)(keepw[c * kWords + r / 64] >> (r % 64) & 1) << c;
            mask[(int64_t)r * (cols / 8) + octet] = (uint8_t)bits;
        }
}

struct Args {
    void *W;
    int64_t rows, cols, ld;
    const float *norms;
    int fmode, along;
    uint32_t n_keep;
    uint8_t *mask;
    hipStream_t stream;
};

template <int DT, int E>
static dass_status launch_e(const char *fn, bool col_lines, const Args &a)
{
    if (!col_lines) {
        hipLaunchKernelGGL((short_rows_kernel<DT, E>), dim3((unsigned)a.rows), dim3(64), 0, a.stream, a.W, a.cols, a.ld,
                           a.norms, a.fmode, a.along, a.n_keep, a.mask);
        return check_launch("short-line unstructured kernel");
    }
    auto lds_of = [](int64_t rows) { return 8 * kWords * 8 + 8 * (size_t)((rows + 15) / 16 * 16 + 8) * (DT == DASS_BF16 ? 2 : 4); };
    const size_t lds = lds_of(a.rows);
    // the same for every call: another thread may set it between this and the launch
    auto k = a.along ? short_cols_kernel<DT, E, true> : short_cols_kernel<DT, E, false>;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_of(64 * E)) != hipSuccess)
        return fail(DASS_ERR_HIP, "%s: cannot reserve %zu bytes of LDS", fn, lds_of(64 * E));
    hipLaunchKernelGGL(k, dim3((unsigned)((a.cols / 8 + 63) / 64 * 64)), dim3(512), lds, a.stream, a.W, a.rows, a.cols, a.ld,
                       a.norms, a.fmode, a.n_keep, a.mask);
    return check_launch("short-line unstructured kernel");
}

// per_lane: positions of a lane, at most 32
template <int DT>
static dass_status launch_dt(const char *fn, bool col_lines, int64_t per_lane, const Args &a)
{
    if (per_lane <= 8)
        return launch_e<DT, 8>(fn, col_lines, a);
    // Lines of 513 to 768 f32 weights, us with 16 positions a lane and with 12: down the rows 520 x 8192 32 26, 768 x 8192
    // 34 28, 688 x 2048 15 13, along them 640 x 4096 lines 18 15, 768 x 8192 lines 28 23.  (bf16 column lines gain as
    // much, 520 x 8192 31 26, and have no such instance; a bf16 row vector has 8 weights, 12 are no whole number.)
    if (DT == DASS_F32 && per_lane <= 12)
        return launch_e<DT, DT == DASS_F32 ? 12 : 16>(fn, col_lines, a);
    if (per_lane <= 16)
        return launch_e<DT, 16>(fn, col_lines, a);
    if (per_lane <= 24)
        return launch_e<DT, 24>(fn, col_lines, a);
    return launch_e<DT, 32>(fn, col_lines, a);
}

}  // namespace shortl

bool short_lines_fit(int64_t rows, int64_t cols, bool col_lines, int64_t longest)
{
    return (col_lines ? rows : cols) <= longest && longest <= shortl::kMaxLine && rows <= 0x7fffffffLL && cols / 8 <= 0x7fffff00LL;
}

dass_status launch_short_lines(const char *fn, void *W, int64_t rows, int64_t cols, int64_t ld, int dt, const float *norms,
                               bool col_lines, bool along, int fmode, uint32_t n_keep, uint8_t *mask_out,
                               hipStream_t stream)
{
    using namespace shortl;
    const Args a{W, rows, cols, ld, norms, fmode, along ? 1 : 0, n_keep, mask_out, stream};
    const int epv = vec_elems(dt);
    const int64_t per_lane = col_lines ? (rows + 63) / 64 : (cols / epv + 63) / 64 * epv;
    return dt == DASS_BF16 ? launch_dt<DASS_BF16>(fn, col_lines, per_lane, a) : launch_dt<DASS_F32>(fn, col_lines, per_lane, a);
}

}  // namespace dass
