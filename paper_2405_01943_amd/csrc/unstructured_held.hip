// Stage 2, unstructured, row lines: the phases of unstructured_rows.hip for matrices of few rows and lines of at most
// 4096 vectors, with the weights in registers between counting and writing: the matrix is read once, and nothing
// waits for 44 KB of factors to be in LDS.  A workgroup owns 4 rows; a thread owns the same J column slots of 16 bytes
// in each of them (slots tid, tid + blockDim, ..; the host makes blockDim J just cover the line).  A slot's factors are
// then read once for 4 rows, straight from the norms into registers, and a row's window and threshold are the same for
// the whole workgroup: scalar registers.  What bounds it is the chain of the phases, with 2 to 16 wavefronts a workgroup:
// 1024 x 5400 bf16 25 -> 21 us a call with the copy of the dense weights, 768 x 14336 50 -> 38, 333 x 16000 f32 48 -> 35.
// Four slots take all of the 128 registers that 16 wavefronts leave each: bf16 keeps 8 of a thread's values in scratch, f32
// with a mask 2 (64 x 32768 bf16 is 57 us all the same, read twice 84).
// (The window, the bin and the ranking stand here and in rowlines_kernel, whose compiled form was 2 to 3 us slower on
// 4096 x 11008 when it called the functions below.  Both texts have to select the same bins: a change to one is made to
// both, and a test runs the same rows through the two kernels.)
#include "unstructured_rows.h"

#include <type_traits>

namespace dass {
namespace rowl {

// The same value, as far as the compiler knows another one: what is computed from it is computed again.
__device__ __forceinline__ uint32_t again(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// LDS accesses before it are done; global ones may be in flight.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The window of a line from its 128 samples, two a lane.
__device__ __forceinline__ Window window_of(uint32_t s0, uint32_t s1, uint32_t n_keep, uint32_t len)
{
    // Ranks (from the top) of the two order statistics: the wanted quantile of the sample give or
    // take six standard deviations of the sampled count above the threshold, and one more.
    const float phi = (float)n_keep / (float)len;
    const float mid = phi * kSamples, dev = 6.0f * sqrtf(kSamples * phi * (1.0f - phi)) + 1.0f;
    const int r_hi = (int)floorf(mid - dev), r_lo = (int)ceilf(mid + dev);
    // the r-th largest sample, cut to its bits 30 .. 19: the largest T with r samples >= T
    auto order_stat = [&](int r) {
        uint32_t t = 0;
        for (int bit = 30; bit >= 19; --bit) {
            const uint32_t trial = t | (1u << bit);
            const int n = __popcll(__ballot(s0 >= trial)) + __popcll(__ballot(s1 >= trial));
            if (n >= r)
                t = trial;
        }
        return t;
    };
    // an end beyond the sample: the sample's extreme serves if the chance that the threshold lies
    // beyond it, phi^128 or (1 - phi)^128, is below 1e-9; else the window is open at that end
    const bool lo_open = r_lo > kSamples && phi > 0.85f, hi_open = r_hi < 1 && phi < 0.15f;
    const uint32_t lo = lo_open ? 0u : order_stat(r_lo <= kSamples ? r_lo : kSamples);
    const uint32_t hi = hi_open ? kInfBits - 1u : (order_stat(r_hi >= 1 ? r_hi : 1) | 0x7ffffu);
    const int width = 32 - __clz((int)(hi - lo) | 1);
    return Window{lo, (uint32_t)(width > 8 ? width - 8 : 0)};
}

// The bin of a row that holds the n_keep-th largest score: the lane whose `out` says so, or -1 if it is outside the
// window or holds more than a list does.  Lane l owns bins 255 - 4 l .. 252 - 4 l, a prefix sum over the lanes counts
// from the top.
__device__ __forceinline__ int bin_of(const uint32_t *h_row, const Window w, uint32_t n_keep, Select &out)
{
    const int lane = threadIdx.x & 63;
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        h[j] = h_row[255 - 4 * lane - j];
    uint32_t above = h_row[kAbove + lane];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        above += __shfl_xor(above, o, 64);
    const uint32_t sum = h[0] + h[1] + h[2] + h[3];
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= o)
            incl += t;
    }
    uint32_t excl = incl - sum;
    bool found = false;
    uint32_t bin = 0, need = 0, inside = 0;
    if (n_keep > above) {
        const uint32_t want = n_keep - above;
        if (excl < want && want <= incl) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!found && want <= excl + h[j]) {
                    found = true;
                    bin = 255 - 4 * lane - j;
                    need = want - excl;
                    inside = h[j];
                }
                excl += h[j];
            }
        }
    }
    const uint64_t who = __ballot(found);
    if (who == 0 || __shfl(inside, __ffsll((long long)who) - 1, 64) > (uint32_t)kCap)
        return -1;
    const uint32_t lo = w.lo + (bin << w.sh);
    out = need == inside ? Select{lo, 0, 0, 0} : Select{lo, 1u << w.sh, need, inside};
    return __ffsll((long long)who) - 1;
}

// Ranks a row's list with one wavefront; an entry with `need` or more entries above it is pruned after all.
template <int DT, bool MASK>
__device__ __forceinline__ void rank_list(const uint32_t *mine_list, uint32_t listed, uint32_t need, char *row,
                                          uint32_t row_index, uint32_t cols, uint8_t *__restrict__ mask)
{
    const int lane = threadIdx.x & 63;
    const uint32_t n = __builtin_amdgcn_readfirstlane(listed < (uint32_t)kCap ? listed : (uint32_t)kCap);
    need = __builtin_amdgcn_readfirstlane(need);
    uint32_t ma[kCap / 64], mb[kCap / 64], mc[kCap / 64];
    uint64_t key[kCap / 64];
#pragma unroll
    for (int j = 0; j < kCap / 64; ++j) {
        const uint32_t k = lane + 64 * j;
        ma[j] = k < n ? mine_list[k * 3] : 0u;
        mb[j] = k < n ? mine_list[k * 3 + 1] : 0u;
        mc[j] = k < n ? mine_list[k * 3 + 2] : 0u;
        key[j] = (uint64_t)ma[j] << 32 | mb[j];
    }
    uint32_t above[kCap / 64] = {0, 0, 0, 0};
    const int slots = (int)((n + 63) / 64);
#pragma unroll
    for (int src = 0; src < kCap / 64; ++src) {
        if (src >= slots)
            break;
        const int in_slot = (int)n - 64 * src < 64 ? (int)n - 64 * src : 64;
        for (int k = 0; k < in_slot; ++k) {
            const uint64_t o = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)ma[src], k) << 32 |
                               (uint32_t)__builtin_amdgcn_readlane((int)mb[src], k);
            const uint32_t oc = (uint32_t)__builtin_amdgcn_readlane((int)mc[src], k);
#pragma unroll
            for (int j = 0; j < kCap / 64; ++j)
                if (j < slots)
                    above[j] += (o > key[j]) | ((o == key[j]) & (oc > mc[j]));
        }
    }
#pragma unroll
    for (int j = 0; j < kCap / 64; ++j) {
        if (lane + 64 * j < n && above[j] >= need) {
            const uint32_t c = 0xFFFFu - mc[j];
            if constexpr (DT == DASS_BF16)
                *reinterpret_cast<uint16_t *>(row + c * 2) = 0;
            else
                *reinterpret_cast<uint32_t *>(row + c * 4) = 0;
            if constexpr (MASK) {
                const size_t byte = (size_t)row_index * (cols / 8) + c / 8;
                atomicAnd(reinterpret_cast<uint32_t *>(mask) + byte / 4, ~(1u << ((byte % 4) * 8 + c % 8)));
            }
        }
    }
}

constexpr int kHeldRows = 4;

// EARLY: the rows are left to the next launch as soon as their samples or a factor say that they will be, before any of
// their weights is requested.  bf16, half of the weights 0, alpha 0.75, mean of eight matrices a size, us: weights
// requested first, behind the decision, and rowlines_kernel: 768 x 8000 148 147 158, 256 x 16384 135 133 135, 512 x 28672
// 345 339 328, 64 x 32768 201 196 197, 1024 x 4096 107 105 113.  (Whether a block's samples lie beyond the two deviations
// is chance, and one block that stays costs all its phases: single matrices differ by 30 % either way.)
template <int DT, int J, bool MASK, bool EARLY>
__global__ __launch_bounds__(kThreads) void held_rows_kernel(void *__restrict__ Wv, uint32_t rows, uint32_t cols, int64_t ld,
                                                             const float *__restrict__ norms, int fmode, uint32_t n_keep,
                                                             uint8_t *__restrict__ mask, uint8_t *__restrict__ todo,
                                                             const uint8_t *__restrict__ out_of_range)
{
    constexpr int EPV = DT == DASS_BF16 ? 8 : 4;
    constexpr int EB = DT == DASS_BF16 ? 2 : 4;
    constexpr int R = kHeldRows;
    __shared__ uint32_t hist[R * kStride];
    __shared__ uint32_t list[R * kCap * 3];
    __shared__ uint32_t cnt[R];
    __shared__ Window win[R];
    __shared__ Select sel[R];
    __shared__ uint32_t fail, zeros;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = blockDim.x, waves = nt / 64;
    const uint32_t row0 = blockIdx.x * R;
    const uint32_t n_rows = rows - row0 < (uint32_t)R ? rows - row0 : (uint32_t)R;
    char *W = static_cast<char *>(Wv) + (size_t)row0 * ld * EB;
    const uint32_t row_bytes = (uint32_t)ld * EB;   // the block's rows span less than 4 GB (host check)
    const uint32_t vpl = cols / EPV;
    auto mark = [&](bool left) {   // a byte of the block's word for every two rows
        if (tid < (R + 1) / 2)
            todo[row0 / 2 + tid] = left;
    };
    if (row0 >= rows) {   // the rest of the last word
        mark(false);
        return;
    }

    // ---- requests, in the order in which they are wanted: samples, factors, weights (EARLY: behind phase A).  A row or
    // slot past the end takes the last one: a load behind a branch could not be counted, and nothing is done with it.
    // rows a wavefront samples: there are two wavefronts or more, R or more with J > 1
    constexpr int S = J == 1 ? (R + 1) / 2 : 1;
    float smp_w[S][2], smp_n[2];
    const uint32_t smp_c = sample_run(lane / 4, cols) + 2 * (lane % 4);   // lane l: columns 2 (l % 4), + 1 of run l / 4
    {
        const float2 n2 = *reinterpret_cast<const float2 *>(norms + smp_c);
        smp_n[0] = n2.x;
        smp_n[1] = n2.y;
    }
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const uint32_t r = wave + k * waves;   // uniform
        smp_w[k][0] = smp_w[k][1] = 0.0f;
        if (r < n_rows) {
            if constexpr (DT == DASS_BF16) {
                const uint32_t two = *reinterpret_cast<const uint32_t *>(W + r * row_bytes + smp_c * 2);
                smp_w[k][0] = __uint_as_float(two << 16);
                smp_w[k][1] = __uint_as_float(two & 0xffff0000u);
            } else {
                const float2 two = *reinterpret_cast<const float2 *>(W + r * row_bytes + smp_c * 4);
                smp_w[k][0] = two.x;
                smp_w[k][1] = two.y;
            }
        }
    }
    uint32_t slot[J];
    float f[J][EPV];
    u32x4 x[J][R];
    auto request = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t cv = tid + j * nt;
            slot[j] = cv < vpl ? cv : vpl - 1;
        }
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int q = 0; q < EPV / 4; ++q) {
                const u32x4 n4 = *reinterpret_cast<const u32x4 *>(norms + slot[j] * EPV + 4 * q);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    f[j][4 * q + i] = __uint_as_float(n4[i]);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int r = 0; r < R; ++r)
                x[j][r] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4 *>(W + (r < (int)n_rows ? r : (int)n_rows - 1) * row_bytes + slot[j] * 16));
        __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (!EARLY)
        request();

    bool leave = false;   // EARLY: the rows are left to the next launch
    if constexpr (EARLY)
        for (uint32_t i = tid; i * kFactorBlock < cols; i += nt)
            leave |= out_of_range[i] != 0;

    // ---- 0: counters cleared
    for (int i = tid; i < R * kStride; i += nt)
        hist[i] = 0;
    if (tid < R)
        cnt[tid] = 0;
    if (tid == 0)
        fail = zeros = 0;
    lds_barrier();

    // ---- A: the rows' windows, one wavefront per row (rowlines_kernel has the reasons)
#pragma unroll
    for (int k = 0; k < S; ++k) {
        const uint32_t r = wave + k * waves;
        if (r >= n_rows)
            break;   // uniform
        uint32_t s[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            s[q] = __float_as_uint(fabsf(smp_w[k][q]) * (factor_of(smp_n[q], fmode) * kFactorScale));
        if constexpr (EARLY) {
            const int n = __popcll(__ballot(s[0] == 0)) + __popcll(__ballot(s[1] == 0));
            if (lane == 0)
                atomicAdd(&zeros, (uint32_t)n);
        }
        const Window w = window_of(s[0], s[1], n_keep, cols);
        if (lane == 0)
            win[r] = w;
    }
    lds_barrier();
    if constexpr (EARLY) {
        const float taken = (float)(n_rows * kSamples), pruned = (float)(cols - n_keep) / (float)cols;
        leave |= (float)zeros >= taken * pruned - 2.0f * sqrtf(taken * pruned * (1.0f - pruned));
        if (__syncthreads_or(leave)) {
            mark(true);
            return;
        }
        request();
    }

    // ---- B: counts
    uint32_t a_max = 0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < J; ++j) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const float u = factor_of(f[j][e], fmode);
            bad |= !factor_in_fast_range(u);
            f[j][e] = u * kFactorScale;
        }
        const bool in = tid + j * nt < (int)vpl;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const Window w = {(uint32_t)__builtin_amdgcn_readfirstlane(win[r].lo),
                              (uint32_t)__builtin_amdgcn_readfirstlane(win[r].sh)};
            __builtin_amdgcn_sched_barrier(0);
            if (in && r < (int)n_rows) {
                uint32_t *const mine = hist + r * kStride;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const uint32_t a = __float_as_uint(fabsf(elem_of<DT>(x[j][r], e)) * f[j][e]);
                    a_max = a > a_max ? a : a_max;
                    int bin = (int)(a - w.lo) >> w.sh;   // negative below the window, 256 or more above it
                    bin = bin < 0 ? kBelow + lane : bin >= kBins ? kAbove + lane : bin;
                    atomicAdd(mine + bin, 1u);
                }
            }
        }
    }
    if (bad || a_max >= kInfBits)   // a factor outside the range of the two-term score, a product that overflowed
        fail = 1;
    lds_barrier();

    // ---- C: each row's bin
    for (uint32_t r = wave; r < n_rows; r += waves) {
        Select t;
        const int found = bin_of(hist + r * kStride, win[r], n_keep, t);
        if (found < 0) {
            if (lane == 0)
                fail = 1;   // threshold outside the window, or more scores in its bin than the list holds
        } else if (lane == found) {
            sel[r] = t;
        }
    }
    lds_barrier();
    if (fail) {   // uniform: the rows stay as they are for the launch that follows
        mark(true);
        return;
    }

    // ---- D: apply and list
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const bool in = tid + j * nt < (int)vpl;
        // the factors again, rather than kept: the registers decide how many workgroups share a compute unit
        float f[EPV];
#pragma unroll
        for (int q = 0; q < EPV / 4; ++q) {
            const u32x4 n4 = *reinterpret_cast<const u32x4 *>(norms + again(slot[j]) * EPV + 4 * q);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                f[4 * q + i] = factor_of(__uint_as_float(n4[i]), fmode) * kFactorScale;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t lo = __builtin_amdgcn_readfirstlane(sel[r].lo);
            const uint32_t width = __builtin_amdgcn_readfirstlane(sel[r].width);
            __builtin_amdgcn_sched_barrier(0);
            const bool live = in && r < (int)n_rows;
            uint32_t kept = 0;
            if (live) {
                uint32_t d[EPV];
                int32_t gone[EPV];
                bool hit = false;
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    d[e] = __float_as_uint(fabsf(elem_of<DT>(x[j][r], e)) * f[e]) - lo;   // negative: pruned
                    hit |= d[e] < width;
                    gone[e] = (int32_t)d[e] >> 31;
                    if constexpr (MASK)
                        kept |= (uint32_t)(~gone[e] & 1) << e;
                }
                if (hit) {   // rarely entered: a few dozen scores per row
                    uint32_t hits = 0;
#pragma unroll
                    for (int e = 0; e < EPV; ++e)
                        hits |= (d[e] < width ? 1u : 0u) << e;
                    while (hits) {
                        const int e = __ffs((int)hits) - 1;
                        hits &= hits - 1;
                        float w = 0.0f, fe = 0.0f;
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            w = k == e ? fabsf(elem_of<DT>(x[j][r], k)) : w;
                            fe = k == e ? f[k] : fe;
                        }
                        const float p = w * fe;
                        const uint32_t at = atomicAdd(&cnt[r], 1u);
                        if (at < (uint32_t)kCap) {
                            uint32_t *entry = list + (r * kCap + at) * 3;
                            entry[0] = __float_as_uint(p);
                            entry[1] = mono(fmaf(w, fe, -p));
                            entry[2] = 0xFFFFu - (slot[j] * EPV + e);
                        }
                    }
                }
                u32x4 y = x[j][r];
                if constexpr (DT == DASS_BF16) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        y[k] &= ~(((uint32_t)gone[2 * k] & 0xffffu) | ((uint32_t)gone[2 * k + 1] & 0xffff0000u));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        y[k] &= ~(uint32_t)gone[k];
                }
                __builtin_nontemporal_store(y, reinterpret_cast<u32x4 *>(W + r * row_bytes + slot[j] * 16));
            }
            if constexpr (MASK) {
                if constexpr (EPV == 8) {
                    if (live)
                        mask[(size_t)(row0 + r) * (cols / 8) + slot[j]] = (uint8_t)kept;
                } else {
                    // f32: a mask byte covers two neighbouring lanes' vectors (vpl is even, the two share every branch)
                    const uint32_t other = __shfl_xor(kept, 1, 64);
                    if (live && (slot[j] & 1) == 0)
                        mask[(size_t)(row0 + r) * (cols / 8) + slot[j] / 2] = (uint8_t)(kept | other << 4);
                }
            }
        }
    }
    // the single stores of E go to lines written just above by other wavefronts of this workgroup: rowlines_kernel
    __syncthreads();

    // ---- E: rank each row's list
    bool short_list = false;
    for (uint32_t r = wave; r < n_rows; r += waves) {
        if (sel[r].width == 0)
            continue;   // uniform
        short_list |= cnt[r] != sel[r].inside;   // ruled out by identical arithmetic in B and D; checked all the same
        rank_list<DT, MASK>(list + r * kCap * 3, cnt[r], sel[r].need, W + r * row_bytes, row0 + r, cols, mask);
    }
    // A short list leaves only weights below the threshold zeroed: redoing the rows selects the same set.
    mark(__syncthreads_or(short_list));
}

}  // namespace rowl

dass_status launch_held_rows(const RowlinesPlan &p, void *W, int64_t rows, int64_t cols, int64_t ld, int dt, const float *norms,
                             int fmode, uint32_t n_keep, uint8_t *mask_out, uint32_t *todo, const uint8_t *out_of_range,
                             hipStream_t stream)
{
    using namespace rowl;
    const bool bf16 = dt == DASS_BF16;
    auto held = [&](auto dt_tag, auto mask_tag, auto early_tag) {
        constexpr int D = decltype(dt_tag)::value;
        constexpr bool M = decltype(mask_tag)::value, E = decltype(early_tag)::value;
        return p.held_slots == 4   ? held_rows_kernel<D, 4, M, E>
               : p.held_slots == 2 ? held_rows_kernel<D, 2, M, E>
                                   : held_rows_kernel<D, 1, M, E>;
    };
    auto pick = [&](auto early_tag) {
        using Bf16 = std::integral_constant<int, DASS_BF16>;
        using F32 = std::integral_constant<int, DASS_F32>;
        return bf16 ? (mask_out ? held(Bf16{}, std::true_type{}, early_tag) : held(Bf16{}, std::false_type{}, early_tag))
                    : (mask_out ? held(F32{}, std::true_type{}, early_tag) : held(F32{}, std::false_type{}, early_tag));
    };
    auto hk = out_of_range ? pick(std::true_type{}) : pick(std::false_type{});
    const int64_t slots = cols / vec_elems(dt), threads = ((slots + p.held_slots - 1) / p.held_slots + 63) / 64 * 64;
    hipLaunchKernelGGL(hk, dim3((unsigned)(p.blocks * (kRows / kHeldRows))), dim3((unsigned)threads), 0, stream, W,
                       (uint32_t)rows, (uint32_t)cols, ld, norms, fmode, n_keep, mask_out,
                       reinterpret_cast<uint8_t *>(todo), out_of_range);
    return check_launch("row-line unstructured kernel");
}

}  // namespace dass
