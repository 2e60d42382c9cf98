// Device setup of the SELL-64 layout with column offsets shared per slice:
// one wavefront per slice builds the slice's sorted offset list and the
// rows' position masks, a scan places the lists, and a fill pass writes the
// values slice by slice.
//
// The passes read CSR once and are bound by that; a row is walked by one lane
// (its entries must be taken in order), so the 64 rows' entries, one
// contiguous CSR range, first go to LDS with coalesced loads.  Creating the
// 7-point 128^3 handle took 41.2 ms with the lists built on the host from a
// copy of the columns, 1.2 ms so (97 x 64 x 81: 8.1 -> 0.84 ms).
#pragma once

#include "spmv.hpp"

namespace spk {

// Totals over the slices, for the decision and the allocations.
struct SharedStats {
    unsigned long long shared;  // sum of the list lengths
    unsigned long long lane;    // sum of the longest rows
    int32_t widest;             // longest list
    int32_t bad;                // slices with over kSellSharedMax offsets, or rows not strictly ascending
};

constexpr int kSharedCap = kSell * kSellSharedMax;  // entries of a slice whose rows all fit

// Least value of a wavefront, in every lane.
__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
    return v;
}

__device__ __forceinline__ int wave_max(int v) { return -wave_min(-v); }

// A wave's own LDS writes before its reads of them.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Offset lists (kSellSharedMax slots per slice) and position masks.  Rows
// have at most kSellSharedMax entries (checked by the caller), so a slice has
// at most kSharedCap.  All lanes step through the merge of their rows'
// ascending offsets: the least offset not yet listed is appended, and the
// rows holding it set its bit and move on.
static __global__ __launch_bounds__(kBlock) void k_shared_lists(int n, const int32_t *__restrict__ rowptr,
                                                                const int32_t *__restrict__ col,
                                                                int32_t *__restrict__ width,
                                                                int32_t *__restrict__ list,
                                                                uint32_t *__restrict__ mask,
                                                                SharedStats *__restrict__ out)
{
    constexpr int kNone = 0x7fffffff;
    __shared__ int32_t stage[kBlock / kWave][kSharedCap];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int ns = (n + kSell - 1) / kSell;
    int32_t *sc = stage[w];
    unsigned long long shared = 0, longest = 0;
    int widest = 0, bad = 0;
    for (int s = blockIdx.x * (kBlock / kWave) + w; s < ns; s += gridDim.x * (kBlock / kWave)) {
        const int row = s * kSell + lane;
        const int base = rowptr[s * kSell], total = rowptr[min(n, (s + 1) * kSell)] - base;
        const int a = rowptr[min(row, n)] - base, e = rowptr[min(row + 1, n)] - base;
        wave_lds_sync();  // the previous slice's reads
        for (int i = lane; i < total; i += kWave) sc[i] = col[base + i];
        wave_lds_sync();
        int k = a, count = 0, wrong = 0;
        uint32_t m = 0;
        int cur = k < e ? sc[k] - row : kNone;
        for (;;) {
            const int least = wave_min(cur);
            if (least == kNone) break;
            if (count == kSellSharedMax) {
                wrong = 1;
                break;
            }
            if (cur == least) {
                m |= 1u << count;
                ++k;
                const int next = k < e ? sc[k] - row : kNone;
                if (next <= cur) wrong = 1;  // not ascending, or twice the same column
                cur = next;
            }
            if (lane == 0) list[(size_t)s * kSellSharedMax + count] = least;
            ++count;
            if (__any(wrong)) break;
        }
        if (row < n) mask[row] = m;
        if (lane == 0) width[s] = count;
        shared += count;
        longest += wave_max(e - a);
        widest = max(widest, count);
        bad += __any(wrong) ? 1 : 0;
    }
    __shared__ unsigned long long sh[2][kBlock / kWave];
    __shared__ int32_t si[2][kBlock / kWave];
    if (lane == 0) {
        sh[0][w] = shared;
        sh[1][w] = longest;
        si[0][w] = widest;
        si[1][w] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / kWave; ++i) {
            shared += sh[0][i];
            longest += sh[1][i];
            widest = max(widest, si[0][i]);
            bad += si[1][i];
        }
        atomicAdd(&out->shared, shared);
        atomicAdd(&out->lane, longest);
        atomicMax(&out->widest, widest);
        if (bad) atomicAdd(&out->bad, bad);
    }
}

// Slice s spans 64 width[s] elements from 64 base[s]; its offsets sit at
// element base[s] of the packed lists (base: the widths' exclusive scan).
static __global__ void k_shared_pack(int ns, const int32_t *__restrict__ base, const int32_t *__restrict__ list,
                                     int32_t *__restrict__ sptr, int32_t *__restrict__ offs)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = t / kSellSharedMax, i = t % kSellSharedMax;
    if (s > ns) return;
    const int b = base[s];
    if (i == 0) sptr[s] = kSell * b;
    if (s < ns && i < base[s + 1] - b) offs[b + i] = list[t];
}

// Shared-offset fill, one wavefront per slice: row i has the positions of
// the set bits of mask[i] in its slice's offset list, in column order; its
// k-th entry goes to the position of the k-th set bit, the other positions
// get zeros.
static __global__ __launch_bounds__(kBlock) void k_shared_fill(int n, const int32_t *__restrict__ rowptr,
                                                               const double *__restrict__ val,
                                                               const int32_t *__restrict__ sptr,
                                                               const uint32_t *__restrict__ mask,
                                                               double *__restrict__ sval)
{
    using DP = typename Pair2<double>::type;
    __shared__ double stage[kBlock / kWave][kSharedCap];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int ns = (n + kSell - 1) / kSell;
    double *sc = stage[w];
    for (int s = blockIdx.x * (kBlock / kWave) + w; s < ns; s += gridDim.x * (kBlock / kWave)) {
        const int row = s * kSell + lane;
        const int base = rowptr[s * kSell], total = rowptr[min(n, (s + 1) * kSell)] - base;
        const int b = sptr[s], slen = (sptr[s + 1] - b) / kSell;
        const uint32_t m = row < n ? mask[row] : 0u;
        int k = rowptr[min(row, n)] - base;
        wave_lds_sync();
        for (int i = lane; i < total; i += kWave) sc[i] = ld_stream(val + base + i);
        wave_lds_sync();
        auto take = [&](int j) { return (m >> j) & 1u ? sc[k++] : 0.0; };
        for (int p = 0; p < slen / 2; ++p) {
            DP v;
            v.x = take(2 * p);
            v.y = take(2 * p + 1);
            reinterpret_cast<DP *>(sval + b)[p * kSell + lane] = v;
        }
        if (slen & 1) sval[(size_t)b + (size_t)(slen - 1) * kSell + lane] = take(slen - 1);
    }
}

// One value per slice position: uval takes, at each offset's index, the value
// of the position's first row; *varied is set when some row's differs (in its
// bits).  Every slice position has a row, so every element is written.
static __global__ __launch_bounds__(kBlock) void k_shared_uniform(int n, const int32_t *__restrict__ rowptr,
                                                                  const double *__restrict__ val,
                                                                  const int32_t *__restrict__ sptr,
                                                                  const uint32_t *__restrict__ mask,
                                                                  double *__restrict__ uval, int32_t *varied)
{
    __shared__ double stage[kBlock / kWave][kSharedCap];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int ns = (n + kSell - 1) / kSell;
    double *sc = stage[w];
    for (int s = blockIdx.x * (kBlock / kWave) + w; s < ns; s += gridDim.x * (kBlock / kWave)) {
        if (__hip_atomic_load(varied, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
        const int row = s * kSell + lane;
        const int base = rowptr[s * kSell], total = rowptr[min(n, (s + 1) * kSell)] - base;
        const int first = sptr[s] / kSell, slen = sptr[s + 1] / kSell - first;
        const uint32_t m = row < n ? mask[row] : 0u;
        int k = rowptr[min(row, n)] - base;
        wave_lds_sync();
        for (int i = lane; i < total; i += kWave) sc[i] = val[base + i];
        wave_lds_sync();
        bool differs = false;
        for (int j = 0; j < slen; ++j) {
            const bool has = (m >> j) & 1u;
            const long long v = has ? __double_as_longlong(sc[k++]) : 0;
            const int holder = __ffsll((unsigned long long)__ballot(has)) - 1;
            const long long v0 = __shfl(v, holder, kWave);
            differs |= has && v != v0;
            if (lane == 0) uval[first + j] = __longlong_as_double(v0);
        }
        if (__any(differs) && lane == 0)
            __hip_atomic_store(varied, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace spk
