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
    int32_t many;               // the matrix has more distinct offsets than the table holds
    int32_t varied;             // entries of one offset differ
    // the matrix's distinct offsets, in no order: offset in the high word,
    // one entry that has it in the low one
    unsigned long long offs[kSell];
};

// A free slot of the table: no offset is -2^31.
constexpr unsigned long long kNoOffset = 0x8000000000000000ull;

// Puts (offset, entry) into the table unless the offset is there.  seen: the
// block's LDS memory of offsets it has put there (kSell slots), which spares
// nearly every slice the look at the table (128^3: 400 -> 118 us).
__device__ __forceinline__ void note_offset(SharedStats *st, int32_t *seen, int off, int entry)
{
    const unsigned at = (uint32_t)off * 2654435761u >> 26;
    if (seen[at] == off) return;
    seen[at] = off;
    if (__hip_atomic_load(&st->many, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
    const unsigned long long v = ((unsigned long long)(uint32_t)off << 32) | (uint32_t)entry;
    unsigned h = at;
    for (int i = 0; i < kSell; ++i, h = (h + 1) & (kSell - 1)) {
        unsigned long long have =
            __hip_atomic_load(&st->offs[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (have == kNoOffset) have = atomicCAS(&st->offs[h], kNoOffset, v);
        if (have == kNoOffset || (have ^ v) >> 32 == 0) return;
    }
    __hip_atomic_store(&st->many, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

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
    __shared__ int32_t seen[kSell];
    if (threadIdx.x < kSell) seen[threadIdx.x] = (int32_t)0x80000000;
    __syncthreads();
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
            const int holder = __ffsll((unsigned long long)__ballot(cur == least)) - 1;
            if (cur == least) {
                m |= 1u << count;
                ++k;
                const int next = k < e ? sc[k] - row : kNone;
                if (next <= cur) wrong = 1;  // not ascending, or twice the same column
                cur = next;
            }
            if (lane == 0) list[(size_t)s * kSellSharedMax + count] = least;
            if (holder == lane) note_offset(out, seen, least, base + k - 1);
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

// The one list of a matrix of one value per offset, ascending, each with an
// entry that has it.
struct StencilList {
    int32_t w;
    int32_t off[kSellUniformMax];
    int32_t entry[kSellUniformMax];
};

// Row masks over the list, the list's offsets and values; *varied is set when
// some entry differs (in its bits) from its offset's.
static __global__ __launch_bounds__(kBlock) void k_stencil_masks(int n, StencilList l,
                                                                 const int32_t *__restrict__ rowptr,
                                                                 const int32_t *__restrict__ col,
                                                                 const double *__restrict__ val,
                                                                 uint32_t *__restrict__ mask,
                                                                 int32_t *__restrict__ offs,
                                                                 double *__restrict__ uval, int32_t *varied)
{
    __shared__ double stage[kBlock / kWave][kSharedCap / 2];
    __shared__ int32_t cols[kBlock / kWave][kSharedCap / 2];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int ns = (n + kSell / 2 - 1) / (kSell / 2);  // half slices, so that both stages fit
    if (blockIdx.x == 0 && (int)threadIdx.x < l.w) {
        int32_t o = 0, k = 0;
#pragma unroll
        for (int j = 0; j < kSellUniformMax; ++j)
            if (j == (int)threadIdx.x) {
                o = l.off[j];
                k = l.entry[j];
            }
        offs[threadIdx.x] = o;
        uval[threadIdx.x] = val[k];
    }
    for (int s = blockIdx.x * (kBlock / kWave) + w; s < ns; s += gridDim.x * (kBlock / kWave)) {
        if (__hip_atomic_load(varied, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
        const int r0 = s * (kSell / 2), row = r0 + (lane & (kSell / 2 - 1));
        const int base = rowptr[r0], total = rowptr[min(n, r0 + kSell / 2)] - base;
        int k = rowptr[min(row, n)] - base;
        const int e = rowptr[min(row + 1, n)] - base;
        wave_lds_sync();
        for (int i = lane; i < total; i += kWave) {
            stage[w][i] = val[base + i];
            cols[w][i] = col[base + i];
        }
        wave_lds_sync();
        uint32_t m = 0;
        bool differs = false;
#pragma unroll
        for (int j = 0; j < kSellUniformMax; ++j) {
            if (j >= l.w) break;
            const double v = val[l.entry[j]];
            if (k < e && cols[w][k] - row == l.off[j]) {
                differs |= __double_as_longlong(stage[w][k]) != __double_as_longlong(v);
                m |= 1u << j;
                ++k;
            }
        }
        if (row < n && lane < kSell / 2) mask[row] = m;
        if (__any(differs || k < e) && lane == 0)
            __hip_atomic_store(varied, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace spk
