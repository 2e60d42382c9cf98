// Binned SpMV for matrices whose columns scatter over a vector larger than one
// XCD's L2 and whose rows are too uneven for a fixed split: products by column,
// sums by row.
//
// An 8-byte gather from the L2 moves a 128-byte line: 154 gathers per ns over
// the chip whatever the cache policy (863 us for the 133 M entries of the 4 M
// row power-law matrix with nothing else done), six times the 258 us that
// streaming the matrix takes.  So x is gathered from LDS: the columns are cut
// into bins of kBinCols (128 KB of x), a first pass walks the entries bin by bin
// and streams out their products, a second walks the rows.
//
// The rows are cut into tiles of kBinItems merge-path items (row ends and
// entries), which bounds a tile's products by its LDS whatever the row lengths.
// Entries are stored by (bin, tile), so a tile's products are one segment per
// bin; `dst`, stored by tile, puts them back in CSR order in LDS, where the
// lanes sum them along the merge path.  28 bytes per entry are moved in FP64
// (10 read and 8 written, then 10 read) instead of 12 and a gather: 1130 us ->
// 510 us for the products (2.7 GB) and 411 for the sums (1.35 GB, 295 us with
// the merge path left out, which a second block on the CU hides in part), FP32
// about 990 -> 600.
#pragma once

#include "spmv.hpp"

namespace spk {

// Bins of 16384 columns: 8192, two blocks a CU, took 539 us for the products
// and 454 for the sums of segments half as long.  Tiles of 4096 items and 512
// threads, four blocks a CU, took 404 us where 8192 and 1024 took 435.
constexpr int kBinCols = 16384;   // columns of a bin
constexpr int kBinMax = 512;      // bins at most: a segment then has 8 products at most on average
                                  // (4096 / 512, less a tile's row ends)
constexpr int kBinProdThreads = 1024;
constexpr int kBinThreads = 512;
constexpr int kBinItems = 4096;   // merge-path items of a tile
constexpr int kBinIpt = kBinItems / kBinThreads;

// Where entry k of a tile is kept in LDS: lanes read kBinIpt consecutive ones
// each, which would meet in a few banks, so groups of eight are permuted within
// by the group's number.
__device__ __forceinline__ int bin_slot(int k) { return k ^ ((k >> 5) & 7); }

// cnt[c * T + t] = entries of tile t in bin c.
static __global__ __launch_bounds__(kBinThreads) void k_bin_count(int nb, int T, const int32_t *__restrict__ tile_k,
                                                                  const int32_t *__restrict__ col,
                                                                  int32_t *__restrict__ cnt)
{
    __shared__ int32_t h[kBinMax];
    const int t = blockIdx.x;
    if ((int)threadIdx.x < nb) h[threadIdx.x] = 0;
    __syncthreads();
    for (int k = tile_k[t] + (int)threadIdx.x; k < tile_k[t + 1]; k += kBinThreads) atomicAdd(&h[col[k] / kBinCols], 1);
    __syncthreads();
    if ((int)threadIdx.x < nb) cnt[(size_t)threadIdx.x * T + t] = h[threadIdx.x];
}

// Exclusive block scan of one int per thread of kBinThreads (sh: one per wave).
__device__ __forceinline__ int bin_scan(int v, int32_t *sh)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int s = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(s, off, kWave);
        if (lane >= off) s += o;
    }
    if (lane == kWave - 1) sh[w] = s;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int i = 0; i < kBinThreads / kWave; ++i) before += i < w ? sh[i] : 0;
    return before + s - v;
}

// Entries to their cells (cp: exclusive scan of cnt), in no particular order
// within one: dst says where a product belongs.  ts[t * nb + c] is where tile
// t's segment of bin c starts; its end is row t + 1's.
static __global__ __launch_bounds__(kBinThreads) void k_bin_fill(int nb, int T, const int32_t *__restrict__ tile_k,
                                                                 const int32_t *__restrict__ col,
                                                                 const double *__restrict__ val,
                                                                 const int32_t *__restrict__ cp, int32_t *__restrict__ ts,
                                                                 uint16_t *__restrict__ bcol, double *__restrict__ bval,
                                                                 uint16_t *__restrict__ dst)
{
    __shared__ int32_t cur[kBinMax], off[kBinMax], sh[kBinThreads / kWave];
    const int t = blockIdx.x, c = threadIdx.x;
    int start = 0, len = 0;
    if (c < nb) {
        start = cp[(size_t)c * T + t];
        const int end = cp[(size_t)c * T + t + 1];
        len = end - start;
        ts[(size_t)t * nb + c] = start;
        if (t == T - 1) ts[(size_t)T * nb + c] = end;
        cur[c] = start;
    }
    const int pre = bin_scan(len, sh);
    if (c < nb) off[c] = pre - start;
    __syncthreads();
    const int k0 = tile_k[t], k1 = tile_k[t + 1];
    for (int k = k0 + (int)threadIdx.x; k < k1; k += kBinThreads) {
        const int j = col[k], b = j / kBinCols;
        const int pos = atomicAdd(&cur[b], 1);
        bcol[pos] = (uint16_t)(j % kBinCols);
        bval[pos] = val[k];
        dst[k0 + pos + off[b]] = (uint16_t)bin_slot(k - k0);
    }
}

// Products of entries [p.y, p.z) of bin p.x, p = piece[blockIdx.x].  bcol, bval
// and prod are 16-byte aligned and two entries longer than the matrix.
template <class V>
__global__ __launch_bounds__(kBinProdThreads) void k_bin_products(int n, const int4 *__restrict__ piece,
                                                              const uint16_t *__restrict__ bcol,
                                                              const V *__restrict__ bval, const V *__restrict__ x,
                                                              V *__restrict__ prod, const SysState *gate_st,
                                                              int gate_mode)
{
    if (gate_st && !gate_open(gate_st, gate_mode)) return;
    constexpr int U = 4;  // pairs of a lane in flight
    typedef V V2 __attribute__((ext_vector_type(2)));
    typedef uint16_t C2 __attribute__((ext_vector_type(2)));
    __shared__ V xs[kBinCols];
    const int4 p = piece[blockIdx.x];
    const V2 *__restrict__ av = reinterpret_cast<const V2 *>(bval);
    const C2 *__restrict__ cv = reinterpret_cast<const C2 *>(bcol);
    const int q1 = (p.z + 1) / 2;
    V2 a[U];
    C2 c[U];
    auto load = [&](int q) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(q + u * kBinProdThreads, q1 - 1);
            c[u] = __builtin_nontemporal_load(cv + i);
            a[u] = __builtin_nontemporal_load(av + i);
        }
    };
    int q = p.y / 2 + (int)threadIdx.x;
    load(q);  // in flight while x arrives
    const int x0 = p.x * kBinCols, nx = min(kBinCols, n - x0);
    {
        constexpr int N = kBinCols / kBinProdThreads;
        V v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = x[x0 + min((int)threadIdx.x + i * kBinProdThreads, nx - 1)];
#pragma unroll
        for (int i = 0; i < N; ++i) xs[(int)threadIdx.x + i * kBinProdThreads] = v[i];
    }
    __syncthreads();
    while (q < q1) {
        V2 y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            y[u][0] = a[u][0] * xs[c[u][0] % kBinCols];
            y[u][1] = a[u][1] * xs[c[u][1] % kBinCols];
        }
        const int qn = q + U * kBinProdThreads;
        load(qn);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = q + u * kBinProdThreads;
            if (2 * i >= p.y && 2 * i + 1 < p.z) *reinterpret_cast<V2 *>(prod + 2 * (int64_t)i) = y[u];
            else if (2 * i >= p.y && 2 * i < p.z) prod[2 * (int64_t)i] = y[u][0];
            else if (2 * i + 1 >= p.y && 2 * i + 1 < p.z) prod[2 * (int64_t)i + 1] = y[u][1];
        }
        q = qn;
    }
}

// Row sums of one tile; a row that goes on past the tile leaves its part as the
// tile's carry (added by k_merge_fixup), as in the merge-path kernel.
template <class V>
__global__ __launch_bounds__(kBinThreads, 8) void k_bin_sum(int n, int nb, int T, const int32_t *__restrict__ rowptr,
                                                            const int32_t *__restrict__ tile_row,
                                                            const int32_t *__restrict__ tile_k,
                                                            const int32_t *__restrict__ ts,
                                                            const uint16_t *__restrict__ dst,
                                                            const V *__restrict__ prod, V *__restrict__ y,
                                                            int32_t *__restrict__ carry_row, V *__restrict__ carry_val,
                                                            const SysState *gate_st, int gate_mode)
{
    if (gate_st && !gate_open(gate_st, gate_mode)) return;
    constexpr int W = kBinThreads / kWave;
    __shared__ V buf[kBinItems + 8];  // products (whole groups of eight), then the row ends
    __shared__ unsigned long long mask[kBinItems / kWave];
    __shared__ int32_t base[kBinItems / kWave], shift[kBinMax], sh[W], wr[W];
    __shared__ V wv[W];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    // neighbours on one XCD: their segments share lines (the grid is T rounded
    // up to a multiple of kXcd)
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    if (t >= T) return;
    const int i0 = tile_row[t], k0 = tile_k[t];
    const int nrows = tile_row[t + 1] - i0, nk = tile_k[t + 1] - k0;
    int32_t *rend = reinterpret_cast<int32_t *>(buf + ((nk + 7) & ~7));
    uint16_t d[kBinIpt];
#pragma unroll
    for (int u = 0; u < kBinIpt; ++u) d[u] = nk > 0 ? dst[k0 + min(tid + u * kBinThreads, nk - 1)] : 0;
    int start = 0, len = 0;
    if (tid < nb) {
        start = ts[(size_t)t * nb + tid];
        len = ts[(size_t)(t + 1) * nb + tid] - start;
    }
    if (tid < kBinItems / kWave) mask[tid] = 0;
    // The segments one after the other: a bit at each one's start, its number at
    // each 64th product, and how far its products lie from their place there.
    const int ex = bin_scan(len | (len > 0) << 16, sh);
    const int pre = ex & 0xffff, rank = ex >> 16;
    if (len > 0) {
        shift[rank] = start - pre;
        atomicOr(&mask[pre / kWave], 1ull << (pre % kWave));
        for (int b = (pre + kWave - 1) / kWave; b * kWave < pre + len; ++b) base[b] = rank;
    }
    for (int r = tid; r <= nrows; r += kBinThreads) rend[r] = i0 + r < n ? rowptr[i0 + r + 1] - k0 : nk;
    __syncthreads();
    if (nk > 0) {
        V v[kBinIpt];
#pragma unroll
        for (int u = 0; u < kBinIpt; ++u) {
            const int f = min(tid + u * kBinThreads, nk - 1);
            const unsigned long long m = mask[f / kWave];
            const int r = base[f / kWave] + __popcll(m & ((2ull << (f % kWave)) - 1) & ~1ull);
            v[u] = prod[f + shift[r]];
        }
#pragma unroll
        for (int u = 0; u < kBinIpt; ++u)
            if (tid + u * kBinThreads < nk) buf[d[u]] = v[u];
    }
    __syncthreads();
    // this lane's start on the tile's merge path
    const int total = nrows + nk;
    const int dd = min(tid * kBinIpt, total);
    int lo = dd > nk ? dd - nk : 0;
    int hi = dd < nrows ? dd : nrows;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (rend[mid] <= dd - mid - 1) lo = mid + 1; else hi = mid;
    }
    int r = lo, kk = dd - lo;
    const int items = min(kBinIpt, total - dd);
    V acc = V(0), head = V(0);
    int head_row = -1;
    int end = rend[r];
    for (int it = 0; it < items; ++it) {
        if (kk < nk && kk < end) {
            acc += buf[bin_slot(kk)];
            ++kk;
        } else {
            if (r >= nrows || i0 + r >= n) break;  // never taken on a consistent path
            if (head_row < 0) { head = acc; head_row = r; }
            else y[i0 + r] = acc;
            acc = V(0);
            end = rend[++r];
        }
    }
    // inclusive sums of the carries of one row over the lanes, then the waves
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const V v = __shfl_up(acc, off, kWave);
        const int o = __shfl_up(r, off, kWave);
        if (lane >= off && o == r) acc = v + acc;
    }
    if (lane == kWave - 1) {
        wr[w] = r;
        wv[w] = acc;
    }
    __syncthreads();
    int br = wr[lane & (W - 1)];
    V bv = wv[lane & (W - 1)];
#pragma unroll
    for (int off = 1; off < W; off <<= 1) {
        const V v = __shfl_up(bv, off, W);
        const int o = __shfl_up(br, off, W);
        if ((lane & (W - 1)) >= off && o == br) bv = v + bv;
    }
    const int pr = __shfl(br, max(w - 1, 0), kWave);
    const V pv = __shfl(bv, max(w - 1, 0), kWave);
    if (w > 0 && pr == r) acc = pv + acc;
    V cin = __shfl_up(acc, 1, kWave);
    if (lane == 0) cin = w > 0 ? pv : V(0);
    if (head_row >= 0) y[i0 + head_row] = cin + head;
    if (tid == kBinThreads - 1) {
        carry_row[t] = i0 + r;
        carry_val[t] = acc;
    }
}

}  // namespace spk
