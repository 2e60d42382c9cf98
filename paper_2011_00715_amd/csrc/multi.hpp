// Multiple right-hand sides (Sec. 4 Response F3: Krylov methods with several
// right-hand sides read the matrix once for all of them and fuse their outer
// loops).  Vectors are row-major n x K (entry (i, j) at i K + j), so a gather
// of row c fetches the K values of all columns with one or two vector loads.
//
//   k_spmm_*        Y = A X
//   k_m_*           K independent Jacobi-PCG recurrences that share every
//                   SpMM: per-column scalars and stopping tests, per-column
//                   per-block partial sums reduced in a fixed order by
//                   one-block finalize kernels, so each column's iterates are
//                   those of its own single-right-hand-side solve up to the
//                   rounding order of the SpMV and the dots.
#pragma once

#include "spmv.hpp"

namespace spk {

constexpr int kMultiMax = 16;

// Purpose of a residual launch: the setup of a solve, or the true residual.
enum { kMultiSetup = 0, kMultiTrue = 1 };

// Columns still iterating (bit j), written by the finalize kernels.
struct MultiCtl {
    int32_t mask;
    int32_t pad_;
};

struct MultiDesc {
    int32_t n, K, nblk, R, ntiles;
    int32_t sell;                // 1: the SELL layout drives the row walk
    const int32_t *rowptr;
    const int32_t *col;
    const double *val;
    const double *dinv;
    SellView sv;
    const double *sell_val;
    const double *B;
    double *X, *Rv, *P, *Q;      // n x K each
    double *partials;            // [kNumPart][K][nblk]
    SysState *st;                // K states
    MultiCtl *ctl;
};

// Y-rows = A X-rows for one row, K columns, entries [a, e) of CSR; U
// entries per round with their gathers issued together.
template <int K>
__device__ __forceinline__ void csr_row_multi(int a, int e, const int32_t *__restrict__ col,
                                              const double *__restrict__ val,
                                              const double *__restrict__ X, double acc[K])
{
    constexpr int U = K >= 8 ? 1 : 8 / K;
#pragma unroll
    for (int q = 0; q < K; ++q) acc[q] = 0.0;
    for (int k0 = a; k0 < e; k0 += U) {
        int c[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + u < e ? k0 + u : e - 1;
            c[u] = ld_stream(col + k);
            v[u] = ld_stream(val + k);
        }
        double xv[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < K; ++q) xv[u][q] = X[(size_t)c[u] * K + q];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < e)
#pragma unroll
                for (int q = 0; q < K; ++q) acc[q] = fma(v[u], xv[u][q], acc[q]);
    }
}

// Same for lane `lane` of a SELL slice (b, slen), the row having rlen
// entries.  The offset and value pairs of up to kMultiPairs pairs are loaded
// together (one paired load of offsets and of values each), then the K
// gathers of pair p + 1 (or of the slice's odd last entry) are issued before
// the FMAs of pair p, so the gathers of consecutive pairs overlap instead of
// costing one memory round trip each (K = 8 on the 7-point 128^3 product:
// 118 -> 95 us with the staged stores below).  K = 16 keeps one pair in
// registers at a time (double buffering would take 128 more VGPRs).  Sums
// run in column order either way.
//
// kOneRound (standalone SpMM): a slice of at most kOneRoundPairs pairs loads
// them and issues every gather (the odd entry's too) before the first FMA,
// one memory round trip per slice at the cost of holding all gathered rows
// (K = 8: 152 VGPRs, three wavefronts per SIMD).  The product inside the
// multi-RHS solve keeps the pipelined walk: there the extra registers cost
// more than the round trips they save.
constexpr int kMultiPairs = 4;
constexpr int kOneRoundPairs = 3;

//
// SH: shared offsets (see the SELL-64 notes): offsets from the slice's list,
// rlen the row's position mask, gathered rows clamped into [0, n).  UNI: one
// value per offset, both from the matrix's one list.
//
// pdiag (the pipelined walk only; null otherwise): where to keep the row's
// own gathered X row, the gather of its diagonal entry (offset 0; the
// solve's matrices have one in every row), so that the caller need not read
// it again.
template <class CI, int K, bool kOneRound = false, bool SH = false, bool UNI = false>
__device__ __forceinline__ void sell_row_multi(const SellView &sv, const double *__restrict__ val,
                                               const double *__restrict__ X, int32_t b, int slen,
                                               int rlen, int lane, int row, int n, double acc[K],
                                               double *pdiag = nullptr)
{
    static_assert(!SH || std::is_same<CI, int32_t>::value, "shared offsets are int32");
    constexpr int PM = K <= 8 ? kMultiPairs : 1;
    using CP = typename Pair2<CI>::type;
    using VP = typename Pair2<double>::type;
    const CP *__restrict__ cp = reinterpret_cast<const CP *>(reinterpret_cast<const CI *>(sv.col) + b) + lane;
    const int32_t first = UNI ? 0 : __builtin_amdgcn_readfirstlane(b) >> 6;  // the slice's first list element
    // lists by scalar loads, whatever the caller's stores may alias
    const auto *ou = as_constant(reinterpret_cast<const int32_t *>(sv.col)) + first;
    const auto *uv = as_constant(val) + first;
    const VP *__restrict__ vp = reinterpret_cast<const VP *>(val + b) + lane;
    auto values = [&](int p) -> VP {
        if constexpr (UNI) {
            VP a;
            a.x = uv[2 * p];
            a.y = uv[2 * p + 1];
            return a;
        } else {
            return ld_stream(vp + (size_t)p * kSell);
        }
    };
    auto offsets = [&](int p) -> CP {
        if constexpr (SH) {
            CP c;
            c.x = ou[2 * p];
            c.y = ou[2 * p + 1];
            return c;
        } else {
            return ld_stream(cp + (size_t)p * kSell);
        }
    };
    auto real = [&](int k) -> bool {
        if constexpr (SH) return ((unsigned)rlen >> k) & 1u;
        else return k < rlen;
    };
    const int np = slen >> 1;
    const bool odd = slen & 1;
    CI ct = CI(0);
    double at = 0.0;
    if (odd) {
        const size_t t = (size_t)b + (size_t)np * (2 * kSell) + lane;
        if constexpr (SH) ct = ou[2 * np];
        else ct = ld_stream(reinterpret_cast<const CI *>(sv.col) + t);
        if constexpr (UNI) at = uv[2 * np];
        else at = ld_stream(val + t);
    }
#pragma unroll
    for (int q = 0; q < K; ++q) acc[q] = 0.0;
    auto gather = [&](int off, double xr[K]) {
        int j = row + off;
        if constexpr (SH) j = min(max(j, 0), n - 1);
#pragma unroll
        for (int q = 0; q < K; ++q) xr[q] = X[(size_t)j * K + q];
    };
    auto madd = [&](double a, const double xr[K]) {
#pragma unroll
        for (int q = 0; q < K; ++q) acc[q] = fma(a, xr[q], acc[q]);
    };
    auto keep = [&](int off, const double xr[K]) {
        if (pdiag && off == 0)
#pragma unroll
            for (int q = 0; q < K; ++q) pdiag[q] = xr[q];
    };
    if (kOneRound && K <= 8 && np <= kOneRoundPairs) {
        // every pair index is clamped into the slice (a slice without pairs
        // loads none: its gathers then fetch the lane's own row, unused)
        constexpr int P1 = kOneRoundPairs;
        CP c[P1];
        VP a[P1];
#pragma unroll
        for (int u = 0; u < P1; ++u) {
            c[u].x = c[u].y = CI(0);
            a[u].x = a[u].y = 0.0;
        }
        if (np > 0)
#pragma unroll
            for (int u = 0; u < P1; ++u) {
                const int p = u < np ? u : np - 1;
                c[u] = offsets(p);
                a[u] = values(p);
            }
        double xv[2 * P1 + 1][K];
#pragma unroll
        for (int u = 0; u < P1; ++u) {
            gather((int)c[u].x, xv[2 * u]);
            gather((int)c[u].y, xv[2 * u + 1]);
        }
        gather((int)ct, xv[2 * P1]);
#pragma unroll
        for (int u = 0; u < P1; ++u)
            if (u < np) {
                if (real(2 * u)) madd(a[u].x, xv[2 * u]);
                if (real(2 * u + 1)) madd(a[u].y, xv[2 * u + 1]);
            }
        if (odd && real(slen - 1)) madd(at, xv[2 * P1]);
        return;
    }
    if (PM > 1 && np >= 1 && np <= PM) {
        // the slice's pairs in one load round, gathers one pair ahead
        CP c[PM];
        VP a[PM];
#pragma unroll
        for (int u = 0; u < PM; ++u) {
            const int p = u < np ? u : np - 1;
            c[u] = offsets(p);
            a[u] = values(p);
        }
        double xa[2][K], xb[2][K];
        gather((int)c[0].x, xa[0]);
        gather((int)c[0].y, xa[1]);
#pragma unroll
        for (int u = 0; u < PM; ++u) {
            if (u + 1 < PM && u + 1 < np) {
                gather((int)c[u + 1].x, xb[0]);
                gather((int)c[u + 1].y, xb[1]);
            }
            if (u < np) {
                if (real(2 * u)) {
                    madd(a[u].x, xa[0]);
                    keep((int)c[u].x, xa[0]);
                }
                if (real(2 * u + 1)) {
                    madd(a[u].y, xa[1]);
                    keep((int)c[u].y, xa[1]);
                }
            }
#pragma unroll
            for (int q = 0; q < K; ++q) {
                xa[0][q] = xb[0][q];
                xa[1][q] = xb[1][q];
            }
        }
    } else {
        // wide slices (or K = 16): one pair per round
        for (int p = 0; p < np; ++p) {
            const CP c = offsets(p);
            const VP a = values(p);
            double x0[K], x1[K];
            gather((int)c.x, x0);
            gather((int)c.y, x1);
            if (real(2 * p)) {
                madd(a.x, x0);
                keep((int)c.x, x0);
            }
            if (real(2 * p + 1)) {
                madd(a.y, x1);
                keep((int)c.y, x1);
            }
        }
    }
    if (odd && real(slen - 1)) {
        double xt[K];
        gather((int)ct, xt);
        madd(at, xt);
        keep((int)ct, xt);
    }
}

// SELL slices of block l with the K products of each row staged in LDS
// (stage: this wave's 64 x K doubles), then handed out flat: flat(e0, cnt)
// for the slice's cnt elements starting at element e0 of the row-major
// n x K layout, which the caller walks with lane t taking elements t, t + 64,
// ... of the stage (so always column t % K, as 64 % K == 0).  A lane's K
// products are 8K contiguous bytes, so storing them from the lanes directly
// writes 64 partial segments per instruction; the flat pass writes whole
// ones (K = 8: 118 -> 99 us on the 7-point 128^3 product).
template <class CI, int K, bool kOneRound, bool SH, bool UNI, class Flat>
__device__ __forceinline__ void multi_sell_walk(const MultiDesc &d, int l, const double *__restrict__ X,
                                                double *stage, double *pstage, Flat &&flat)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int ns = (d.n + kSell - 1) / kSell;
    for (int s = l * (kBlock / kWave) + (int)threadIdx.x / kWave; s < ns; s += d.nblk * (kBlock / kWave)) {
        int32_t b = 0, e = (d.sv.plain >> kSellWidthShift) * kSell;
        if constexpr (!UNI) {
            b = d.sv.ptr[s];
            e = d.sv.ptr[s + 1];
        }
        const int row = s * kSell + lane;
        if (row < d.n) {
            double acc[K];
            const int rl = SH ? (int)d.sv.mask[row] : (int)d.sv.len[row];
            sell_row_multi<CI, K, kOneRound, SH, UNI>(d.sv, d.sell_val, X, b, (e - b) / kSell, rl, lane, row, d.n,
                                                 acc, pstage ? pstage + lane * K : nullptr);
#pragma unroll
            for (int q = 0; q < K; ++q) stage[lane * K + q] = acc[q];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        flat((int64_t)s * kSell * K, (min(d.n, (s + 1) * kSell) - s * kSell) * K);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <class CI, int K, bool kOneRound, class Flat>
__device__ __forceinline__ void multi_sell_staged(const MultiDesc &d, int l, const double *__restrict__ X,
                                                  double *stage, double *pstage, Flat &&flat)
{
    if constexpr (std::is_same<CI, Stencil>::value) {
        multi_sell_walk<int32_t, K, kOneRound, true, true>(d, l, X, stage, pstage, flat);
    } else {
        if constexpr (std::is_same<CI, int32_t>::value) {
            if (d.sv.mask) {
                multi_sell_walk<CI, K, kOneRound, true, false>(d, l, X, stage, pstage, flat);
                return;
            }
        }
        multi_sell_walk<CI, K, kOneRound, false, false>(d, l, X, stage, pstage, flat);
    }
}

// Row walk of block l (of nblk) of a multi kernel: SELL slices in
// round-robin order, or CSR rows of the block's contiguous tile range with
// one row per lane.  fn(row, acc) gets the K products of the row.
template <class CI, int K, class Fn>
__device__ __forceinline__ void multi_rows(const MultiDesc &d, int l, int j, const double *__restrict__ X,
                                           Fn &&fn)
{
    double acc[K];
    if (d.sell) {
        const int lane = threadIdx.x & (kWave - 1);
        const int ns = (d.n + kSell - 1) / kSell;
        for (int s = l * (kBlock / kWave) + (int)threadIdx.x / kWave; s < ns; s += d.nblk * (kBlock / kWave)) {
            const int row = s * kSell + lane;
            if (row >= d.n) continue;
            if constexpr (std::is_same<CI, Stencil>::value) {
                sell_row_multi<int32_t, K, false, true, true>(d.sv, d.sell_val, X, 0, d.sv.plain >> kSellWidthShift,
                                                              (int)d.sv.mask[row], lane, row, d.n, acc);
            } else {
                const int32_t b = d.sv.ptr[s], e = d.sv.ptr[s + 1];
                bool done = false;
                if constexpr (std::is_same<CI, int32_t>::value) {
                    if (d.sv.mask) {
                        sell_row_multi<CI, K, false, true>(d.sv, d.sell_val, X, b, (e - b) / kSell,
                                                           (int)d.sv.mask[row], lane, row, d.n, acc);
                        done = true;
                    }
                }
                if (!done)
                    sell_row_multi<CI, K>(d.sv, d.sell_val, X, b, (e - b) / kSell, d.sv.len[row], lane, row, d.n, acc);
            }
            fn(row, acc);
        }
    } else {
        int t0, t1;
        block_tiles(j, d.nblk, d.ntiles, t0, t1);
        const int rb = t0 * d.R, re = min(t1 * d.R, d.n);
        for (int row = rb + (int)threadIdx.x; row < re; row += kBlock) {
            csr_row_multi<K>(d.rowptr[row], d.rowptr[row + 1], d.col, d.val, X, acc);
            fn(row, acc);
        }
    }
}

// Block sums of K per-lane values, one partial per column: part[q * nblk + j].
template <int K>
__device__ __forceinline__ void block_partials(double v[K], double *sh /* [4][K] */, double *part,
                                               int nblk, int j)
{
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = wave_sum(v[q]);
    const int w = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0)
#pragma unroll
        for (int q = 0; q < K; ++q) sh[w * K + q] = v[q];
    __syncthreads();
    if ((int)threadIdx.x < K) {
        const int q = threadIdx.x;
        double s = sh[q];
#pragma unroll
        for (int ww = 1; ww < kBlock / kWave; ++ww) s += sh[ww * K + q];
        part[(size_t)q * nblk + j] = s;
    }
}

// Two elements of the flat n x K layout (one where K is 1): a lane's columns are
// kCols * (t % (K / kCols)) and, for two, the next one, in every walk below.
template <int K>
struct Flat {
    static constexpr int kCols = K > 1 ? 2 : 1;
    static constexpr int kLanes = K / kCols;  // lanes per row
    typedef double Elem __attribute__((ext_vector_type(kCols)));
    static __device__ __forceinline__ int col(int t) { return t % kLanes * kCols; }
};

// Block sums per column of what the lanes hold for their columns: lanes of one
// column are combined by the butterfly levels at distances >= kLanes, then the
// waves in order.
template <int K>
__device__ __forceinline__ void block_partials_elem(typename Flat<K>::Elem v, double *sh /* [4][K] */, double *part,
                                                    int nblk, int j)
{
    constexpr int C = Flat<K>::kCols, L = Flat<K>::kLanes;
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    // K = 2 sums two columns over all six levels: with shuffles the update of
    // 152,000 rows took 5.2 us, with the lane swaps and rotations 4.2 (for K = 8
    // they cost the product 86.0 -> 87.3)
    if constexpr (L == 1) {
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = wave_sum((double)v[c]);
    } else {
#pragma unroll
        for (int off = kWave / 2; off >= L; off >>= 1)
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] += __shfl_xor(v[c], off, kWave);
    }
    __syncthreads();
    if (lane < L)
#pragma unroll
        for (int c = 0; c < C; ++c) sh[w * K + lane * C + c] = v[c];
    __syncthreads();
    if ((int)threadIdx.x < K) {
        const int q = threadIdx.x;
        double s = sh[q];
#pragma unroll
        for (int ww = 1; ww < kBlock / kWave; ++ww) s += sh[ww * K + q];
        part[(size_t)q * nblk + j] = s;
    }
}

// Elements [e0, e1) of the flat layout (multiples of K), kCols at a time with a
// stride of kBlock lanes: ld(t, i) loads what lane-element t of row i needs,
// st(t, v) uses it; a chunk's loads are issued before its stores.
template <int K, class Ld, class St>
__device__ __forceinline__ void flat_walk(int64_t e0, int64_t e1, Ld &&ld, St &&st)
{
    constexpr int U = 4, C = Flat<K>::kCols;
    using T = decltype(ld(int64_t(0), int64_t(0)));
    const int64_t t0 = e0 / C, t1 = e1 / C;
    for (int64_t tb = t0 + threadIdx.x; tb < t1; tb += (int64_t)kBlock * U) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = min(tb + (int64_t)u * kBlock, t1 - 1);  // past the end: the last one, unused
            v[u] = ld(t, t / Flat<K>::kLanes);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = tb + (int64_t)u * kBlock;
            if (t < t1) st(t, v[u]);
        }
    }
}

// The flat range of block j's rows.
__device__ __forceinline__ void flat_range(const MultiDesc &d, int j, int64_t &e0, int64_t &e1)
{
    int t0, t1;
    block_tiles(j, d.nblk, d.ntiles, t0, t1);
    e0 = (int64_t)t0 * d.R * d.K;
    e1 = (int64_t)min(t1 * d.R, d.n) * d.K;
}

constexpr int kMultiAhead = 2;

// Row walk for a matrix of one value per offset (K even): with the values in
// scalar registers a row's product is the same for all its columns, so the
// flat layout is walked like a vector, two elements a lane, and every gather is
// one contiguous kilobyte per wavefront.  (A lane per row reads 8 K bytes of
// each gathered row, a line per lane and instruction.)  A wave takes slices
// s0, s0 + stride, ... of 64 rows, 64 lane-elements at a time (the order of the
// staged walk, so sums over a lane's elements have its bits); fn(t, row, y, own)
// gets lane-element t of the flat layout, own being what pre(t) loaded, once
// go() holds.  X is 16-byte aligned.  The walk waits on the latency of its
// rounds (16 waves a CU), so kMultiAhead pieces are loaded before the first is
// used: with p.q on the 7-point 128^3 matrix, K = 8, 107.8 us with one, 95.7
// with two, 100.7 with four (registers).  Neighbours a few rows away by lane
// moves instead of loads: 127.6.
template <int K, int W, class Go, class Pre, class Fn>
__device__ __forceinline__ void multi_stencil(const MultiDesc &d, int s0, int stride, const double *__restrict__ X,
                                              Go &&go, Pre &&pre, Fn &&fn)
{
    using E = typename Flat<K>::Elem;
    constexpr int L = Flat<K>::kLanes;
    constexpr int kRows = kWave / L;                       // rows of 64 lane-elements
    constexpr int U = L > 1 ? kMultiAhead : 1;             // such pieces at a time
    const int n = d.n, lane = threadIdx.x & (kWave - 1);
    const int ns = (n + kSell - 1) / kSell;
    const int w = d.sv.plain >> kSellWidthShift;
    const uint32_t *__restrict__ masks = d.sv.mask;
    // constant for the kernel's life: read by scalar loads; positions past the
    // list repeat its last one, no mask has their bits
    const auto *ou = as_constant(reinterpret_cast<const int32_t *>(d.sv.col));
    const auto *uv = as_constant(d.sell_val);
    const int64_t lo = ou[0], hi = ou[w - 1];
    const E *__restrict__ Xe = reinterpret_cast<const E *>(X);
    int ok[W];
    double vk[W];
    auto list = [&](int k0) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
            ok[k] = ou[min(k0 + k, w - 1)];
            vk[k] = uv[min(k0 + k, w - 1)];
        }
    };
    list(0);
    int s = __builtin_amdgcn_readfirstlane(s0);
    if (!go()) return;
    for (; s < ns; s += stride) {
        const int re = min((s + 1) * kSell, n);
        for (int r0 = s * kSell; r0 < re; r0 += U * kRows) {
            const bool in = r0 + lo >= 0 && r0 + (U * kRows - 1) + hi < n;
            uint32_t m[U];
            decltype(pre(int64_t(0))) own[U];
            E acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int row = r0 + u * kRows + lane / L;
                m[u] = row < n ? masks[min(row, n - 1)] : 0u;
                own[u] = pre(min((int64_t)(r0 + u * kRows) * L + lane, (int64_t)n * L - 1));
                acc[u] = E(0.0);
            }
            for (int k0 = 0; k0 < w; k0 += W) {
                E xv[U][W];
                if (in) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int k = 0; k < W; ++k)
                            xv[u][k] = (Xe + ((int64_t)(r0 + u * kRows) + ok[k]) * L)[(unsigned)lane];
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
#pragma unroll
                        for (int k = 0; k < W; ++k) {
                            const int c = min(max(r0 + u * kRows + lane / L + ok[k], 0), n - 1);
                            xv[u][k] = Xe[(int64_t)c * L + lane % L];
                        }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < W; ++k)
#pragma unroll
                        for (int c = 0; c < Flat<K>::kCols; ++c) {
                            const double t = fma(vk[k], xv[u][k][c], acc[u][c]);
                            acc[u][c] = (m[u] >> k) & 1u ? t : acc[u][c];
                        }
                if (w <= W) break;
#pragma unroll
                for (int u = 0; u < U; ++u) m[u] >>= W;
                list(k0 + W < w ? k0 + W : 0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int row = r0 + u * kRows + lane / L;
                if (row < n) fn((int64_t)(r0 + u * kRows) * L + lane, row, acc[u], own[u]);
            }
        }
    }
}

__device__ __forceinline__ int multi_block(const MultiDesc &d, int &j)
{
    if ((int)blockIdx.x >= d.nblk) return -1;
    j = xcd_remap(blockIdx.x, d.nblk);
    return blockIdx.x;
}

// ------------------------------------------------------------------ SpMM
// Physical block l runs on XCD l % 8.  Logical blocks in runs of R per XCD:
// ((l / 8) / R) 8R + (l % 8) R + (l / 8) % R, a bijection when nblk is a
// multiple of 8R (else the identity), so that R consecutive logical blocks
// (4R consecutive slices for the SpMM) share an L2.
__device__ __forceinline__ int xcd_runs(int l, int nblk, int R)
{
    if (nblk % (kXcd * R)) return l;
    const int x = l % kXcd, k = l / kXcd;
    return (k / R) * (kXcd * R) + x * R + k % R;
}

// Consecutive blocks per XCD of the stencil walk: 4, 16, 64 and a whole eighth
// of the rows measured alike (101.6 to 104.1 us).
constexpr int kStencilRun = 16;

template <class CI, int K>
__global__ __launch_bounds__(kBlock) void k_spmm(MultiDesc d, const double *__restrict__ X, double *__restrict__ Y)
{
    __shared__ double stage[(kBlock / kWave) * kWave * (K > 1 ? K : 1)];
    int j;
    int l = multi_block(d, j);
    if (l < 0) return;
    if (d.sell && K > 1) {
        // runs of 4 blocks (16 slices) per XCD keep the +-1-line gathers of
        // neighbouring slices in one L2
        l = xcd_runs(l, d.nblk, 4);
        // flat stores of two elements (K is even): 1 KB per instruction
        using VP = typename Pair2<double>::type;
        const int lane = threadIdx.x & (kWave - 1);
        double *st = stage + (threadIdx.x / kWave) * kWave * K;
        multi_sell_staged<CI, K, true>(d, l, X, st, nullptr, [&](int64_t e0, int cnt) {
            const VP *src = reinterpret_cast<const VP *>(st);
            VP *dst = reinterpret_cast<VP *>(Y + e0);
            for (int t = lane; t < cnt / 2; t += kWave) __builtin_nontemporal_store(src[t], dst + t);
        });
        return;
    }
    multi_rows<CI, K>(d, l, j, X, [&](int row, const double *acc) {
#pragma unroll
        for (int q = 0; q < K; ++q) Y[(size_t)row * K + q] = acc[q];
    });
}

// The same for a matrix of one value per offset, K even, X and Y 16-byte aligned.
template <int K, int W>
__global__ __launch_bounds__(kBlock) void k_spmm_stencil(MultiDesc d, const double *__restrict__ X,
                                                         double *__restrict__ Y)
{
    using E = typename Flat<K>::Elem;
    const int l = xcd_runs((int)blockIdx.x, (int)gridDim.x, kStencilRun);
    E *Ye = reinterpret_cast<E *>(Y);
    multi_stencil<K, W>(d, l * (kBlock / kWave) + (int)threadIdx.x / kWave, (int)gridDim.x * (kBlock / kWave), X,
                        [] { return true; }, [](int64_t) { return 0; },
                        [&](int64_t t, int, E y, int) { __builtin_nontemporal_store(y, Ye + t); });
}

// ------------------------------------------------------------------ residual
// R = B - A X for the columns in `mask` (others untouched), per-column
// per-block r.r and b.b.
template <class CI, int K>
__global__ __launch_bounds__(kBlock) void k_m_resid(MultiDesc d, int32_t mask)
{
    __shared__ double sh[(kBlock / kWave) * K];
    int j;
    const int l = multi_block(d, j);
    if (l < 0) return;
    const double *__restrict__ X = d.X;
    const double *__restrict__ Bv = d.B;
    double *__restrict__ Rv = d.Rv;
    double rr[K], bb[K];
#pragma unroll
    for (int q = 0; q < K; ++q) rr[q] = bb[q] = 0.0;
    multi_rows<CI, K>(d, l, j, X, [&](int row, const double *acc) {
        double br[K];  // the row of B, loaded before any store of R
#pragma unroll
        for (int q = 0; q < K; ++q) br[q] = Bv[(size_t)row * K + q];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            if (!((mask >> q) & 1)) continue;
            const double bi = br[q];
            const double ri = bi - acc[q];
            Rv[(size_t)row * K + q] = ri;
            rr[q] = fma(ri, ri, rr[q]);
            bb[q] = fma(bi, bi, bb[q]);
        }
    });
    block_partials<K>(rr, sh, d.partials + (size_t)kPartRr * K * d.nblk, d.nblk, j);
    block_partials<K>(bb, sh, d.partials + (size_t)kPartBb * K * d.nblk, d.nblk, j);
}

// The finalize kernels run one block per column (q = blockIdx.x): the block
// sums the column's nblk partials in a fixed order (reduce_partials), thread
// 0 runs the column's scalar logic, and a column that stops clears its bit
// of the running mask with an integer atomic (the only cross-block write).
__device__ __forceinline__ const double *col_part(const MultiDesc &d, int part, int q)
{
    return d.partials + ((size_t)part * d.K + q) * d.nblk;
}

__device__ __forceinline__ void stop_column(const MultiDesc &d, int q)
{
    atomicAnd(&d.ctl->mask, ~(1 << q));
}

// purpose kMultiSetup: norms, thresholds, stop at start; kMultiTrue: store the
// true residual norm of the columns in mask.
static __global__ __launch_bounds__(kBlock) void k_m_fin_resid(MultiDesc d, int purpose, int32_t mask)
{
    __shared__ double red[kBlock / kWave];
    const int q = blockIdx.x;
    if (q >= d.K || !((mask >> q) & 1)) return;
    double RR, BB;
    reduce_partials2(col_part(d, kPartRr, q), col_part(d, kPartBb, q), d.nblk, red, RR, BB);
    if (threadIdx.x != 0) return;
    SysState *st = d.st + q;
    const double rn = sqrt(RR);
    if (purpose == kMultiTrue) {
        st->rnorm_true = rn;
        return;
    }
    const double bn = sqrt(BB);
    st->bnorm = bn;
    st->thresh = fmax(st->rtol * bn, st->atol);
    st->rnorm = rn;
    st->rnorm0 = rn;
    if (bn == 0.0) st->status = SPK_CONVERGED_ATOL;
    else if (!isfinite(rn) || !isfinite(bn)) st->status = SPK_DIVERGED_NANORINF;
    else if (rn <= st->thresh) st->status = rn <= st->rtol * bn ? SPK_CONVERGED_RTOL : SPK_CONVERGED_ATOL;
    if (st->status != SPK_RUNNING) stop_column(d, q);
}

// ------------------------------------------------------------------ setup
// z = D^-1 r is formed where it is needed (the dots, p): reading r and D^-1 again
// costs a K-th more than z would, and z is never stored (8 n K bytes an
// iteration less).

// P = Z for the running columns in mask, per-block r.z.
template <int K>
__global__ __launch_bounds__(kBlock) void k_m_setup(MultiDesc d, int32_t mask)
{
    using E = typename Flat<K>::Elem;
    constexpr int C = Flat<K>::kCols;
    __shared__ double sh[(kBlock / kWave) * K];
    int j;
    if (multi_block(d, j) < 0) return;
    const int q = Flat<K>::col(threadIdx.x);
    bool run[C];
#pragma unroll
    for (int c = 0; c < C; ++c) run[c] = ((mask >> (q + c)) & 1) && d.st[q + c].status == SPK_RUNNING;
    const E *__restrict__ Re = reinterpret_cast<const E *>(d.Rv);
    const double *__restrict__ dinv = d.dinv;
    E *__restrict__ Pe = reinterpret_cast<E *>(d.P);
    struct In {
        E r, p;
        double dinv;
    };
    E rz = E(0.0);
    int64_t e0, e1;
    flat_range(d, j, e0, e1);
    flat_walk<K>(e0, e1, [&](int64_t t, int64_t i) { return In{Re[t], Pe[t], dinv[i]}; },
                 [&](int64_t t, const In &v) {
                     E p = v.p;
#pragma unroll
                     for (int c = 0; c < C; ++c)
                         if (run[c]) {
                             const double zi = v.dinv * v.r[c];
                             p[c] = zi;
                             rz[c] = fma(v.r[c], zi, rz[c]);
                         }
                     Pe[t] = p;
                 });
    block_partials_elem<K>(rz, sh, d.partials + (size_t)kPartRz * K * d.nblk, d.nblk, j);
}

static __global__ __launch_bounds__(kBlock) void k_m_fin_setup(MultiDesc d, int32_t mask)
{
    __shared__ double red[kBlock / kWave];
    const int q = blockIdx.x;
    if (q >= d.K || !((mask >> q) & 1)) return;
    SysState *st = d.st + q;
    if (st->status != SPK_RUNNING) return;
    const double RZ = reduce_partials(col_part(d, kPartRz, q), d.nblk, red);
    if (threadIdx.x != 0) return;
    st->cmode = 0;
    if (!isfinite(RZ)) st->status = SPK_DIVERGED_NANORINF;
    else if (RZ < 0.0) st->status = SPK_DIVERGED_INDEFINITE_PC;
    else if (RZ == 0.0) st->status = SPK_DIVERGED_BREAKDOWN;
    else if (st->iter >= st->maxit) { st->status = SPK_DIVERGED_ITS; st->rho = RZ; }
    else st->rho = RZ;
    if (st->status != SPK_RUNNING) stop_column(d, q);
}

// Restart the columns in mask from their true residual (already in R).
static __global__ void k_m_restart(MultiDesc d, int32_t mask)
{
    const int q = threadIdx.x;
    if (q < d.K && ((mask >> q) & 1)) {
        d.st[q].status = SPK_RUNNING;
        d.st[q].cmode = 0;
    }
    if (q == 0) d.ctl->mask |= mask;
}

// ------------------------------------------------------------------ iteration
// A: Q = A P, per-column per-block p.q (columns that stopped are multiplied
// too: the matrix is read once either way; their partials are ignored).
template <class CI, int K>
__global__ __launch_bounds__(kBlock, K <= 8 ? 4 : 1) void k_m_spmm_pq(MultiDesc d)
{
    __shared__ double sh[(kBlock / kWave) * K];
    __shared__ double stage[(kBlock / kWave) * kWave * (K > 1 ? K : 1)];
    // each row's own P row, kept from its diagonal gather (every row of a
    // solved matrix has one): the flat pass's p.q reads it here instead of
    // fetching P a second time (the rows were gathered moments before, but
    // read again from memory they cost a third of the kernel's traffic)
    __shared__ double pstage[(kBlock / kWave) * kWave * (K > 1 ? K : 1)];
    int j;
    const int l = multi_block(d, j);
    if (l < 0) return;
    if (d.ctl->mask == 0) return;
    // Q never aliases P: without the qualifiers the compiler orders every
    // gather of P behind the stores of Q
    const double *__restrict__ P = d.P;
    double *__restrict__ Q = d.Q;
    if (d.sell && K > 1) {
        // flat pass, two elements a lane
        using E = typename Flat<K>::Elem;
        E pqv = E(0.0);
        const int lane = threadIdx.x & (kWave - 1);
        const E *st = reinterpret_cast<const E *>(stage + (threadIdx.x / kWave) * kWave * K);
        const E *pst = reinterpret_cast<const E *>(pstage + (threadIdx.x / kWave) * kWave * K);
        multi_sell_staged<CI, K, false>(d, l, P, stage + (threadIdx.x / kWave) * kWave * K,
                                        pstage + (threadIdx.x / kWave) * kWave * K,
                                        [&](int64_t e0, int cnt) {
                                            E *q = reinterpret_cast<E *>(Q + e0);
                                            for (int t = lane; t < cnt / Flat<K>::kCols; t += kWave) {
                                                const E v = st[t], pe = pst[t];
                                                q[t] = v;
#pragma unroll
                                                for (int c = 0; c < Flat<K>::kCols; ++c)
                                                    pqv[c] = fma(v[c], pe[c], pqv[c]);
                                            }
                                        });
        block_partials_elem<K>(pqv, sh, d.partials + (size_t)kPartPq * K * d.nblk, d.nblk, j);
        return;
    }
    double pq[K];
#pragma unroll
    for (int q = 0; q < K; ++q) pq[q] = 0.0;
    multi_rows<CI, K>(d, l, j, P, [&](int row, const double *acc) {
        double pr[K];  // the row of P, loaded before any store of Q
#pragma unroll
        for (int q = 0; q < K; ++q) pr[q] = P[(size_t)row * K + q];
#pragma unroll
        for (int q = 0; q < K; ++q) {
            Q[(size_t)row * K + q] = acc[q];
            pq[q] = fma(acc[q], pr[q], pq[q]);
        }
    });
    block_partials<K>(pq, sh, d.partials + (size_t)kPartPq * K * d.nblk, d.nblk, j);
}

// A for a matrix of one value per offset, K even: 103.8 us a row per lane ->
// 95.7 on the 7-point 128^3 matrix with K = 8 (444 MB moved; P is fetched 2.3
// times, the planes of the grid being 1 MB apart).
template <int K, int W>
__global__ __launch_bounds__(kBlock) void k_m_spmm_pq_stencil(MultiDesc d)
{
    using E = typename Flat<K>::Elem;
    __shared__ double sh[(kBlock / kWave) * K];
    if ((int)blockIdx.x >= d.nblk) return;
    const int mask = d.ctl->mask;
    const E *__restrict__ Pe = reinterpret_cast<const E *>(d.P);
    E *__restrict__ Qe = reinterpret_cast<E *>(d.Q);
    E pq = E(0.0);
    const int l = xcd_runs((int)blockIdx.x, d.nblk, kStencilRun);
    const int j = xcd_remap(l, d.nblk);  // the partial that the general kernel gives these slices
    multi_stencil<K, W>(d, l * (kBlock / kWave) + (int)threadIdx.x / kWave, d.nblk * (kBlock / kWave), d.P,
                        [&] { return mask != 0; }, [&](int64_t t) { return Pe[t]; },
                        [&](int64_t t, int, E y, E p) {
                            Qe[t] = y;
#pragma unroll
                            for (int c = 0; c < Flat<K>::kCols; ++c) pq[c] = fma(y[c], p[c], pq[c]);
                        });
    if (mask != 0) block_partials_elem<K>(pq, sh, d.partials + (size_t)kPartPq * K * d.nblk, d.nblk, j);
}

// F_A: eta = p.q and alpha per running column; eta <= 0 stops the column.
static __global__ __launch_bounds__(kBlock) void k_m_fin_pq(MultiDesc d)
{
    __shared__ double red[kBlock / kWave];
    const int q = blockIdx.x;
    if (q >= d.K) return;
    SysState *st = d.st + q;
    if (st->status != SPK_RUNNING) return;
    const double eta = reduce_partials(col_part(d, kPartPq, q), d.nblk, red);
    if (threadIdx.x != 0) return;
    st->eta = eta;
    st->cmode = 0;
    if (!isfinite(eta)) st->status = SPK_DIVERGED_NANORINF;
    else if (eta <= 0.0) st->status = SPK_DIVERGED_INDEFINITE_MAT;
    else st->alpha = st->rho / eta;
    if (st->status != SPK_RUNNING) stop_column(d, q);
}

// B: R -= alpha Q for the running columns, per-block r.z and r.r (z = D^-1 r).
// 128^3, K = 8: 98 us with z stored and one element a lane -> 73.6 (420 MB).
template <int K>
__global__ __launch_bounds__(kBlock) void k_m_update(MultiDesc d)
{
    using E = typename Flat<K>::Elem;
    constexpr int C = Flat<K>::kCols;
    __shared__ double sh[(kBlock / kWave) * K];
    int j;
    if (multi_block(d, j) < 0) return;
    const int mask = d.ctl->mask;
    if (mask == 0) return;
    const int q = Flat<K>::col(threadIdx.x);
    bool run[C];
    double nal[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        run[c] = (mask >> (q + c)) & 1;
        nal[c] = run[c] ? -d.st[q + c].alpha : 0.0;
    }
    const E *__restrict__ Qe = reinterpret_cast<const E *>(d.Q);
    const double *__restrict__ dinv = d.dinv;
    E *__restrict__ Re = reinterpret_cast<E *>(d.Rv);
    struct In {
        E r, q;
        double dinv;
    };
    E rz = E(0.0), rr = E(0.0);
    int64_t e0, e1;
    flat_range(d, j, e0, e1);
    flat_walk<K>(e0, e1, [&](int64_t t, int64_t i) { return In{Re[t], Qe[t], dinv[i]}; },
                 [&](int64_t t, const In &v) {
                     E r = v.r;
#pragma unroll
                     for (int c = 0; c < C; ++c)
                         if (run[c]) {  // a stopped column keeps its r
                             const double ri = fma(nal[c], v.q[c], v.r[c]);
                             r[c] = ri;
                             rz[c] = fma(ri, v.dinv * ri, rz[c]);
                             rr[c] = fma(ri, ri, rr[c]);
                         }
                     Re[t] = r;
                 });
    block_partials_elem<K>(rz, sh, d.partials + (size_t)kPartRz * K * d.nblk, d.nblk, j);
    block_partials_elem<K>(rr, sh, d.partials + (size_t)kPartRr * K * d.nblk, d.nblk, j);
}

// F_B: per running column: iteration count, convergence, breakdowns, beta;
// cmode 2 (x and p updates) or 1 (the last x update), as in the single
// solve; a column that is not running gets cmode 0, so the p/x kernel of a
// later replay leaves it alone.
static __global__ __launch_bounds__(kBlock) void k_m_fin_update(MultiDesc d)
{
    __shared__ double red[kBlock / kWave];
    const int q = blockIdx.x;
    if (q >= d.K) return;
    SysState *st = d.st + q;
    if (st->status != SPK_RUNNING) {
        if (threadIdx.x == 0) st->cmode = 0;
        return;
    }
    double RZ, RR;
    reduce_partials2(col_part(d, kPartRz, q), col_part(d, kPartRr, q), d.nblk, red, RZ, RR);
    if (threadIdx.x != 0) return;
    const int k = ++st->iter;
    const double rn = sqrt(RR);
    st->rnorm = rn;
    st->cmode = 1;
    if (!isfinite(rn)) st->status = SPK_DIVERGED_NANORINF;
    else if (rn <= st->thresh)
        st->status = rn <= st->rtol * st->bnorm ? SPK_CONVERGED_RTOL : SPK_CONVERGED_ATOL;
    else if (k >= st->maxit) st->status = SPK_DIVERGED_ITS;
    else if (!isfinite(RZ)) st->status = SPK_DIVERGED_NANORINF;
    else if (RZ < 0.0) st->status = SPK_DIVERGED_INDEFINITE_PC;
    else if (RZ == 0.0) st->status = SPK_DIVERGED_BREAKDOWN;
    else { st->beta = RZ / st->rho; st->rho = RZ; st->cmode = 2; }
    if (st->status != SPK_RUNNING) stop_column(d, q);
}

// C: per column, cmode 2: x += alpha p, p = z + beta p; cmode 1: x += alpha p.
// It keeps no partial sums, so it runs on a grid of its own (kMultiPxBlocks
// at most): block b takes the b-th chunk of the flat n x K range, a multiple
// of 256 elements, in physical block order (a streaming pass gains nothing
// from XCD-contiguous ranges; on the 128^3 k = 8 block, 1024 blocks with
// those ranges took 131.5 us, 8192 in order 120.8; 111.4 with two elements a
// lane and z formed here: 690 MB at 6.2 TB/s).
constexpr int kMultiPxBlocks = 8192;
template <int K>
__global__ __launch_bounds__(kBlock) void k_m_px(MultiDesc d)
{
    using E = typename Flat<K>::Elem;
    constexpr int C = Flat<K>::kCols;
    const int q = Flat<K>::col(threadIdx.x);
    int cm[C], any = 0;
    double al[C], be[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        cm[c] = d.st[q + c].cmode;
        al[c] = d.st[q + c].alpha;
        be[c] = d.st[q + c].beta;
        any |= cm[c];
    }
    if (any == 0) return;  // no barrier follows
    E *__restrict__ Xe = reinterpret_cast<E *>(d.X);
    E *__restrict__ Pe = reinterpret_cast<E *>(d.P);
    const E *__restrict__ Re = reinterpret_cast<const E *>(d.Rv);
    const double *__restrict__ dinv = d.dinv;
    const int64_t nk = (int64_t)d.n * K;
    constexpr int64_t kStep = (int64_t)kBlock * C;
    const int64_t per = ((nk + gridDim.x - 1) / gridDim.x + kStep - 1) / kStep * kStep;
    const int64_t e0 = min(nk, (int64_t)blockIdx.x * per), e1 = min(nk, e0 + per);
    struct In {
        E p, x, r;
        double dinv;
    };
    flat_walk<K>(e0, e1, [&](int64_t t, int64_t i) { return In{Pe[t], Xe[t], Re[t], dinv[i]}; },
                 [&](int64_t t, const In &v) {
                     E x = v.x, p = v.p;
#pragma unroll
                     for (int c = 0; c < C; ++c) {
                         if (cm[c]) x[c] = fma(al[c], v.p[c], v.x[c]);
                         if (cm[c] == 2) p[c] = fma(be[c], v.p[c], v.dinv * v.r[c]);
                     }
                     Xe[t] = x;
                     Pe[t] = p;
                 });
}

// Per-column state for a new solve (FP64, one thread per column), all
// columns running until the setup kernels decide otherwise.
static __global__ void k_m_init(MultiDesc d, double rtol, double atol, int maxit)
{
    const int q = threadIdx.x;
    if (q < d.K) {
        SysState *st = d.st + q;
        *st = SysState{};
        st->status = SPK_RUNNING;
        st->phase = kPhaseInner;
        st->maxit = maxit;
        st->rtol = rtol;
        st->atol = atol;
    }
    if (q == 0) {
        d.ctl->mask = (1 << d.K) - 1;
        d.ctl->pad_ = 0;
    }
    if (q < d.K) d.st[q].cmode = 0;
}

// x = 0 for the columns in mask (right-hand sides that are zero).
template <int K>
__global__ void k_m_zero_cols(MultiDesc d, int32_t mask)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < d.n; i += gridDim.x * blockDim.x)
#pragma unroll
        for (int q = 0; q < K; ++q)
            if ((mask >> q) & 1) d.X[(size_t)i * K + q] = 0.0;
}

// The running-column mask to pinned host memory (one thread's store).
static __global__ void k_m_publish(const MultiCtl *ctl, int32_t *host)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) host[0] = ctl->mask;
}

}  // namespace spk
