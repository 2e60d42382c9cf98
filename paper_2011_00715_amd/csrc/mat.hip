// Matrix handle, SpMV dispatch, vector kernels and utilities of libspk.so.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include <time.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "runtime.hpp"
#include "scan.hpp"
#include "sellset.hpp"
#include "spmv.hpp"

namespace spk {

// ------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int hip_fail(hipError_t e, const char *what, const char *file, int line)
{
    // the runtime keeps an error until it is read: left there, the launch checks
    // of a fallback, or of the program's own kernels, would report it again
    (void)hipGetLastError();
    set_error("%s failed: %s (%s:%d)", what, hipGetErrorString(e), file, line);
    return e == hipErrorOutOfMemory ? SPK_ENOMEM : SPK_EHIP;
}

// ------------------------------------------------------------------ analysis kernels
__global__ void k_row_stats(int n, int64_t nnz, const int32_t *__restrict__ rowptr,
                            RowStats *__restrict__ out)
{
    __shared__ int32_t hist[33];
    __shared__ unsigned long long s1, s2;
    __shared__ int32_t mx, mn, bad, tmax[6];
    if (threadIdx.x < 33) hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) { s1 = 0; s2 = 0; mx = 0; mn = 0x7fffffff; bad = 0; }
    if (threadIdx.x < 6) tmax[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long a1 = 0, a2 = 0;
    int amx = 0, amn = 0x7fffffff, abad = 0, bin0 = 0, cnt = 0;
    int at[6] = {0, 0, 0, 0, 0, 0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int64_t a = rowptr[i], e = rowptr[i + 1];
        if (e < a || a < 0 || e > nnz || (i == 0 && a != 0) || (i == n - 1 && e != nnz)) {
            ++abad;
            continue;
        }
        const int len = (int)(e - a);
        a1 += (unsigned long long)len;
        a2 += (unsigned long long)len * (unsigned long long)len;
        amx = max(amx, len);
        amn = min(amn, len);
        const int bin = len == 0 ? 0 : 32 - __clz(len);
        if (bin != bin0) {  // a thread's rows mostly fall into one bin
            if (cnt) atomicAdd(&hist[bin0], cnt);
            bin0 = bin;
            cnt = 0;
        }
        ++cnt;
#pragma unroll
        for (int t = 0; t < 6; ++t) {
            const int R = t == 0 ? 256 : (t == 1 ? 128 : (t == 2 ? 64 : (t == 3 ? 32 : (t == 4 ? 16 : 8))));
            if (i % R == 0) {
                const int ie = min(i + R, n);
                const int64_t te = rowptr[ie];
                if (te >= a && te <= nnz) at[t] = max(at[t], (int)(te - a));
            }
        }
    }
    // one lane per wavefront: on one LDS address the atomics of a block's
    // threads queue up (192 us of 7-point 128^3)
    auto wsum = [](unsigned long long v) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
        return v;
    };
    auto wmax = [](int v) {
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
        return v;
    };
    a1 = wsum(a1);
    a2 = wsum(a2);
    abad = (int)wsum((unsigned long long)abad);
    amx = wmax(amx);
    amn = -wmax(-amn);
#pragma unroll
    for (int t = 0; t < 6; ++t) at[t] = wmax(at[t]);
    if (cnt) atomicAdd(&hist[bin0], cnt);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&s1, a1);
        atomicAdd(&s2, a2);
        atomicMax(&mx, amx);
        atomicMin(&mn, amn);
        atomicAdd(&bad, abad);
#pragma unroll
        for (int t = 0; t < 6; ++t) atomicMax(&tmax[t], at[t]);
    }
    __syncthreads();
    if (threadIdx.x < 33 && hist[threadIdx.x]) atomicAdd(&out->hist[threadIdx.x], hist[threadIdx.x]);
    if (threadIdx.x < 6) atomicMax(&out->tile_max[threadIdx.x], tmax[threadIdx.x]);
    if (threadIdx.x == 0) {
        atomicAdd(&out->sum_len, s1);
        atomicAdd(&out->sum_len2, s2);
        atomicMax(&out->max_len, mx);
        atomicMin(&out->min_len, mn);
        atomicAdd(&out->bad_rowptr, bad);
    }
}

// Column range and (optionally) strict ascending order; needs a valid rowptr.
// Entries of a SELL-64 layout: one thread per slice of 64 rows adds 64 x the
// slice's longest row (rowptr already validated).
__global__ void k_slice_pad(int n, const int32_t *__restrict__ rowptr, RowStats *__restrict__ out)
{
    const int ns = (n + 63) / 64;
    unsigned long long acc = 0;
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < ns; s += gridDim.x * blockDim.x) {
        const int r0 = s * 64, r1 = min(r0 + 64, n);
        int mx = 0;
        int prev = rowptr[r0];
        for (int i = r0; i < r1; ++i) {
            const int e = rowptr[i + 1];
            mx = max(mx, e - prev);
            prev = e;
        }
        acc += 64ULL * (unsigned long long)mx;
    }
    if (acc) atomicAdd(&out->sell_padded, acc);
}

__global__ void k_check_cols(int n, const int32_t *__restrict__ rowptr,
                             const int32_t *__restrict__ col, int check_sorted,
                             RowStats *__restrict__ out)
{
    int badc = 0, uns = 0, md = 0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        int prev = -1;
        for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
            const int c = col[k];
            if (c < 0 || c >= n) ++badc;
            if (check_sorted && c <= prev) ++uns;
            prev = c;
            md = max(md, abs(c - i));
        }
    }
    if (badc) atomicAdd(&out->bad_col, badc);
    if (uns) atomicAdd(&out->unsorted, uns);
    if (md) atomicMax(&out->max_delta, md);
}

// dinv_i = 1 / a_ii (duplicates of the diagonal are summed).
__global__ void k_diag_inv(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                           const double *__restrict__ val, double *__restrict__ dinv,
                           RowStats *__restrict__ out)
{
    int bad = 0;
    double gmax = 0.0;  // Gershgorin bound of D^-1 A: max_i sum_j |a_ij| / |a_ii|
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        double d = 0.0, sabs = 0.0;
        for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
            const double v = val[k];
            sabs += fabs(v);
            if (col[k] == i) d += v;
        }
        if (d == 0.0) { ++bad; dinv[i] = 0.0; }
        else {
            dinv[i] = 1.0 / d;
            gmax = fmax(gmax, sabs / fabs(d));
        }
    }
    if (bad) atomicAdd(&out->zero_diag, bad);
    // non-negative doubles order like their bit patterns: one atomic per wave
    gmax = fmax(gmax, 0.0);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) gmax = fmax(gmax, __shfl_xor(gmax, off, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0 && gmax > 0.0)
        atomicMax(&out->gersh_bits, (unsigned long long)__double_as_longlong(gmax));
}

__global__ void k_to_f32(int64_t m, const double *__restrict__ a, float *__restrict__ b)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        b[i] = (float)a[i];
}

// ------------------------------------------------------------------ vector kernels
__global__ void k_fill0(int64_t m, double *__restrict__ a)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0.0;
}

// out = f(a, b) element by element, kPairs: two a lane (16-byte aligned
// operands; an odd last element is the last lane's alone).  One launch lane per
// element or pair.  1.9 M elements (cached): axpy 9.6 -> 8.4 us,
// aypx 8.7 -> 7.5, the pointwise product 9.4 -> 8.2.
template <bool kPairs, class F>
__global__ __launch_bounds__(kBlock) void k_map(int n, const double *a, const double *b, double *out, F f)
{
    typedef double D2 __attribute__((ext_vector_type(2)));
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if constexpr (kPairs) {
        if (2 * t + 1 < n) {
            const D2 x = reinterpret_cast<const D2 *>(a)[t], y = reinterpret_cast<const D2 *>(b)[t];
            reinterpret_cast<D2 *>(out)[t] = D2{f(x[0], y[0]), f(x[1], y[1])};
        } else if (2 * t < n) {
            out[2 * t] = f(a[2 * t], b[2 * t]);
        }
    } else {
        for (int64_t i = t; i < n; i += (int64_t)gridDim.x * blockDim.x) out[i] = f(a[i], b[i]);
    }
}

struct Axpy {
    double alpha;
    __device__ double operator()(double x, double y) const { return fma(alpha, x, y); }
};
struct Aypx {
    double beta;
    __device__ double operator()(double x, double y) const { return fma(beta, y, x); }
};
struct Mul {
    __device__ double operator()(double d, double r) const { return d * r; }
};

// Single-pass dots: per-block partials of x.y (and x.w) over a contiguous
// chunk per block; k_dot_fin sums them in a fixed order.  A lane's next
// kDotAhead elements are loaded before the first is added: a chunk is a few
// steps long, and one load a step waited out the memory's latency each time
// (1.9 M elements, cached: 8.7 -> 7.2 to 8.0 us).  Two dots gain from that at
// every size (2^24: 87.4 us with one element ahead, 77.9 with four); a single
// one of longer chunks loses by it (nrm2 of 2^23 15.1 against 16.4, x.y of 2^25
// 91.7 against 95.2).
constexpr int kDotAhead = 4;
constexpr int kDotAheadMax = 1 << 22;  // elements of a single dot, exclusive
template <int kAhead>
__global__ __launch_bounds__(kBlock) void k_dot(int n, const double *__restrict__ x,
                                                const double *__restrict__ y,
                                                const double *__restrict__ w,
                                                double *__restrict__ part)
{
    __shared__ double red[kBlock / kWave];
    const int nb = gridDim.x;
    const int j = xcd_remap(blockIdx.x, nb);
    const int64_t chunk = ((int64_t)n + nb - 1) / nb;
    const int rb = (int)min((int64_t)n, j * chunk);
    const int re = (int)min((int64_t)n, (j + 1) * chunk);
    double a = 0.0, b = 0.0;
    for (int64_t i0 = rb + (int)threadIdx.x; i0 < re; i0 += kAhead * kBlock) {
        double xv[kAhead], yv[kAhead], wv[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t i = min(i0 + u * kBlock, (int64_t)re - 1);  // past the end: the last one, unused
            xv[u] = x[i];
            yv[u] = y[i];
        }
        if (w) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) wv[u] = w[min(i0 + u * kBlock, (int64_t)re - 1)];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (i0 + u * kBlock >= re) break;
            a = fma(xv[u], yv[u], a);
            if (w) b = fma(xv[u], wv[u], b);
        }
    }
    a = block_sum(a, red);
    if (w) b = block_sum(b, red);
    if (threadIdx.x == 0) { part[j] = a; part[nb + j] = b; }
}

// result[0] = x.y, result[1] = x.w (if two), or ||x|| (mode 2).
__global__ __launch_bounds__(kBlock) void k_dot_fin(int nb, int two, int mode,
                                                    const double *__restrict__ part,
                                                    double *__restrict__ result)
{
    __shared__ double red[kBlock / kWave];
    const double A = reduce_partials(part, nb, red);
    const double B = two ? reduce_partials(part + nb, nb, red) : 0.0;
    if (threadIdx.x == 0) {
        if (mode == 2) result[0] = sqrt(A);
        else {
            result[0] = A;
            if (two) result[1] = B;
        }
    }
}

typedef double dvec2 __attribute__((ext_vector_type(2)));

// Bandwidth calibration: plain stream copy (2 accesses per entry, Sec. 5.1),
// one 16-byte pair per thread, launched with grid_stream.
__global__ __launch_bounds__(kBlock) void k_copy(int64_t m, const dvec2 *__restrict__ a,
                                                 dvec2 *__restrict__ b)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        __builtin_nontemporal_store(__builtin_nontemporal_load(a + i), b + i);
}

// Cache eviction by reading: the Infinity Cache ends up holding clean lines
// of the scratch buffer, so the next kernel finds none of its data cached and
// pays no write-back of dirty lines left by the eviction itself.  The store
// only happens for a sum no real buffer of finite values produces; it keeps
// the loads from being optimised away.
__global__ __launch_bounds__(kBlock) void k_evict(int64_t m, dvec2 *__restrict__ b)
{
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x) {
        const dvec2 v = b[i];
        s += v.x + v.y;
    }
    if (s == -1.0e308) b[0] = dvec2{s, s};
}

// ------------------------------------------------------------------ SpMV dispatch
template <class V, int L>
static void launch_vector_l(const spk_mat *A, const V *val, const V *x, V *y, hipStream_t s,
                            const SysState *gst, int gmode)
{
    constexpr int rpb = kBlock / L;
    int grid = ceil_div(A->n, rpb);
    if (grid > kMaxBlocksSingle) grid = kMaxBlocksSingle;
    if (grid >= kXcd) grid -= grid % kXcd;
    hipLaunchKernelGGL((k_spmv_vector<V, L>), dim3(grid), dim3(kBlock), 0, s, A->n, A->rowptr,
                       A->col, val, x, y, gst, gmode);
}

template <class V>
int launch_spmv(const spk_mat *A, const V *val, const V *x, V *y, hipStream_t s,
                const SysState *gst, int gmode)
{
    if (A->n == 0) return SPK_OK;
    switch (A->kernel) {
    case SPK_KERNEL_STREAM:
        if (gst) {
            set_error("internal: gated stream SpMV");
            return SPK_EINVAL;
        }
        hipLaunchKernelGGL((k_spmv_stream<V>), dim3(A->nblk), dim3(kBlock), 0, s, A->n, A->R,
                           A->ntiles, A->nblk, A->rowptr, A->col, val, x, y);
        break;
    case SPK_KERNEL_VECTOR:
        switch (A->lanes) {
        case 1: launch_vector_l<V, 1>(A, val, x, y, s, gst, gmode); break;
        case 2: launch_vector_l<V, 2>(A, val, x, y, s, gst, gmode); break;
        case 4: launch_vector_l<V, 4>(A, val, x, y, s, gst, gmode); break;
        case 8: launch_vector_l<V, 8>(A, val, x, y, s, gst, gmode); break;
        case 16: launch_vector_l<V, 16>(A, val, x, y, s, gst, gmode); break;
        case 32: launch_vector_l<V, 32>(A, val, x, y, s, gst, gmode); break;
        default: launch_vector_l<V, 64>(A, val, x, y, s, gst, gmode); break;
        }
        break;
    case SPK_KERNEL_SELL: {
        if (gst || !A->sell_cw) {
            set_error("internal: gated SELL SpMV or no SELL layout");
            return SPK_EINVAL;
        }
        const SellView sv{A->sell_ptr, A->sell_col, A->sell_len, A->sell_plain_spmv, A->sell_len16, A->sell_perm,
                          A->sell_mask};
        const V *sval = std::is_same<V, double>::value ? (const V *)A->sell_val : (const V *)A->sell_val32;
        (void)val;
        // up to one wavefront per slice
        const dim3 grid(std::max(1, std::min(ceil_div(ceil_div(A->n, kSell), kBlock / kWave), 16384)));
        const int n = A->n;
        with_sell(A, [&](auto ci, auto uc) {
            using CI = decltype(ci);
            constexpr int U = decltype(uc)::value;
            hipLaunchKernelGGL((k_spmv_sell<V, CI, U>), grid, dim3(kBlock), 0, s, n, sv, sval, x, y);
        });
        break;
    }
    case SPK_KERNEL_SLICED:
        return launch_sliced<V>(A, x, y, s, gst, gmode);
    case SPK_KERNEL_MERGE: {
        V *cv = reinterpret_cast<V *>(A->carry_val);
        hipLaunchKernelGGL((k_spmv_merge<V>), dim3(A->mtiles), dim3(kBlock), 0, s, A->n,
                           (int)A->nnz, A->rowptr, A->col, val, x, y, A->tile_row, A->tile_k,
                           A->carry_row, cv, gst, gmode);
        hipLaunchKernelGGL((k_merge_fixup<V>), dim3(ceil_div(A->mtiles, kBlock)), dim3(kBlock), 0,
                           s, A->n, A->mtiles, A->carry_row, (const V *)cv, y, gst, gmode);
        break;
    }
    default:
        set_error("internal: unknown kernel %d", A->kernel);
        return SPK_EINVAL;
    }
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

template int launch_spmv<double>(const spk_mat *, const double *, const double *, double *,
                                 hipStream_t, const SysState *, int);
template int launch_spmv<float>(const spk_mat *, const float *, const float *, float *,
                                hipStream_t, const SysState *, int);

// Elementwise kernels: one element per thread and one block per 256 of them
// (up to 2^22 blocks, grid-stride beyond).  On gfx950 a launch of many
// short blocks streams faster than a grid-stride loop over a resident grid
// (2 GiB copy: 6.6 against 5.0 TB/s with 8192 blocks).
static int grid_stream(int64_t m)
{
    int64_t g = (m + kBlock - 1) / kBlock;
    if (g > (1 << 22)) g = 1 << 22;
    if (g < 1) g = 1;
    return (int)g;
}

// Pairs where the operands (at most three vectors) stay in the Infinity Cache;
// streamed from HBM one element a lane is the faster by 2 % (2^27 elements: 537
// against 549 us).
constexpr int kPairsMax = 1 << 23;

template <class F>
static void launch_map(int n, const double *a, const double *b, double *out, F f, void *stream)
{
    const int64_t pairs = ((int64_t)n + 1) / 2;
    if (n <= kPairsMax && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)out) & 15) == 0)
        hipLaunchKernelGGL((k_map<true, F>), dim3((unsigned)((pairs + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                           (hipStream_t)stream, n, a, b, out, f);
    else
        hipLaunchKernelGGL((k_map<false, F>), dim3(grid_stream(n)), dim3(kBlock), 0, (hipStream_t)stream, n, a, b, out,
                           f);
}

static int grid_for(int64_t m)
{
    int64_t g = (m + kBlock - 1) / kBlock;
    if (g > kMaxBlocksSingle) g = kMaxBlocksSingle;
    if (g < 1) g = 1;
    return (int)g;
}

void update_info(spk_mat *A)
{
    spk_mat_info &I = A->info;
    const RowStats &S = A->stats;
    I.n = A->n;
    I.nnz = A->nnz;
    I.kernel = A->kernel == SPK_KERNEL_SELL && A->sell_sigma ? SPK_KERNEL_SELL_SIGMA : A->kernel;
    I.sell_sigma = A->kernel == SPK_KERNEL_SELL ? A->sell_sigma : 0;
    I.lanes = A->kernel == SPK_KERNEL_SLICED ? (A->xs_merge ? kMergeItems : A->lanes)
              : A->kernel == SPK_KERNEL_VECTOR ? A->lanes
              : A->kernel == SPK_KERNEL_STREAM ? A->R
              : A->kernel == SPK_KERNEL_SELL ? (A->sell_mask ? 0 : 8 * A->sell_cw) : kMergeItems;
    I.has_f32 = A->val32 != nullptr;
    I.row_min = A->n ? S.min_len : 0;
    I.row_max = S.max_len;
    const double n = A->n > 0 ? (double)A->n : 1.0;
    I.row_mean = (double)S.sum_len / n;
    const double var = (double)S.sum_len2 / n - I.row_mean * I.row_mean;
    I.row_cv = I.row_mean > 0 ? sqrt(var > 0 ? var : 0) / I.row_mean : 0.0;
    // percentiles: upper bound of the log2 bin holding the 50% / 99% rank
    int64_t acc = 0;
    I.row_p50 = I.row_p99 = 0;
    bool got50 = false;
    for (int b = 0; b < 33; ++b) {
        acc += S.hist[b];
        const int ub = b == 0 ? 0 : (int)((1ll << b) - 1);
        if (!got50 && acc * 2 >= A->n) { I.row_p50 = std::min(ub, S.max_len); got50 = true; }
        if (acc * 100 >= (int64_t)A->n * 99) { I.row_p99 = std::min(ub, S.max_len); break; }
    }
    const int64_t nn = A->n, nz = A->nnz;
    I.bytes_spmv_f64 = 12 * nz + 4 * (nn + 1) + 16 * nn;
    I.bytes_spmv_f32 = 8 * nz + 4 * (nn + 1) + 8 * nn;
    I.bytes_pcg_iter_f64 = 12 * nz + 4 * (nn + 1) + 88 * nn;
    I.bytes_pcg_iter_f32 = 8 * nz + 4 * (nn + 1) + 44 * nn;
    I.device_bytes = A->bytes + (A->ws ? A->ws->bytes : 0);
    I.zero_diag_rows = S.zero_diag;
    I.cached_loads = A->kernel == SPK_KERNEL_SELL ? (A->sell_plain & 3) | (A->sell_plain_spmv & 3) << 2 : 0;
    double g = 0.0;
    memcpy(&g, &S.gersh_bits, sizeof g);  // bits of a non-negative double
    I.gershgorin = S.zero_diag ? 0.0 : g;
    if (A->kernel == SPK_KERNEL_SELL && A->sell_cw) {
        const int64_t ns = (nn + kSell - 1) / kSell;
        I.stored_nnz = A->sell_nnz;
        // offsets and row lengths (or shared offsets and row masks), plus the
        // row permutation of SELL-C-sigma
        const int64_t extra = A->sell_idx_bytes + (A->sell_perm ? 4 * nn : 0) + (A->sell_ptr ? 4 * (ns + 1) : 0);
        I.format_bytes_spmv_f64 = 8 * A->sell_nnz + 16 * nn + extra;
        I.format_bytes_spmv_f32 = 4 * A->sell_nnz + 8 * nn + extra;
    } else if (A->kernel == SPK_KERNEL_SLICED && A->xs_merge && A->bn_slab) {
        // per entry the column within its bin, the value, the place in its tile
        // and the product written and read; per tile its segments' starts
        I.stored_nnz = nz;
        const int64_t per = 4 * (nn + 1) + 8 * (int64_t)A->bn_tiles * A->bn_bins;
        I.format_bytes_spmv_f64 = 28 * nz + 16 * nn + per;
        I.format_bytes_spmv_f32 = 16 * nz + 8 * nn + per;
    } else if (A->kernel == SPK_KERNEL_SLICED && A->xs_ptr) {
        // stacked slices: 8n + 1 row pointers; the 8n partial products are
        // written once and read once by the summing pass
        I.stored_nnz = nz;
        I.format_bytes_spmv_f64 = 12 * nz + 4 * (8 * nn + 1) + 8 * nn + 2 * 8 * 8 * nn + 8 * nn;
        I.format_bytes_spmv_f32 = 8 * nz + 4 * (8 * nn + 1) + 4 * nn + 2 * 4 * 8 * nn + 4 * nn;
    } else {
        I.stored_nnz = nz;
        I.format_bytes_spmv_f64 = I.bytes_spmv_f64;
        I.format_bytes_spmv_f32 = I.bytes_spmv_f32;
    }
}

int ensure_f32(spk_mat *A, hipStream_t s)
{
    if (A->sell_cw && !A->sell_val32 && A->sell_nnz > 0) {
        SPK_HIP(hipMalloc(&A->sell_val32, sizeof(float) * A->sell_nnz));
        hipLaunchKernelGGL(k_to_f32, dim3(grid_for(A->sell_nnz)), dim3(kBlock), 0, s, A->sell_nnz,
                           A->sell_val, A->sell_val32);
        SPK_HIP(hipGetLastError());
        A->bytes += 4 * A->sell_nnz;
    }
    if (A->xs_ptr || A->bn_slab) {
        const int rc = ensure_sliced_f32(A, s);
        if (rc) return rc;
    }
    if (A->val32 || A->n == 0) return SPK_OK;
    // val32 says that both are there
    if (!A->dinv32) SPK_HIP(hipMalloc(&A->dinv32, sizeof(float) * A->n));
    SPK_HIP(hipMalloc(&A->val32, sizeof(float) * (A->nnz > 0 ? A->nnz : 1)));
    A->bytes += 4 * A->nnz + 4 * (int64_t)A->n;
    if (A->nnz > 0)
        hipLaunchKernelGGL(k_to_f32, dim3(grid_for(A->nnz)), dim3(kBlock), 0, s, A->nnz, A->val,
                           A->val32);
    hipLaunchKernelGGL(k_to_f32, dim3(grid_for(A->n)), dim3(kBlock), 0, s, (int64_t)A->n, A->dinv,
                       A->dinv32);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

static int pow2_ceil(double v)
{
    int L = 1;
    while (L < v && L < 64) L <<= 1;
    return L;
}

// Merge-path diagonals are int32: n + nnz must stay below 2^31.
static bool merge_fits(const spk_mat *A) { return (int64_t)A->n + A->nnz < 0x7fff0000LL; }

// Row-length statistics -> kernel family (stream for short, even rows; vector
// for long, even rows; merge-path for skewed lengths).
// The sliced layout pays when x does not fit one XCD's 4 MB L2 and rows
// reach across it (scattered columns).  For 4M skewed power-law rows of 32
// entries on average 0.90 ms binned and 1.14 with the merge path over the
// slices against 1.94 ms (merge); lanes per slice row take 1.95 ms.  Below the
// line the product gains little (270 k rows of 32, FP64: 72 us against 65 of the
// stream kernel; 450 k power-law rows: 104 against 116) for a copy of the matrix.
// Banded matrices keep their x window in L2 anyway.
static bool sliced_wanted(const spk_mat *A)
{
    const double mean = A->n ? (double)A->stats.sum_len / A->n : 0.0;
    return sliced_fits(A) && A->n >= (1 << 19) && mean >= 8.0 &&
           (int64_t)A->stats.max_delta * kXcd >= A->n && (!sliced_skewed(A) || sliced_merge_fits(A));
}

static void choose_kernel(spk_mat *A, bool allow_sell = true, bool allow_sliced = true)
{
    const RowStats &S = A->stats;
    const double mean = A->n ? (double)S.sum_len / A->n : 0.0;
    const int cap = TileLds<double>::kCap;
    int R = 0;
    for (int t = 0; t < 6; ++t)
        if (S.tile_max[t] <= cap) { R = kTileRs[t]; break; }
    // SELL-64: short rows of similar length within each slice (stencils).
    // No LDS staging; column offsets shared per slice where the slices' rows
    // use at most 32 of them (8 bytes per FP64 nonzero and 4 per row instead
    // of CSR's 12), else int16 offsets per entry in a band of +-32767 (10
    // bytes; wider bands keep int32 offsets and still beat the stream
    // kernel: 171 against 195 us on a 200^3 7-point stencil)
    const bool sell_ok = allow_sell && A->n >= kSell && S.max_len <= 64 &&
                         (double)S.sell_padded <= 1.15 * (double)A->nnz &&
                         S.sell_padded < 0x7fff0000ULL;
    if (sell_ok) {
        A->kernel = SPK_KERNEL_SELL;
        A->R = 256;
    } else if (S.max_len <= 64 && R >= 32) {
        A->kernel = SPK_KERNEL_STREAM;
        A->R = R;
    } else if ((mean >= 8 && S.max_len <= 8 * mean + 8) || !merge_fits(A)) {
        A->kernel = SPK_KERNEL_VECTOR;
        A->lanes = pow2_ceil(mean < 2 ? 2 : mean);
        A->R = 256;
    } else {
        A->kernel = SPK_KERNEL_MERGE;
        A->R = 256;
    }
    if (allow_sliced && sliced_wanted(A)) {
        A->kernel = SPK_KERNEL_SLICED;
        A->lanes = sliced_lanes(A);
        A->xs_merge = sliced_merge_fits(A) ? 1 : 0;
        A->R = 256;
    }
}

static int apply_partition(spk_mat *A)
{
    A->ntiles = ceil_div(A->n, A->R);
    A->nblk = pick_nblk(A->ntiles, A->kernel == SPK_KERNEL_SELL ? kPcgBlocksSell : kMaxBlocksSingle);
    return SPK_OK;
}

static int setup_merge(spk_mat *A, hipStream_t s)
{
    if (A->tile_row) return SPK_OK;
    const int64_t items = (int64_t)A->n + A->nnz;
    A->mtiles = (int)((items + kMergeItems - 1) / kMergeItems);
    const int mt = A->mtiles > 0 ? A->mtiles : 1;
    hipError_t e = hipMalloc(&A->tile_row, sizeof(int32_t) * (mt + 1));
    if (e == hipSuccess) e = hipMalloc(&A->tile_k, sizeof(int32_t) * (mt + 1));
    if (e == hipSuccess) e = hipMalloc(&A->carry_row, sizeof(int32_t) * mt);
    if (e == hipSuccess) e = hipMalloc(&A->carry_val, sizeof(double) * mt);
    if (e != hipSuccess) {  // all four or none: tile_row says that they are there
        hipFree(A->tile_row);
        hipFree(A->tile_k);
        hipFree(A->carry_row);
        hipFree(A->carry_val);
        A->tile_row = A->tile_k = A->carry_row = nullptr;
        A->carry_val = nullptr;
        return hip_fail(e, "merge path", __FILE__, __LINE__);
    }
    A->bytes += (int64_t)mt * 20 + 8;
    hipLaunchKernelGGL(k_merge_partition, dim3(ceil_div(A->mtiles + 1, kBlock)), dim3(kBlock), 0, s,
                       A->n, (int)A->nnz, A->rowptr, A->mtiles, kMergeItems, A->tile_row, A->tile_k);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

void free_workspace(spk_mat *A);

static void free_sell(spk_mat *A)
{
    if (A->sell_cw) {
        const int64_t ns = (A->n + kSell - 1) / kSell;
        A->bytes -= (A->sell_ptr ? 4 * (ns + 1) : 0) + 8 * A->sell_nnz + A->sell_idx_bytes;
        if (A->sell_perm) A->bytes -= 4ll * A->n;
        if (A->sell_val32) A->bytes -= 4 * A->sell_nnz;
    }
    hipFree(A->sell_mask);
    A->sell_mask = nullptr;
    A->sell_idx_bytes = 0;
    A->sell_req = -1;
    hipFree(A->sell_ptr);
    hipFree(A->sell_col);
    hipFree(A->sell_len);
    hipFree(A->sell_len16);
    hipFree(A->sell_perm);
    hipFree(A->sell_val);
    hipFree(A->sell_val32);
    A->sell_ptr = nullptr;
    A->sell_col = nullptr;
    A->sell_len = nullptr;
    A->sell_len16 = nullptr;
    A->sell_perm = nullptr;
    A->sell_val = nullptr;
    A->sell_val32 = nullptr;
    A->sell_cw = 0;
    A->sell_sigma = 0;
    A->sell_nnz = 0;
    A->sell_plain = 0;
    A->sell_plain_spmv = 0;
}


// The shared-offset layout of rows in matrix order, built on the device:
// every slice's rows must have strictly increasing columns and use between
// them at most kSellSharedMax distinct offsets, and the padding may grow by at
// most 1/16 over the per-lane layout.  *fits says whether it is so; if not,
// nothing is left behind.  Slice s spans 64 u[s] elements (u: the list
// lengths); its offsets sit at element sell_ptr[s] / 64 of sell_col (int32).
// With may_unify a matrix of one value per offset stores one list for all
// slices (kSellUniform), if that leaves the gathers of positions that rows do
// not use below a quarter.
static int build_sell_shared(spk_mat *A, hipStream_t s, bool may_unify, bool *fits)
{
    *fits = false;
    const int n = A->n;
    const int ns = ceil_div(n, kSell);
    const int g = scan_blocks(ns);
    struct Temp {
        void *p[5] = {};
        SharedStats *host = nullptr;
        ~Temp()
        {
            for (void *q : p) hipFree(q);
            hipHostFree(host);
        }
    } t;
    const size_t sizes[5] = {sizeof(SharedStats), sizeof(int32_t) * (size_t)ns,
                             sizeof(int32_t) * (size_t)ns * kSellSharedMax, sizeof(int32_t) * ((size_t)ns + 1),
                             sizeof(long long) * ((size_t)g + 1)};
    for (int i = 0; i < 5; ++i) SPK_HIP(hipMalloc(&t.p[i], sizes[i]));
    SPK_HIP(hipHostMalloc((void **)&t.host, sizeof(SharedStats), hipHostMallocDefault));
    SPK_HIP(hipMalloc(&A->sell_mask, sizeof(uint32_t) * (size_t)n));
    auto *stats = (SharedStats *)t.p[0];
    auto *width = (int32_t *)t.p[1], *list = (int32_t *)t.p[2], *base = (int32_t *)t.p[3];
    const int blocks = std::min(ceil_div(ns, kBlock / kWave), kMaxBlocksSingle);
    *t.host = SharedStats{};
    std::fill(t.host->offs, t.host->offs + kSell, kNoOffset);
    SPK_HIP(hipMemcpyAsync(stats, t.host, sizeof(SharedStats), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_shared_lists, dim3(blocks), dim3(kBlock), 0, s, n, A->rowptr, A->col, width, list,
                       A->sell_mask, stats);
    SPK_HIP(scan_exclusive(ns, width, base, (long long *)t.p[4], s));
    SPK_HIP(hipMemcpyAsync(t.host, stats, sizeof(SharedStats), hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    const SharedStats st = *t.host;
    int64_t acc = (int64_t)kSell * (int64_t)st.shared;
    if (st.bad || st.shared * 16 > st.lane * 17) {
        hipFree(A->sell_mask);
        A->sell_mask = nullptr;
        return SPK_OK;
    }
    *fits = true;
    if (acc > 0x7fffffffLL) { set_error("SELL layout exceeds 2^31 entries"); return SPK_EINVAL; }
    // one list for the whole matrix?
    StencilList l{};
    if (may_unify && !st.many) {
        std::vector<std::pair<int32_t, int32_t>> all;
        for (const unsigned long long v : st.offs)
            if (v != kNoOffset) all.emplace_back((int32_t)(v >> 32), (int32_t)v);
        std::sort(all.begin(), all.end());
        if ((int)all.size() <= kSellUniformMax && 4 * (uint64_t)all.size() * ns <= 5 * st.shared) {
            l.w = (int)all.size();
            for (int j = 0; j < l.w; ++j) {
                l.off[j] = all[j].first;
                l.entry[j] = all[j].second;
            }
        }
    }
    bool uniform = false;
    if (l.w > 0) {
        uint32_t *mask = nullptr;
        SPK_HIP(hipMalloc(&A->sell_col, sizeof(int32_t) * l.w));
        SPK_HIP(hipMalloc(&A->sell_val, sizeof(double) * l.w));
        SPK_HIP(hipMalloc(&mask, sizeof(uint32_t) * (size_t)n));
        hipLaunchKernelGGL(k_stencil_masks, dim3(std::min(ceil_div(2 * ns, kBlock / kWave), kMaxBlocksSingle)),
                           dim3(kBlock), 0, s, n, l, A->rowptr, A->col, A->val, mask, (int32_t *)A->sell_col,
                           A->sell_val, &stats->varied);
        hipError_t e = hipMemcpyAsync(&t.host->varied, &stats->varied, sizeof(int32_t), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        uniform = e == hipSuccess && t.host->varied == 0;
        if (uniform) std::swap(mask, A->sell_mask);
        hipFree(mask);
        if (e != hipSuccess) return hip_fail(e, "stencil masks", __FILE__, __LINE__);
        if (!uniform) {
            hipFree(A->sell_col);
            hipFree(A->sell_val);
            A->sell_col = nullptr;
            A->sell_val = nullptr;
        }
    }
    // the load policy below is that of a value per entry either way
    const int64_t entries = acc, offsets = uniform ? l.w : (int64_t)st.shared;
    if (uniform) acc = l.w;
    const size_t m = acc > 0 ? (size_t)acc : 1;
    if (!uniform) {
        SPK_HIP(hipMalloc(&A->sell_ptr, sizeof(int32_t) * ((size_t)ns + 1)));
        SPK_HIP(hipMalloc(&A->sell_col, sizeof(int32_t) * (st.shared > 0 ? (size_t)st.shared : 1)));
        SPK_HIP(hipMalloc(&A->sell_val, sizeof(double) * m));
        hipLaunchKernelGGL(k_shared_pack, dim3(ceil_div((int64_t)(ns + 1) * kSellSharedMax, kBlock)), dim3(kBlock), 0,
                           s, ns, (const int32_t *)base, (const int32_t *)list, A->sell_ptr, (int32_t *)A->sell_col);
        hipLaunchKernelGGL(k_shared_fill, dim3(blocks), dim3(kBlock), 0, s, n, A->rowptr, A->val,
                           (const int32_t *)A->sell_ptr, (const uint32_t *)A->sell_mask, A->sell_val);
    }
    SPK_HIP(hipGetLastError());
    A->sell_cw = 4;
    A->sell_sigma = 0;
    A->sell_u = pick_sell_u(uniform ? l.w : st.widest);
    A->sell_nnz = acc;
    A->sell_idx_bytes = 4 * offsets + 4ll * n;
    // the load policy counts cw bytes per entry plus one byte per row:
    // here no bytes per entry and the rest of the index bytes in the budget
    const int64_t extra = 4 * (int64_t)st.shared + 3ll * n;
    A->sell_plain = A->stream_loads ? 0 : sell_load_policy(entries, 0, ns, n, 6, kIterCacheBudget - extra);
    A->sell_plain_spmv = A->stream_loads ? 0 : sell_load_policy(entries, 0, ns, n, 2, kSpmvCacheBudget - extra);
    if (uniform) {
        A->sell_plain |= kSellUniform | l.w << kSellWidthShift;
        A->sell_plain_spmv |= kSellUniform | l.w << kSellWidthShift;
    }
    A->bytes += (uniform ? 0 : 4 * ((int64_t)ns + 1)) + 8 * acc + A->sell_idx_bytes;
    if (A->val32) {
        SPK_HIP(hipMalloc(&A->sell_val32, sizeof(float) * m));
        hipLaunchKernelGGL(k_to_f32, dim3(grid_for((int64_t)m)), dim3(kBlock), 0, s, (int64_t)m, A->sell_val,
                           A->sell_val32);
        SPK_HIP(hipGetLastError());
        A->bytes += 4 * acc;
    }
    SPK_HIP(hipStreamSynchronize(s));  // the passes above read the temporaries
    return SPK_OK;
}

// Build the SELL-64 copy: slice widths from rowptr on the host (setup only),
// entries filled by one device lane per layout position.  cw: 2 (int16
// offsets), 4 (int32), 1 (offsets shared per slice; SPK_EINVAL when the
// matrix does not qualify) or 0 (shared when the matrix qualifies, else int16
// when every |col - row| fits, else int32).  sigma > 0 builds SELL-C-sigma:
// within each window of sigma rows the rows are ordered by length, longest
// first (ties in row order), so that the rows sharing a slice have similar
// lengths and the padding shrinks on skewed matrices; the layout then
// carries the permutation.  Rows longer than 255 entries store their
// lengths in 16 bits.
static int setup_sell(spk_mat *A, hipStream_t s, int cw, int sigma = 0)
{
    if (A->sell_cw && A->sell_req == cw && A->sell_sigma == sigma) return SPK_OK;
    const int req = cw;
    const bool try_shared = (cw == 0 || cw == 1) && sigma == 0 && A->n > 0 && A->stats.max_len <= kSellSharedMax;
    if (cw == 1 && !try_shared) {
        set_error("shared SELL offsets need rows in matrix order of at most %d entries", kSellSharedMax);
        return SPK_EINVAL;
    }
    if (cw == 0 || cw == 1) cw = A->stats.max_delta <= 32767 ? 2 : 4;
    if (cw == 2 && A->stats.max_delta > 32767) {
        set_error("column offsets up to %d do not fit int16", A->stats.max_delta);
        return SPK_EINVAL;
    }
    if (A->stats.max_len > 65535) {
        set_error("SELL needs rows of at most 65535 entries (max %d)", A->stats.max_len);
        return SPK_EINVAL;
    }
    free_sell(A);
    const int n = A->n;
    if (try_shared) {
        bool fits = false;
        const int rc = build_sell_shared(A, s, req == 0, &fits);
        if (rc != SPK_OK) return rc;
        if (fits) {
            A->sell_req = req;
            return SPK_OK;
        }
        if (req == 1) {
            set_error("the rows of a slice use more than %d distinct column offsets (or are unsorted)",
                      kSellSharedMax);
            return SPK_EINVAL;
        }
    }
    std::vector<int32_t> rp((size_t)n + 1);
    SPK_HIP(hipMemcpyAsync(rp.data(), A->rowptr, sizeof(int32_t) * ((size_t)n + 1), hipMemcpyDeviceToHost, s));
    SPK_HIP(hipStreamSynchronize(s));
    std::vector<int32_t> perm;
    if (sigma > 0) {
        perm.resize((size_t)n);
        for (int i = 0; i < n; ++i) perm[i] = i;
        for (int w0 = 0; w0 < n; w0 += sigma) {
            const int w1 = (int)std::min<int64_t>((int64_t)w0 + sigma, n);
            std::stable_sort(perm.begin() + w0, perm.begin() + w1, [&](int32_t x, int32_t y) {
                return rp[x + 1] - rp[x] > rp[y + 1] - rp[y];
            });
        }
    }
    auto rlen = [&](int j) {
        const int r = sigma > 0 ? perm[j] : j;
        return rp[r + 1] - rp[r];
    };
    const int ns = ceil_div(n, kSell);
    std::vector<int32_t> sp((size_t)ns + 1);
    int64_t acc = 0;
    int wmax = 0;
    for (int k = 0; k < ns; ++k) {
        int mx = 0;
        for (int j = k * kSell; j < std::min(n, (k + 1) * kSell); ++j) mx = std::max(mx, rlen(j));
        wmax = std::max(wmax, mx);
        sp[k] = (int32_t)acc;
        acc += (int64_t)kSell * mx;
        if (acc > 0x7fffffffLL) { set_error("SELL layout exceeds 2^31 entries"); return SPK_EINVAL; }
    }
    sp[ns] = (int32_t)acc;
    const bool len16 = A->stats.max_len > 255;
    const size_t m = acc > 0 ? (size_t)acc : 1;
    SPK_HIP(hipMalloc(&A->sell_ptr, sizeof(int32_t) * ((size_t)ns + 1)));
    SPK_HIP(hipMalloc(&A->sell_col, (size_t)cw * m));
    if (len16) SPK_HIP(hipMalloc(&A->sell_len16, sizeof(uint16_t) * (size_t)(n > 0 ? n : 1)));
    else SPK_HIP(hipMalloc(&A->sell_len, (size_t)(n > 0 ? n : 1)));
    if (sigma > 0) SPK_HIP(hipMalloc(&A->sell_perm, sizeof(int32_t) * (size_t)(n > 0 ? n : 1)));
    SPK_HIP(hipMalloc(&A->sell_val, sizeof(double) * m));
    SPK_HIP(hipMemcpyAsync(A->sell_ptr, sp.data(), sizeof(int32_t) * ((size_t)ns + 1), hipMemcpyHostToDevice, s));
    if (sigma > 0)
        SPK_HIP(hipMemcpyAsync(A->sell_perm, perm.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, s));
    if (cw == 2)
        hipLaunchKernelGGL(k_sell_fill<int16_t>, dim3(grid_for(n)), dim3(kBlock), 0, s, n, A->rowptr, A->col,
                           A->val, A->sell_ptr, (const int32_t *)A->sell_perm, (int16_t *)A->sell_col, A->sell_val,
                           A->sell_len, A->sell_len16);
    else
        hipLaunchKernelGGL(k_sell_fill<int32_t>, dim3(grid_for(n)), dim3(kBlock), 0, s, n, A->rowptr, A->col,
                           A->val, A->sell_ptr, (const int32_t *)A->sell_perm, (int32_t *)A->sell_col, A->sell_val,
                           A->sell_len, A->sell_len16);
    SPK_HIP(hipGetLastError());
    A->sell_cw = cw;
    A->sell_req = req;
    A->sell_sigma = sigma;
    A->sell_u = pick_sell_u(wmax);
    A->sell_nnz = acc;
    A->sell_idx_bytes = (int64_t)cw * acc + n + (len16 ? n : 0);
    const int64_t extra = (len16 ? n : 0) + (sigma > 0 ? 4ll * n : 0);
    A->sell_plain = A->stream_loads ? 0 : sell_load_policy(acc, cw, ns, n, 6, kIterCacheBudget - extra);
    A->sell_plain_spmv = A->stream_loads ? 0 : sell_load_policy(acc, cw, ns, n, 2, kSpmvCacheBudget - extra);
    A->bytes += 4 * ((int64_t)ns + 1) + 8 * acc + A->sell_idx_bytes + (sigma > 0 ? 4ll * n : 0);
    if (A->val32) {
        SPK_HIP(hipMalloc(&A->sell_val32, sizeof(float) * m));
        hipLaunchKernelGGL(k_to_f32, dim3(grid_for((int64_t)m)), dim3(kBlock), 0, s, (int64_t)m, A->sell_val,
                           A->sell_val32);
        SPK_HIP(hipGetLastError());
        A->bytes += 4 * acc;
    }
    // the (sigma-sorted) layout is read in the fill above: wait before the
    // host vectors go
    SPK_HIP(hipStreamSynchronize(s));
    return SPK_OK;
}

}  // namespace spk

using namespace spk;

// ================================================================== C ABI
extern "C" {

const char *spk_last_error(void) { return g_err; }

const char *spk_status_str(int st)
{
    switch (st) {
    case SPK_OK: return "SPK_OK";
    case SPK_EINVAL: return "SPK_EINVAL";
    case SPK_ENOMEM: return "SPK_ENOMEM";
    case SPK_EHIP: return "SPK_EHIP";
    case SPK_EZERODIAG: return "SPK_EZERODIAG";
    case SPK_EBUSY: return "SPK_EBUSY";
    case SPK_EBUDGET: return "SPK_EBUDGET";
    case SPK_ENOTFOUND: return "SPK_ENOTFOUND";
    }
    return "SPK_UNKNOWN_STATUS";
}

const char *spk_reason_str(int r)
{
    switch (r) {
    case SPK_CONVERGED_RTOL: return "CONVERGED_RTOL";
    case SPK_CONVERGED_ATOL: return "CONVERGED_ATOL";
    case SPK_RUNNING: return "RUNNING";
    case SPK_DIVERGED_ITS: return "DIVERGED_ITS";
    case SPK_DIVERGED_INDEFINITE_MAT: return "DIVERGED_INDEFINITE_MAT";
    case SPK_DIVERGED_INDEFINITE_PC: return "DIVERGED_INDEFINITE_PC";
    case SPK_DIVERGED_NANORINF: return "DIVERGED_NANORINF";
    case SPK_DIVERGED_BREAKDOWN: return "DIVERGED_BREAKDOWN";
    case SPK_DIVERGED_STAGNATION: return "DIVERGED_STAGNATION";
    }
    return "UNKNOWN_REASON";
}

double spk_now(void)
{
    struct timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    return (double)ts.tv_sec + 1e-9 * (double)ts.tv_nsec;
}

int spk_runtime_version(void)
{
    int v = 0;
    if (hipRuntimeGetVersion(&v) != hipSuccess) return -1;
    return v;
}

static int create_impl(int32_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colind,
                       const double *values, int memtype, uint32_t flags, hipStream_t s,
                       spk_mat *A)
{
    A->n = n;
    A->nnz = nnz;
    A->stream_loads = (flags & SPK_MAT_STREAM) != 0;
    SPK_HIP(hipGetDevice(&A->device));
    const bool borrow = (flags & SPK_MAT_BORROW) != 0;
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t nzb = nnz > 0 ? (size_t)nnz : 1;
    const size_t b_val = borrow ? 0 : up(sizeof(double) * nzb), b_col = borrow ? 0 : up(sizeof(int32_t) * nzb),
                 b_ptr = borrow ? 0 : up(sizeof(int32_t) * ((size_t)n + 1)), b_inv = sizeof(double) * (n > 0 ? n : 1);
    SPK_HIP(hipMalloc(&A->slab, b_val + b_col + b_ptr + b_inv));
    char *slab = (char *)A->slab;
    A->dinv = (double *)(slab + b_val + b_col + b_ptr);
    if (borrow) {
        A->own_csr = false;
        A->rowptr = const_cast<int32_t *>(rowptr);
        A->col = const_cast<int32_t *>(colind);
        A->val = const_cast<double *>(values);
    } else {
        A->val = (double *)slab;
        A->col = (int32_t *)(slab + b_val);
        A->rowptr = (int32_t *)(slab + b_val + b_col);
        A->bytes += 4 * ((int64_t)n + 1) + 12 * nnz;
        const hipMemcpyKind kind = memtype == SPK_MEM_HOST ? hipMemcpyHostToDevice
                                                           : hipMemcpyDeviceToDevice;
        if (memtype == SPK_MEM_HOST) {
            // stage through pinned memory in chunks (Response A4: pinned transfers)
            const size_t chunk = 64u << 20;
            char *pin = nullptr;
            SPK_HIP(hipHostMalloc((void **)&pin, chunk, hipHostMallocDefault));
            struct Part { void *dst; const void *src; size_t bytes; } parts[3] = {
                {A->rowptr, rowptr, sizeof(int32_t) * ((size_t)n + 1)},
                {A->col, colind, sizeof(int32_t) * (size_t)nnz},
                {A->val, values, sizeof(double) * (size_t)nnz}};
            int rc = SPK_OK;
            for (auto &pt : parts) {
                for (size_t off = 0; off < pt.bytes && rc == SPK_OK; off += chunk) {
                    const size_t len = std::min(chunk, pt.bytes - off);
                    memcpy(pin, (const char *)pt.src + off, len);
                    hipError_t e = hipMemcpyAsync((char *)pt.dst + off, pin, len,
                                                  hipMemcpyHostToDevice, s);
                    if (e == hipSuccess) e = hipStreamSynchronize(s);
                    if (e != hipSuccess) rc = hip_fail(e, "pinned upload", __FILE__, __LINE__);
                }
            }
            hipHostFree(pin);
            if (rc) return rc;
        } else {
            SPK_HIP(hipMemcpyAsync(A->rowptr, rowptr, sizeof(int32_t) * ((size_t)n + 1), kind, s));
            if (nnz > 0) {
                SPK_HIP(hipMemcpyAsync(A->col, colind, sizeof(int32_t) * nnz, kind, s));
                SPK_HIP(hipMemcpyAsync(A->val, values, sizeof(double) * nnz, kind, s));
            }
        }
    }
    A->bytes += 8 * (int64_t)n;

    // statistics + structural checks (memory safety of every later kernel)
    RowStats *dst = nullptr, *hst = nullptr;
    SPK_HIP(hipMalloc(&dst, sizeof(RowStats)));
    SPK_HIP(hipHostMalloc((void **)&hst, sizeof(RowStats), hipHostMallocDefault));
    RowStats init{};
    init.min_len = 0x7fffffff;
    int rc = SPK_OK;
    auto fail = [&](int code) { rc = code; };
    do {
        hipError_t e = hipMemcpyAsync(dst, &init, sizeof(RowStats), hipMemcpyHostToDevice, s);
        if (e != hipSuccess) { fail(hip_fail(e, "stats init", __FILE__, __LINE__)); break; }
        if (n > 0)
            hipLaunchKernelGGL(k_row_stats, dim3(grid_for(n)), dim3(kBlock), 0, s, n, nnz, A->rowptr,
                               dst);
        e = hipMemcpyAsync(hst, dst, sizeof(RowStats), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { fail(hip_fail(e, "row statistics", __FILE__, __LINE__)); break; }
        if (hst->bad_rowptr) {
            set_error("malformed rowptr: %d rows out of order or outside [0, nnz] "
                      "(rowptr[0] must be 0 and rowptr[n] = nnz)", hst->bad_rowptr);
            fail(SPK_EINVAL);
            break;
        }
        if (n > 0) {
            hipLaunchKernelGGL(k_slice_pad, dim3(grid_for(ceil_div(n, 64))), dim3(kBlock), 0, s, n,
                               A->rowptr, dst);
            hipLaunchKernelGGL(k_check_cols, dim3(grid_for(n)), dim3(kBlock), 0, s, n, A->rowptr,
                               A->col, (flags & SPK_MAT_VALIDATE) ? 1 : 0, dst);
            hipLaunchKernelGGL(k_diag_inv, dim3(grid_for(n)), dim3(kBlock), 0, s, n, A->rowptr,
                               A->col, A->val, A->dinv, dst);
        }
        e = hipMemcpyAsync(hst, dst, sizeof(RowStats), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) { fail(hip_fail(e, "column checks", __FILE__, __LINE__)); break; }
        if (hst->bad_col) {
            set_error("%d column indices outside [0, n)", hst->bad_col);
            fail(SPK_EINVAL);
            break;
        }
        if (hst->unsorted) {
            set_error("%d entries not strictly ascending within their row", hst->unsorted);
            fail(SPK_EINVAL);
            break;
        }
        A->stats = *hst;
    } while (0);
    hipFree(dst);
    hipHostFree(hst);
    if (rc) return rc;

    choose_kernel(A);
    if (const char *f = getenv("SPK_FORCE_KERNEL")) {
        if (!strncmp(f, "stream", 6)) A->kernel = SPK_KERNEL_STREAM;
        else if (!strncmp(f, "merge", 5) && merge_fits(A)) A->kernel = SPK_KERNEL_MERGE;
        else if (!strncmp(f, "sell", 4) && A->stats.max_len <= 255) A->kernel = SPK_KERNEL_SELL;
        else if (!strncmp(f, "vector", 6)) {
            A->kernel = SPK_KERNEL_VECTOR;
            const char *c = strchr(f, ':');
            A->lanes = c ? atoi(c + 1) : 32;
        }
    }
    if (A->kernel != SPK_KERNEL_STREAM) A->R = 256;
    if (A->kernel == SPK_KERNEL_STREAM && A->R == 0) A->R = 32;
    if (A->kernel == SPK_KERNEL_SLICED && setup_sliced(A, A->xs_merge, s) != SPK_OK) {
        choose_kernel(A, true, false);  // no room for the copy: the unsliced family
        if (A->kernel != SPK_KERNEL_STREAM) A->R = 256;
    }
    apply_partition(A);
    if (A->kernel == SPK_KERNEL_MERGE) {
        rc = setup_merge(A, s);
        if (rc) return rc;
    }
    if (A->kernel == SPK_KERNEL_SELL) {
        rc = setup_sell(A, s, 0);
        if (rc) {
            if (getenv("SPK_FORCE_KERNEL")) return rc;
            free_sell(A);  // the layout did not fit: take the next family that needs no copy
            choose_kernel(A, false, false);
            if (A->kernel != SPK_KERNEL_STREAM) A->R = 256;
            apply_partition(A);
            if (A->kernel == SPK_KERNEL_MERGE) {
                rc = setup_merge(A, s);
                if (rc) return rc;
            }
        }
    }
    if (flags & SPK_MAT_MIXED) {
        rc = ensure_f32(A, s);
        if (rc) return rc;
    }
    SPK_HIP(hipStreamSynchronize(s));
    update_info(A);
    return SPK_OK;
}

int spk_mat_create_csr(int32_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colind,
                       const double *values, int memtype, uint32_t flags, void *stream,
                       spk_mat **out)
{
    if (!out) { set_error("out is NULL"); return SPK_EINVAL; }
    *out = nullptr;
    if (n < 0 || nnz < 0 || nnz > 0x7fffffffLL) {
        set_error("n = %d, nnz = %lld: need 0 <= n and 0 <= nnz < 2^31", n, (long long)nnz);
        return SPK_EINVAL;
    }
    if (!rowptr || (nnz > 0 && (!colind || !values))) { set_error("NULL array"); return SPK_EINVAL; }
    if (memtype != SPK_MEM_HOST && memtype != SPK_MEM_DEVICE) {
        set_error("memtype %d", memtype);
        return SPK_EINVAL;
    }
    if ((flags & SPK_MAT_BORROW) && memtype != SPK_MEM_DEVICE) {
        set_error("SPK_MAT_BORROW needs SPK_MEM_DEVICE");
        return SPK_EINVAL;
    }
    if (flags & ~(uint32_t)(SPK_MAT_MIXED | SPK_MAT_VALIDATE | SPK_MAT_BORROW | SPK_MAT_STREAM)) {
        set_error("unknown flags 0x%x", flags);
        return SPK_EINVAL;
    }
    if (memtype == SPK_MEM_HOST) {
        if (rowptr[0] != 0 || rowptr[n] != nnz) {
            set_error("rowptr[0] = %d, rowptr[n] = %d, nnz = %lld", rowptr[0], rowptr[n],
                      (long long)nnz);
            return SPK_EINVAL;
        }
    }
    spk_mat *A = new (std::nothrow) spk_mat();
    if (!A) { set_error("out of host memory"); return SPK_ENOMEM; }
    A->stream = (hipStream_t)stream;
    const int rc = create_impl(n, nnz, rowptr, colind, values, memtype, flags,
                               (hipStream_t)stream, A);
    if (rc) {
        spk_mat_destroy(A);
        return rc;
    }
    *out = A;
    return SPK_OK;
}

static int set_kernel(spk_mat *A, int kernel, int32_t param, hipStream_t s)
{
    switch (kernel) {
    case SPK_KERNEL_AUTO: choose_kernel(A); break;
    case SPK_KERNEL_STREAM: {
        int R = param;
        if (R == 0) {
            for (int t = 0; t < 6; ++t)
                if (A->stats.tile_max[t] <= TileLds<double>::kCap) { R = kTileRs[t]; break; }
            if (R == 0) R = 8;
        }
        if (R < 1 || R > kBlock) { set_error("stream rows per tile %d not in [1, 256]", R); return SPK_EINVAL; }
        A->kernel = SPK_KERNEL_STREAM;
        A->R = R;
        break;
    }
    case SPK_KERNEL_VECTOR:
        if (param < 1 || param > 64 || (param & (param - 1))) {
            set_error("lanes %d not a power of two in [1, 64]", param);
            return SPK_EINVAL;
        }
        A->kernel = SPK_KERNEL_VECTOR;
        A->lanes = param;
        A->R = 256;
        break;
    case SPK_KERNEL_MERGE:
        if (!merge_fits(A)) { set_error("merge path needs n + nnz < 2^31"); return SPK_EINVAL; }
        A->kernel = SPK_KERNEL_MERGE;
        A->R = 256;
        break;
    case SPK_KERNEL_SELL: {
        if (param != 0 && param != 1 && param != 16 && param != 32) {
            set_error("SELL column offsets %d not in {0, 1, 16, 32}", param);
            return SPK_EINVAL;
        }
        const int rc = setup_sell(A, s, param == 1 ? 1 : param / 8);
        if (rc) return rc;
        if (A->val32) {
            const int r2 = ensure_f32(A, s);
            if (r2) return r2;
            SPK_HIP(hipStreamSynchronize(s));
        }
        A->kernel = SPK_KERNEL_SELL;
        A->R = 256;
        break;
    }
    case SPK_KERNEL_SELL_SIGMA: {
        const int sigma = param == 0 ? 4096 : param;
        if (sigma < kSell || sigma % kSell != 0) {
            set_error("SELL-C-sigma window %d: a positive multiple of %d", param, kSell);
            return SPK_EINVAL;
        }
        const int rc = setup_sell(A, s, 0, sigma);
        if (rc) return rc;
        if (A->val32) {
            const int r2 = ensure_f32(A, s);
            if (r2) return r2;
            SPK_HIP(hipStreamSynchronize(s));
        }
        A->kernel = SPK_KERNEL_SELL;
        A->R = 256;
        break;
    }
    case SPK_KERNEL_SLICED: {
        const bool lanes_ok = param >= 1 && param <= 64 && !(param & (param - 1));
        if (param != 0 && param != kMergeItems && !lanes_ok) {
            set_error("sliced parameter %d: 0, a power of two in [1, 64] or %d (merge path)", param, kMergeItems);
            return SPK_EINVAL;
        }
        const int merge = param == kMergeItems || (param == 0 && sliced_merge_fits(A));
        const int rc = setup_sliced(A, merge, s);
        if (rc) return rc;
        A->kernel = SPK_KERNEL_SLICED;
        A->xs_merge = merge;
        A->lanes = lanes_ok ? param : sliced_lanes(A);
        A->R = 256;
        break;
    }
    default:
        set_error("unknown kernel %d", kernel);
        return SPK_EINVAL;
    }
    if (A->kernel == SPK_KERNEL_MERGE) {
        const int rc = setup_merge(A, s);
        if (rc) return rc;
        SPK_HIP(hipStreamSynchronize(s));
    }
    if (kernel == SPK_KERNEL_AUTO && A->kernel == SPK_KERNEL_SLICED) {
        if (setup_sliced(A, A->xs_merge, s) != SPK_OK) {
            choose_kernel(A, true, false);
            if (A->kernel == SPK_KERNEL_MERGE) {
                const int r2 = setup_merge(A, s);
                if (r2) return r2;
                SPK_HIP(hipStreamSynchronize(s));
            }
        }
    }
    if (kernel == SPK_KERNEL_AUTO && A->kernel == SPK_KERNEL_SELL) {
        int rc = setup_sell(A, s, 0);
        if (rc == SPK_OK && A->val32) rc = ensure_f32(A, s);
        if (rc == SPK_OK) rc = hipStreamSynchronize(s) == hipSuccess ? SPK_OK : SPK_EHIP;
        if (rc) {
            free_sell(A);
            choose_kernel(A, false, false);
            if (A->kernel == SPK_KERNEL_MERGE) {
                const int r2 = setup_merge(A, s);
                if (r2) return r2;
                SPK_HIP(hipStreamSynchronize(s));
            }
        }
    }
    return SPK_OK;
}

// After a refused set_kernel: the family and layout of before it (`was`), or,
// where that layout is gone and does not fit any more, a family without one.
struct KernelChoice {
    int kernel, R, lanes, xs_merge, sell_req, sell_sigma;
};
static void keep_kernel(spk_mat *A, const KernelChoice &was, hipStream_t s)
{
    A->kernel = was.kernel;
    A->R = was.R;
    A->lanes = was.lanes;
    A->xs_merge = was.xs_merge;
    bool there = true;
    if (was.kernel == SPK_KERNEL_SELL) {
        // (built again if the request took it down)
        there = setup_sell(A, s, was.sell_req, was.sell_sigma) == SPK_OK &&
                (!A->val32 || (ensure_f32(A, s) == SPK_OK && hipStreamSynchronize(s) == hipSuccess));
    } else if (was.kernel == SPK_KERNEL_SLICED) {
        there = A->xs_merge ? A->bn_slab || A->xs_tiles : A->xs_ptr != nullptr;
    }
    if (!there || A->sell_req < 0) free_sell(A);  // half a layout
    if (there) return;
    choose_kernel(A, false, false);
    if (A->kernel == SPK_KERNEL_MERGE && setup_merge(A, s) != SPK_OK) {
        A->kernel = SPK_KERNEL_VECTOR;  // the one that needs no memory at all
        A->lanes = 32;
    }
}

int spk_mat_set_kernel(spk_mat *A, int kernel, int32_t param, void *stream)
{
    if (!A) { set_error("A is NULL"); return SPK_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    ++A->layout_gen;
    // solver graphs and partials depend on the partition: release them after
    // the handle's earlier work has finished
    free_workspace(A);
    free_multi(A);
    A->stream = s;
    const KernelChoice was{A->kernel, A->R, A->lanes, A->xs_merge, A->sell_req, A->sell_sigma};
    const int rc = set_kernel(A, kernel, param, s);
    if (rc != SPK_OK) {
        char why[sizeof g_err];
        memcpy(why, g_err, sizeof why);
        keep_kernel(A, was, s);
        memcpy(g_err, why, sizeof why);
    }
    apply_partition(A);
    update_info(A);
    return rc;
}

int spk_mat_mult(const spk_mat *A, const double *x, double *y, void *stream)
{
    if (!A || (A->n > 0 && (!x || !y))) { set_error("NULL argument"); return SPK_EINVAL; }
    if (x == y && A->n > 0) { set_error("x and y must not alias"); return SPK_EINVAL; }
    A->stream = (hipStream_t)stream;
    return launch_spmv<double>(A, A->val, x, y, (hipStream_t)stream, nullptr, 0);
}

int spk_mat_mult_f32(const spk_mat *A, const float *x, float *y, void *stream)
{
    if (!A || (A->n > 0 && (!x || !y))) { set_error("NULL argument"); return SPK_EINVAL; }
    if (x == y && A->n > 0) { set_error("x and y must not alias"); return SPK_EINVAL; }
    A->stream = (hipStream_t)stream;
    if (!A->val32 && A->n > 0) { set_error("matrix has no FP32 values (create with SPK_MAT_MIXED)"); return SPK_EINVAL; }
    return launch_spmv<float>(A, A->val32, x, y, (hipStream_t)stream, nullptr, 0);
}

int spk_mat_get_info(const spk_mat *A, spk_mat_info *info)
{
    if (!A || !info) { set_error("NULL argument"); return SPK_EINVAL; }
    update_info(const_cast<spk_mat *>(A));
    *info = A->info;
    return SPK_OK;
}

int spk_pc_jacobi_apply(const spk_mat *A, const double *r, double *z, void *stream)
{
    if (!A || (A->n > 0 && (!r || !z))) { set_error("NULL argument"); return SPK_EINVAL; }
    if (A->n == 0) return SPK_OK;
    if (A->stats.zero_diag) {
        set_error("%d rows have no stored or a zero diagonal", A->stats.zero_diag);
        return SPK_EZERODIAG;
    }
    A->stream = (hipStream_t)stream;
    launch_map(A->n, (const double *)A->dinv, r, z, Mul{}, stream);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

int spk_mat_destroy(spk_mat *A)
{
    if (!A) return SPK_OK;
    // the handle's work is queued on the stream of its last call; HIP's
    // hipFree below waits for the device as HIP documents
    hipStreamSynchronize(A->stream);
    free_workspace(A);
    free_multi(A);
    hipFree(A->slab);
    hipFree(A->val32);
    hipFree(A->dinv32);
    hipFree(A->tile_row);
    hipFree(A->tile_k);
    hipFree(A->carry_row);
    hipFree(A->carry_val);
    free_sell(A);
    free_sliced(A);
    delete A;
    return SPK_OK;
}

// ------------------------------------------------------------------ vectors
int spk_vec_axpy(int32_t n, double alpha, const double *x, double *y, void *stream)
{
    if (n < 0 || (n > 0 && (!x || !y))) { set_error("bad argument"); return SPK_EINVAL; }
    if (n == 0) return SPK_OK;
    launch_map(n, x, y, y, Axpy{alpha}, stream);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

int spk_vec_aypx(int32_t n, double beta, const double *x, double *y, void *stream)
{
    if (n < 0 || (n > 0 && (!x || !y))) { set_error("bad argument"); return SPK_EINVAL; }
    if (n == 0) return SPK_OK;
    launch_map(n, x, y, y, Aypx{beta}, stream);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

// Per-stream reduction scratch (partials + counter), created on first use.
struct DotScratch {
    double *part = nullptr;
};
static std::mutex g_dot_mu;
static std::map<std::pair<int, void *>, DotScratch> g_dot;

// The two dot kernels on partials `part` (2 x kMaxBlocksSingle doubles).
static int dot_enqueue(int32_t n, const double *x, const double *y, const double *w, int mode,
                       double *result, double *part, void *stream)
{
    int grid = grid_for(n > 0 ? n : 1);
    if (grid >= kXcd) grid -= grid % kXcd;
    auto dot = w || n < kDotAheadMax ? k_dot<kDotAhead> : k_dot<1>;
    hipLaunchKernelGGL(dot, dim3(grid), dim3(kBlock), 0, (hipStream_t)stream, n, x, mode == 2 ? x : y, w, part);
    hipLaunchKernelGGL(k_dot_fin, dim3(1), dim3(kBlock), 0, (hipStream_t)stream, grid,
                       w ? 1 : 0, mode, part, result);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

static int dot_launch(int32_t n, const double *x, const double *y, const double *w, int mode,
                      double *result, void *stream)
{
    if (n < 0 || !x || !result || (mode != 2 && !y)) { set_error("bad argument"); return SPK_EINVAL; }
    int dev = 0;
    SPK_HIP(hipGetDevice(&dev));
    DotScratch sc;
    {
        std::lock_guard<std::mutex> lk(g_dot_mu);
        auto it = g_dot.find({dev, stream});
        if (it == g_dot.end()) {
            SPK_HIP(hipMalloc(&sc.part, sizeof(double) * 2 * kMaxBlocksSingle));
            g_dot[{dev, stream}] = sc;
        } else {
            sc = it->second;
        }
    }
    return dot_enqueue(n, x, y, w, mode, result, sc.part, stream);
}

// Partials of the allocation-free fused dot: one launch has at most
// kMaxBlocksSingle blocks and two sums per block, so every n fits.  Each GPU
// holds its own copy for the life of the process; host code never passes this
// name to a kernel (on the host it is a stand-in, not a device address) but
// the address hipGetSymbolAddress returns for the current device.
constexpr int kScratchDoubles = 2 * kMaxBlocksSingle;
static __device__ __align__(256) double scratch[kScratchDoubles];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static double *g_scratch_ptr[kMaxDevices];  // device -> its copy of `scratch`

static int scratch_on_device(double **out)
{
    int dev = 0;
    SPK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("device %d: the allocation-free entry points serve devices 0..%d", dev, kMaxDevices - 1);
        return SPK_EINVAL;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        SPK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) { set_error("hipGetSymbolAddress returned no address for the scratch array"); return SPK_EHIP; }
        g_scratch_ptr[dev] = (double *)p;
    }
    *out = g_scratch_ptr[dev];
    return SPK_OK;
}

int spk_vec_dot(int32_t n, const double *x, const double *y, double *result, void *stream)
{
    return dot_launch(n, x, y, nullptr, 0, result, stream);
}

int spk_vec_dot2(int32_t n, const double *x, const double *y, const double *w, double *result,
                 void *stream)
{
    if (!w) { set_error("w is NULL"); return SPK_EINVAL; }
    return dot_launch(n, x, y, w, 1, result, stream);
}

int spk_vec_dot2_noalloc(int32_t n, const double *x, const double *y, const double *w, double *result,
                         void *stream)
{
    if (n < 0 || !x || !y || !w || !result) { set_error("bad argument"); return SPK_EINVAL; }
    const int grid = grid_for(n > 0 ? n : 1);
    if (2 * grid > kScratchDoubles) {  // cannot happen while grid_for caps the grid
        set_error("n = %d needs %d partials, more than the %d of the static scratch", n, 2 * grid,
                  kScratchDoubles);
        return SPK_EINVAL;
    }
    double *part = nullptr;
    const int rc = scratch_on_device(&part);
    if (rc != SPK_OK) return rc;
    return dot_enqueue(n, x, y, w, 1, result, part, stream);
}

int spk_vec_nrm2(int32_t n, const double *x, double *result, void *stream)
{
    return dot_launch(n, x, nullptr, nullptr, 2, result, stream);
}

int spk_bw_copy(int64_t n, const double *src, double *dst, void *stream)
{
    if (n < 0 || (n & 1) || (n > 0 && (!src || !dst))) { set_error("n must be even and >= 0"); return SPK_EINVAL; }
    if (n == 0) return SPK_OK;
    const int64_t m = n / 2;
    hipLaunchKernelGGL(k_copy, dim3(grid_stream(m)), dim3(kBlock), 0, (hipStream_t)stream, m,
                       (const dvec2 *)src, (dvec2 *)dst);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

int spk_cache_flush(void *scratch, int64_t bytes, void *stream)
{
    if (!scratch || bytes < 16) { set_error("bad argument"); return SPK_EINVAL; }
    const int64_t m = bytes / 16;
    int64_t g = (m + kBlock - 1) / kBlock;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL(k_evict, dim3((int)g), dim3(kBlock), 0, (hipStream_t)stream, m, (dvec2 *)scratch);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

}  // extern "C"
