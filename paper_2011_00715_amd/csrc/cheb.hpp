// Jacobi-preconditioned Chebyshev smoother kernels (the multigrid smoother of
// Sec. 5.3).  The three-term recurrence has coefficients known before the
// first step, so each step is one pass with no inner product:
//   x += d_k;  r -= A d_k;  d_{k+1} = c1 d_k + c2 D^-1 r
// For the SELL and stream families that pass is a single kernel (the update
// runs in the SpMV's row epilogue); d is double-buffered because every block
// gathers d_k while it writes d_{k+1} for its own rows.
//
// The passes are bound by HBM, so the vector-only passes around the steps are
// folded into them:
//  * a start from zero (x = 0, r = b, d_0 = D^-1 b / theta) is formed where
//    the first step gathers it, on SELL: two more gathers that the L2 serves
//    instead of 40n bytes written and 24n read back;
//  * the closing x += d_{k+1} (no residual wanted) needs no neighbour, so the
//    step before it adds both: x = (x + d_k) + d_{k+1}, and neither r nor
//    d_{k+1} is stored (24n bytes of a pass of its own and 16n of stores).
// Two steps from zero, the multigrid default, are then one pass over the
// matrix that reads b and D^-1 and writes x: 7-point 128^3 64.5 -> 39.6 us a smoothing
// (each on other buffers), the V-cycle solve on it 5.42 -> 4.90 ms.
// The sums and their order are those of the separate passes.
#pragma once

#include "spmv.hpp"

namespace spk {

template <class V>
struct ChebStep {
    const V *dk;  // d_k (gathered); unused in a first step from zero
    V *dn;        // d_{k+1}, or null on the last step
    V *r;
    V *x;
    const V *dinv;
    V c1, c2;
    const SysState *gate = nullptr;  // inside a captured solve: run only while it iterates
    // first step from zero (SELL): the right-hand side, in V or (an FP32
    // cycle's finest level) in FP64, then also stored rounded into bcopy
    const V *b = nullptr;
    const double *b64 = nullptr;
    V *bcopy = nullptr;
    V inv_theta = V(0);
    // the closing x += d_{k+1} folded in; with z the result goes there in
    // FP64, and with part also the per-block sums of rcg . z
    bool close = false;
    double *z = nullptr;
    const double *rcg = nullptr;
    double *part = nullptr;
};

__device__ __forceinline__ bool cheb_go(const SysState *gate)
{
    return !gate || gate_open(gate, kGateInner64);
}

// A row's own operands of a step: d_k, x, r, D^-1, and rcg where a closing
// step sums rcg . z.
template <class V>
struct ChebOwn {
    V d, x, r, dinv;
    double rcg;
};

// kOneDiag: the matrix has one value per offset, so one D^-1.
template <class V, bool kOneDiag = false>
__device__ __forceinline__ ChebOwn<V> cheb_own(const ChebStep<V> &c, int i)
{
    return ChebOwn<V>{c.dk[i], c.x[i], c.r[i], kOneDiag ? (V)*as_constant(c.dinv) : c.dinv[i],
                      c.part ? c.rcg[i] : 0.0};
}

// Row i of a step whose product is y.  Returns its term of rcg . z (0 when
// none is wanted).
template <class V>
__device__ __forceinline__ double cheb_row(const ChebStep<V> &c, int i, V y, const ChebOwn<V> &o)
{
#pragma clang fp contract(off)  // x = (x + d_k) + d_{k+1}, each sum rounded
    const V r1 = o.r - y;
    const V x1 = o.x + o.d;
    const V dn = fma(c.c1, o.d, c.c2 * (o.dinv * r1));
    if (c.close) {
        const V x2 = x1 + dn;
        if (!c.z) {
            c.x[i] = x2;
            return 0.0;
        }
        const double zi = (double)x2;
        c.z[i] = zi;
        return o.rcg * zi;
    }
    c.r[i] = r1;
    c.x[i] = x1;
    if (c.dn) c.dn[i] = dn;
    return 0.0;
}

template <class V>
__device__ __forceinline__ double cheb_row(const ChebStep<V> &c, int i, V y)
{
    return cheb_row(c, i, y, cheb_own(c, i));
}

// Per-block sums of a closing step's rcg . z terms.
__device__ __forceinline__ void cheb_part(double acc, double *part)
{
    __shared__ double sh[kBlock / kWave];
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

template <class V, class CI, int U>
__global__ __launch_bounds__(kBlock) void k_cheb_sell(int n, SellView sv, const V *__restrict__ val,
                                                      ChebStep<V> c)
{
    double acc = 0.0;
    bool run = true;
    sell_slices<V, CI, U>(n, blockIdx.x * (kBlock / kWave) + (int)threadIdx.x / kWave,
                          gridDim.x * (kBlock / kWave), sv, val, c.dk, [&] { return run = cheb_go(c.gate); },
                          [&](int i) { return cheb_own<V, std::is_same<CI, Stencil>::value>(c, i); },
                          [&](int i, V y, const ChebOwn<V> &o) { acc += cheb_row(c, i, y, o); });
    if (c.part && run) cheb_part(acc, c.part);
}

// d_0 = (D^-1 b) / theta of a start from zero; kOneDiag: D^-1 is `one`.
template <class V, class B, bool kOneDiag>
struct GatherD0 {
    const V *__restrict__ dinv;
    const B *__restrict__ b;
    V it, one;
    struct Raw {
        V dinv;
        B b;
    };
    __device__ Raw at(int j) const { return Raw{kOneDiag ? one : dinv[j], b[j]}; }
    __device__ Raw sh(int64_t base, unsigned l) const
    {
        return Raw{kOneDiag ? one : (dinv + base)[l], (b + base)[l]};
    }
    __device__ V of(const Raw &r) const
    {
#pragma clang fp contract(off)
        return r.dinv * (V)r.b * it;
    }
};

// The first step from zero: d_0 is formed at every gather.
template <class V, class B, class CI, int U>
__global__ __launch_bounds__(kBlock) void k_cheb_sell_zero(int n, SellView sv, const V *__restrict__ val,
                                                           ChebStep<V> c, const B *__restrict__ b)
{
    constexpr bool kOneDiag = std::is_same<CI, Stencil>::value;
    const V one = kOneDiag ? (V)*as_constant(c.dinv) : V(0);
    const GatherD0<V, B, kOneDiag> d0{c.dinv, b, c.inv_theta, one};
    double acc = 0.0;
    bool run = true;
    sell_slices_g<V, CI, U>(n, blockIdx.x * (kBlock / kWave) + (int)threadIdx.x / kWave,
                            gridDim.x * (kBlock / kWave), sv, val, d0, [&] { return run = cheb_go(c.gate); },
                            [&](int i) {
#pragma clang fp contract(off)
                                const V bi = (V)b[i], di = kOneDiag ? one : c.dinv[i];
                                return ChebOwn<V>{di * bi * c.inv_theta, V(0), bi, di, c.part ? c.rcg[i] : 0.0};
                            },
                            [&](int i, V y, const ChebOwn<V> &o) {
                                if (c.bcopy) c.bcopy[i] = o.r;
                                acc += cheb_row(c, i, y, o);
                            });
    if (c.part && run) cheb_part(acc, c.part);
}

template <class V>
__global__ __launch_bounds__(kBlock) void k_cheb_stream(int n, int R, int ntiles, int nblk,
                                                        const int32_t *__restrict__ rowptr,
                                                        const int32_t *__restrict__ col,
                                                        const V *__restrict__ val, ChebStep<V> c)
{
    if (!cheb_go(c.gate)) return;
    __shared__ TileLds<V> sm;
    const int j = xcd_remap(blockIdx.x, nblk);
    int t0, t1;
    block_tiles(j, nblk, ntiles, t0, t1);
    double acc = 0.0;
    for (int t = t0; t < t1; ++t) {
        const int r0 = t * R;
        const int r1 = min(r0 + R, n);
        stream_tile<V>(r0, r1, rowptr, col, val, c.dk, sm, [&](int i, V y) { acc += cheb_row(c, i, y); });
    }
    if (c.part) cheb_part(acc, c.part);
}

// Other families: y = A d_k was written by the standalone SpMV.
template <class V>
__global__ __launch_bounds__(kBlock) void k_cheb_update(int n, const V *__restrict__ y, ChebStep<V> c)
{
    if (!cheb_go(c.gate)) return;
    double acc = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        acc += cheb_row(c, i, y[i]);
    if (c.part) cheb_part(acc, c.part);
}

// r = b - A x (ax holds A x; null for x = 0, which is then stored), and
// d_0 = D^-1 r / theta.  B is the right-hand side's type: a double b with
// float vectors also stores the rounded b into bcopy (the FP32 cycle of a
// multigrid preconditioner inside FP64 CG).
template <class V, class B>
__global__ void k_cheb_init(int n, const B *__restrict__ b, const V *__restrict__ ax, V *__restrict__ x,
                            V *__restrict__ r, V *__restrict__ d0, const V *__restrict__ dinv, V inv_theta,
                            const SysState *gate, V *__restrict__ bcopy)
{
    if (!cheb_go(gate)) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const V bi = (V)b[i];
        if (bcopy) bcopy[i] = bi;
        V ri;
        if (ax) ri = bi - ax[i];
        else {
            ri = bi;
            x[i] = V(0);
        }
        r[i] = ri;
        d0[i] = dinv[i] * ri * inv_theta;
    }
}

// One step from zero without a residual: x = D^-1 b / theta.
template <class V>
__global__ void k_cheb_one(int n, const V *__restrict__ b, const V *__restrict__ dinv, V inv_theta, V *__restrict__ x)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = V(0) + dinv[i] * b[i] * inv_theta;
}

// The last step without a residual: x += d.
template <class V>
__global__ void k_cheb_last(int n, const V *__restrict__ d, V *__restrict__ x, const SysState *gate)
{
    if (!cheb_go(gate)) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        x[i] = x[i] + d[i];
}

}  // namespace spk
