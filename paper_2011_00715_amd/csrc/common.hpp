// Internal definitions shared by the HIP translation units of libspk.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "spk.h"

namespace spk {

// ------------------------------------------------------------------ launch shape
constexpr int kBlock = 256;              // threads per block (4 wavefronts of 64)
constexpr int kWave = 64;
constexpr int kXcd = 8;                  // MI355X: 8 accelerator complex dies
constexpr int kMaxBlocksSingle = 2048;   // 256 CUs x 8 resident blocks
constexpr int kTileBytes = 16384;        // LDS bytes for one tile of products
constexpr int kMergeItems = 2048;        // merge-path items per tile (256 x 8)
constexpr int kMergeIpt = kMergeItems / kBlock;

// ------------------------------------------------------------------ solver state
// Phase of a system inside a solve (FP64 solves stay in kPhaseInner).
enum : int32_t {
    kPhaseInner = 0,   // Krylov iterations (FP64, or FP32 inner for mixed)
    kPhaseResid = 1,   // mixed: form r = b - A x in FP64
    kPhaseSetup = 2,   // mixed: scale/cast r, start the FP32 inner solve
    kPhaseUpdate = 3,  // mixed: x += s d, then kPhaseResid
};

// Slots of the per-block partial sums (each B doubles).
enum { kPartPq = 0, kPartRz = 1, kPartRr = 2, kPartBb = 3, kNumPart = 4 };

// Device-resident scalars of one system.  Written by one block only: the
// one-block finalize kernels, the one-thread init kernel, block 0 of the
// PCG update pass (the snap_* fields) and block 0 of the p/x pass (the rest);
// no kernel's blocks read a field that a block of the same kernel writes.
// Every later kernel turns into a no-op once `status` is no longer
// SPK_RUNNING.
struct SysState {
    int32_t status;       // SPK_RUNNING or a reason
    int32_t phase;        // kPhase*
    int32_t iter;         // Krylov iterations done (inner ones for mixed)
    int32_t inner_iter;   // iterations of the current inner solve
    int32_t outer;        // mixed: refinement steps done
    int32_t cmode;        // next x/p update: 2 both, 1 x only (last), 0 none
    int32_t maxit;
    int32_t inner_maxit;
    int32_t max_outer;
    int32_t stagnant;     // mixed: consecutive weak outer reductions
    int32_t mixed;        // 1: mixed-precision solve
    int32_t hist_len;
    int32_t ru;           // mixed: 1 keeps p across refinements (reliable updates)
    int32_t fresh_p;      // mixed: the next refinement starts p from z
    // the scalars of the current iteration as the update pass saw them: the
    // p/x pass decides from these while its block 0 rewrites the live ones
    int32_t snap_status, snap_phase, snap_iter, snap_inner_iter;
    // fused p/x + product kernel (F): p lives in one of two buffers, pbuf
    // (written by F's block 0) naming the current one; snap_pbuf is the
    // copy F's blocks read.  snap_mode says what the next F does: 1 take the
    // decision recorded by the update pass, then (while iterating) the
    // product with p = z + beta p; 0 start: p = z; 3 continue after a
    // reliable update: p = z + beta p with beta from the refinement
    int32_t pbuf, snap_pbuf, snap_mode, pad_f;
    double scale;         // mixed: r32 = r / scale, x += scale d
    double rho, alpha, beta, eta;
    double rnorm, rnorm0, bnorm, thresh, rtol, atol;
    double inner_rtol, inner_thresh;
    double s;             // mixed: ||r|| of the current outer residual
    double s_prev;        // mixed: previous outer ||r||
    double rnorm_true;    // result of the last true-residual kernel
    double snap_rho, snap_eta;
};

// One linear system as seen by the batched kernels.
struct SysDesc {
    int32_t n;
    int32_t R;            // rows per tile
    int32_t ntiles;
    int32_t nblk;         // logical blocks (a multiple of kXcd when >= kXcd)
    const int32_t *rowptr;
    const int32_t *col;
    const double *val;
    const float *val32;
    const double *dinv;
    const float *dinv32;
    const double *b;
    double *x;
    double *r, *z, *p, *q;            // FP64 Krylov vectors
    float *r32, *z32, *p32, *q32, *d32;  // FP32 inner vectors (mixed)
    double *p2;                       // second p buffer of the fused kernels
    float *p2_32;                     //   (null: the three-kernel iteration)
    double *partials;                 // kNumPart * nblk
    SysState *st;
    double *hist;                     // device history (hist_len) or null
    // SELL-64 copy of the matrix (used when `sell_cw` is nonzero)
    int32_t sell_cw;
    int32_t sell_plain;  // kSellPlain64/32 load-policy bits
    const int32_t *sell_ptr;
    const void *sell_col;
    const uint8_t *sell_len;
    const double *sell_val;
    const float *sell_val32;
    const uint16_t *sell_len16;  // row lengths when some row has more than 255 entries
    const int32_t *sell_perm;    // SELL-C-sigma: matrix row of each sorted position
    const uint32_t *sell_mask;   // shared offsets: per-row position masks, or null
};

// ------------------------------------------------------------------ host helpers
void set_error(const char *fmt, ...);
int hip_fail(hipError_t e, const char *what, const char *file, int line);

#define SPK_HIP(call)                                                        \
    do {                                                                     \
        hipError_t e_ = (call);                                              \
        if (e_ != hipSuccess) return ::spk::hip_fail(e_, #call, __FILE__, __LINE__); \
    } while (0)

#define SPK_TRY(x)                  \
    do {                            \
        const int rc_ = (x);        \
        if (rc_ != SPK_OK) return rc_; \
    } while (0)

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Logical blocks for a system of `ntiles` tiles, at most `maxb`: a multiple of
// kXcd when there are at least kXcd tiles, so that the XCD-aware remap below
// is a bijection.
inline int pick_nblk(int ntiles, int maxb)
{
    if (ntiles <= 0) return 0;
    if (ntiles < kXcd) return ntiles;
    int b = ntiles < maxb ? ntiles : maxb;
    return b - b % kXcd;
}

// ------------------------------------------------------------------ device helpers
// Workgroups are dispatched round-robin over the 8 XCDs.  Physical block `l`
// of a system therefore runs on XCD l % 8; give XCD x the contiguous logical
// range [x*B/8, (x+1)*B/8) so each XCD's L2 sees a contiguous band of rows
// (and of the gathered x window of banded matrices).
__device__ __forceinline__ int xcd_remap(int l, int nblk)
{
    if (nblk < kXcd || (nblk % kXcd) != 0) return l;
    return (l % kXcd) * (nblk / kXcd) + l / kXcd;
}

// Tiles handled by logical block j of nblk: a balanced contiguous chunk.
__device__ __forceinline__ void block_tiles(int j, int nblk, int ntiles, int &t0, int &t1)
{
    t0 = (int)(((int64_t)j * ntiles) / nblk);
    t1 = (int)(((int64_t)(j + 1) * ntiles) / nblk);
}

// Find the system of physical block b: blk_start is ascending, nsys+1 entries.
__device__ __forceinline__ int find_sys(const int32_t *blk_start, int nsys, int b)
{
    int lo = 0, hi = nsys - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (blk_start[mid] <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Two registers' halves (D = 32) or rows of 16 lanes (D = 16) exchanged: lane
// by lane, a then holds the lower and b the upper partner of each pair at
// distance D, of x where that bit of the lane is clear and of y where it is
// set.
template <int D, class T>
__device__ __forceinline__ void lane_swap(T x, T y, T &a, T &b)
{
    constexpr int W = sizeof(T) / 4;
    union { T t; uint32_t w[W]; } ux, uy, ua, ub;
    ux.t = x;
    uy.t = y;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        if constexpr (D == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(ux.w[i], uy.w[i], false, false);
            ua.w[i] = r[0];
            ub.w[i] = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane16_swap(ux.w[i], uy.w[i], false, false);
            ua.w[i] = r[0];
            ub.w[i] = r[1];
        }
    }
    a = ua.t;
    b = ub.t;
}

// The value D lanes on within a row of 16 (D < 16).
template <int D, class T>
__device__ __forceinline__ T row_ror(T v)
{
    constexpr int W = sizeof(T) / 4;
    union { T t; uint32_t w[W]; } u;
    u.t = v;
#pragma unroll
    for (int i = 0; i < W; ++i)
        u.w[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.w[i], 0x120 + D, 0xf, 0xf, true);
    return u.t;
}

// One level of the butterfly: lane i's value plus lane i ^ D's.  Below 16 a
// rotation by D is i ^ D once the values repeat every 2 D lanes, which the
// levels 32, 16, 8, 4, 2, 1, taken in this order, give (at D = 8 a row is two
// halves).
template <int D, class T>
__device__ __forceinline__ T wave_level(T v)
{
    if constexpr (D >= 16) {
        T a, b;
        lane_swap<D>(v, v, a, b);
        return a + b;
    } else {
        return v + row_ror<D>(v);
    }
}

// The levels 8, 4, 2, 1: sums of the rows of 16 lanes.
template <class T>
__device__ __forceinline__ T row_sum(T v)
{
    v = wave_level<8>(v);
    v = wave_level<4>(v);
    v = wave_level<2>(v);
    return wave_level<1>(v);
}

// Butterfly sum over a wavefront; every lane ends with the same bits
// (each level adds two values whose sum is commutative, hence identical).
// Lane swaps and rotations instead of shuffles through the LDS pipe: a level
// is three vector instructions instead of an LDS round trip.
template <class T>
__device__ __forceinline__ T wave_sum(T v)
{
    return row_sum(wave_level<16>(wave_level<32>(v)));
}

// Two butterfly sums at once, x's in the lower and y's in the upper half of
// the lanes; four at once, w's, y's, x's and z's in rows 0 to 3.  The first
// levels halve what a register needs, so the sums share the later ones; each
// sum has wave_sum's bits.
template <class T>
__device__ __forceinline__ T wave_sum2(T x, T y)
{
    T a, b;
    lane_swap<32>(x, y, a, b);
    return row_sum(wave_level<16>(a + b));
}

template <class T>
__device__ __forceinline__ T wave_sum4(T w, T x, T y, T z)
{
    T a, b, c, d, e, f;
    lane_swap<32>(w, x, a, b);
    lane_swap<32>(y, z, c, d);
    lane_swap<16>(a + b, c + d, e, f);
    return row_sum(e + f);
}

__device__ __forceinline__ double read_lane(double v, int lane)
{
    union { double d; int w[2]; } u;
    u.d = v;
    u.w[0] = __builtin_amdgcn_readlane(u.w[0], lane);
    u.w[1] = __builtin_amdgcn_readlane(u.w[1], lane);
    return u.d;
}

// Deterministic block sum: wave butterflies, then wave 0..3 in order.
// Result valid in every thread.  `sh` holds kBlock/kWave values.
template <class T>
__device__ __forceinline__ T block_sum(T v, T *sh)
{
    v = wave_sum(v);
    const int w = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) sh[w] = v;
    __syncthreads();
    T s = sh[0];
#pragma unroll
    for (int i = 1; i < kBlock / kWave; ++i) s += sh[i];
    return s;
}

// Fixed-order sum of nblk partials by one block (all threads get the result).
// Each lane sums part[tid], part[tid + 256], ... in that order; the loads of a
// chunk are issued together so the reduction costs one memory latency.
__device__ __forceinline__ double reduce_partials(const double *part, int nblk, double *sh)
{
    constexpr int U = 8;
    double s = 0.0;
    for (int i0 = threadIdx.x; i0 < nblk; i0 += kBlock * U) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kBlock;
            v[u] = i < nblk ? part[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) s += v[u];
    }
    return block_sum(s, sh);
}

// Three partial arrays reduced together (same order as reduce_partials); all
// loads of a chunk are in flight at once.
__device__ __forceinline__ void reduce_partials3(const double *pa, const double *pb,
                                                 const double *pc, int nblk, double *sh,
                                                 double &A, double &B, double &C)
{
    constexpr int U = 8;
    double s = 0.0, t = 0.0, w = 0.0;
    for (int i0 = threadIdx.x; i0 < nblk; i0 += kBlock * U) {
        double u0[U], u1[U], u2[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kBlock;
            u0[u] = i < nblk ? pa[i] : 0.0;
            u1[u] = i < nblk ? pb[i] : 0.0;
            u2[u] = i < nblk ? pc[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s += u0[u];
            t += u1[u];
            w += u2[u];
        }
    }
    A = block_sum(s, sh);
    B = block_sum(t, sh);
    C = block_sum(w, sh);
}

// Two partial arrays reduced together (same order as reduce_partials).
__device__ __forceinline__ void reduce_partials2(const double *pa, const double *pb, int nblk,
                                                 double *sh, double &A, double &B)
{
    constexpr int U = 8;
    double s = 0.0, t = 0.0;
    for (int i0 = threadIdx.x; i0 < nblk; i0 += kBlock * U) {
        double v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kBlock;
            v[u] = i < nblk ? pa[i] : 0.0;
            w[u] = i < nblk ? pb[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s += v[u];
            t += w[u];
        }
    }
    A = block_sum(s, sh);
    B = block_sum(t, sh);
}

template <class T>
__device__ __forceinline__ T ld_stream(const T *p)
{
    return __builtin_nontemporal_load(p);
}

}  // namespace spk
