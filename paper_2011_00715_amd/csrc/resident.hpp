// The FP64 Jacobi-PCG iterations of a small SELL system in one launch.
//
// A system of up to 2^18 rows stays in the caches, and its two kernels per
// iteration then cost launches and ramp-up, not bandwidth (64 x 64 five-point:
// 10.4 us an iteration for 0.5 MB of data).  Here the blocks stay for the whole
// solve: a row's x, r, p, q and D^-1 live in its lane's registers, and the
// iteration's two reductions are the only meetings.
//
//  * One block (up to kResidentRows1 rows): p and q live in LDS, nothing
//    leaves the CU, a reduction costs one barrier.  An iteration takes 2.5 us at
//    1,024 rows and 4.7 at 4,096 (10.4 as two launches), where what every wave
//    issues sets the time.
//  * Several blocks (two tiles of 256 rows each, launched cooperatively so that
//    all are resident): the product gathers z and the previous p from memory and forms
//    p' = z + beta p as the fused kernel F does, so the update's reduction
//    also orders the exchange of z and no third meeting is needed.  What one
//    block writes and another reads (z, p, partial sums) is stored and loaded
//    with agent scope, past the per-XCD L2s: no cache is written back or
//    invalidated.  An iteration takes 6.5 us at 4,550 rows, 7.3 at 40,000, 9.8 at
//    262,144 (12.0, 12.1 and 16.8 as two launches): two meetings and a product
//    from beyond the L2s.  One block is faster up to the rows it holds.
//
// The operations are those of k_pcg_update and k_pcg_fused_sell, and so are the
// sums: a tile of 256 rows is one block there (the FP64 partition of these
// sizes, see fp64_blocks), so a tile's partial sum is the butterflies of its
// four slices added in order, and the partials are added as partials_sum adds
// them.  A solve gives the same bits on either path.
#pragma once

#include "krylov.hpp"

namespace spk {

constexpr int kResTile = kBlock / kWave;         // slices of a tile
// one block: 8 wavefronts, so that what every wave does for itself (totals,
// the decision) is done twice per SIMD, and up to 8 rows per lane
constexpr int kResOne = 512;
constexpr int kResOneWaves = kResOne / kWave;
constexpr int kResRows1 = 8;
constexpr int kResidentRows1 = kResOne * kResRows1;
constexpr int kResSlices1 = kResidentRows1 / kSell;
// several blocks: two tiles each, at most two blocks per CU
constexpr int kResMany = 512;
constexpr int kResManyTiles = kResMany / kBlock;
constexpr int kResPerCu = 2;
constexpr int kResidentTiles = 1024;
constexpr int kResidentRowsN = kResidentTiles * kBlock;
// partials_sum's first level: lanes t, t + 1, ... of wave g add the tiles
// t, t + 256, ..., so group g is 64 such lanes
constexpr int kResGroups = kBlock / kWave;
constexpr int kResMaxU = 4;                      // pairs per round: rows of up to 9 entries in one

// Partial sums of one reduction: a slot per tile and sum, three in turn.
constexpr int kResRing = 3;
// An empty slot: a NaN that a published sum never is (NaNs are published as
// the canonical one).
constexpr unsigned long long kResEmpty = 0x7ff4dead00c0ffeeull;
// Polls of a slot before a block gives up (seconds): every wait ends, also where
// something else holds the CUs that the other blocks need.
constexpr int kResPolls = 1 << 21;

struct ResidentArgs {
    SysDesc d;
    unsigned long long *slots;  // [kResRing][2][nblk + kResGroups], all kResEmpty on entry
    int32_t *gave_up;           // set when a wait ran out
    int polls;                  // of a slot, before a block gives up
};

template <class T>
__device__ __forceinline__ T ld_agent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_agent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the product of several blocks gathers.
struct GatherRes {
    const double *z, *p;
    double beta;
    bool fresh;
    struct Raw {
        double z, p;
    };
    __device__ Raw at(int j) const { return Raw{ld_agent(z + j), ld_agent(p + j)}; }
    __device__ Raw sh(int64_t base, unsigned l) const
    {
        return Raw{ld_agent(z + base + l), ld_agent(p + base + l)};
    }
    __device__ double of(const Raw &r) const { return fresh ? r.z : fma(beta, r.p, r.z); }
};

// What the product of one block gathers: p in LDS.
struct GatherLds {
    const double *p;
    using Raw = double;
    __device__ double at(int j) const { return p[j]; }
    __device__ double sh(int64_t base, unsigned l) const { return p[(int)base + (int)l]; }
    __device__ double of(double v) const { return v; }
};

// The scalars of the iteration's decision.
struct ResScalars {
    double rho, alpha = 0.0, beta = 0.0, rn;
    int iter, status = SPK_RUNNING;
    bool fresh = true;  // no iteration yet: p = z
};

// pcg_decide for an FP64 solve; identical in every thread.
__device__ __forceinline__ void res_decide(ResScalars &c, bool step, double eta, double rz, double rr,
                                           const SysState &ss, double *hist, bool first)
{
    if (!step) {
        c.status = finite(eta) ? SPK_DIVERGED_INDEFINITE_MAT : SPK_DIVERGED_NANORINF;
        return;
    }
    ++c.iter;
    c.rn = sqrt(rr);
    if (first && hist && c.iter < ss.hist_len) hist[c.iter] = c.rn;
    if (!finite(c.rn)) c.status = SPK_DIVERGED_NANORINF;
    else if (c.rn <= ss.thresh)
        c.status = c.rn <= ss.rtol * ss.bnorm ? SPK_CONVERGED_RTOL : SPK_CONVERGED_ATOL;
    else if (c.iter >= ss.maxit) c.status = SPK_DIVERGED_ITS;
    else if (!finite(rz)) c.status = SPK_DIVERGED_NANORINF;
    else if (rz < 0.0) c.status = SPK_DIVERGED_INDEFINITE_PC;
    else if (rz == 0.0) c.status = SPK_DIVERGED_BREAKDOWN;
    else {
        c.beta = rz / c.rho;
        c.rho = rz;
        c.fresh = false;
    }
}

__device__ __forceinline__ void res_store(SysState *st, const ResScalars &c, double eta)
{
    st->status = c.status;
    st->iter = c.iter;
    st->rnorm = c.rn;
    st->rho = c.rho;
    st->eta = eta;
    st->alpha = c.alpha;
    st->beta = c.beta;
}

// One block: the iterations of a solve from the state the setup kernels left
// (r, z, rho) to its stop.  Thread's k-th row: slice 8 k + wave.
template <class CI, int U>
__global__ __launch_bounds__(kResOne) void k_pcg_resident_one(ResidentArgs a)
{
    constexpr int R = kResRows1;
    extern __shared__ double lds[];
    // slices' sums, three kinds; two sets in turn, so that a sum costs one barrier
    __shared__ double ws[2][3][kResSlices1];
    __shared__ SysState ss;
    const SysDesc &d = a.d;
    const int n = d.n, ns = (n + kSell - 1) / kSell, ntiles = d.nblk;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int used = (ns + kResOneWaves - 1) / kResOneWaves;  // rows per thread
    double *ql = lds;                            // q of the thread's k-th row at k * kResOne + tid
    double *pl = lds + (size_t)used * kResOne;   // p by row
    if (tid == 0) {
        ss = *d.st;
        *a.gave_up = 0;
    }
    __syncthreads();
    if (ss.status != SPK_RUNNING) return;
    double x[R], r[R], dinv[R], p[R];
    auto row_of = [&](int k) { return (w + k * kResOneWaves) * kSell + lane; };
#pragma unroll
    for (int k = 0; k < R; ++k) {
        x[k] = r[k] = dinv[k] = p[k] = 0.0;
        const int i = row_of(k);
        if (i < n) {
            x[k] = d.x[i];
            r[k] = d.r[i];
            dinv[k] = d.dinv[i];
            p[k] = d.z[i];  // p = z starts the sequence
            pl[i] = p[k];
        }
    }
    for (int i = tid; i < 6 * kResSlices1; i += kResOne) (&ws[0][0][0])[i] = 0.0;
    __syncthreads();
    const SellView sv{d.sell_ptr, d.sell_col, d.sell_len, d.sell_plain, d.sell_len16, d.sell_perm, d.sell_mask};
    // the slices' sums of v[0..R) into set `to`, four at a time
    const int kk = ((lane >> 4) & 1) * 2 + (lane >> 5);  // which of the four this row of lanes ends with
    auto put = [&](const double (&v)[R], double *to) {
#pragma unroll
        for (int g = 0; g < R; g += 4)
            if (g < used) {
                const double s = wave_sum4(v[g], v[g + 1], v[g + 2], v[g + 3]);
                if ((lane & 15) == 0) to[(g + kk) * kResOneWaves + w] = s;
            }
    };
    // the tile at this lane's place among the partials: p.q's stand in the
    // order of the product's blocks
    const int per = ntiles / kXcd;
    const int tile_pq = lane < ntiles && ntiles >= kXcd && ntiles % kXcd == 0 ? lane % per * kXcd + lane / per : lane;
    auto tile_sum = [&](const double *v, int t) {
        double s = 0.0;
        if (lane < ntiles) {
            s = v[kResTile * t];
#pragma unroll
            for (int i = 1; i < kResTile; ++i) s += v[kResTile * t + i];
        }
        return s;
    };
    ResScalars c;
    c.rho = ss.rho;
    c.rn = ss.rnorm;
    c.iter = ss.iter;
    double eta = 0.0;
    int set = 0;
    while (c.status == SPK_RUNNING) {
        // A: q = A p and p.q
        int k = 0;
        sell_slices_g<double, CI, U>(n, w, kResOneWaves, sv, d.sell_val, GatherLds{pl}, [] { return true; }, NoOwn{},
                                     [&](int, double y, int) { ql[k++ * kResOne + tid] = y; });
        double q[R], t0[R], t1[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            q[u] = row_of(u) < n ? ql[u * kResOne + tid] : 0.0;
            t0[u] = fma(q[u], p[u], 0.0);
        }
        put(t0, ws[set][0]);
        __syncthreads();
        eta = wave_sum(tile_sum(ws[set][0], tile_pq));
        // B: r -= alpha q, z = D^-1 r, r.z and r.r; x += alpha p
        double rz = 0.0, rr = 0.0;
        const bool step = eta > 0.0 && finite(eta);
        if (step) {
            c.alpha = c.rho / eta;
#pragma unroll
            for (int u = 0; u < R; ++u) {  // rows past n hold zeros and keep them
                r[u] = fma(-c.alpha, q[u], r[u]);
                q[u] = dinv[u] * r[u];
                x[u] = fma(c.alpha, p[u], x[u]);
                t0[u] = fma(r[u], q[u], 0.0);
                t1[u] = fma(r[u], r[u], 0.0);
            }
            put(t0, ws[set][1]);
            put(t1, ws[set][2]);
            __syncthreads();
            const double both = wave_sum2(tile_sum(ws[set][1], lane), tile_sum(ws[set][2], lane));
            rz = read_lane(both, 0);
            rr = read_lane(both, kWave / 2);
        }
        set ^= 1;
        res_decide(c, step, eta, rz, rr, ss, d.hist, tid == 0);
        if (c.status == SPK_RUNNING) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                p[u] = fma(c.beta, p[u], q[u]);
                if (row_of(u) < n) pl[row_of(u)] = p[u];
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (row_of(k) < n) {
            d.x[row_of(k)] = x[k];
            d.r[row_of(k)] = r[k];
        }
    if (tid == 0) res_store(d.st, c, eta);
}

// Several blocks' meeting: publishes this block's tile sums and returns the
// sums over all tiles in every thread.  Before it, every thread's own
// agent-scope stores are waited for, so who leaves the meeting sees them.
// Two levels: a wave per group (and sum) collects the group's tiles and
// publishes their sum, and all blocks read the groups' sums, one line.  With
// every block reading every tile, all blocks' polls met on the few memory
// channels that hold the slots: 152 k rows took 18.6 us an iteration with
// blocks of one tile, 10.2 with blocks of four.
// A block whose wait runs out leaves for good, and so do those that wait for it
// at this meeting or the next.  At a solve's last meeting some may leave and
// others finish: x, r and the state are then of no use.
struct Meeting {
    unsigned long long *slots;
    int32_t *gave_up;
    int polls;
    double *ws;     // [2][kResMany / kWave]
    double *group;  // [2][kResGroups]
    int nblk, turn = 0;
    bool lost = false;

    __device__ __forceinline__ unsigned long long *ring(int t) const
    {
        return slots + (size_t)t * 2 * (nblk + kResGroups);
    }

    // Waits for P slots, stride apart, of which this lane has the first cnt;
    // all of a round's loads are in flight together.
    template <int P>
    __device__ __forceinline__ void wait_slots(unsigned long long *p, int stride, int cnt,
                                               unsigned long long (&v)[P], bool &ok) const
    {
#pragma unroll
        for (int u = 0; u < P; ++u) v[u] = u < cnt ? ld_agent(p + (size_t)u * stride) : 0;
        bool all = false;
        for (int k = 0; k < polls; ++k) {
            all = true;
#pragma unroll
            for (int u = 0; u < P; ++u) all &= v[u] != kResEmpty;
            if (all) break;
#pragma unroll
            for (int u = 0; u < P; ++u)
                if (v[u] == kResEmpty) v[u] = ld_agent(p + (size_t)u * stride);
        }
        ok &= all;
    }

    // remap: partials in the order of the product's blocks
    __device__ __forceinline__ void sums(double a, double b, bool two, bool remap, double &A, double &B)
    {
        constexpr int kWaves = kResMany / kWave;
        const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
        const double v = two ? wave_sum2(a, b) : wave_sum(a);
        if (lane == 0) ws[w] = v;
        if (two && lane == kWave / 2) ws[kWaves + w] = v;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's stores have arrived
        __syncthreads();
        unsigned long long *cur = ring(turn);
        // the block's tiles: thread 2 i + sum
        const int tile = (int)blockIdx.x * kResManyTiles + tid / 2;
        if (tid < 2 * kResManyTiles && tile < nblk && (tid & 1) <= (two ? 1 : 0)) {
            const double *m = ws + (tid & 1) * kWaves + tid / 2 * kResTile;
            st_agent(cur + (size_t)(tid & 1) * nblk + (remap ? xcd_remap(tile, nblk) : tile),
                     bits(((m[0] + m[1]) + m[2]) + m[3]));
        }
        bool ok = true;
        const int jobs = two ? 2 * kResGroups : kResGroups;
        for (int job = (int)blockIdx.x + w * (int)gridDim.x; job < jobs; job += kWaves * (int)gridDim.x) {
            const int g = job % kResGroups, which = job / kResGroups;
            constexpr int P = kResidentTiles / kBlock;
            const int i = g * kWave + lane;
            unsigned long long v[P];
            wait_slots(cur + (size_t)which * nblk + i, kBlock, i < nblk ? (nblk - i + kBlock - 1) / kBlock : 0, v, ok);
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < P; ++u) s += __longlong_as_double((long long)v[u]);
            s = wave_sum(s);
            if (lane == 0) st_agent(cur + 2 * (size_t)nblk + job, bits(s));
        }
        if (tid < jobs) {
            unsigned long long v[1];
            wait_slots(cur + 2 * (size_t)nblk + tid, 0, 1, v, ok);
            group[tid] = __longlong_as_double((long long)v[0]);
        }
        if (!__syncthreads_and(ok)) {
            lost = true;
            if (tid == 0) st_agent(gave_up, 1);
            return;
        }
        // leaving meeting t, all blocks have arrived at it and so have left
        // meeting t - 1: its slots may be emptied for meeting t + 2, and are
        // before this block arrives at t + 1 (by place here, whoever filled it)
        unsigned long long *old = ring(turn == 0 ? kResRing - 1 : turn - 1);
        if (tid < 2 * kResManyTiles && tile < nblk) st_agent(old + (size_t)(tid & 1) * nblk + tile, kResEmpty);
        if (blockIdx.x == 0 && tid < 2 * kResGroups) st_agent(old + 2 * (size_t)nblk + tid, kResEmpty);
        A = ((group[0] + group[1]) + group[2]) + group[3];
        if (two) B = ((group[4] + group[5]) + group[6]) + group[7];
        turn = turn == kResRing - 1 ? 0 : turn + 1;
    }

    static __device__ __forceinline__ unsigned long long bits(double v)
    {
        return v == v ? (unsigned long long)__double_as_longlong(v) : 0x7ff8000000000000ull;
    }
};

// Several blocks, two tiles each: the same iterations, a row per thread.
template <class CI, int U>
__global__ __launch_bounds__(kResMany, kResPerCu * kResMany / kWave / 4) void k_pcg_resident_many(ResidentArgs a)
{
    __shared__ double ws[2 * kResMany / kWave];
    __shared__ double group[2 * kResGroups];
    __shared__ SysState ss;
    const SysDesc &d = a.d;
    const int n = d.n, ns = (n + kSell - 1) / kSell, nblk = d.nblk;
    const int tid = threadIdx.x;
    const int s0 = (int)blockIdx.x * (kResMany / kWave) + tid / kWave;
    const int row = (int)blockIdx.x * kResMany + tid;
    const bool own = row < n;
    if (tid == 0) ss = *d.st;
    __syncthreads();
    if (ss.status != SPK_RUNNING) return;  // the same in all blocks: nobody waits
    double x = 0.0, r = 0.0, dinv = 0.0, p = 0.0;
    if (own) {
        x = d.x[row];
        r = d.r[row];
        dinv = d.dinv[row];
    }
    const SellView sv{d.sell_ptr, d.sell_col, d.sell_len, d.sell_plain, d.sell_len16, d.sell_perm, d.sell_mask};
    Meeting meet{a.slots, a.gave_up, a.polls, ws, group, nblk};
    ResScalars c;
    c.rho = ss.rho;
    c.rn = ss.rnorm;
    c.iter = ss.iter;
    double eta = 0.0, none = 0.0, z = dinv * r;
    bool flip = false;
    while (c.status == SPK_RUNNING) {
        // A: q = A p and p.q
        const double *pold = flip ? d.p2 : d.p;
        double *pnew = flip ? d.p : d.p2;
        flip = !flip;
        p = c.fresh ? z : fma(c.beta, p, z);
        if (own) st_agent(pnew + row, p);
        double q = 0.0;
        sell_slices_g<double, CI, U>(n, s0, ns, sv, d.sell_val, GatherRes{d.z, pold, c.beta, c.fresh},
                                     [] { return true; }, NoOwn{}, [&](int, double y, int) { q = y; });
        meet.sums(fma(q, p, 0.0), 0.0, false, true, eta, none);
        if (meet.lost) return;
        // B: r -= alpha q, z = D^-1 r, r.z and r.r; x += alpha p
        double rz = 0.0, rr = 0.0;
        const bool step = eta > 0.0 && finite(eta);
        if (step) {
            c.alpha = c.rho / eta;
            r = fma(-c.alpha, q, r);
            z = dinv * r;
            if (own) st_agent(d.z + row, z);
            x = fma(c.alpha, p, x);
            meet.sums(fma(r, z, 0.0), fma(r, r, 0.0), true, false, rz, rr);
            if (meet.lost) return;
        }
        res_decide(c, step, eta, rz, rr, ss, d.hist, blockIdx.x == 0 && tid == 0);
    }
    if (own) {
        d.x[row] = x;
        d.r[row] = r;
    }
    if (blockIdx.x == 0 && tid == 0) res_store(d.st, c, eta);
}

static __global__ void k_res_empty(unsigned long long *slots, int count, int32_t *gave_up)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) slots[i] = kResEmpty;
    if (blockIdx.x == 0 && threadIdx.x == 0) *gave_up = 0;
}

}  // namespace spk
