// Launches of the Krylov iterations of one system, FP64 or FP32.
//
// A process loads the code of a source file, all its instances, when it first
// launches one of its kernels (about 3 ms a megabyte), so what is used apart is
// compiled apart: the iterations of either precision (iter64.hip, iter32.hip),
// the smoother's steps (cheb.hip, cheb32.hip), the one-launch solves
// (resident.hip), and the rest of the solves (ksp.hip).  The first call of a
// process, with all but the one-launch solves in one file of 4.6 MB and apart:
// smoothing of 7-point 128^3 15.0 -> 8.0 ms, a solve of 64^2 17.6 -> 6.9, of
// 61 x 47 x 53 22.3 -> 12.6, of 128^3 34.3 -> 26.3, with multigrid 14.8 -> 5.5.
#pragma once

#include "krylov.hpp"
#include "runtime.hpp"

namespace spk {

// Every pointer of the descriptor is owned by the workspace (b is copied in),
// so the descriptor travels by value in the kernel arguments and captured
// graphs stay valid from one solve to the next.  A profiled solve times the
// product kernel alone, so it runs the three-kernel iteration: its
// descriptor has no second p buffer (the results are the same bits).
inline bool use_fused(const Workspace *w, bool mixed) { return (mixed ? w->fused32 : w->fused64) && !w->prof; }
inline One batch_of(Workspace *w, bool mixed)
{
    One b{w->hdesc};
    if (!mixed) b.d.nblk = w->nblk64;
    if (!use_fused(w, false)) b.d.p2 = nullptr;
    if (!use_fused(w, true)) b.d.p2_32 = nullptr;
    return b;
}

// The next event pair of a profiled solve (created on first use).
inline int prof_pair(Workspace *w, hipEvent_t *e0, hipEvent_t *e1)
{
    const size_t k = 2 * (size_t)w->pev_used;
    while (w->pev.size() < k + 2) {
        hipEvent_t e = nullptr;
        SPK_HIP(hipEventCreate(&e));
        w->pev.push_back(e);
    }
    if (w->alive.size() < (size_t)w->pev_used + 1) w->alive.resize(w->pev_used + 1);
    w->alive[w->pev_used] = 1;
    *e0 = w->pev[k];
    *e1 = w->pev[k + 1];
    ++w->pev_used;
    return SPK_OK;
}

template <class V>
int launch_iteration(spk_mat *A, Workspace *w, hipStream_t s)
{
    const One b = batch_of(w, Vecs<V>::mixed);
    const dim3 g(b.d.nblk), t(kBlock), one(1);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (w->prof) {
        SPK_TRY(prof_pair(w, &e0, &e1));
        SPK_HIP(hipEventRecord(e0, s));
    }
    if (A->kernel == SPK_KERNEL_STREAM) {
        hipLaunchKernelGGL((k_pcg_spmv_stream<V, One>), g, t, 0, s, b);
    } else if (A->kernel == SPK_KERNEL_SELL && w->wpart) {
        const dim3 gw(w->nwpart);
        with_sell(A, [&](auto ci, auto uc) {
            using CI = decltype(ci);
            constexpr int U = decltype(uc)::value;
            // (a list for the whole matrix streams too little for the rule)
            if constexpr (!std::is_same<CI, Stencil>::value)
                hipLaunchKernelGGL((k_pcg_spmv_sell_wide<V, CI, U>), gw, t, 0, s, b, w->wpart);
        });
        // the pair times the slice kernel, which moves the bytes; the fold
        // of its per-block partials (one block, a few microseconds) is outside
        if (e1) {
            SPK_HIP(hipEventRecord(e1, s));
            e1 = nullptr;
        }
        hipLaunchKernelGGL((k_fin_pq<V>), one, dim3(kFinPqThreads), 0, s, b, (const double *)w->wpart, w->nwpart);
    } else if (A->kernel == SPK_KERNEL_SELL) {
        with_sell(A, [&](auto ci, auto uc) {
            using CI = decltype(ci);
            constexpr int U = decltype(uc)::value;
            hipLaunchKernelGGL((k_pcg_spmv_sell<V, CI, U, One>), g, t, 0, s, b);
        });
    } else {
        const V *val = std::is_same<V, double>::value ? (const V *)A->val : (const V *)A->val32;
        V *p = std::is_same<V, double>::value ? (V *)w->p : (V *)w->p32;
        V *q = std::is_same<V, double>::value ? (V *)w->q : (V *)w->q32;
        SPK_TRY(launch_spmv<V>(A, val, p, q, s, w->st, Vecs<V>::gate));
        hipLaunchKernelGGL((k_pcg_pq<V, One>), g, t, 0, s, b);
    }
    if (e1) SPK_HIP(hipEventRecord(e1, s));
    hipLaunchKernelGGL((k_pcg_update<V, One>), g, t, 0, s, b);
    hipLaunchKernelGGL((k_pcg_px<V, One>), g, t, 0, s, b);
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

// B of the fused iteration.
template <class V>
void launch_update(spk_mat *A, Workspace *w, hipStream_t s)
{
    const One b = batch_of(w, Vecs<V>::mixed);
    const dim3 g(b.d.nblk), t(kBlock);
    if (one_diag(A)) hipLaunchKernelGGL((k_pcg_update<V, One, true>), g, t, 0, s, b);
    else hipLaunchKernelGGL((k_pcg_update<V, One>), g, t, 0, s, b);
}

// Pairs per round of F for a matrix whose walk takes u.  A start runs once a
// sequence: one size will do for it (the list for a whole matrix has to fit its
// round).  In FP32, 27 z and p in flight hold 169 registers, two waves to a SIMD;
// two rounds, of 9 and 4 pairs, hold 122, four waves.  Mixed solves of 27-point
// 96^3 11.1 -> 9.7 ms, 61 x 47 x 53 3.34 -> 3.02, 30^3 1.39 -> 1.36 (rounds of 7: 9.4,
// 3.03 and 1.42; of 5: 9.7, 2.99 and 1.39).  In FP64 27 of them leave two waves
// either way; 15 leave three, where two rounds of 4 leave five, which pays once
// the persistent grid's waves take more than one slice each (15-point 96^3, 60
// iterations: 3.20 -> 2.78 ms; 30^3 0.81 -> 0.84).
template <class V, class CI, bool kStart>
constexpr int fused_round(int u)
{
    if (std::is_same<CI, Stencil>::value) return u;
    if (kStart) return 4;
    return std::is_same<V, float>::value && std::is_same<CI, int32_t>::value && u == 13 ? 9 : u;
}

// F of the fused iteration (the C part, then the next product).
template <class V, bool kStart>
void launch_fused(spk_mat *A, Workspace *w, hipStream_t s)
{
    const One b = batch_of(w, Vecs<V>::mixed);
    const dim3 g(b.d.nblk), t(kBlock);
    with_sell(A, [&](auto ci, auto uc) {
        using CI = decltype(ci);
        constexpr int U = fused_round<V, CI, kStart>(decltype(uc)::value);
        if constexpr (std::is_same<V, double>::value && std::is_same<CI, int32_t>::value && U == 7)
            if (ceil_div(A->n, kSell) > b.d.nblk * (kBlock / kWave)) {
                hipLaunchKernelGGL((k_pcg_fused_sell<V, CI, 4, kStart, One>), g, t, 0, s, b);
                return;
            }
        hipLaunchKernelGGL((k_pcg_fused_sell<V, CI, U, kStart, One>), g, t, 0, s, b);
    });
}

// K iterations of a batch.  Fused: a start kernel (a no-op unless a setup
// finalizer just ran) and K times B, F.
template <class V>
int launch_iterations(spk_mat *A, Workspace *w, int K, hipStream_t s)
{
    constexpr bool mixed = Vecs<V>::mixed;
    if (use_fused(w, mixed)) {
        launch_fused<V, true>(A, w, s);
        for (int k = 0; k < K; ++k) {
            launch_update<V>(A, w, s);
            launch_fused<V, false>(A, w, s);
        }
    } else {
        if constexpr (mixed)
            hipLaunchKernelGGL((k_pcg_p_continue<float, One>), dim3(A->nblk), dim3(kBlock), 0, s, batch_of(w, true));
        for (int k = 0; k < K; ++k) SPK_TRY(launch_iteration<V>(A, w, s));
    }
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

// each in a file of its own
extern template int launch_iterations<double>(spk_mat *, Workspace *, int, hipStream_t);
extern template int launch_iterations<float>(spk_mat *, Workspace *, int, hipStream_t);

}  // namespace spk
