// Launch of one Chebyshev step (cheb.hpp), FP64 or FP32.
#pragma once

#include <algorithm>

#include "cheb.hpp"
#include "runtime.hpp"

namespace spk {

inline int grid_n(int64_t n)
{
    int64_t g = (n + kBlock - 1) / kBlock;
    if (g > kMaxBlocksSingle) g = kMaxBlocksSingle;
    return (int)(g < 1 ? 1 : g);
}

// One Chebyshev step: fused SpMV + update for the SELL and stream families,
// SpMV into tmp then the update pass for the others (V = double, or float
// with the handle's FP32 values).
template <class V>
int cheb_step(spk_mat *A, const ChebStep<V> &c, V *tmp, hipStream_t s, int *np)
{
    constexpr bool f64 = std::is_same<V, double>::value;
    const dim3 g(A->nblk), t(kBlock);
    if ((c.b || c.b64) && !cheb_zero_fused(A)) {
        set_error("internal: Chebyshev start from zero without a SELL layout");
        return SPK_EINVAL;
    }
    if (A->kernel == SPK_KERNEL_SELL) {
        const SellView sv{A->sell_ptr, A->sell_col, A->sell_len, A->sell_plain, A->sell_len16, A->sell_perm, A->sell_mask};
        // up to one wavefront per slice (no partial sums to keep per block)
        const dim3 gs(std::max(1, std::min(ceil_div(ceil_div(A->n, kSell), kBlock / kWave), 16384)));
        const int n = A->n;
        const V *sval = f64 ? (const V *)A->sell_val : (const V *)A->sell_val32;
        if (!sval) { set_error("internal: no SELL values of this precision"); return SPK_EINVAL; }
        auto from_zero = [&](auto *b) {
            using B = std::remove_const_t<std::remove_pointer_t<decltype(b)>>;
            with_sell(A, [&](auto ci, auto uc) {
                using CI = decltype(ci);
                constexpr int U = decltype(uc)::value;
                hipLaunchKernelGGL((k_cheb_sell_zero<V, B, CI, U>), gs, t, 0, s, n, sv, sval, c, b);
            });
        };
        if (c.b64) from_zero(c.b64);
        else if (c.b) from_zero(c.b);
        else
            with_sell(A, [&](auto ci, auto uc) {
                using CI = decltype(ci);
                constexpr int U = decltype(uc)::value;
                hipLaunchKernelGGL((k_cheb_sell<V, CI, U>), gs, t, 0, s, n, sv, sval, c);
            });
        if (np) *np = (int)gs.x;
    } else if (A->kernel == SPK_KERNEL_STREAM) {
        const V *val = f64 ? (const V *)A->val : (const V *)A->val32;
        hipLaunchKernelGGL((k_cheb_stream<V>), g, t, 0, s, A->n, A->R, A->ntiles, A->nblk, A->rowptr, A->col, val,
                           c);
        if (np) *np = A->nblk;
    } else {
        const V *val = f64 ? (const V *)A->val : (const V *)A->val32;
        SPK_TRY(launch_spmv<V>(A, val, c.dk, tmp, s, c.gate, c.gate ? kGateInner64 : kGateNone));
        hipLaunchKernelGGL((k_cheb_update<V>), dim3(grid_n(A->n)), t, 0, s, A->n, (const V *)tmp, c);
        if (np) *np = grid_n(A->n);
    }
    SPK_HIP(hipGetLastError());
    return SPK_OK;
}

}  // namespace spk
