// Launch of the one-launch PCG iterations (resident.hpp).
#include <algorithm>
#include <cstdlib>

#include "resident.hpp"
#include "runtime.hpp"

namespace spk {

// Stencil-like rows (one round of the walk) in matrix order, few enough for
// the blocks that the device holds at once.  Larger systems keep two kernels
// per iteration: they would need more rows per lane than registers hold, and
// there bandwidth, not launches, sets the time.
bool resident_fits(const spk_mat *A)
{
    if (A->kernel != SPK_KERNEL_SELL || !A->sell_cw || A->sell_perm || A->sell_u > kResMaxU) return false;
    if (A->n <= kResidentRows1) return true;
    int cus = 0, coop = 0;
    if (A->n > kResidentRowsN ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, A->device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, A->device) != hipSuccess)
        return false;
    return coop && ceil_div(A->n, kResMany) <= cus * kResPerCu;
}

int64_t resident_slots(const spk_mat *A) 
{
    return (int64_t)kResRing * 2 * (ceil_div(A->n, kBlock) + kResGroups);
}

template <class CI, int U>
static hipError_t launch(const spk_mat *A, ResidentArgs a, int nslots, hipStream_t s)
{
    if (A->n <= kResidentRows1) {
        const int used = ceil_div(ceil_div(A->n, kSell), kResOneWaves);
        const size_t lds = sizeof(double) * ((size_t)used * kResOne + (size_t)A->n);
        const void *f = (const void *)k_pcg_resident_one<CI, U>;
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_pcg_resident_one<CI, U>), dim3(1), dim3(kResOne), lds, s, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_res_empty, dim3(ceil_div(nslots, kBlock)), dim3(kBlock), 0, s, a.slots, nslots, a.gave_up);
    void *args[] = {&a};
    return hipLaunchCooperativeKernel((const void *)k_pcg_resident_many<CI, U>, dim3(ceil_div(A->n, kResMany)),
                                      dim3(kResMany), args, 0u, s);
}

int resident_polls()
{
    const char *e = getenv("SPK_RESIDENT_POLLS");
    return e ? std::max(atoi(e), 0) : kResPolls;
}

// Runs the iterations of the FP64 solve whose descriptor is d (p2 set, one
// tile per block) on the stream; *done says whether it was launched (the
// caller iterates otherwise).  gave_up (device) is nonzero afterwards if the
// blocks lost each other; x, r and the state then hold nothing of use.
// d.q is not touched.
int launch_resident(const spk_mat *A, const SysDesc &d, unsigned long long *slots, int32_t *gave_up, int polls,
                    hipStream_t s, bool *done)
{
    const ResidentArgs a{d, slots, gave_up, polls};
    hipError_t e = hipErrorInvalidValue;
    with_sell_ci(A->sell_cw, A->sell_plain, [&](auto ci) {
        using CI = decltype(ci);
        const int ns = (int)resident_slots(A);
        if (A->sell_u == 2) e = launch<CI, 2>(A, a, ns, s);
        else if (A->sell_u == 3) e = launch<CI, 3>(A, a, ns, s);
        else if (A->sell_u == 4) e = launch<CI, 4>(A, a, ns, s);
    });
    *done = e == hipSuccess;
    if (e != hipSuccess) (void)hipGetLastError();  // refused (no room for all blocks): nothing ran
    return SPK_OK;
}

}  // namespace spk
