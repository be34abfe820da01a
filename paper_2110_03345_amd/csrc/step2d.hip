// 2D step kernels (both directions, every mode), their batched form, and the
// sweeps that keep the state on the chip.
#include "step_kernels.h"

namespace stride {
namespace {
#include "step2d_resident.h"

template <int R, int MODE, int J, int T>
hipError_t resident_t(const Dims& d, const StencilCoef& cf, const ResidentShape& rs,
                      const ResidentBatch& b, hipStream_t s)
{
    const void* k = reinterpret_cast<const void*>(step2d_resident<R, MODE, J, T>);
    const int lds = resident_lds_bytes(R, rs, b.p[0].injects, MODE == kImageV);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess)
        return e;
    Dims d_ = d;
    StencilCoef cf_ = cf;
    ResidentShape rs_ = rs;
    ResidentBatch b_ = b;
    void* args[] = {&d_, &cf_, &rs_, &b_};
    return hipLaunchCooperativeKernel(k, dim3((b.n * rs.tiles + kXcds - 1) / kXcds * kXcds),
                                      dim3(kResidentThreads), args, (unsigned)lds, s);
}

template <int R, int MODE>
hipError_t resident_m(const Dims& d, const StencilCoef& cf, const ResidentShape& rs,
                      const ResidentBatch& b, hipStream_t s)
{
    constexpr int J = kResidentItems;
    const bool one = resident_items(R, rs) <= kResidentThreads;     // quads per thread
    if (rs.t == 1)
        return one ? resident_t<R, MODE, 1, 1>(d, cf, rs, b, s) : resident_t<R, MODE, J, 1>(d, cf, rs, b, s);
    if constexpr (R == 4)       // (two steps per exchange: order 8, one quad)
        if (one)
            return resident_t<R, MODE, 1, 2>(d, cf, rs, b, s);
    return hipErrorInvalidValue;
}

template <int R>
hipError_t resident_r(int mode, const Dims& d, const StencilCoef& cf, const ResidentShape& rs,
                      const ResidentBatch& b, hipStream_t s)
{
    return mode == kStep    ? resident_m<R, kStep>(d, cf, rs, b, s)
           : mode == kStepV ? resident_m<R, kStepV>(d, cf, rs, b, s)
                            : resident_m<R, kImageV>(d, cf, rs, b, s);
}

}  // namespace

hipError_t launch_resident(const Dims& d, int R, int mode, const StencilCoef& cf,
                           const ResidentShape& rs, const ResidentBatch& b, hipStream_t s)
{
    return R == 4 ? resident_r<4>(mode, d, cf, rs, b, s)
                  : resident_r<5>(mode, d, cf, rs, b, s);
}

void launch_family_2d(bool adjoint, int R, int mode, const Dims& d, const StencilCoef& cf,
                      const SpongeCoef& sp, const LaunchShape& ls, const StepParams& p, hipStream_t s)
{
    if (adjoint)
        R == 4 ? launch_mode_r<false, true, 4>(mode, d, cf, sp, ls, p, s)
               : launch_mode_r<false, true, 5>(mode, d, cf, sp, ls, p, s);
    else
        R == 4 ? launch_mode_r<false, false, 4>(mode, d, cf, sp, ls, p, s)
               : launch_mode_r<false, false, 5>(mode, d, cf, sp, ls, p, s);
}

void launch_batched_2d(bool adjoint, int R, int mode, const Dims& d, const StencilCoef& cf,
                       const LaunchShape& ls, const SlotStep* table, int nslots, int max_samples,
                       hipStream_t s)
{
    if (adjoint)
        R == 4 ? batched_mode_r<false, true, 4>(mode, d, cf, ls, table, nslots, max_samples, s)
               : batched_mode_r<false, true, 5>(mode, d, cf, ls, table, nslots, max_samples, s);
    else
        R == 4 ? batched_mode_r<false, false, 4>(mode, d, cf, ls, table, nslots, max_samples, s)
               : batched_mode_r<false, false, 5>(mode, d, cf, ls, table, nslots, max_samples, s);
}

}  // namespace stride
