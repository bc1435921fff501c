// Brick step kernel instances for double state.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "brick.hpp"

namespace tdse {

namespace {

template <int W, int BX, int BY>
hipError_t go(BrickOp op, bool rec, dim3 grid, size_t lds, hipStream_t st, const BrickArgs<double>& a,
              hipEvent_t e0, hipEvent_t e1) {
    const dim3 all((BX + 2 * BRICK_HALO) / W, BY + 2 * BRICK_HALO, BRICK_NG);
    const dim3 owners(BX / W, BY, 2);
    auto run = [&](auto kern, dim3 block) -> hipError_t {
        if (lds > 65536) {
            // more than 64 KiB of dynamic LDS has to be allowed per kernel
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        if (e0)
            hipExtLaunchKernelGGL(kern, grid, block, lds, st, e0, e1, 0, a);
        else
            hipLaunchKernelGGL(kern, grid, block, lds, st, a);
        return hipGetLastError();
    };
    switch (op) {
        case BRICK_TWO:
            return rec ? run(brick_kernel<double, W, BX, BY, true, true>, all)
                       : run(brick_kernel<double, W, BX, BY, false, true>, all);
        case BRICK_ONE:
            return rec ? run(brick_kernel<double, W, BX, BY, true, false>, all)
                       : run(brick_kernel<double, W, BX, BY, false, false>, all);
        case BRICK_HALF_I: return run(brick_half_kernel<double, W, BX, BY, false, false>, owners);
        default:
            return rec ? run(brick_half_kernel<double, W, BX, BY, true, true>, owners)
                       : run(brick_half_kernel<double, W, BX, BY, true, false>, owners);
    }
}

}  // namespace

hipError_t launch_brick_f64(int w, int bx, int by, BrickOp op, bool rec, dim3 grid, size_t lds,
                            hipStream_t st, const BrickArgs<double>& a, hipEvent_t e0, hipEvent_t e1) {
    if (w == 2 && bx == 16 && by == 8) return go<2, 16, 8>(op, rec, grid, lds, st, a, e0, e1);
    if (w == 2 && bx == 8 && by == 8) return go<2, 8, 8>(op, rec, grid, lds, st, a, e0, e1);
    if (w == 1 && bx == 8 && by == 8) return go<1, 8, 8>(op, rec, grid, lds, st, a, e0, e1);
    return hipErrorInvalidValue;
}

}  // namespace tdse
