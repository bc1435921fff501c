// Two-step (temporally blocked) sweep kernel instances for double state:
// (rows per thread, threads per workgroup) in {(2, 256), (3, 256), (1, 512), (2, 512), (1, 1024)}.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "fused2.hpp"

namespace tdse {

namespace {

template <int W, int M, int NT, bool MARCH = false>
hipError_t go2(bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st, const Fused2Args<double>& a,
               hipEvent_t e0, hipEvent_t e1) {
    auto run = [&](auto kern) -> hipError_t {
        if (lds > 65536) {
            // more than 64 KiB of dynamic LDS has to be allowed per kernel
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        if (e0)
            hipExtLaunchKernelGGL(kern, grid, dim3(NT), lds, st, e0, e1, 0, a);
        else
            hipLaunchKernelGGL(kern, grid, dim3(NT), lds, st, a);
        return hipGetLastError();
    };
    if (pf)
        return rec ? run(fused2_kernel<double, W, M, true, true, NT, MARCH>) : run(fused2_kernel<double, W, M, false, true, NT, MARCH>);
    return rec ? run(fused2_kernel<double, W, M, true, false, NT, false>) : run(fused2_kernel<double, W, M, false, false, NT, false>);
}

template <int W>
hipError_t go2_m(int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                 const Fused2Args<double>& a, hipEvent_t e0, hipEvent_t e1) {
    if (m == 2 && nt == 256) return go2<W, 2, 256>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 3 && nt == 256) return go2<W, 3, 256>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 1 && nt == 512) return go2<W, 1, 512>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 2 && nt == 512) return go2<W, 2, 512>(rec, pf, grid, lds, st, a, e0, e1);
    // the march loop: not with a zero boundary in x or y (nothing could take
    // it).  Vectors of one gain in short chunks without absorption too (us a
    // step with and without: 301x300x200 in 32 planes 155 and 165, in 20 164
    // and 164, 165x88x410 in 32 56.1 and 57.2, in 44 69.1 and 74.1).
    const bool no_march = a.bcx || a.bcy;
    if (m == 1 && nt == 1024)
        return no_march ? go2<W, 1, 1024>(rec, pf, grid, lds, st, a, e0, e1)
                        : go2<W, 1, 1024, true>(rec, pf, grid, lds, st, a, e0, e1);
    return hipErrorInvalidValue;
}

template <int W, int M, int NT, bool MARCH = false>
hipError_t gob2(bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st, const Batch2Step<double>& b) {
    if (pf) {
        if (rec) hipLaunchKernelGGL((fused2_batch_kernel<double, W, M, true, true, NT, MARCH>), grid, dim3(NT), lds, st, b);
        else hipLaunchKernelGGL((fused2_batch_kernel<double, W, M, false, true, NT, MARCH>), grid, dim3(NT), lds, st, b);
    } else {
        if (rec) hipLaunchKernelGGL((fused2_batch_kernel<double, W, M, true, false, NT, false>), grid, dim3(NT), lds, st, b);
        else hipLaunchKernelGGL((fused2_batch_kernel<double, W, M, false, false, NT, false>), grid, dim3(NT), lds, st, b);
    }
    return hipGetLastError();
}

template <int W>
hipError_t gob2_m(int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                  const Batch2Step<double>& b) {
    if (m == 2 && nt == 256) return gob2<W, 2, 256>(rec, pf, grid, lds, st, b);
    if (m == 3 && nt == 256) return gob2<W, 3, 256>(rec, pf, grid, lds, st, b);
    if (m == 1 && nt == 512) return gob2<W, 1, 512>(rec, pf, grid, lds, st, b);
    if (m == 2 && nt == 512) return gob2<W, 2, 512>(rec, pf, grid, lds, st, b);
    if (m == 1 && nt == 1024)
        return b.zero_xy ? gob2<W, 1, 1024>(rec, pf, grid, lds, st, b)
                         : gob2<W, 1, 1024, true>(rec, pf, grid, lds, st, b);
    return hipErrorInvalidValue;
}

template <int W, int M, int NT, bool MARCH = false>
hipError_t allow2(size_t lds) {
    const void* k[4] = {reinterpret_cast<const void*>(fused2_batch_kernel<double, W, M, true, true, NT, MARCH>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<double, W, M, false, true, NT, MARCH>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<double, W, M, true, false, NT, false>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<double, W, M, false, false, NT, false>)};
    for (const void* f : k) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int W>
hipError_t allow2_m(int m, int nt, size_t lds) {
    if (m == 2 && nt == 256) return allow2<W, 2, 256>(lds);
    if (m == 3 && nt == 256) return allow2<W, 3, 256>(lds);
    if (m == 1 && nt == 512) return allow2<W, 1, 512>(lds);
    if (m == 2 && nt == 512) return allow2<W, 2, 512>(lds);
    if (m == 1 && nt == 1024) {
        const hipError_t e = allow2<W, 1, 1024>(lds);
        return e == hipSuccess ? allow2<W, 1, 1024, true>(lds) : e;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fused2_f64(int w, int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                             const Fused2Args<double>& a, hipEvent_t e0, hipEvent_t e1) {
    switch (w) {
        case 2: return go2_m<2>(m, nt, rec, pf, grid, lds, st, a, e0, e1);
        case 1: return go2_m<1>(m, nt, rec, pf, grid, lds, st, a, e0, e1);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fused2_batch_f64(int w, int m, int nt, bool rec, bool pf, dim3 grid, size_t lds,
                                   hipStream_t st, const Batch2Step<double>& b) {
    switch (w) {
        case 2: return gob2_m<2>(m, nt, rec, pf, grid, lds, st, b);
        case 1: return gob2_m<1>(m, nt, rec, pf, grid, lds, st, b);
        default: return hipErrorInvalidValue;
    }
}

// Allow the batch instances more than 64 KiB of dynamic LDS (before capture).
hipError_t fused2_batch_allow_lds_f64(int w, int m, int nt, size_t lds) {
    switch (w) {
        case 2: return allow2_m<2>(m, nt, lds);
        case 1: return allow2_m<1>(m, nt, lds);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tdse
