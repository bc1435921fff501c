// Two-step (temporally blocked) sweep kernel instances for float state:
// (rows per thread, threads per workgroup) in {(2, 256), (3, 256), (1, 512), (2, 512), (1, 1024)}.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "fused2.hpp"

namespace tdse {

namespace {

template <int W, int M, int NT, bool MARCH = false>
hipError_t go2(bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st, const Fused2Args<float>& a,
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
        return rec ? run(fused2_kernel<float, W, M, true, true, NT, MARCH>) : run(fused2_kernel<float, W, M, false, true, NT, MARCH>);
    return rec ? run(fused2_kernel<float, W, M, true, false, NT, false>) : run(fused2_kernel<float, W, M, false, false, NT, false>);
}

template <int W>
hipError_t go2_m(int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                 const Fused2Args<float>& a, hipEvent_t e0, hipEvent_t e1) {
    if (m == 2 && nt == 256) return go2<W, 2, 256>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 3 && nt == 256) return go2<W, 3, 256>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 1 && nt == 512) return go2<W, 1, 512>(rec, pf, grid, lds, st, a, e0, e1);
    if (m == 2 && nt == 512) return go2<W, 2, 512>(rec, pf, grid, lds, st, a, e0, e1);
    // the march loop: not with a zero boundary in x or y (nothing could take
    // it), nor, for vectors of two, where chunks of fewer than 48 planes have
    // no absorption: a chunk with a detection face breaks its few runs of six
    // planes, and with all workgroups in one round that chunk is the time of
    // the launch (us a step with and without: 166x88x410 in 32 planes 34.9
    // and 29.7, with the face in the last plane 26.5 and 29.0; 202x190x300 in
    // 44 planes 40.2 and 37.4; 250x200x200 in 40 planes 35.5 and 35.0; in two
    // rounds it is level, 202x190x300 in 30 planes 52.4 and 55.1, 250x200x200
    // in 25 planes 49.7 and 48.9).  With CAP planes the other iterations are
    // the slower ones (166x88x410 33.3 with, 44.0 without), and vectors of
    // one gain in any chunk (201x200x250 in 32 planes 71.3 and 81.2, in 42
    // planes 53.4 and 64.8).
    const bool no_march = a.bcx || a.bcy || (W == 2 && a.zc < 48 && a.ulo <= 0 && a.uhi >= a.nz);
    if (m == 1 && nt == 1024)
        return no_march ? go2<W, 1, 1024>(rec, pf, grid, lds, st, a, e0, e1)
                        : go2<W, 1, 1024, true>(rec, pf, grid, lds, st, a, e0, e1);
    return hipErrorInvalidValue;
}

template <int W, int M, int NT, bool MARCH = false>
hipError_t gob2(bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st, const Batch2Step<float>& b) {
    if (pf) {
        if (rec) hipLaunchKernelGGL((fused2_batch_kernel<float, W, M, true, true, NT, MARCH>), grid, dim3(NT), lds, st, b);
        else hipLaunchKernelGGL((fused2_batch_kernel<float, W, M, false, true, NT, MARCH>), grid, dim3(NT), lds, st, b);
    } else {
        if (rec) hipLaunchKernelGGL((fused2_batch_kernel<float, W, M, true, false, NT, false>), grid, dim3(NT), lds, st, b);
        else hipLaunchKernelGGL((fused2_batch_kernel<float, W, M, false, false, NT, false>), grid, dim3(NT), lds, st, b);
    }
    return hipGetLastError();
}

template <int W>
hipError_t gob2_m(int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                  const Batch2Step<float>& b) {
    if (m == 2 && nt == 256) return gob2<W, 2, 256>(rec, pf, grid, lds, st, b);
    if (m == 3 && nt == 256) return gob2<W, 3, 256>(rec, pf, grid, lds, st, b);
    if (m == 1 && nt == 512) return gob2<W, 1, 512>(rec, pf, grid, lds, st, b);
    if (m == 2 && nt == 512) return gob2<W, 2, 512>(rec, pf, grid, lds, st, b);
    // (the members of a batch share many rounds, in which short chunks without
    // absorption lose nothing: six grids of 166x88x200 in 32 planes 62.4 us a
    // step, 64.6 without the march)
    if (m == 1 && nt == 1024)
        return b.zero_xy ? gob2<W, 1, 1024>(rec, pf, grid, lds, st, b)
                         : gob2<W, 1, 1024, true>(rec, pf, grid, lds, st, b);
    return hipErrorInvalidValue;
}

template <int W, int M, int NT, bool MARCH = false>
hipError_t allow2(size_t lds) {
    const void* k[4] = {reinterpret_cast<const void*>(fused2_batch_kernel<float, W, M, true, true, NT, MARCH>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<float, W, M, false, true, NT, MARCH>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<float, W, M, true, false, NT, false>),
                        reinterpret_cast<const void*>(fused2_batch_kernel<float, W, M, false, false, NT, false>)};
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

hipError_t launch_fused2_f32(int w, int m, int nt, bool rec, bool pf, dim3 grid, size_t lds, hipStream_t st,
                             const Fused2Args<float>& a, hipEvent_t e0, hipEvent_t e1) {
    switch (w) {
        case 4: return go2_m<4>(m, nt, rec, pf, grid, lds, st, a, e0, e1);
        case 2: return go2_m<2>(m, nt, rec, pf, grid, lds, st, a, e0, e1);
        case 1: return go2_m<1>(m, nt, rec, pf, grid, lds, st, a, e0, e1);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fused2_batch_f32(int w, int m, int nt, bool rec, bool pf, dim3 grid, size_t lds,
                                   hipStream_t st, const Batch2Step<float>& b) {
    switch (w) {
        case 4: return gob2_m<4>(m, nt, rec, pf, grid, lds, st, b);
        case 2: return gob2_m<2>(m, nt, rec, pf, grid, lds, st, b);
        case 1: return gob2_m<1>(m, nt, rec, pf, grid, lds, st, b);
        default: return hipErrorInvalidValue;
    }
}

// Allow the batch instances more than 64 KiB of dynamic LDS (before capture).
hipError_t fused2_batch_allow_lds_f32(int w, int m, int nt, size_t lds) {
    switch (w) {
        case 4: return allow2_m<4>(m, nt, lds);
        case 2: return allow2_m<2>(m, nt, lds);
        case 1: return allow2_m<1>(m, nt, lds);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tdse
