// One or two leapfrog steps of a small grid per launch: eqs. (9), (8) and,
// for two steps, (9), (8) again (arXiv 2401.07416 section 2.1) on bricks held
// on the chip.
//
// What bounds it.  On grids up to a few million cells the arrays sit in the
// caches and a step kernel's time is latency: the launch, then a chain of
// dependent loads and barriers.  A z march pays one barrier (and, without
// prefetch, one load latency) per plane, four to ten of them even in the
// shortest chunks.  Here every load of a workgroup is issued at once, and
// the launch has one barrier per half-step.
//
// Mapping.  A workgroup owns a brick of bx x by x bz cells and works on it
// extended by four cells on every side, the reach of two steps; each
// half-step is exact one cell less far out, and the rim is computed
// redundantly instead of exchanged.  A thread owns one W-wide x vector
// column of NV consecutive planes: its R, I and potential term stay in
// registers, z neighbours inside the column are its own registers, and all
// other neighbours come from the two LDS images (R and I of the extended
// brick).  A half-step reads one image and updates the other in place at
// the thread's own cells, so one barrier separates half-steps.
//
// A single step (TWO = false) runs the last two half-steps in the same
// geometry: each cell of the brick belongs to the same thread as in the
// two-step form, so the FP64 sums of a step have the same order, and the
// same bits, whichever form took it.
//
// Measured (microseconds per step, against the one-pass step): 64^3 FP64 5.8
// (9.0), 64x64x128 FP32 4.8 (8.5).  Of the 11.6 us of a 64^3 launch about 3 are
// the launch, 3.5 the kernel's start and its loads (18 wavefront loads per
// SIMD and a latency), 4.5 the four half-steps, whose instruction issue (the
// rim triples the cells) sets their time.  Eight cells and four planes
// a thread in z: taller bricks need more registers than two rounds of
// wavefronts leave, shorter ones more rim.
//
// The cell arithmetic is vterm / hterm / upd_* of kernels.hpp: the states
// are bitwise those of the other step kernels.
#pragma once

#include <type_traits>

#include "kernels.hpp"

namespace tdse {

constexpr int BRICK_HALO = 4;
constexpr int BRICK_NV = 4;   // planes per thread
constexpr int BRICK_NG = 4;   // threads per column
constexpr int BRICK_BZ = BRICK_NV * BRICK_NG - 2 * BRICK_HALO;

template <typename T>
struct BrickArgs {
    const T* R0;  // R^n
    const T* I0;  // I^{n-1/2}
    T* R1;        // R^{n+2} (R^{n+1} for a single step)
    T* I1;        // I^{n+3/2} (I^{n+1/2})
    const T* V;
    const T* ca;
    const T* cb;
    T cx, cy, cz, cv;
    T d0, dlo;             // 2 (cx + cy + cz) as hi + lo parts
    int nx, ny, nz;
    int bytes;             // of one array
    int ntx, ntiles, nwg;  // bricks along x, per layer, in all
    unsigned mtiles, mtx;  // ceil(2^32 / ntiles), ceil(2^32 / ntx): exact quotients below 2^16
    int bcx, bcy, bcz;
    int ulo, uhi;          // planes [ulo, uhi) have no absorption (ca = cb = 1)
    int k_det, k_up;
    double* flux_a;        // [2][ntiles], the first of two steps
    double* flux_b;        // [2][ntiles], the last step
    // record of the last level (REC instances only)
    T* rec_plane;
    double* part_q;        // [nzc][ntiles]
    double* part_naive;
    double* part_plane;    // [ntiles]
    double* pixel;
    double pixel_w;
};

// Sums of N values over the workgroup in a fixed order (butterflies, then
// the wavefronts in order), the N trees side by side behind one barrier:
// one after the other they would lengthen the launch by half a microsecond
// each.  Thread j < N returns sum j.
template <int N>
__device__ __forceinline__ double block_sums(double (&v)[N], double* red, int tid, int nwaves) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] += __shfl_xor(v[j], o, 64);
    if ((tid & 63) == 0)
#pragma unroll
        for (int j = 0; j < N; ++j) red[j * 16 + (tid >> 6)] = v[j];
    __syncthreads();
    double s = 0.0;
    if (tid < N)
        for (int w = 0; w < nwaves; ++w) s += red[tid * 16 + w];
    return s;
}

// BX x BY x 8 cells per brick; blockDim = ((BX + 8) / W, BY + 8, NG).
// The shape is compiled in, so that every LDS neighbour is an immediate
// offset from the thread's own cell: the half-steps are bound by
// instruction issue.
template <typename T, int W, int BX, int BY, bool REC, bool TWO>
__global__ __launch_bounds__((BX + 8) / W * (BY + 8) * BRICK_NG) void brick_kernel(BrickArgs<T> a) {
    using VT = vec_t<T, W>;
    constexpr int H = BRICK_HALO, NV = BRICK_NV, NG = BRICK_NG;
    constexpr int D0 = TWO ? 0 : 2;   // half-steps left out at the start
    constexpr int EX = BX + 2 * H, EY = BY + 2 * H, EZ = NV * NG, BZ = EZ - 2 * H;
    constexpr int SZ = EX * EY, PAD = 16 / (int)sizeof(T);
    constexpr int NW = EX / W * EY * NG / 64;
    static_assert(EX / W * EY * NG % 64 == 0, "whole wavefronts");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[7 * 16];
    // the two images, each with a vector of padding at both ends (the x
    // neighbours of the first and last cell)
    T* const Rl = reinterpret_cast<T*>(smem_raw) + PAD;
    T* const Il = Rl + SZ * EZ + PAD;

    const int L = xcd_remap(blockIdx.x, a.nwg);
    const int zchunk = a.ntiles == 1 ? L : (int)__umulhi((unsigned)L, a.mtiles);
    const int tile = L - zchunk * a.ntiles;
    const int tyi = a.ntx == 1 ? tile : (int)__umulhi((unsigned)tile, a.mtx);
    const int txi = tile - tyi * a.ntx;
    const int x0 = txi * BX, y0 = tyi * BY, k0 = zchunk * BZ;
    const int k1 = min(k0 + BZ, a.nz);
    // uniform over the workgroup
    const bool z_inner = k0 >= H && k0 + BZ + H <= a.nz;
    const bool unit = z_inner && k0 - H >= a.ulo && k0 + BZ + H <= a.uhi;
    const bool any_zero = a.bcx || a.bcy || a.bcz;
    const bool has_det = a.k_det >= k0 && a.k_det < k1;
    const bool has_up = a.k_up >= k0 && a.k_up < k1;
    const bool has_face = has_det || has_up;

    const int c0 = threadIdx.x * W, yl = threadIdx.y, zb = threadIdx.z * NV;
    // grid index of an extended coordinate: one wrap reaches every cell that
    // a stored cell depends on (n >= 4); further out nothing is needed, and
    // outside a zero boundary the field is zero (-1: reads as zero)
    auto wrap = [](int g, int n, int zero) -> int {
        if (g < 0) return zero ? -1 : g + n;
        if (g >= n) return zero || g >= n + H ? -1 : g - n;
        return g;
    };
    const int gx = x0 - H + c0, gy = y0 - H + yl;
    const int cx = wrap(gx, a.nx, a.bcx), cy = wrap(gy, a.ny, a.bcy);
    const bool xy_zero = (a.bcx && cx < 0) || (a.bcy && cy < 0);
    const bool xy_in = c0 >= H && c0 < H + BX && gx < a.nx && yl >= H && yl < H + BY && gy < a.ny;
    constexpr int es = (int)sizeof(T);
    const int xyoff = (cx | cy) < 0 ? OOB : (cy * a.nx + cx) * es;
    const int pbytes = a.nx * a.ny * es;
    // half-step d (1 .. 4) is exact and needed d cells inside the extension
    auto xy_box = [&](int d) -> bool { return c0 + W > d && c0 < EX - d && yl >= d && yl < EY - d; };
    // planes zb + i of the thread inside the box of half-step d: only the
    // first and last threads of a column have any outside it
    auto z_box = [&](int i, int d) -> bool { return zb >= d - i && zb < EZ - d - i; };

    const auto rR = plane_rsrc(a.R0, a.bytes), rI = plane_rsrc(a.I0, a.bytes), rV = plane_rsrc(a.V, a.bytes);
    VT r[NV], im[NV], vt[NV];
    int off[NV];
    const int g0 = k0 - H + zb;
    if (z_inner) {
#pragma unroll
        for (int i = 0; i < NV; ++i) off[i] = (int)((unsigned)xyoff + (unsigned)(g0 + i) * (unsigned)pbytes);
        if (xyoff == OOB) {
#pragma unroll
            for (int i = 0; i < NV; ++i) off[i] = OOB;
        }
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int gz = wrap(g0 + i, a.nz, a.bcz);
            off[i] = xyoff == OOB || gz < 0 ? OOB : gz * pbytes + xyoff;
        }
    }
    const bool bi = xy_box(D0 + 1), br = xy_box(D0);
#pragma unroll
    for (int i = 0; i < NV; ++i) r[i] = bload<T, W>(rR, br && z_box(i, D0) ? off[i] : OOB);
#pragma unroll
    for (int i = 0; i < NV; ++i) im[i] = bload<T, W>(rI, bi && z_box(i, D0 + 1) ? off[i] : OOB);
#pragma unroll
    for (int i = 0; i < NV; ++i) vt[i] = bload<T, W>(rV, bi && z_box(i, D0 + 1) ? off[i] : OOB);
    T ca[NV], cb[NV];
    if (!unit) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int gz = max(wrap(g0 + i, a.nz, a.bcz), 0);
            ca[i] = a.ca[gz];
            cb[i] = a.cb[gz];
        }
    }
    // outside a zero boundary: the field stays zero there
    auto is_zero = [&](int i) -> bool { return xy_zero || (a.bcz && (g0 + i < 0 || g0 + i >= a.nz)); };
    const int lofs = (zb * EY + yl) * EX + c0;
    T* const Rt = Rl + lofs;
    T* const It = Il + lofs - SZ;   // the image of I starts at plane 1
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<VT*>(Rt + i * SZ) = r[i];
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int e = 0; e < W; ++e) vt[i].v[e] = vterm(vt[i].v[e], a.cv, a.d0);
    __syncthreads();

    // flux through the detection face: faces of the first step, of the
    // last; then the record sums
    double fs[4] = {0.0, 0.0, 0.0, 0.0};
    double rs[3] = {0.0, 0.0, 0.0};
    // half-step d: U (own registers u, image Ut) from the stencil of S (own
    // registers s, image St)
    auto phase = [&](auto is_r, auto dc, auto un, VT(&u)[NV], const VT(&s)[NV], const T* St, T* Ut) {
        constexpr bool IS_R = decltype(is_r)::value, UNIT = decltype(un)::value;
        constexpr int d = decltype(dc)::value;
        if (xy_box(d)) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (!z_box(i, d)) continue;
                const T* p = St + i * SZ;
                const VT ylv = *reinterpret_cast<const VT*>(p - EX);
                const VT yrv = *reinterpret_cast<const VT*>(p + EX);
                const VT zlv = i > 0 ? s[i > 0 ? i - 1 : 0] : *reinterpret_cast<const VT*>(p - SZ);
                const VT zrv = i < NV - 1 ? s[i < NV - 1 ? i + 1 : i] : *reinterpret_cast<const VT*>(p + SZ);
                const T xle = p[-1], xre = p[W];
                VT o;
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const T c = s[i].v[e];
                    const T xl = e > 0 ? s[i].v[e - 1] : xle;
                    const T xr = e < W - 1 ? s[i].v[e + 1] : xre;
                    const T hx = hterm(c, xl, xr, ylv.v[e], yrv.v[e], zlv.v[e], zrv.v[e], vt[i].v[e], a.cx,
                                       a.cy, a.cz, a.dlo);
                    if constexpr (UNIT)
                        o.v[e] = IS_R ? upd_R_unit(hx, u[i].v[e]) : upd_I_unit(hx, u[i].v[e]);
                    else
                        o.v[e] = IS_R ? upd_R(hx, u[i].v[e], ca[i], cb[i]) : upd_I(hx, u[i].v[e], ca[i], cb[i]);
                }
                if (any_zero) {
                    const bool zr = is_zero(i);
#pragma unroll
                    for (int e = 0; e < W; ++e) o.v[e] = zr ? T(0) : o.v[e];
                }
                if (IS_R && (has_face || (REC && d == 4))) {
                    const int gz = g0 + i;
                    if (xy_in && gz >= k0 && gz < k1) {
                        if (gz == a.k_det || gz == a.k_up) {
                            const bool det = gz == a.k_det, up = gz == a.k_up;
#pragma unroll
                            for (int e = 0; e < W; ++e) {
                                const double sm = (double)u[i].v[e] + (double)o.v[e];
                                if (det) fs[d == 4 ? 2 : 0] += (double)zrv.v[e] * sm;
                                if (up) fs[d == 4 ? 3 : 1] += (double)zlv.v[e] * sm;
                            }
                        }
                        if (REC && d == 4) {
#pragma unroll
                            for (int e = 0; e < W; ++e) {
                                const double dc_ = (double)s[i].v[e], du = (double)u[i].v[e];
                                const double dn = (double)o.v[e];
                                rs[0] += dc_ * dc_ + du * dn;
                                rs[1] += dn * dn + dc_ * dc_;
                            }
                            if (gz == a.k_det) {
                                VT rv;
                                const long poff = xyoff / es;
#pragma unroll
                                for (int e = 0; e < W; ++e) {
                                    const double dn = (double)o.v[e], dc_ = (double)s[i].v[e];
                                    const double rho = dn * dn + dc_ * dc_;
                                    rv.v[e] = (T)rho;
                                    rs[2] += rho;
                                    if (a.pixel) a.pixel[poff + e] += a.pixel_w * rho;
                                }
                                stv<T, W>(a.rec_plane + poff, rv);
                            }
                        }
                    }
                }
                u[i] = o;
                if (d < 4) *reinterpret_cast<VT*>(Ut + i * SZ) = o;
            }
        }
        if (d < 4) __syncthreads();
    };
    using IsR = std::integral_constant<bool, true>;
    using IsI = std::integral_constant<bool, false>;
    auto steps = [&](auto un) {
        if constexpr (TWO) {
            phase(IsI{}, std::integral_constant<int, 1>{}, un, im, r, Rt, It);
            phase(IsR{}, std::integral_constant<int, 2>{}, un, r, im, It, Rt);
        }
        phase(IsI{}, std::integral_constant<int, 3>{}, un, im, r, Rt, It);
        // I is final: its stores go out under the last half-step
        const auto oI = plane_rsrc(a.I1, a.bytes);
#pragma unroll
        for (int i = 0; i < NV; ++i)
            bstore<T, W>(oI, xy_in && g0 + i >= k0 && g0 + i < k1 ? off[i] : OOB, im[i]);
        phase(IsR{}, std::integral_constant<int, 4>{}, un, r, im, It, Rt);
    };
    if (unit)
        steps(std::true_type{});
    else
        steps(std::false_type{});
    const auto oR = plane_rsrc(a.R1, a.bytes);
#pragma unroll
    for (int i = 0; i < NV; ++i)
        bstore<T, W>(oR, xy_in && g0 + i >= k0 && g0 + i < k1 ? off[i] : OOB, r[i]);

    // fixed-order sums of the partials; the branches are uniform
    const int tid = threadIdx.x + EX / W * (threadIdx.y + EY * threadIdx.z);
    if (has_face) {
        const double s = block_sums<4>(fs, red, tid, NW);
        // sums 0, 1: faces det, up of the first step; 2, 3: of the last
        if (tid < 4 && ((tid & 1) ? has_up : has_det) && (TWO || tid >= 2))
            (tid >= 2 ? a.flux_b : a.flux_a)[(tid & 1) * a.ntiles + tile] = s;
    }
    if (REC) {
        const double s = block_sums<3>(rs, red + 4 * 16, tid, NW);
        const long slot = (long)zchunk * a.ntiles + tile;
        if (tid == 0) a.part_q[slot] = s;
        if (tid == 1) a.part_naive[slot] = s;
        if (tid == 2 && has_det) a.part_plane[tile] = s;
    }
}

}  // namespace tdse
