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
// geometry, and brick_half_kernel one half-step in place: each cell of the
// brick belongs to the same thread as in the two-step form, so the FP64 sums
// of a step have the same order, and the same bits, whichever form took it.
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

// What a launch does: two steps or one into the second state pair, or one
// half-step in place.
enum BrickOp : int { BRICK_TWO, BRICK_ONE, BRICK_HALF_I, BRICK_HALF_R };

template <typename T>
struct BrickArgs {
    const T* R0;  // R^n
    const T* I0;  // I^{n-1/2}
    T* R1;        // R^{n+2} (R^{n+1} for a single step; R0 in place)
    T* I1;        // I^{n+3/2} (I^{n+1/2}; I0 in place)
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
    double* flux_a;        // [2][ntiles], the first of two steps (BRICK_TWO only)
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

// block_sums<N> of brick_kernel's workgroup by a smaller one of only the
// threads that own cells: each wavefront of the larger one is put together
// from the owners' values and zeros and summed by the same tree, all trees of
// a value side by side in one wavefront.  Value j is zero outside the larger
// workgroup's threads of z place z0[j] .. z0[j] + NZ - 1 (1 and 2 own cells);
// its wavefronts with none of them add nothing.  put(j, sum j) once each.
template <int N, int NZ, int W, int BX, int BY, typename Put>
__device__ __forceinline__ void owner_sums(const double (&v)[N], const int (&z0)[N], double* val, int tid, Put put) {
    constexpr int H = BRICK_HALO, PX = BX / W, VX = PX + 2 * H / W, S = VX * (BY + 2 * H), NT = PX * BY * 2;
    // wavefronts that NZ places can touch
    constexpr int NWV = NZ * S % 64 == 0 && S % 64 == 0 ? NZ * S / 64 : (NZ * S + 62) / 64 + 1;
#pragma unroll
    for (int j = 0; j < N; ++j) val[j * NT + tid] = v[j];
    __syncthreads();
    for (int j = tid >> 6; j < N; j += NT / 64) {
        int zj = z0[0];
#pragma unroll
        for (int i = 1; i < N; ++i) zj = j == i ? z0[i] : zj;
        double x[NWV];
#pragma unroll
        for (int q = 0; q < NWV; ++q) {
            const int p = (zj * S / 64 + q) * 64 + (tid & 63);
            const int z = p / S, y = p % S / VX - H, c = p % VX - H / W;
            const bool own = z >= 1 && z <= 2 && y >= 0 && y < BY && c >= 0 && c < PX;
            x[q] = own ? val[j * NT + c + PX * (y + BY * (z - 1))] : 0.0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int q = 0; q < NWV; ++q) x[q] += __shfl_xor(x[q], o, 64);
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NWV; ++q) s += x[q];
        if ((tid & 63) == 0) put(j, s);
    }
}

// One half-step in place on the bricks' geometry: eq. (9) into I or (IS_R)
// eq. (8) into R.  A call with an odd number of steps takes its last one this
// way, so that the state ends in the arrays it began in.
//
// Bound by latency: every load of a thread is issued at once, the neighbours
// straight from the caches, and nothing is exchanged, so the launch has no
// barrier but those of the sums, in the bricks that have any.  A cell's old
// value is read and its new one written by its own thread only, and the other
// array is only read: in place without a race.  Of brick_kernel's threads
// only those that own cells of the brick are launched (with the others idle
// a half-step of 64^3 FP64 took 7.0 us); their sums are added in the lanes
// that brick_kernel adds them in.  blockDim = (BX / W, BY, 2).
// 64^3 FP64: 4.0 us eq. (9), 4.9 us eq. (8) with the flux; a call of one step
// 11.9 us, as with the half-step kernels of any grid (12.0), where one step
// into the second pair and two copies of the state took 16.4.
template <typename T, int W, int BX, int BY, bool IS_R, bool REC>
__global__ __launch_bounds__(BX / W * BY * 2) void brick_half_kernel(BrickArgs<T> a) {
    using VT = vec_t<T, W>;
    constexpr int H = BRICK_HALO, NV = BRICK_NV, NG = BRICK_NG;
    constexpr int BZ = NV * NG - 2 * H;
    constexpr int NT = BX / W * BY * 2;
    static_assert(H == NV && BZ == 2 * NV && NT % 64 == 0, "the owned planes are two threads of a column");
    __shared__ double val[5 * NT];

    const int L = xcd_remap(blockIdx.x, a.nwg);
    const int zchunk = a.ntiles == 1 ? L : (int)__umulhi((unsigned)L, a.mtiles);
    const int tile = L - zchunk * a.ntiles;
    const int tyi = a.ntx == 1 ? tile : (int)__umulhi((unsigned)tile, a.mtx);
    const int txi = tile - tyi * a.ntx;
    const int k0 = zchunk * BZ, k1 = min(k0 + BZ, a.nz);
    const int g0 = k0 + (int)threadIdx.z * NV;
    const int gx = txi * BX + (int)threadIdx.x * W, gy = tyi * BY + (int)threadIdx.y;
    const bool xy_in = gx < a.nx && gy < a.ny;
    constexpr int es = (int)sizeof(T);
    const unsigned pbytes = (unsigned)(a.nx * a.ny) * es;
    const auto rS = plane_rsrc(IS_R ? a.I0 : a.R0, a.bytes), rU = plane_rsrc(IS_R ? a.R0 : a.I0, a.bytes);
    const auto rV = plane_rsrc(a.V, a.bytes);
    const auto rca = plane_rsrc(a.ca, a.nz * es), rcb = plane_rsrc(a.cb, a.nz * es);
    // Byte offsets in plane g0, a plane's bytes further on in each of the
    // next three: past the end (reads as zero, stores nothing) from plane nz
    // on, and for cells outside the grid or a zero boundary (OOB and three
    // planes of a grid of four or more stay below 2^32).  They are formed
    // once: a wavefront has a SIMD to itself, and every instruction before
    // the loads is waited for
    auto at = [&](int x, int y, int z) -> unsigned {
        return !xy_in || x < 0 || y < 0 || z < 0 ? (unsigned)OOB : (unsigned)z * pbytes + (unsigned)(y * a.nx + x) * es;
    };
    const unsigned oc = at(gx, gy, g0);
    const unsigned ol = at(gx > 0 ? gx - 1 : a.bcx ? -1 : a.nx - 1, gy, g0);
    const unsigned orr = at(gx + W < a.nx ? gx + W : a.bcx ? -1 : 0, gy, g0);
    const unsigned ou = at(gx, gy > 0 ? gy - 1 : a.bcy ? -1 : a.ny - 1, g0);
    const unsigned od = at(gx, gy + 1 < a.ny ? gy + 1 : a.bcy ? -1 : 0, g0);
    // the planes below the thread's first and above its last
    const unsigned ob = at(gx, gy, g0 > 0 ? g0 - 1 : a.bcz ? -1 : a.nz - 1);
    const unsigned ot = at(gx, gy, g0 + NV < a.nz ? g0 + NV : a.bcz ? -1 : 0);
    VT s[NV + 2], u[NV], v[NV], sl[NV], sr[NV];
    vec_t<T, 1> el[NV], er[NV], ca[NV], cb[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const unsigned z = (unsigned)i * pbytes;
        s[i + 1] = bload<T, W>(rS, (int)(oc + z));
        sl[i] = bload<T, W>(rS, (int)(ou + z));
        sr[i] = bload<T, W>(rS, (int)(od + z));
        el[i] = bload<T, 1>(rS, (int)(ol + z));
        er[i] = bload<T, 1>(rS, (int)(orr + z));
        u[i] = bload<T, W>(rU, (int)(oc + z));
        v[i] = bload<T, W>(rV, (int)(oc + z));
        ca[i] = bload<T, 1>(rca, (g0 + i) * es);
        cb[i] = bload<T, 1>(rcb, (g0 + i) * es);
    }
    s[0] = bload<T, W>(rS, (int)ob);
    s[NV + 1] = bload<T, W>(rS, (int)ot);
    // all of them in flight before the first use
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NV - 1; ++i)
        if (g0 + i == a.nz - 1) s[i + 2] = s[NV + 1];
    double fs[2] = {0.0, 0.0}, rs[3] = {0.0, 0.0, 0.0};
    const auto oU = plane_rsrc(IS_R ? a.R1 : a.I1, a.bytes);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int gz = g0 + i;
        VT o;
#pragma unroll
        for (int e = 0; e < W; ++e) {
            const T c = s[i + 1].v[e];
            const T hx = hterm(c, e > 0 ? s[i + 1].v[e > 0 ? e - 1 : 0] : el[i].v[0],
                               e < W - 1 ? s[i + 1].v[e < W - 1 ? e + 1 : e] : er[i].v[0], sl[i].v[e], sr[i].v[e],
                               s[i].v[e], s[i + 2].v[e], vterm(v[i].v[e], a.cv, a.d0), a.cx, a.cy, a.cz, a.dlo);
            o.v[e] = IS_R ? upd_R(hx, u[i].v[e], ca[i].v[0], cb[i].v[0]) : upd_I(hx, u[i].v[e], ca[i].v[0], cb[i].v[0]);
        }
        bstore<T, W>(oU, (int)(oc + (unsigned)i * pbytes), o);
        if (!IS_R || !xy_in || gz >= a.nz) continue;
        if (gz == a.k_det || gz == a.k_up) {
            const bool det = gz == a.k_det, up = gz == a.k_up;
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const double sm = (double)u[i].v[e] + (double)o.v[e];
                if (det) fs[0] += (double)s[i + 2].v[e] * sm;
                if (up) fs[1] += (double)s[i].v[e] * sm;
            }
        }
        if (REC) {
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const double dc = (double)s[i + 1].v[e], du = (double)u[i].v[e], dn = (double)o.v[e];
                rs[0] += dc * dc + du * dn;
                rs[1] += dn * dn + dc * dc;
            }
            if (gz == a.k_det) {
                VT rv;
                const long poff = (long)gy * a.nx + gx;
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const double dn = (double)o.v[e], dc = (double)s[i + 1].v[e];
                    const double rho = dn * dn + dc * dc;
                    rv.v[e] = (T)rho;
                    rs[2] += rho;
                    if (a.pixel) a.pixel[poff + e] += a.pixel_w * rho;
                }
                stv<T, W>(a.rec_plane + poff, rv);
            }
        }
    }
    if constexpr (IS_R) {
        const int tid = threadIdx.x + BX / W * (threadIdx.y + BY * threadIdx.z);
        const bool has_det = a.k_det >= k0 && a.k_det < k1, has_up = a.k_up >= k0 && a.k_up < k1;
        if (has_det || has_up) {
            const int zd = has_det ? (a.k_det - k0) / NV + 1 : 1, zu = has_up ? (a.k_up - k0) / NV + 1 : 1;
            owner_sums<2, 1, W, BX, BY>(fs, {zd, zu}, val, tid, [&](int j, double t) {
                if (j ? has_up : has_det) a.flux_b[j * a.ntiles + tile] = t;
            });
        }
        if constexpr (REC) {
            const long slot = (long)zchunk * a.ntiles + tile;
            owner_sums<3, 2, W, BX, BY>(rs, {1, 1, 1}, val + 2 * NT, tid, [&](int j, double t) {
                if (j < 2) (j ? a.part_naive : a.part_q)[slot] = t;
                else if (has_det) a.part_plane[tile] = t;
            });
        }
    }
}

}  // namespace tdse
