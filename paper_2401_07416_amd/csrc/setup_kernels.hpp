// Device code of libtdse outside the half-step kernels: the fixed-order
// finalisation of the FP64 partial sums and the setup passes (potential,
// Gaussian packet, min/max of V).  Included by the runtime only.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"

namespace tdse {

// Fixed-order FP64 sum over a workgroup of 256 threads (wavefront
// butterflies, then the four wavefront totals in order).
__device__ __forceinline__ double block_sum256(double v, double* red) { return block_sum(v, red, 4); }

struct FinArgs {
    const double* flux_ring;  // [n_pending][2][ytiles]
    int n_pending, ytiles, has_up, record;
    long rec_idx;
    double dv_cz, dV;
    double* acc;              // acc[0] = accumulated flux
    const double* part_q;
    const double* part_naive;
    long n_part;
    const double* part_plane;
    double* scalars;          // [max_records][4]
};

// Folds the pending per-step flux partials into the accumulator in step
// order and, on record steps, writes {plane_sum, naive_norm, Q, flux_acc}.
//
// One workgroup, so what bounds it is latency: a wavefront per step (beyond
// 16 steps four at a time, their loads in flight together) instead of the
// whole workgroup step by step, and the record sums eight loads deep.  20
// pending steps with a record on 64x64x128 FP32 13.2 -> 4.3 us, 50 on
// 128x128x256 32.5 -> 6.5, the 131072 partials of a record 0 on 512x512x1024
// 204 -> 64; one step without a record 1.7.  The order of every sum is fixed,
// and a step's sum depends on its own partials only.
constexpr int FIN_THREADS = 1024;
constexpr int FIN_WAVES = FIN_THREADS / 64;
constexpr int FIN_MAX_PENDING = 256;   // steps the flux ring holds

__device__ __forceinline__ void finalize_body(const FinArgs& a) {
    __shared__ double red[3 * FIN_WAVES];
    __shared__ double step_flux[FIN_MAX_PENDING];
    // (the wavefront's number as a scalar: its steps' addresses are then formed
    // on the scalar unit, not by 64-bit vector products in front of the loads)
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    double acc = a.acc[0];   // here, so that it arrives under the sums
    auto fold = [&](auto steps) {
        constexpr int N = decltype(steps)::value;
        for (int s0 = N * wv; s0 < a.n_pending; s0 += N * FIN_WAVES) {
            double v[N] = {};
            for (int i = lane; i < a.ytiles; i += 64)
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const double* f = a.flux_ring + (long)min(s0 + j, a.n_pending - 1) * 2 * a.ytiles;
                    v[j] += f[i] - f[a.ytiles + i];
                }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
#pragma unroll
                for (int j = 0; j < N; ++j) v[j] += __shfl_xor(v[j], o, 64);
            if (lane == 0)
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (s0 + j < a.n_pending) step_flux[s0 + j] = v[j];
        }
    };
    // one step each while there are wavefronts for it: the exchanges of four
    // side by side cost a call of one step 0.3 us
    if (a.n_pending <= FIN_WAVES)
        fold(std::integral_constant<int, 1>{});
    else
        fold(std::integral_constant<int, 4>{});
    if (a.record) {
        // eight independent sums each, added in order below
        double q[8] = {}, n[8] = {}, p = 0.0;
        for (long i0 = t; i0 < a.n_part; i0 += 8 * FIN_THREADS)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const long i = i0 + j * FIN_THREADS;
                if (i < a.n_part) {
                    q[j] += a.part_q[i];
                    n[j] += a.part_naive[i];
                }
            }
        for (int i = t; i < a.ytiles; i += FIN_THREADS) p += a.part_plane[i];
        double v[3] = {((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7])),
                       ((n[0] + n[1]) + (n[2] + n[3])) + ((n[4] + n[5]) + (n[6] + n[7])), p};
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < 3; ++j) v[j] += __shfl_xor(v[j], o, 64);
        if (lane == 0)
#pragma unroll
            for (int j = 0; j < 3; ++j) red[j * FIN_WAVES + wv] = v[j];
    }
    __syncthreads();
    if (t == 0) {
        if (a.has_up)
            for (int s = 0; s < a.n_pending; ++s) acc += a.dv_cz * step_flux[s];
        a.acc[0] = acc;
        if (a.record) a.scalars[4 * a.rec_idx + 3] = acc;
    } else if (a.record && t >= 64 && t < 67) {
        const int j = t - 64;
        double s = 0.0;
        for (int w = 0; w < FIN_WAVES; ++w) s += red[j * FIN_WAVES + w];
        // sums q, naive, plane -> columns 2, 1, 0
        a.scalars[4 * a.rec_idx + 2 - j] = a.dV * s;
    }
}

__global__ __launch_bounds__(FIN_THREADS) void finalize_kernel(FinArgs a) { finalize_body(a); }

// One workgroup per configuration of a batch; pending count, record flag and
// the device record counter are shared by the launch.
struct BatchFin {
    const FinArgs* cfg;
    const long* rec_idx;
    int n_pending, record;
};

__global__ __launch_bounds__(FIN_THREADS) void finalize_batch_kernel(BatchFin b) {
    FinArgs a = b.cfg[blockIdx.x];
    a.n_pending = b.n_pending;
    a.record = b.record;
    a.rec_idx = b.record ? *b.rec_idx : 0;
    finalize_body(a);
}

// Advance / set the device record counter of a batch (one lane, vector store).
__global__ void bump_counter_kernel(long* c) {
    if (threadIdx.x == 0) c[0] = c[0] + 1;
}

__global__ void set_counter_kernel(long* c, long v) {
    if (threadIdx.x == 0) c[0] = v;
}

// ---------------------------------------------------------------------------
// Setup kernels
// ---------------------------------------------------------------------------

// Per-block min, max and non-finite count of V, for E_max.  A streaming
// read: 16-byte vectors, four in flight per thread, compared in the state's
// precision (512x512x1024 FP32: 322 us element by element, 184 us now).
template <typename T>
__global__ __launch_bounds__(256) void minmax_kernel(const T* V, long n, double* out) {
    constexpr int W = 16 / (int)sizeof(T);
    __shared__ double smin[4], smax[4], sbad[4];
    const int t = threadIdx.x;
    const T big = sizeof(T) == 4 ? (T)3.402823466e38 : (T)1.7976931348623157e308;
    T mn = big, mx = -big;
    int bad = 0;
    auto see = [&](T v) {
        const bool fin = fabs(v) <= big;   // false for NaN and infinities
        bad += !fin;
        mn = fin && v < mn ? v : mn;
        mx = fin && v > mx ? v : mx;
    };
    const long nv = n / W, step = (long)gridDim.x * 256;
    for (long i = (long)blockIdx.x * 256 + t; i < nv; i += 4 * step) {
        vec_t<T, W> x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = ldv_nt<T, W>(V + W * min(i + j * step, nv - 1));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j * step < nv)
#pragma unroll
                for (int e = 0; e < W; ++e) see(x[j].v[e]);
    }
    // the cells past the last whole vector
    if (blockIdx.x == 0 && t < (int)(n - nv * W)) see(V[nv * W + t]);
    double a = (double)mn, b = (double)mx, c = (double)bad;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a = fmin(a, __shfl_xor(a, o, 64));
        b = fmax(b, __shfl_xor(b, o, 64));
        c += __shfl_xor(c, o, 64);
    }
    if ((t & 63) == 0) {
        smin[t >> 6] = a;
        smax[t >> 6] = b;
        sbad[t >> 6] = c;
    }
    __syncthreads();
    if (t == 0) {
        out[3 * blockIdx.x + 0] = fmin(fmin(smin[0], smin[1]), fmin(smin[2], smin[3]));
        out[3 * blockIdx.x + 1] = fmax(fmax(smax[0], smax[1]), fmax(smax[2], smax[3]));
        out[3 * blockIdx.x + 2] = (sbad[0] + sbad[1]) + (sbad[2] + sbad[3]);
    }
}

// Tile of a workgroup of the potential kernel: 32 x 8 columns of TZ planes.
constexpr int POT_TX = 32, POT_TY = 8;

struct PotArgs {
    int nx, ny, nz;
    int ntx;                // tiles along x
    double dx, dy, dz, Lx, Ly, Lz;
    int bcx, bcy, bcz, screened;
    // one image of every atom serves a whole tile on the axis (a zero
    // boundary, or a period of at least twice the cutoff plus the tile, and
    // no atom a million periods out, where rounding moves cells and images)
    int fixx, fixy, fixz;
    // what an atom's distance from a tile's centre is allowed beyond the half
    // tile: the cutoff and rounding, without limit for atoms that far out
    double reachx, reachy;
    const double* atoms;    // [n][5] in caller order
    const int* slab_ptr;    // [slabs + 1], slabs of TZ planes
    const int* slab_idx;    // candidate atoms per slab, ascending atom index
    double soft, cutoff, kappa, a0;
};

__device__ __forceinline__ double min_image(double u, double L) { return u - L * rint(u / L); }

// V(r) = sum_a amp_a v_Z(d_a) over the atoms nearer than the cutoff, in atom
// order, v_Z(d) = -Z kappa exp(-d/lam_Z) / sqrt(d^2 + s^2), lam_Z = 0.8853 a0
// Z^(-1/3).
//
// What bounds it: the FP64 exponential, roots and divisions of the pairs
// inside the cutoff (about 90 instructions each), once the pairs outside it
// cost next to nothing.  The workgroup keeps, 256 at a time and in order,
// the candidates of its slab whose image comes within the cutoff of its
// tile, with their screening length and image shift formed once per tile; a
// thread holds a column of TZ planes, so a pair's x and y parts are
// formed once per column, and a root is taken only of squared distances not
// beyond the cutoff.  The arithmetic of a pair and the order of the sum are
// those of a plain loop over all atoms: the same bits.  1200 atoms on
// 256x256x512 FP32: 13.6 ms testing every atom near a plane at every cell,
// 0.78 ms now (192 atoms on 128x128x256: 1.39 and 0.22).
template <typename T, int TZ>
__global__ __launch_bounds__(256) void potential_kernel(PotArgs p, T* V) {
    // per kept atom: x, y, z, their image shifts, lam, -Z kappa, amp
    __shared__ double at[256][9];
    __shared__ int wcount[4];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int ty = blockIdx.x / p.ntx, tx = blockIdx.x - ty * p.ntx;
    const int i0 = tx * POT_TX, j0 = ty * POT_TY, k0 = blockIdx.y * TZ;
    // a wavefront takes 8 x 8 columns: the more compact, the fewer idle lanes
    // at the rim of a cutoff sphere
    const int i = i0 + 8 * wv + (lane & 7), j = j0 + (lane >> 3);
    const double r0 = i * p.dx, r1 = j * p.dy;
    const double hx = 0.5 * (POT_TX - 1) * p.dx, hy = 0.5 * (POT_TY - 1) * p.dy, hz = 0.5 * (TZ - 1) * p.dz;
    const double mx = i0 * p.dx + hx, my = j0 * p.dy + hy, mz = k0 * p.dz + hz;
    const double far2 = p.cutoff * p.cutoff * (1.0 + 1e-12);
    double v[TZ];
#pragma unroll
    for (int k = 0; k < TZ; ++k) v[k] = 0.0;
    const int q1 = p.slab_ptr[blockIdx.y + 1];
    for (int q0 = p.slab_ptr[blockIdx.y]; q0 < q1; q0 += 256) {
        bool keep = false;
        double a[5], sh[3] = {0.0, 0.0, 0.0};
        if (q0 + t < q1) {
            const double* src = p.atoms + 5 * (long)p.slab_idx[q0 + t];
#pragma unroll
            for (int c = 0; c < 5; ++c) a[c] = src[c];
            const double u0 = mx - a[0], u1 = my - a[1], u2 = mz - a[2];
            if (!p.bcx) sh[0] = p.Lx * rint(u0 / p.Lx);
            if (!p.bcy) sh[1] = p.Ly * rint(u1 / p.Ly);
            if (!p.bcz) sh[2] = p.Lz * rint(u2 / p.Lz);
            // what this admits in excess, the exact test below rejects
            keep = fabs(u0 - sh[0]) <= p.reachx + hx && fabs(u1 - sh[1]) <= p.reachy + hy;
        }
        const unsigned long long m = __ballot(keep);
        if (lane == 0) wcount[wv] = __popcll(m);
        __syncthreads();
        int slot = __popcll(m & ((1ull << lane) - 1));
        for (int w = 0; w < wv; ++w) slot += wcount[w];
        if (keep) {
            double* o = at[slot];
            o[0] = a[0];
            o[1] = a[1];
            o[2] = a[2];
            o[3] = sh[0];
            o[4] = sh[1];
            o[5] = sh[2];
            o[6] = p.screened ? 0.8853 * p.a0 * pow(a[3], -1.0 / 3.0) : 1.0;
            o[7] = -a[3] * p.kappa;
            o[8] = a[4];
        }
        const int n = (wcount[0] + wcount[1]) + (wcount[2] + wcount[3]);
        __syncthreads();
        for (int e = 0; e < n; ++e) {
            const double* o = at[e];
            double u0 = r0 - o[0], u1 = r1 - o[1];
            if (p.fixx)
                u0 = u0 - o[3];
            else
                u0 = min_image(u0, p.Lx);
            if (p.fixy)
                u1 = u1 - o[4];
            else
                u1 = min_image(u1, p.Ly);
            const double a2 = u0 * u0 + u1 * u1;
            if (!(a2 < far2)) continue;
#pragma unroll
            for (int k = 0; k < TZ; ++k) {
                double u2 = (k0 + k) * p.dz - o[2];
                if (p.fixz)
                    u2 = u2 - o[5];
                else
                    u2 = min_image(u2, p.Lz);
                const double d2 = a2 + u2 * u2;
                if (!(d2 < far2)) continue;
                const double d = sqrt(d2);
                if (d >= p.cutoff) continue;
                const double ex = p.screened ? exp(-d / o[6]) : 1.0;
                v[k] += o[8] * (o[7] * ex / sqrt(d * d + p.soft * p.soft));
            }
        }
        __syncthreads();
    }
    if (i >= p.nx || j >= p.ny) return;
    T* out = V + ((long)k0 * p.ny + j) * p.nx + i;
#pragma unroll
    for (int k = 0; k < TZ; ++k)
        if (k0 + k < p.nz) out[(long)k * p.nx * p.ny] = (T)v[k];
}

struct GaussAxisArgs {
    int n[3];
    double d[3], L[3], r0[3], k0[3];
    int periodic[3];
    double sigma, hbar, mass, t0, t1;
    double* fac;  // [2 times][nx + ny + nz][2] complex
};

// One factor of eq. (3) evolved freely to time t (closed form), summed over
// periodic images |m| <= 2:
//   phi = (pi s^2)^(-1/4) (1 + i tau)^(-1/2)
//         exp(-(x - x0 - v t)^2 / (2 s^2 (1 + i tau)) + i k (x - x0) - i hbar k^2 t / 2m)
__device__ void gauss_phi(double x, double x0, double k, double s, double t, double hbar,
                          double mass, double* re, double* im) {
    const double tau = hbar * t / (mass * s * s);
    const double v = hbar * k / mass;
    const double u = x - x0 - v * t;
    const double den = 2.0 * s * s * (1.0 + tau * tau);
    const double are = -(u * u) / den;
    const double aim = (u * u) * tau / den + k * (x - x0) - hbar * k * k * t / (2.0 * mass);
    // (1 + i tau)^(-1/2) = (1 + tau^2)^(-1/4) exp(-i atan(tau) / 2)
    const double mod = pow(1.0 + tau * tau, -0.25) * pow(M_PI * s * s, -0.25) * exp(are);
    const double ph = aim - 0.5 * atan(tau);
    double sn, cs;
    sincos(ph, &sn, &cs);
    *re = mod * cs;
    *im = mod * sn;
}

__global__ __launch_bounds__(256) void gauss_axis_kernel(GaussAxisArgs a) {
    const int tot = a.n[0] + a.n[1] + a.n[2];
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= 2 * tot) return;
    const int which = idx / tot;
    int m = idx % tot;
    int ax = 0;
    while (m >= a.n[ax]) {
        m -= a.n[ax];
        ++ax;
    }
    const double t = which ? a.t1 : a.t0;
    const double x = m * a.d[ax];
    double sre = 0.0, sim = 0.0;
    const int ni = a.periodic[ax] ? 2 : 0;
    for (int im = -ni; im <= ni; ++im) {
        double re, imv;
        gauss_phi(x + im * a.L[ax], a.r0[ax], a.k0[ax], a.sigma, t, a.hbar, a.mass, &re, &imv);
        sre += re;
        sim += imv;
    }
    a.fac[2 * idx] = sre;
    a.fac[2 * idx + 1] = sim;
}

struct GaussCellArgs {
    int nx, ny, nz;
    const double* fac;  // as written by gauss_axis_kernel
    double scale;
    int zc;             // planes per workgroup
    int nt_out;         // non-temporal stores
};

__device__ __forceinline__ void cmul(double ar, double ai, double br, double bi, double* cr,
                                     double* ci) {
    *cr = ar * br - ai * bi;
    *ci = ar * bi + ai * br;
}

// Partial sums of |psi(r, 0)|^2, one per (256-cell block, plane), on zc
// planes per workgroup.  Bound by FP64 issue and the lane exchanges of the
// sums: the x and y factors are formed once, and eight planes are summed
// together, each exchange handing over the half of the planes that the lane
// drops (10 exchanges for eight planes instead of 48; 512x512x1024: 671 us
// with a workgroup per plane, 406 us now).  P is 8, fewer on grids of fewer
// planes, where the sums of planes that are not there cost as much as the
// others: 2048x2048 cells in 1, 2, 4 planes 53 us each with eight, 12.5, 15.1
// and 23.4 with as many as there are; five planes take 52 with eight, and 50
// with a workgroup per plane.
// A plane's sum is the butterfly of wave_sum and the wavefronts in order for
// every P: the same bits.
template <int P>
__global__ __launch_bounds__(256) void gauss_norm_kernel(GaussCellArgs a, double* partial, int nblk) {
    __shared__ double red[2][4][P];
    const int t = threadIdx.x, lane = t & 63;
    const int c = blockIdx.x * 256 + t;
    double pr = 0.0, pi = 0.0;
    if (c < a.nx * a.ny) {
        const int j = c / a.nx, ox = 2 * (c - j * a.nx), oy = 2 * (a.nx + j);
        cmul(a.fac[ox], a.fac[ox + 1], a.fac[oy], a.fac[oy + 1], &pr, &pi);
    }
    const int k0 = blockIdx.y * a.zc, k1 = min(k0 + a.zc, a.nz);
    for (int k = k0, par = 0; k < k1; k += P, par ^= 1) {
        double v[P];
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int oz = 2 * (a.nx + a.ny + min(k + q, k1 - 1));
            double re, im;
            cmul(pr, pi, ld_uniform(a.fac, oz), ld_uniform(a.fac, oz + 1), &re, &im);
            v[q] = re * re + im * im;
        }
        // the lane's top bits (5, 4, 3 for eight) come to select the plane
#pragma unroll
        for (int o = 32, n = P / 2; n > 0; o >>= 1, n >>= 1) {
            const bool up = lane & o;
#pragma unroll
            for (int q = 0; q < n; ++q) {
                const double give = up ? v[q] : v[q + n], own = up ? v[q + n] : v[q];
                v[q] = own + __shfl_xor(give, o, 64);
            }
        }
#pragma unroll
        for (int o = 32 / P; o > 0; o >>= 1) v[0] += __shfl_xor(v[0], o, 64);
        if (lane % (64 / P) == 0) red[par][t >> 6][lane / (64 / P)] = v[0];
        __syncthreads();   // two buffers: the next planes' sums wait for no reader
        if (t < P && k + t < k1)
            partial[(long)(k + t) * nblk + blockIdx.x] =
                ((red[par][0][t] + red[par][1][t]) + red[par][2][t]) + red[par][3][t];
    }
}

// R = s Re psi(r, t0), I = s Im psi(r, t1).  Bound by its two written
// streams: a thread keeps the x and y factors of W cells and writes them on
// zc planes, whose z factors are scalar loads, with vector stores.
// 512x512x1024 FP32: 634 us with a thread per cell, 360 us (6.0 TB/s) now.
template <typename T, int W>
__global__ __launch_bounds__(256) void gauss_write_kernel(GaussCellArgs a, T* R, T* I) {
    const int nv = a.nx * a.ny / W;   // vectors per plane
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= nv) return;
    const int j = c / (a.nx / W), i = (c - j * (a.nx / W)) * W;
    const double* f0 = a.fac;
    const double* f1 = a.fac + 2 * (long)(a.nx + a.ny + a.nz);
    const int oy = 2 * (a.nx + j);
    double r0[W], m0[W], r1[W], m1[W];
#pragma unroll
    for (int e = 0; e < W; ++e) {
        const int ox = 2 * (i + e);
        cmul(f0[ox], f0[ox + 1], f0[oy], f0[oy + 1], &r0[e], &m0[e]);
        cmul(f1[ox], f1[ox + 1], f1[oy], f1[oy + 1], &r1[e], &m1[e]);
    }
    const int k0 = blockIdx.y * a.zc, k1 = min(k0 + a.zc, a.nz);
    const int bytes = a.nx * a.ny * (int)sizeof(T);   // below 2^31 for every supported plane
    for (int k = k0; k < k1; ++k) {
        const int oz = 2 * (a.nx + a.ny + k);
        const double zr0 = ld_uniform(f0, oz), zi0 = ld_uniform(f0, oz + 1);
        const double zr1 = ld_uniform(f1, oz), zi1 = ld_uniform(f1, oz + 1);
        vec_t<T, W> vr, vi;
#pragma unroll
        for (int e = 0; e < W; ++e) {
            double re0, im0, re1, im1;
            cmul(r0[e], m0[e], zr0, zi0, &re0, &im0);
            cmul(r1[e], m1[e], zr1, zi1, &re1, &im1);
            vr.v[e] = (T)(a.scale * re0);
            vi.v[e] = (T)(a.scale * im1);
        }
        const long plane = (long)k * a.nx * a.ny;
        bstore_out<T, W>(plane_rsrc(R + plane, bytes), c * W * (int)sizeof(T), vr, a.nt_out);
        bstore_out<T, W>(plane_rsrc(I + plane, bytes), c * W * (int)sizeof(T), vi, a.nt_out);
    }
}

}  // namespace tdse

namespace tdse {

struct VjpArgs {
    int nx, ny, nz;
    double dx, dy, dz, Lx, Ly, Lz;
    int bcx, bcy, bcz, screened;
    const double* atoms;  // [n][5]
    const double* gV;     // dL/dV [nz][ny][nx]
    double soft, cutoff, kappa, a0;
    double* out;          // [n][4]: dL/dx, dL/dy, dL/dz, dL/damp
};

// Index range of one axis around coordinate x within the cutoff: the cells
// i0 .. i0 + cnt - 1 (wrapped on a periodic axis, clipped on a zero one),
// each cell of the axis at most once.
__device__ __forceinline__ void axis_range(double x, double cut, double d, int n, int zero,
                                           int* i0, int* cnt) {
    int lo = (int)ceil((x - cut) / d), hi = (int)floor((x + cut) / d);
    if (zero) {
        lo = max(lo, 0);
        hi = min(hi, n - 1);
        *i0 = lo;
        *cnt = max(0, hi - lo + 1);
        return;
    }
    if (hi - lo + 1 >= n) {
        *i0 = 0;
        *cnt = n;
        return;
    }
    *i0 = lo;
    *cnt = hi - lo + 1;
}

// Chain rule from dL/dV to the atoms:
//   dL/dX_a = sum_r gV(r) (-amp_a v'(d) u / d),  dL/damp_a = sum_r gV(r) v(d),
// u = r - X_a (minimum image), d = |u| < cutoff; a cell exactly on the atom
// adds nothing to dL/dX_a (cusp of the screened potential).  One workgroup
// per atom, fixed-order reduction.
__global__ __launch_bounds__(256) void potential_vjp_kernel(VjpArgs p) {
    __shared__ double red[256];
    const double* at = p.atoms + 5 * (long)blockIdx.x;
    int i0, ci, j0, cj, k0, ck;
    axis_range(at[0], p.cutoff, p.dx, p.nx, p.bcx, &i0, &ci);
    axis_range(at[1], p.cutoff, p.dy, p.ny, p.bcy, &j0, &cj);
    axis_range(at[2], p.cutoff, p.dz, p.nz, p.bcz, &k0, &ck);
    const long tot = (long)ci * cj * ck;
    double sx = 0.0, sy = 0.0, sz = 0.0, sa = 0.0;
    const double Z = at[3], amp = at[4];
    const double lam = 0.8853 * p.a0 * pow(Z, -1.0 / 3.0);
    for (long c = threadIdx.x; c < tot; c += 256) {
        const int ii = (int)(c % ci), jj = (int)((c / ci) % cj), kk = (int)(c / ((long)ci * cj));
        int i = i0 + ii, j = j0 + jj, k = k0 + kk;
        if (!p.bcx) i = ((i % p.nx) + p.nx) % p.nx;
        if (!p.bcy) j = ((j % p.ny) + p.ny) % p.ny;
        if (!p.bcz) k = ((k % p.nz) + p.nz) % p.nz;
        double ux = i * p.dx - at[0], uy = j * p.dy - at[1], uz = k * p.dz - at[2];
        if (!p.bcx) ux = min_image(ux, p.Lx);
        if (!p.bcy) uy = min_image(uy, p.Ly);
        if (!p.bcz) uz = min_image(uz, p.Lz);
        const double d = sqrt(ux * ux + uy * uy + uz * uz);
        if (d >= p.cutoff) continue;
        const double w = p.gV[((long)k * p.ny + j) * p.nx + i];
        const double e = p.screened ? exp(-d / lam) : 1.0;
        const double v = -Z * p.kappa * e / sqrt(d * d + p.soft * p.soft);
        sa += w * v;
        if (d > 0.0) {
            const double inv_lam = p.screened ? 1.0 / lam : 0.0;
            const double dv = v * (-inv_lam - d / (d * d + p.soft * p.soft));
            const double f = -amp * dv / d;
            sx += w * f * ux;
            sy += w * f * uy;
            sz += w * f * uz;
        }
    }
    sx = block_sum256(sx, red);
    sy = block_sum256(sy, red);
    sz = block_sum256(sz, red);
    sa = block_sum256(sa, red);
    if (threadIdx.x == 0) {
        double* o = p.out + 4 * (long)blockIdx.x;
        o[0] = sx;
        o[1] = sy;
        o[2] = sz;
        o[3] = sa;
    }
}

// Potential from a table over one unit cell (section 2.3: the cell's
// potential is repeated in x and y and interpolated onto the mesh points),
// trilinear.  Sample (a, b, c) of the table [uz][uy][ux] sits at origin +
// (a sx, b sy, c sz); the cell repeats in x and y, and the table is held
// constant beyond its first and last z planes.
struct InterpArgs {
    const double* table;
    int ux, uy, uz;
    double sx, sy, sz, ox, oy, oz;
    int nx, ny, nz;
    double dx, dy, dz;
};

// Per-axis samples and weight of one mesh index: the lower table sample a0,
// the upper a1 and the weight t of a1.
struct AxisW {
    int a0, a1;
    double t;
};

// fractional table coordinate u -> lower sample (wrapped), upper sample and weight
__device__ __forceinline__ AxisW cell_axis(double u, int n) {
    const double f = floor(u);
    AxisW w;
    w.t = u - f;
    long a = (long)f % n;
    if (a < 0) a += n;
    w.a0 = (int)a;
    w.a1 = (int)((a + 1) % n);
    return w;
}

// The weights of every mesh index of the three axes, once per call:
// ax[0 .. nx) for x, ax[nx .. nx+ny) for y (both periodic over the cell),
// ax[nx+ny .. nx+ny+nz) for z (clamped to the table's z range).
__global__ __launch_bounds__(256) void interp_axes_kernel(InterpArgs a, AxisW* ax) {
    const long n = (long)a.nx + a.ny + a.nz;
    for (long c = (long)blockIdx.x * 256 + threadIdx.x; c < n; c += (long)gridDim.x * 256) {
        AxisW w{0, 0, 0.0};
        if (c < a.nx) {
            w = cell_axis(((double)c * a.dx - a.ox) / a.sx, a.ux);
        } else if (c < (long)a.nx + a.ny) {
            w = cell_axis(((double)(c - a.nx) * a.dy - a.oy) / a.sy, a.uy);
        } else if (a.uz > 1) {
            const long k = c - a.nx - a.ny;
            double u = ((double)k * a.dz - a.oz) / a.sz;
            u = fmin(fmax(u, 0.0), (double)(a.uz - 1));
            w.a0 = min((int)floor(u), a.uz - 2);
            w.t = u - (double)w.a0;
            w.a1 = w.a0 + 1;
        }
        ax[c] = w;
    }
}

// One workgroup: plane k = blockIdx.y, a segment of 256 x columns and rows
// [j0, j0 + rows) (blockIdx.x = segment + nseg * row group).  Each thread
// holds its column's x weights and reads the row's y and the plane's z
// weights as wave-uniform values, so a cell costs its eight table samples
// (four table rows that the whole row shares, from the caches), the blends
// in x, then y, then z, and one coalesced store.
template <typename T>
__global__ __launch_bounds__(256) void interp_potential_kernel(InterpArgs a, const AxisW* ax, int nseg,
                                                               int rows, T* V) {
    const int seg = blockIdx.x % nseg;
    const int j0 = (blockIdx.x / nseg) * rows;
    const int k = blockIdx.y;
    const int i = seg * 256 + threadIdx.x;
    if (i >= a.nx) return;   // no barriers below
    const AxisW wx = ax[i];
    const AxisW wz = ax[a.nx + a.ny + k];
    const double tx = wx.t, sx = 1.0 - tx;
    const double tz = wz.t;
    const long plane = (long)a.uy * a.ux;
    const double* p0 = a.table + (long)wz.a0 * plane;
    const double* p1 = a.table + (long)wz.a1 * plane;
    T* out = V + ((long)k * a.ny) * a.nx + i;
    const int j1 = min(j0 + rows, a.ny);
    for (int j = j0; j < j1; ++j) {
        const AxisW wy = ax[a.nx + j];
        const double ty = wy.t;
        const long r0 = (long)wy.a0 * a.ux, r1 = (long)wy.a1 * a.ux;
        const double b00 = sx * p0[r0 + wx.a0] + tx * p0[r0 + wx.a1];
        const double b10 = sx * p0[r1 + wx.a0] + tx * p0[r1 + wx.a1];
        const double b01 = sx * p1[r0 + wx.a0] + tx * p1[r0 + wx.a1];
        const double b11 = sx * p1[r1 + wx.a0] + tx * p1[r1 + wx.a1];
        const double c0 = (1.0 - ty) * b00 + ty * b10;
        const double c1 = (1.0 - ty) * b01 + ty * b11;
        out[(long)j * a.nx] = (T)((1.0 - tz) * c0 + tz * c1);
    }
}

// The same with the z blend of the workgroup's mesh plane done once per
// table sample, Z[b][a] = (1 - tz) T[c0][b][a] + tz T[c1][b][a], and then
// the y blend of each of its rows once per sample of the row,
// Y[r][a] = (1 - ty_r) Z[b0_r][a] + ty_r Z[b1_r][a], both staged in LDS
// when they fit (rows of ux + 1 samples, the last a copy of the first, so
// the upper x sample is always the next one).  A cell then costs one paired
// LDS read and the x blend (3 FP64 operations instead of 21).  The same
// trilinear value, blended z, y, x instead of x, y, z: it differs from that
// order by FP64 rounding only.
template <typename T>
__global__ __launch_bounds__(256) void interp_potential_lds_kernel(InterpArgs a, const AxisW* ax, int nseg,
                                                                   int rows, T* V) {
    extern __shared__ double zl[];   // Z: [uy][ux + 1], then Y: [rows][ux + 1]
    const int seg = blockIdx.x % nseg;
    const int j0 = (blockIdx.x / nseg) * rows;
    const int k = blockIdx.y;
    const int ux1 = a.ux + 1;
    const int per = a.uy * ux1;
    const int j1 = min(j0 + rows, a.ny);
    const AxisW wz = ax[a.nx + a.ny + k];
    const long plane = (long)a.uy * a.ux;
    const double* t0 = a.table + (long)wz.a0 * plane;
    const double* t1 = a.table + (long)wz.a1 * plane;
    for (int t = threadIdx.x; t < per; t += 256) {
        const int r = t / ux1, q = t - r * ux1;
        const long src = (long)r * a.ux + (q == a.ux ? 0 : q);
        zl[t] = (1.0 - wz.t) * t0[src] + wz.t * t1[src];
    }
    __syncthreads();
    double* yl = zl + per;
    const int ny1 = (j1 - j0) * ux1;
    for (int t = threadIdx.x; t < ny1; t += 256) {
        const int r = t / ux1, q = t - r * ux1;
        const AxisW wy = ax[a.nx + j0 + r];
        yl[t] = (1.0 - wy.t) * zl[wy.a0 * ux1 + q] + wy.t * zl[wy.a1 * ux1 + q];
    }
    __syncthreads();
    const int i = seg * 256 + threadIdx.x;
    if (i >= a.nx) return;   // after the last barrier
    const AxisW wx = ax[i];
    const double tx = wx.t, sx = 1.0 - tx;
    const double* yx = yl + wx.a0;
    T* out = V + ((long)k * a.ny) * a.nx + i;
    for (int j = j0; j < j1; ++j) {
        const double* y = yx + (j - j0) * ux1;
        __builtin_nontemporal_store((T)(sx * y[0] + tx * y[1]), out + (long)j * a.nx);
    }
}

}  // namespace tdse
