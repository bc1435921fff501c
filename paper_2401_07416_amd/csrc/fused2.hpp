// Two leapfrog steps per sweep: eqs. (9), (8), (9), (8) of arXiv 2401.07416
// section 2.1 chained in one z-marching pass (temporal blocking of depth
// two).  The sweep reads (R^n, I^{n-1/2}, V) once and writes (R^{n+2},
// I^{n+3/2}) once, 20 B per cell in FP32 for two steps, where the one-pass
// step moves 20 B per step.  The intermediate level (I^{n+1/2}, R^{n+1})
// never leaves the chip.
//
// Mapping.  A workgroup (NT = 256, 512 or 1024 threads) owns an interior
// tile of tx x ty cells of every plane of a z chunk, and works on the tile
// extended by four cells on each side in x and y (ex = tx + 8, ey = ty + 8,
// ey = M rows per thread x the rows one pass of NT threads covers): each of
// the four half-steps needs its input one cell further out than its output,
// so the region on which a phase result is exact shrinks by one cell per
// phase, from the whole extension for the loaded R^n to the interior for
// R^{n+2}.  Results on the shrinking rim are computed and discarded.
//
// Per iteration k of the z march the four phases run one plane apart:
//   A1  I^{n+1/2}(k+3)  from R^n(k+2..k+4)
//   B1  R^{n+1}(k+2)    from I^{n+1/2}(k+1..k+3)
//   A2  I^{n+3/2}(k+1)  from R^{n+1}(k..k+2)
//   B2  R^{n+2}(k)      from I^{n+3/2}(k-1..k+1)
// Each thread keeps the z windows of the four fields (the new plane of each
// plus the two below it that the next phases read, in rings of three
// register slots) and four planes of the potential term vterm(V) in
// registers (its W-wide x vectors of M extended rows).  The x and y
// neighbours of each phase's centre plane come from LDS, where the previous
// iteration left them: every phase reads the LDS buffers of parity k and
// writes those of parity k + 1, so one barrier per iteration orders all
// reads and writes.  The march starts six planes before the chunk so
// that every stored plane is exact.
//
// The cell arithmetic is vterm / hterm / upd_* of kernels.hpp, so the
// states are bitwise identical to those of the one-pass and two-pass steps.
// The flux partials of both steps (every step) and, on the second step only,
// the record fields are reduced per workgroup in a fixed order.
#pragma once

#include <type_traits>

#include "kernels.hpp"

namespace tdse {

template <typename T>
struct Fused2Args {
    const T* R0;  // R^n
    const T* I0;  // I^{n-1/2}
    T* R1;        // R^{n+2}
    T* I1;        // I^{n+3/2}
    const T* V;
    const T* ca;
    const T* cb;
    T cx, cy, cz, cv;
    T d0, dlo;            // 2 (cx + cy + cz) as hi + lo parts
    int nx, ny, nz;
    int tx, ty, ex, ey;   // interior and extended tile extents
    int tpr, rpp;         // threads per extended row, extended rows per pass
    int ntx, ntiles, zc, nzc, nwg;
    int bcx, bcy, bcz;
    int k_det, k_up;
    int ulo, uhi;         // planes [ulo, uhi) have no absorption (ca = cb = 1)
    double* flux_a;       // [2][ntiles], step n -> n+1
    double* flux_b;       // [2][ntiles], step n+1 -> n+2
    // record of level n+2 (REC instances only)
    T* rec_plane;
    double* part_q;       // [nzc][ntiles]
    double* part_naive;
    double* part_plane;   // [ntiles]
    double* pixel;
    double pixel_w;
    int nt_out;           // non-temporal hint on the R^{n+2}, I^{n+3/2} stores
};

// Bytes of one LDS buffer of a 1024-thread workgroup: the most eight of them
// can take of a CU's 160 KB (such a workgroup has the CU to itself), at a
// distance known to the compiler.
constexpr int FUSED2_BUF = 20448;

// MARCH (1024 threads, one row each, prefetch): the instance for grids
// periodic in x and y, whose common iterations run in the march loop.  With a
// zero boundary there nothing could take that loop, and the other instance
// runs its iterations unrolled by three without moves (256x256x512 FP32 with
// zero boundaries: 80 us a step, 101 in the instance with the loop).
template <typename T, int W, int M, bool REC, bool PF, int NT, bool MARCH>
__device__ __forceinline__ void fused2_body(const Fused2Args<T>& a, int L, unsigned char* smem_raw) {
    using VT = vec_t<T, W>;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int ex = a.ex, ey = a.ey;
    const int pbytes = (int)((long)nx * ny * (long)sizeof(T));
    // one LDS buffer with a pad row on each side
    const long fstride = NT == 1024 ? FUSED2_BUF / (int)sizeof(T) : (long)(ey + 2) * ex;
    T* lds = reinterpret_cast<T*>(smem_raw);
    // field f (0 R^n, 1 I^{n+1/2}, 2 R^{n+1}, 3 I^{n+3/2}), parity q: row 0
    auto buf = [&](int f, int q) -> T* { return lds + (f + 4 * q) * fstride + ex; };

    const int zchunk = L / a.ntiles;
    const int tile = L - zchunk * a.ntiles;
    const int tyi = tile / a.ntx;
    const int txi = tile - tyi * a.ntx;
    const int x0 = txi * a.tx, y0 = tyi * a.ty;
    const int k0 = zchunk * a.zc;
    const int k1 = min(k0 + a.zc, nz);
    const int tid = threadIdx.x;
    const int rs0 = tid / a.tpr;
    const bool live = rs0 < a.rpp;             // threads past the last full row idle
    const int rs = live ? rs0 : 0;
    const int c0 = (live ? tid - rs0 * a.tpr : 0) * W;   // extended column of the vector
    const int gx = x0 - 4 + c0;                          // unwrapped grid column
    int colg = gx;
    if (gx < 0 || gx >= nx) colg = a.bcx ? -1 : ((gx % nx) + nx) % nx;
    const bool xin = c0 >= 4 && c0 < 4 + a.tx && gx < nx;

    int rowb[M], voff[M], soff[M], voff_iv[M];
    bool zc_cell[M];   // cell outside a zero-boundary axis (or idle thread): forced to 0
#pragma unroll
    for (int i = 0; i < M; ++i) {
        rowb[i] = rs + i * a.rpp;
        const int gy = y0 - 4 + rowb[i];
        int rj = gy;
        if (gy < 0 || gy >= ny) rj = a.bcy ? -1 : ((gy % ny) + ny) % ny;
        const bool ok = live && rj >= 0 && colg >= 0;
        zc_cell[i] = !ok;
        voff[i] = ok ? (rj * nx + colg) * (int)sizeof(T) : OOB;
        const bool st = live && xin && rowb[i] >= 4 && rowb[i] < 4 + a.ty && gy < ny;
        soff[i] = st ? voff[i] : OOB;
        // I^{n-1/2} and V of the outermost extended rows feed only the
        // first phase's results there, which are discarded: not read
        voff_iv[i] = (rowb[i] >= 1 && rowb[i] < ey - 1) ? voff[i] : OOB;
    }
    auto gplane = [&](int p) -> int {
        if (p < 0) {
            if (a.bcz) return -1;
            do p += nz; while (p < 0);
        } else if (p >= nz) {
            if (a.bcz) return -1;
            do p -= nz; while (p >= nz);
        }
        return p;
    };
    auto prs = [&](const T* base, int gp) {
        return plane_rsrc(base + (long)(gp < 0 ? 0 : gp) * nx * ny, gp < 0 ? 0 : pbytes);
    };
    auto zero_vec = [&]() {
        VT z;
#pragma unroll
        for (int e = 0; e < W; ++e) z.v[e] = T(0);
        return z;
    };

    // z windows.  The four fields live in rings of three register slots,
    // plane p of a field in slot (p + off) mod 3, so that an iteration
    // writes each new plane over the one that has gone out of use and
    // nothing moves between iterations; the march is unrolled three times
    // so that every slot index is a compile-time constant.  At iteration k:
    // R^n holds planes k+2, k+3 and receives k+4; I^{n+1/2} holds k+1, k+2
    // and receives k+3; R^{n+1} holds k, k+1 and receives k+2; I^{n+3/2}
    // holds k-1, k and receives k+1.  Vw[0..3] holds the potential term of
    // V(k..k+3) (V(k+3) arrives in the iteration), io I^{n-1/2}(k+3).
    VT Rn[3][M], Ia[3][M], Rb[3][M], Ib[3][M], Vw[4][M], io[M];
    VT pR[M], pI[M], pV[M];   // prefetched inputs of the next iteration
#pragma unroll
    for (int i = 0; i < M; ++i) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            Ia[s][i] = zero_vec();
            Rb[s][i] = zero_vec();
            Ib[s][i] = zero_vec();
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) Vw[s][i] = zero_vec();
    }

    // one phase on plane p: centre c, z neighbours zl / zr, x / y neighbours
    // from LDS buffer src (the centre plane), old value uo, potential term
    // vterm(V) in vtv;
    // IS_R selects eq. (8), else eq. (9).  The result goes to out and, from
    // live threads, to LDS buffer dst (if not null).  A plane outside a zero
    // z boundary is zero.  Workgroups of 512 and 1024 threads (one or two
    // per CU, where the VALU work is least hidden) also take two uniform
    // shortcuts: no zero-boundary select without zero x / y boundaries (idle
    // threads' results are never stored or read), and no CAP factors on
    // planes without absorption (ca = cb = 1); the bits are the same.
    const bool sel_xy = NT < 512 || a.bcx || a.bcy;
    // Phase d (1..4) is exact on extended rows [d, ey - d); with one row per
    // thread, a wavefront none of whose rows lie there skips it (its rows
    // are all discarded rim, and no needed cell of the next phase reads
    // them): two of 16 wavefronts in the last phase of a 1024-thread tile.
    const int wbase = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int wlo = wbase / a.tpr;
    const int whi = min((wbase + 63) / a.tpr, a.rpp - 1);
    auto wave_needed = [&](int d) -> bool {
#pragma unroll
        for (int i = 0; i < M; ++i)
            if (whi + i * a.rpp >= d && wlo + i * a.rpp < ey - d) return true;
        return false;
    };
    auto phase = [&](auto is_r, int depth, int p, const VT(&zl)[M], const VT(&c)[M], const VT(&zr)[M],
                     const T* src, const VT(&uo)[M], const VT(&vtv)[M], VT(&out)[M], T* dst) {
        constexpr bool IS_R = decltype(is_r)::value;
        // the march's first iterations reach planes below those the stored
        // planes [k0, k1) depend on: phase d needs planes >= k0 - (4 - d)
        if (p < k0 - (4 - depth) || (M == 1 && !wave_needed(depth))) {
#pragma unroll
            for (int i = 0; i < M; ++i) out[i] = zero_vec();
            return;
        }
        const int gp = gplane(p);
        if (gp < 0) {
#pragma unroll
            for (int i = 0; i < M; ++i) {
                out[i] = zero_vec();
                if (dst && live) *reinterpret_cast<VT*>(dst + rowb[i] * ex + c0) = out[i];
            }
            return;
        }
        const T cap = ld_uniform(a.ca, gp);
        const T cbp = ld_uniform(a.cb, gp);
        auto cells = [&](auto sel, auto unit) {
            constexpr bool SEL = decltype(sel)::value, UNIT = decltype(unit)::value;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const T* row = src + rowb[i] * ex + c0;
                const VT yl = *reinterpret_cast<const VT*>(row - ex);
                const VT yr = *reinterpret_cast<const VT*>(row + ex);
                const T xle = row[-1], xre = row[W];
                VT o;
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const T cc = c[i].v[e];
                    const T xl = e > 0 ? c[i].v[e - 1] : xle;
                    const T xr = e < W - 1 ? c[i].v[e + 1] : xre;
                    const T hx = hterm(cc, xl, xr, yl.v[e], yr.v[e], zl[i].v[e], zr[i].v[e], vtv[i].v[e],
                                       a.cx, a.cy, a.cz, a.dlo);
                    T u;
                    if constexpr (UNIT)
                        u = IS_R ? upd_R_unit(hx, uo[i].v[e]) : upd_I_unit(hx, uo[i].v[e]);
                    else
                        u = IS_R ? upd_R(hx, uo[i].v[e], cap, cbp) : upd_I(hx, uo[i].v[e], cap, cbp);
                    if constexpr (SEL)
                        o.v[e] = zc_cell[i] ? T(0) : u;
                    else
                        o.v[e] = u;
                }
                out[i] = o;
                if (dst && live) *reinterpret_cast<VT*>(dst + rowb[i] * ex + c0) = o;
            }
        };
        using Yes = std::true_type;
        using No = std::false_type;
        const bool unit = NT >= 512 && cap == T(1) && cbp == T(1);
        if (sel_xy) {
            if (unit) cells(Yes{}, Yes{});
            else cells(Yes{}, No{});
        } else {
            if (unit) cells(No{}, Yes{});
            else cells(No{}, No{});
        }
    };
    using IsR = std::integral_constant<bool, true>;
    using IsI = std::integral_constant<bool, false>;

    // The straight-line iteration (one row per thread, 512 or 1024
    // threads): the cells of one phase on plane p from their neighbours in
    // LDS, without CAP factors where they are all one (unit), and the write
    // slot of each buffer (wslot + buffer index x wstep; idle threads: the
    // slot past the eight buffers, wstep 0).
    constexpr bool FAST = M == 1 && NT >= 512;
    struct Nb {
        VT yl, yr;
        T xl, xr;
    };
    static_assert(!MARCH || (FAST && PF && NT == 1024));
    const bool fast_grid = !sel_xy;
    const bool need4 = M != 1 || wave_needed(4);
    const bool wave_live = wlo < a.rpp;   // some thread of the wavefront owns a row
    T* const wslot = live ? buf(0, 0) + rowb[0] * ex + c0 : lds + 8 * fstride;
    const long wstep = live ? fstride : 0;
    const int rofs = rowb[0] * ex + c0;
    auto fast_cells = [&](auto is_r, bool unit, int p, const VT& zl, const VT& c, const VT& zr, const Nb& n,
                          const VT& uo, const VT& vtv, VT& out) {
        constexpr bool IS_R = decltype(is_r)::value;
        auto cells = [&](auto with_cap, T cap, T cbp) {
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const T xl = e > 0 ? c.v[e > 0 ? e - 1 : 0] : n.xl;
                const T xr = e < W - 1 ? c.v[e < W - 1 ? e + 1 : e] : n.xr;
                const T hx = hterm(c.v[e], xl, xr, n.yl.v[e], n.yr.v[e], zl.v[e], zr.v[e], vtv.v[e], a.cx,
                                   a.cy, a.cz, a.dlo);
                if constexpr (decltype(with_cap)::value)
                    out.v[e] = IS_R ? upd_R(hx, uo.v[e], cap, cbp) : upd_I(hx, uo.v[e], cap, cbp);
                else
                    out.v[e] = IS_R ? upd_R_unit(hx, uo.v[e]) : upd_I_unit(hx, uo.v[e]);
            }
        };
        if (unit)
            cells(std::false_type{}, T(1), T(1));
        else
            cells(std::true_type{}, ld_uniform(a.ca, p), ld_uniform(a.cb, p));
    };
    auto read_nb = [&](const T* src) -> Nb {
        const T* row = src + rofs;
        Nb n;
        n.yl = *reinterpret_cast<const VT*>(row - ex);
        n.yr = *reinterpret_cast<const VT*>(row + ex);
        n.xl = row[-1];
        n.xr = row[W];
        return n;
    };

    auto load3 = [&](int pr, int pi, VT(&r)[M], VT(&iv)[M], VT(&vv)[M]) {
        const int gr = gplane(pr), gi = gplane(pi);
        const auto rR = prs(a.R0, gr), rI = prs(a.I0, gi), rV = prs(a.V, gi);
#pragma unroll
        for (int i = 0; i < M; ++i) {
            r[i] = bload<T, W>(rR, voff[i]);
            iv[i] = bload<T, W>(rI, voff_iv[i]);
            vv[i] = bload<T, W>(rV, voff_iv[i]);
        }
    };

    const int ks = k0 - 6;
    // ring slot of plane p: R^n and I^{n+1/2} by (p - ks) mod 3, R^{n+1} and
    // I^{n+3/2} the same (their planes trail by one and two); as a
    // compile-time function of the unrolled iteration u = (k - ks) mod 3
    // and the plane's offset j from k
    auto slot = [](int u, int j) -> int { return ((u + j) % 3 + 3) % 3; };
    // prologue: R^n(ks+2), R^n(ks+3) into the ring, R^n(ks+3) staged for A1
    {
        const auto r2 = prs(a.R0, gplane(ks + 2)), r3 = prs(a.R0, gplane(ks + 3));
#pragma unroll
        for (int i = 0; i < M; ++i) {
            Rn[slot(0, 2)][i] = bload<T, W>(r2, voff[i]);
            Rn[slot(0, 3)][i] = bload<T, W>(r3, voff[i]);
        }
        if (live) {
#pragma unroll
            for (int i = 0; i < M; ++i)
                *reinterpret_cast<VT*>(buf(0, 0) + rowb[i] * ex + c0) = Rn[slot(0, 3)][i];
        }
        if (PF) load3(ks + 4, ks + 3, pR, pI, pV);
    }
    __syncthreads();

    // fixed-order workgroup sums
    __shared__ double red[NT / 64];
    auto wg_sum = [&](double v) -> double { return block_sum(v, red, NT / 64); };
    double fa0 = 0.0, fa1 = 0.0, fb0 = 0.0, fb1 = 0.0, q = 0.0, nv = 0.0, pl = 0.0;
    // one iteration of the march; U = (k - ks) mod 3 as a type
    auto iteration = [&](auto uc, int k) {
        constexpr int U = decltype(uc)::value;
        const int par = (k - ks) & 1;
        VT(&rN)[M] = Rn[slot(U, 4)];   // R^n(k+4), arriving
        VT(&rC)[M] = Rn[slot(U, 3)];
        VT(&rL)[M] = Rn[slot(U, 2)];
        VT(&nA)[M] = Ia[slot(U, 3)];   // I^{n+1/2}(k+3), formed by A1
        VT(&iC)[M] = Ia[slot(U, 2)];
        VT(&iL)[M] = Ia[slot(U, 1)];
        VT(&nB)[M] = Rb[slot(U, 2)];   // R^{n+1}(k+2), formed by B1
        VT(&bC)[M] = Rb[slot(U, 1)];
        VT(&bL)[M] = Rb[slot(U, 0)];
        VT(&nC)[M] = Ib[slot(U, 1)];   // I^{n+3/2}(k+1), formed by A2
        VT(&jC)[M] = Ib[slot(U, 0)];
        VT(&jL)[M] = Ib[slot(U, -1)];
        if (PF) {
#pragma unroll
            for (int i = 0; i < M; ++i) {
                rN[i] = pR[i];
                io[i] = pI[i];
                Vw[3][i] = pV[i];
            }
            if (k + 1 < k1) load3(k + 5, k + 4, pR, pI, pV);
        } else {
            load3(k + 4, k + 3, rN, io, Vw[3]);
        }
        // the window keeps the potential term of the update (vterm),
        // formed once per plane instead of per phase
#pragma unroll
        for (int i = 0; i < M; ++i)
#pragma unroll
            for (int e = 0; e < W; ++e) Vw[3][i].v[e] = vterm(Vw[3][i].v[e], a.cv, a.d0);
        VT nD[M];   // R^{n+2}(k), formed by B2
        if constexpr (MARCH) nD[0] = zero_vec();
        const bool unit = k >= a.ulo && k + 3 < a.uhi;
        if (FAST && fast_grid &&
            (MARCH ? !a.bcz || (k >= 0 && k + 3 < nz)
                   // (formed here for FP64: with the value from above the
                   // compiler's loop is 1% slower, in FP32 1% faster)
                   : k >= k0 && (sizeof(T) == 8 ? k >= a.ulo && k + 3 < a.uhi : unit))) {
            // periodic x and y, all four planes inside the grid (without
            // the march also inside the chunk's dependence range and without
            // absorption: the branches for the others cost a kernel of 512
            // threads more than they give, 192x192x384 FP32 53 us a step
            // without them, 62 with): the phases as
            // straight lines.  Every LDS read comes before the first LDS
            // write (the reads take parity k, the writes parity k + 1), so
            // the compiler may issue a phase's neighbour reads ahead of the
            // previous phase's arithmetic; idle threads write a slot past the
            // buffers instead of branching around the writes.  Same bits as
            // the phases below.
            if (wave_live) {
                const bool no_cap = !MARCH || unit;
                fast_cells(IsI{}, no_cap, gplane(k + 3), rL[0], rC[0], rN[0], read_nb(buf(0, par)), io[0],
                           Vw[3][0], nA[0]);
                if (!MARCH || k >= k0 - 4)
                    fast_cells(IsR{}, no_cap, gplane(k + 2), iL[0], iC[0], nA[0], read_nb(buf(1, par)), rL[0],
                               Vw[2][0], nB[0]);
                if (!MARCH || k >= k0 - 2)
                    fast_cells(IsI{}, no_cap, gplane(k + 1), bL[0], bC[0], nB[0], read_nb(buf(2, par)), iL[0],
                               Vw[1][0], nC[0]);
                if ((!MARCH || k >= k0) && need4)
                    fast_cells(IsR{}, no_cap, k, jL[0], jC[0], nC[0], read_nb(buf(3, par)), bL[0], Vw[0][0],
                               nD[0]);
                else if (!MARCH)
                    nD[0] = zero_vec();
                *reinterpret_cast<VT*>(wslot + (0 + 4 * (par ^ 1)) * wstep) = rN[0];
                *reinterpret_cast<VT*>(wslot + (1 + 4 * (par ^ 1)) * wstep) = nA[0];
                *reinterpret_cast<VT*>(wslot + (2 + 4 * (par ^ 1)) * wstep) = nB[0];
                *reinterpret_cast<VT*>(wslot + (3 + 4 * (par ^ 1)) * wstep) = nC[0];
            } else if (!MARCH) {
                // a wavefront of idle threads (a tile shorter than the
                // threads cover): nothing of it is stored or read
                nA[0] = nB[0] = nC[0] = nD[0] = zero_vec();
            }
        } else {
            // stage R^n(k+4) for the next iteration's A1
            if (live) {
#pragma unroll
                for (int i = 0; i < M; ++i)
                    *reinterpret_cast<VT*>(buf(0, par ^ 1) + rowb[i] * ex + c0) = rN[i];
            }
            // A1: I^{n+1/2}(k+3)
            phase(IsI{}, 1, k + 3, rL, rC, rN, buf(0, par), io, Vw[3], nA, buf(1, par ^ 1));
            // B1: R^{n+1}(k+2)
            phase(IsR{}, 2, k + 2, iL, iC, nA, buf(1, par), rL, Vw[2], nB, buf(2, par ^ 1));
            // A2: I^{n+3/2}(k+1)
            phase(IsI{}, 3, k + 1, bL, bC, nB, buf(2, par), iL, Vw[1], nC, buf(3, par ^ 1));
            // B2: R^{n+2}(k)
            phase(IsR{}, 4, k, jL, jC, nC, buf(3, par), bL, Vw[0], nD, nullptr);
        }
        const int pB = k + 2, pC = k + 1, pD = k;
        if (pC >= k0 && pC < k1) {
            const auto rI = prs(a.I1, pC);
#pragma unroll
            for (int i = 0; i < M; ++i) bstore_out<T, W>(rI, soff[i], nC[i], a.nt_out);
        }
        if (pD >= k0) {
            const auto rR = prs(a.R1, pD);
#pragma unroll
            for (int i = 0; i < M; ++i) bstore_out<T, W>(rR, soff[i], nD[i], a.nt_out);
        }
        // flux partials of both steps over the stored cells (the two faces
        // are the same plane when nz = 1).  With the march they are summed
        // over the workgroup where they arise: accumulators kept through it
        // would take eight of its registers.
        auto flux = [&](int p, const VT(&up)[M], const VT(&lo)[M], const VT(&ro)[M], const VT(&rn)[M],
                        double& acc0, double& acc1, double* slots) {
            double l0 = 0.0, l1 = 0.0;
            double& f0 = MARCH ? l0 : acc0;
            double& f1 = MARCH ? l1 : acc1;
            const bool det = p == a.k_det, at_up = p == a.k_up;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if (soff[i] == OOB) continue;
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const double s = (double)ro[i].v[e] + (double)rn[i].v[e];
                    if (det) f0 += (double)up[i].v[e] * s;
                    if (at_up) f1 += (double)lo[i].v[e] * s;
                }
            }
            if constexpr (MARCH) {
                if (det) {
                    const double s = wg_sum(f0);
                    if (tid == 0) slots[tile] = s;
                }
                if (at_up) {
                    const double s = wg_sum(f1);
                    if (tid == 0) slots[a.ntiles + tile] = s;
                }
            }
        };
        if (pB >= k0 && pB < k1 && (pB == a.k_det || pB == a.k_up))
            flux(pB, nA, iL, rL, nB, fa0, fa1, a.flux_a);
        if (pD >= k0 && (pD == a.k_det || pD == a.k_up)) flux(pD, nC, jL, bL, nD, fb0, fb1, a.flux_b);
        if (REC && pD >= k0) {
            double lp = 0.0;
            double& plane_sum = MARCH ? lp : pl;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                if (soff[i] == OOB) continue;
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const double dc = (double)jC[i].v[e], du = (double)bL[i].v[e];
                    const double dn = (double)nD[i].v[e];
                    q += dc * dc + du * dn;
                    nv += dn * dn + dc * dc;
                }
                if (pD == a.k_det) {
                    VT rv;
                    const long poff = soff[i] / (int)sizeof(T);
#pragma unroll
                    for (int e = 0; e < W; ++e) {
                        const double dn = (double)nD[i].v[e], dc = (double)jC[i].v[e];
                        const double rho = dn * dn + dc * dc;
                        rv.v[e] = (T)rho;
                        plane_sum += rho;
                        if (a.pixel) a.pixel[poff + e] += a.pixel_w * rho;
                    }
                    stv<T, W>(a.rec_plane + poff, rv);
                }
            }
            if (MARCH && pD == a.k_det) {
                const double sp = wg_sum(plane_sum);
                if (tid == 0) a.part_plane[tile] = sp;
            }
        }
        // shift the potential window one plane up
#pragma unroll
        for (int i = 0; i < M; ++i) {
            Vw[0][i] = Vw[1][i];
            Vw[1][i] = Vw[2][i];
            Vw[2][i] = Vw[3][i];
        }
        __syncthreads();
    };
    using U0 = std::integral_constant<int, 0>;
    using U1 = std::integral_constant<int, 1>;
    using U2 = std::integral_constant<int, 2>;

    // The march proper: runs of six iterations inside the grid and the chunk
    // with no detection face among their stored planes, periodic x and y,
    // 1024 threads.  What bounds an iteration is instruction issue, so here
    // it is stripped to the arithmetic: R^n and the potential term in rings
    // of four slots, loads landing in the slot that has gone out of use, so
    // that nothing is moved; LDS buffers at compile-time distances from four
    // offsets that swap parity with one addition each; running pointers for
    // the five streams.  164 vector instructions per iteration (FP32, W = 4),
    // of which 148 are arithmetic, where the phase-by-phase iteration took
    // 213.  512x512x1024 FP32 1130 -> 990 us per launch, 240x240x520 FP32
    // 15.8 -> 14.3 ms and 256x256x512 FP64 31.0 -> 28.2 ms a run, 12 films
    // of 128..256 squared 94.2 -> 90.8 ms.  The loop exists once, with the
    // store hint and the CAP factors as branches, and reads a phase's
    // neighbours only when it begins: two copies of the loop, or neighbours
    // read one phase ahead, took the kernel past the 128 registers that 1024
    // threads have, and the spills alone made it two to five times slower.
    // CAP planes are part of the march because the chunks at both ends of z
    // hold them and the slowest workgroup is the time of the launch (left to
    // the other iterations: 240x240x520 18.0 ms).  Same bits as the phases
    // above.
    VT mR[4], mV[4];
    // byte offsets of the thread's cells and the rows beside them in the
    // buffers that the iteration reads, and of its cells in those it writes
    // (idle threads of a live wavefront write into the pad row above): the
    // two sets of four change places every iteration
    int rd_c = 0, rd_l = 0, rd_r = 0, wr = 0, turn_by = 0;
    auto neighbours = [&](auto fc) -> Nb {
        constexpr int F = decltype(fc)::value * FUSED2_BUF, ES = (int)sizeof(T);
        Nb n;
        n.yl = *reinterpret_cast<const VT*>(smem_raw + rd_l + F);
        n.yr = *reinterpret_cast<const VT*>(smem_raw + rd_r + F);
        // (rd_c lies a vector before the cells)
        n.xl = *reinterpret_cast<const T*>(smem_raw + rd_c + F + (W - 1) * ES);
        n.xr = *reinterpret_cast<const T*>(smem_raw + rd_c + F + 2 * W * ES);
        return n;
    };
    auto put = [&](auto fc, const VT& v) {
        constexpr int F = decltype(fc)::value * FUSED2_BUF;
        *reinterpret_cast<VT*>(smem_raw + wr + F) = v;
    };
    // streams of the march at its current plane
    const long plane = (long)nx * ny;
    const T *gR = nullptr, *gI = nullptr, *gV = nullptr;
    T *oI = nullptr, *oR = nullptr;
    // iteration k + J of the march; slot of plane k + J + j of R^n and V:
    // (J + j) mod 4, of the other fields: (J + j) mod 3
    auto march = [&](auto jc, int k) {
        constexpr int J = decltype(jc)::value, U = J % 3;
        using F0 = std::integral_constant<int, 0>;
        using F1 = std::integral_constant<int, 1>;
        using F2 = std::integral_constant<int, 2>;
        using F3 = std::integral_constant<int, 3>;
        const bool unit = k + J >= a.ulo && k + J + 3 < a.uhi;
        const Nb n0 = neighbours(F0{});
        VT& v3 = mV[(J + 3) % 4];
#pragma unroll
        for (int e = 0; e < W; ++e) v3.v[e] = vterm(pV[0].v[e], a.cv, a.d0);
        mR[(J + 5) % 4] = bload<T, W>(plane_rsrc(gR, pbytes), voff[0]);
        pV[0] = bload<T, W>(plane_rsrc(gV, pbytes), voff_iv[0]);
        put(F0{}, mR[(J + 4) % 4]);
        __builtin_amdgcn_sched_barrier(0);
        VT& nA = Ia[(U + 3) % 3][0];
        fast_cells(IsI{}, unit, k + J + 3, mR[(J + 2) % 4], mR[(J + 3) % 4], mR[(J + 4) % 4], n0, pI[0], v3,
                   nA);
        pI[0] = bload<T, W>(plane_rsrc(gI, pbytes), voff_iv[0]);
        __builtin_amdgcn_sched_barrier(0);
        put(F1{}, nA);
        __builtin_amdgcn_sched_barrier(0);
        const Nb n1 = neighbours(F1{});
        VT& nB = Rb[(U + 2) % 3][0];
        fast_cells(IsR{}, unit, k + J + 2, Ia[(U + 1) % 3][0], Ia[(U + 2) % 3][0], nA, n1,
                   mR[(J + 2) % 4], mV[(J + 2) % 4], nB);
        __builtin_amdgcn_sched_barrier(0);
        put(F2{}, nB);
        __builtin_amdgcn_sched_barrier(0);
        const Nb n2 = neighbours(F2{});
        VT& nC = Ib[(U + 1) % 3][0];
        fast_cells(IsI{}, unit, k + J + 1, Rb[U % 3][0], Rb[(U + 1) % 3][0], nB, n2,
                   Ia[(U + 1) % 3][0], mV[(J + 1) % 4], nC);
        __builtin_amdgcn_sched_barrier(0);
        put(F3{}, nC);
        __builtin_amdgcn_sched_barrier(0);
        if (need4) {
            bstore_out<T, W>(plane_rsrc(oI, pbytes), soff[0], nC, a.nt_out);
            const Nb n3 = neighbours(F3{});
            VT nD;
            fast_cells(IsR{}, unit, k + J, Ib[(U + 2) % 3][0], Ib[U % 3][0], nC, n3, Rb[U % 3][0],
                       mV[J % 4], nD);
            bstore_out<T, W>(plane_rsrc(oR, pbytes), soff[0], nD, a.nt_out);
            if (REC && soff[0] != OOB) {
#pragma unroll
                for (int e = 0; e < W; ++e) {
                    const double dc = (double)Ib[U % 3][0].v[e], du = (double)Rb[U % 3][0].v[e];
                    const double dn = (double)nD.v[e];
                    q += dc * dc + du * dn;
                    nv += dn * dn + dc * dc;
                }
            }
        }
        gR += plane;
        gI += plane;
        gV += plane;
        oI += plane;
        oR += plane;
        rd_c += turn_by;
        rd_l += turn_by;
        rd_r += turn_by;
        wr -= turn_by;
        turn_by = -turn_by;
        // kept as four registers: as constants of the unrolled iterations the
        // compiler would hold every buffer's addresses at once
        asm volatile("" : "+v"(rd_c), "+v"(rd_l), "+v"(rd_r), "+v"(wr));
        __syncthreads();
    };
    // how many iterations from k on (a multiple of six, 0 if none) the march
    // may take
    auto march_len = [&](int k) -> int {
        if (!fast_grid || k < k0) return 0;
        int last = min(k1 - 2, nz - 6);
        for (int f : {a.k_det, a.k_up})
            for (int sp : {f - 2, f})
                if (sp >= k) last = min(last, sp - 1);
        return last < k ? 0 : (last - k + 1) / 6 * 6;
    };
    // k1 - ks >= 7 iterations; every branch is uniform over the workgroup.
    // Without the march the loop is left through its breaks only: with a test
    // of k at its head as well it took 1-9% longer (zero boundaries, us a
    // step: 37x500x1400 FP32 433 against 398, 301x300x200 209 and 193,
    // 200x180x300 on 512 threads 53.5 and 51.6)
    for (int k = ks; !MARCH || k < k1;) {
        if constexpr (MARCH) {
            int n = march_len(k);
            if (n > 0) {
                mR[2] = Rn[2][0];
                mR[3] = Rn[0][0];
                mR[0] = pR[0];
                mV[0] = Vw[0][0];
                mV[1] = Vw[1][0];
                mV[2] = Vw[2][0];
                gR = a.R0 + (k + 5) * plane;
                gI = a.I0 + (k + 4) * plane;
                gV = a.V + (k + 4) * plane;
                oI = a.I1 + (k + 1) * plane;
                oR = a.R1 + k * plane;
                const int at = (ex + rofs) * (int)sizeof(T);   // past the pad row
                const int pb = ((k - ks) & 1) * 4 * FUSED2_BUF;
                rd_c = pb + at - W * (int)sizeof(T);
                rd_l = pb + at - ex * (int)sizeof(T);
                rd_r = pb + at + ex * (int)sizeof(T);
                wr = 4 * FUSED2_BUF - pb + (live ? at : 0);
                turn_by = 4 * FUSED2_BUF - 2 * pb;
                asm volatile("" : "+v"(rd_c), "+v"(rd_l), "+v"(rd_r), "+v"(wr));
                if (!wave_live) {
                    // a wavefront of idle threads keeps the barriers
                    for (k += n; n > 0; --n) __syncthreads();
                }
                for (; n > 0; n -= 6, k += 6) {
                    march(std::integral_constant<int, 0>{}, k);
                    march(std::integral_constant<int, 1>{}, k);
                    march(std::integral_constant<int, 2>{}, k);
                    march(std::integral_constant<int, 3>{}, k);
                    march(std::integral_constant<int, 4>{}, k);
                    march(std::integral_constant<int, 5>{}, k);
                    // six iterations turn the rings of four by two slots
                    const VT r0 = mR[0], r1 = mR[1], v0 = mV[0];
                    mR[0] = mR[2];
                    mR[1] = mR[3];
                    mR[2] = r0;
                    mR[3] = r1;
                    mV[0] = mV[2];
                    mV[2] = v0;
                    mV[1] = mV[3];
                }
                Rn[2][0] = mR[2];
                Rn[0][0] = mR[3];
                pR[0] = mR[0];
                Vw[0][0] = mV[0];
                Vw[1][0] = mV[1];
                Vw[2][0] = mV[2];
                continue;
            }
        }
        if constexpr (MARCH) {
            iteration(U0{}, k);
            auto turn = [&](VT(&r)[3][M]) {
                const VT t = r[0][0];
                r[0][0] = r[1][0];
                r[1][0] = r[2][0];
                r[2][0] = t;
            };
            turn(Rn);
            turn(Ia);
            turn(Rb);
            turn(Ib);
            ++k;
        } else {
            iteration(U0{}, k);
            if (k + 1 >= k1) break;
            iteration(U1{}, k + 1);
            if (k + 2 >= k1) break;
            iteration(U2{}, k + 2);
            if (k + 3 >= k1) break;
            k += 3;
        }
    }

    // fixed-order workgroup sums of the partials
    const bool has_det = a.k_det >= k0 && a.k_det < k1;
    const bool has_up = a.k_up >= k0 && a.k_up < k1;
    if (!MARCH && has_det) {
        const double sa = wg_sum(fa0);
        const double sb = wg_sum(fb0);
        if (tid == 0) {
            a.flux_a[tile] = sa;
            a.flux_b[tile] = sb;
        }
    }
    if (!MARCH && has_up) {
        const double sa = wg_sum(fa1);
        const double sb = wg_sum(fb1);
        if (tid == 0) {
            a.flux_a[a.ntiles + tile] = sa;
            a.flux_b[a.ntiles + tile] = sb;
        }
    }
    if (REC) {
        const double sq = wg_sum(q);
        const double sn = wg_sum(nv);
        const long slot = (long)zchunk * a.ntiles + tile;
        if (tid == 0) {
            a.part_q[slot] = sq;
            a.part_naive[slot] = sn;
        }
        if (!MARCH && has_det) {
            const double sp = wg_sum(pl);
            if (tid == 0) a.part_plane[tile] = sp;
        }
    }
}

template <typename T, int W, int M, bool REC, bool PF, int NT, bool MARCH>
__global__ __launch_bounds__(NT) void fused2_kernel(Fused2Args<T> a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    fused2_body<T, W, M, REC, PF, NT, MARCH>(a, xcd_remap(blockIdx.x, a.nwg), smem_raw);
}

// Two steps of many grids in one launch (the batch form of the sweep).
// cfg[c] describes grid c from its state pair 0 into pair 1 (parity 0) or
// back (parity 1), with flux_a at its ring's slot 0; the launch takes ring
// slots flux_slot and flux_slot + 1.  Workgroups wg_start[c] ..
// wg_start[c+1]-1 of the launch (after an XCD remap over the whole launch)
// belong to grid c.  The record slot comes from the device counter so a
// captured graph can be replayed.
template <typename T>
struct Batch2Step {
    const Fused2Args<T>* cfg;
    const int* wg_start;
    const long* rec_idx;
    int n, total_wg, parity, flux_slot;
    int zero_xy;   // some grid has a zero x or y boundary
};

template <typename T, int W, int M, bool REC, bool PF, int NT, bool MARCH>
__global__ __launch_bounds__(NT) void fused2_batch_kernel(Batch2Step<T> b) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int Lg = xcd_remap(blockIdx.x, b.total_wg);
    int lo = 0, hi = b.n;  // wg_start[lo] <= Lg < wg_start[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (b.wg_start[mid] <= Lg) lo = mid; else hi = mid;
    }
    Fused2Args<T> a = b.cfg[lo];
    if (b.parity) {
        const T* r0 = a.R0;
        const T* i0 = a.I0;
        a.R0 = a.R1;
        a.I0 = a.I1;
        a.R1 = const_cast<T*>(r0);
        a.I1 = const_cast<T*>(i0);
    }
    a.flux_a += (long)b.flux_slot * 2 * a.ntiles;
    a.flux_b = a.flux_a + 2 * a.ntiles;
    if (REC) a.rec_plane += (*b.rec_idx) * (long)a.nx * a.ny;
    fused2_body<T, W, M, REC, PF, NT, MARCH>(a, Lg - b.wg_start[lo], smem_raw);
}

}  // namespace tdse
