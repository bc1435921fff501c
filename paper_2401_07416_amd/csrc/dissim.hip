// Trajectory dissimilarity of eq. (16), arXiv 2401.07416 section 3.2: for
// every pair (k, j) of trajectories, the time average of the L2 distance
// between their detector-plane densities,
//   d_kj = sum_t w_t sqrt(dA sum_p (rho_k,t,p - rho_j,t,p)^2),
// with the quadrature weights w_t carrying 1 / (t1 - t0).
//
// FP32 frames (the records) go to the FP64 matrix cores as a Gram
// contraction of shifted frames (dissim_gram_kernel, below).  FP64 frames
// keep the direct form on the vector ALU, where an FP64 Gram expansion
// would lose close pairs to cancellation: register tiled like a GEMM, a
// workgroup owns a 64 x 64 block of pairs, each thread a 4 x 4 sub-block,
// pixels stream through LDS in chunks of 32, and the squared differences of
// a chunk are summed with fused multiply-adds.  Each workgroup covers a
// range of frames and writes its partial time sums; a second kernel adds
// the partials in a fixed order, so the result is bitwise reproducible and
// exactly symmetric.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "../../include/tdse.h"

namespace {

constexpr int BK = 64;   // trajectories per block side
constexpr int PC = 32;   // pixels per LDS chunk
constexpr int LS = BK + 4;  // LDS row stride (pixel-major rows of BK values)

template <typename T>
struct alignas(4 * sizeof(T)) vec_of {
    T v[4];
};

struct DissimArgs {
    const void* frames;   // [K][T][P]
    const double* w;      // [T]
    double dA;
    int K, T;
    long P;
    int nb;               // row blocks
    int npb;              // pair blocks (upper triangle with diagonal)
    int tpc;              // frames per workgroup
    double* part;         // [ntc][K][K]
};

// e * e + s with one rounding (a fused multiply-add): two instructions per
// pair and pixel with the subtraction, and a sum at least as accurate as
// the separately rounded product and add.
__device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

// pair block index -> (row block, column block), column >= row
__device__ __forceinline__ void pair_block(int q, int nb, int* bi, int* bj) {
    int r = 0;
    while (q >= nb - r) {
        q -= nb - r;
        ++r;
    }
    *bi = r;
    *bj = r + q;
}

// LDS tiles are pixel-major ([PC][BK], stride LS) so that each thread reads
// its 4 consecutive trajectories of a pixel with one vector read.
template <typename T>
__global__ __launch_bounds__(256) void dissim_kernel(DissimArgs a) {
    __shared__ __align__(16) T As[PC * LS];
    __shared__ __align__(16) T Bs[PC * LS];
    using V4 = vec_of<T>;
    const T* F = static_cast<const T*>(a.frames);
    const int q = blockIdx.x % a.npb;
    const int tc = blockIdx.x / a.npb;
    int bi, bj;
    pair_block(q, a.nb, &bi, &bj);
    const int r0 = bi * BK, c0 = bj * BK;
    const int tid = threadIdx.x;
    const int tr = tid >> 4, tcl = tid & 15;   // rows 4 tr .. 4 tr + 3, columns 4 tcl .. 4 tcl + 3
    const int t0 = tc * a.tpc;
    const int t1 = min(t0 + a.tpc, a.T);
    double acc[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[x][y] = 0.0;

    // chunks of PC pixels of the workgroup's frames, in (frame, pixel) order;
    // the next chunk's values are loaded into registers while the current
    // one is summed from LDS
    constexpr int PER = BK * PC / 256;   // values per thread and tile
    const long cpt = (a.P + PC - 1) / PC;  // chunks per frame
    const long nch = cpt * (t1 - t0);
    T ra[PER], rb[PER];
    // value i of a thread's tile share: row (tid / PC) + i (256 / PC), pixel tid % PC
    constexpr int RSTEP = 256 / PC;
    const int row0 = tid / PC, col = tid - row0 * PC;
    const long rstride = (long)RSTEP * a.T * a.P;
    const T* pa = F + ((long)(r0 + row0) * a.T) * a.P + col;
    const T* pb = F + ((long)(c0 + row0) * a.T) * a.P + col;
    auto fetch = [&](long c) {
        const int t = t0 + (int)(c / cpt);
        const long p0 = (c % cpt) * PC;
        const bool pin = p0 + col < a.P;
        const long off = (long)t * a.P + p0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            ra[i] = (pin && r0 + row0 + RSTEP * i < a.K) ? pa[off + i * rstride] : T(0);
            rb[i] = (pin && c0 + row0 + RSTEP * i < a.K) ? pb[off + i * rstride] : T(0);
        }
    };
    double s64[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) s64[x][y] = 0.0;
    if (nch > 0) fetch(0);
    for (long c = 0; c < nch; ++c) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            As[col * LS + row0 + RSTEP * i] = ra[i];
            Bs[col * LS + row0 + RSTEP * i] = rb[i];
        }
        __syncthreads();
        if (c + 1 < nch) fetch(c + 1);
        T s[4][4];
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) s[x][y] = T(0);
#pragma unroll 8
        for (int p = 0; p < PC; ++p) {
            const V4 av = *reinterpret_cast<const V4*>(As + p * LS + 4 * tr);
            const V4 bv = *reinterpret_cast<const V4*>(Bs + p * LS + 4 * tcl);
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const T e = av.v[x] - bv.v[y];
                    s[x][y] = fma_of(e, e, s[x][y]);
                }
        }
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) s64[x][y] += (double)s[x][y];
        if (c % cpt == cpt - 1) {
            // the frame is complete
            const double wt = a.w[t0 + (int)(c / cpt)];
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    acc[x][y] += wt * sqrt(a.dA * s64[x][y]);
                    s64[x][y] = 0.0;
                }
        }
        __syncthreads();
    }
    double* out = a.part + (long)tc * a.K * a.K;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int k = r0 + 4 * tr + x, j = c0 + 4 * tcl + y;
            if (k < a.K && j < a.K) {
                out[(long)k * a.K + j] = acc[x][y];
                out[(long)j * a.K + k] = acc[x][y];
            }
        }
}

// FP32 frames on the matrix cores.  The distance does not change when every
// frame of a time t is shifted by the same image c_t, and with x_k = rho_k - c
//   sum_p (rho_k - rho_j)^2 = |x_k|^2 + |x_j|^2 - 2 x_k . x_j,
// a Gram contraction.  Formed in FP64 from FP32 frames: x = rho - c is exact
// in FP64 with the shift c_t = the frame of trajectory 0, and the
// cancellation in the expansion costs a few FP64 ulps of |x_k|^2 + |x_j|^2:
// a squared frame distance d^2 carries a relative error of about
// eps64 (|x_k|^2 + |x_j|^2) / d^2, tiny while a pair's distance is not far
// below the distances to trajectory 0 (1e-15 for random frames), larger for
// a tight cluster far from trajectory 0 (pairs 1e-6 apart at unit distance
// from it: about 1e-4 in d^2); the FP64-frame form below has no such
// cancellation.  The Gram block of a workgroup (GB x GB pairs, sixteen wavefronts
// of 32 x 32 pairs: four per SIMD) accumulates on v_mfma_f64_16x16x4_f64
// over chunks of GPC pixels staged in LDS as FP64 rows; the squared norms
// come from the same FP64 values as they are staged.
constexpr int GB = 128;           // trajectories per block side
constexpr int GPC = 32;           // pixels per LDS chunk
constexpr int GLS = GPC + 2;      // LDS row stride in doubles (16-byte rows, spread banks)
constexpr int GTHREADS = 1024;
constexpr int GQ = GPC / 4;       // 4-pixel vectors per row and chunk
constexpr int GSTEPS = GPC / 4;   // matrix steps per chunk
static_assert(GB * GQ == GTHREADS, "each thread stages one vector of a row of each side");
static_assert((GB / 32) * (GB / 32) * 64 == GTHREADS, "a wavefront per 32 x 32 pairs");

typedef double dbl4 __attribute__((ext_vector_type(4)));

// Work is counted in quarters of an off-diagonal block's frame.  A diagonal
// block's frame is three: ten of its sixteen wavefronts have pairs k <= j, at
// most three of them on one SIMD.
constexpr int GFULL = 4, GDIAG = 3;

// How the frames of the pair blocks are shared out, in one of two ways:
//  chunks (tpc > 0): a workgroup takes tpc frames of one block, and each of
//    the ntc chunks has a slab of [K][K] time sums (its pairs k <= j);
//  spans (tpc = 0): the frames, block after block, are one sequence, cut into
//    `spans` equal parts of work, a workgroup each; a frame belongs to the
//    part that holds its first unit, and a block has one slab of [GB][GB] per
//    workgroup that works on it.
struct GramPlan {
    int nb, npb;       // row blocks, pair blocks
    int K, T;
    int tpc, ntc;      // chunks
    int slots;         // spans: slabs per block, the most any block needs
    long spans, units; // workgroups; spans: units of work in all
};

__host__ __device__ inline int block_cost(int bi, int bj) { return bi == bj ? GDIAG : GFULL; }

// index of block (bi, bj), row by row, and its first unit (every row of
// blocks up to it has a diagonal one)
__host__ __device__ inline long block_index(const GramPlan& p, int bi, int bj) {
    return (long)bi * p.nb - (long)bi * (bi - 1) / 2 + (bj - bi);
}
__host__ __device__ inline long block_start(const GramPlan& p, int bi, int bj) {
    return p.T * (block_index(p, bi, bj) * GFULL - (long)(bi + (bj > bi)) * (GFULL - GDIAG));
}

// first unit of span w, and the span that holds unit u
__host__ __device__ inline long span_start(const GramPlan& p, long w) { return (w * p.units + p.spans - 1) / p.spans; }
__host__ __device__ inline long span_of(const GramPlan& p, long u) { return u * p.spans / p.units; }

// slabs that hold a block's time sums: all chunks, or from its first
// frame's span to its last one's
__host__ __device__ inline int block_slots(const GramPlan& p, int bi, int bj) {
    if (p.tpc) return p.ntc;
    const long s = block_start(p, bi, bj);
    return (int)(span_of(p, s + (long)(p.T - 1) * block_cost(bi, bj)) - span_of(p, s)) + 1;
}

// where a block's slab begins, its row stride, and the distance to its next
__host__ __device__ inline long slab_at(const GramPlan& p, long slot, int bi, int bj) {
    return p.tpc ? (slot * p.K + (long)bi * GB) * p.K + (long)bj * GB
                 : (slot * p.npb + block_index(p, bi, bj)) * (GB * GB);
}
__host__ __device__ inline int slab_ld(const GramPlan& p) { return p.tpc ? p.K : GB; }
__host__ __device__ inline long slab_step(const GramPlan& p) {
    return p.tpc ? (long)p.K * p.K : (long)p.npb * (GB * GB);
}

struct GramArgs {
    const float* frames;  // [K][T][P]
    const double* w;      // [T]
    double dA;
    long P;
    GramPlan p;
    double tau;           // a frame's d^2 below tau (|x_k|^2 + |x_j|^2) marks the pair
    double* part;         // the slabs
    unsigned* count;      // length of the list of marked pairs (zeroed here)
};

// four consecutive pixels p0 .. p0 + 3 of a row (zero past P)
template <bool VEC>
__device__ __forceinline__ float4 load4(const float* row, long p0, long P) {
    if (VEC) {
        if (p0 < P) return *reinterpret_cast<const float4*>(row + p0);
        return make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float4 r;
    r.x = p0 < P ? row[p0] : 0.f;
    r.y = p0 + 1 < P ? row[p0 + 1] : 0.f;
    r.z = p0 + 2 < P ? row[p0 + 2] : 0.f;
    r.w = p0 + 3 < P ? row[p0 + 3] : 0.f;
    return r;
}

// LOAD: 0, P is no multiple of 4 or the frames are not 16-byte aligned; 1,
// whole float4 loads; 2, whole chunks too (P a multiple of GPC), so that a row's
// chunks follow one another across frames and a fetch is three loads.
//
// What bounds it: the FP64 matrix cores, which share their datapath with the
// FP64 vector instructions, so every conversion of the staging costs matrix
// time (17.5 ms without any staging on 879 x 77 x 16384, of 20.4).  A wavefront
// carries its matrix steps through the chunk with one slice of the staging
// between two of them, the next step's fragments read a step ahead, no branch
// in the way, and the barrier where two steps' fragments are still in
// registers (19.4 ms); the equal spans of work instead of whole rounds of
// equal workgroups take it to 17.3 ms.
template <int LOAD>
__global__ __launch_bounds__(GTHREADS) void dissim_gram_kernel(GramArgs a) {
    __shared__ __align__(16) double As[2 * GB * GLS];
    __shared__ __align__(16) double Bs[2 * GB * GLS];
    __shared__ double nrm[2 * 2 * GB];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const long TP = (long)a.p.T * a.P;
    const long cpt = (a.P + GPC - 1) / GPC;
    // the reduction that follows on the stream appends the marked pairs
    if (blockIdx.x == 0 && tid == 0) *a.count = 0u;
    // staging: row srow of each side, pixels 4 quad .. 4 quad + 3
    const int quad = tid % GQ, srow = tid / GQ;
    double2* const sa = reinterpret_cast<double2*>(As + srow * GLS + 4 * quad);
    double2* const sb = reinterpret_cast<double2*>(Bs + srow * GLS + 4 * quad);
    constexpr int BUF = GB * GLS;   // doubles per buffer

    const int K = a.p.K;
    long u0 = 0, u1 = 0;            // spans: the workgroup's units
    int ci = -1, cj = -1, ct0 = 0;  // chunks: its block and first frame
    if (a.p.tpc) {
        pair_block(blockIdx.x % a.p.npb, a.p.nb, &ci, &cj);
        ct0 = blockIdx.x / a.p.npb * a.p.tpc;
    } else {
        u0 = span_start(a.p, blockIdx.x);
        u1 = span_start(a.p, (long)blockIdx.x + 1);
    }
    for (int bi = a.p.tpc ? ci : 0; bi < (a.p.tpc ? ci + 1 : a.p.nb); ++bi) {
        if (!a.p.tpc) {
            // rows of blocks wholly before or behind the span
            if (block_start(a.p, bi + 1, bi + 1) <= u0) continue;
            if (block_start(a.p, bi, bi) >= u1) break;
        }
        for (int bj = a.p.tpc ? cj : bi; bj < (a.p.tpc ? cj + 1 : a.p.nb); ++bj) {
            const long us = block_start(a.p, bi, bj);
            const int cost = block_cost(bi, bj);
            // frames t0 .. t1 - 1 of this block: the chunk's, or those that
            // start inside the span
            int t0 = ct0, t1 = min(ct0 + a.p.tpc, a.p.T);
            if (!a.p.tpc) {
                t0 = u0 <= us ? 0 : (int)min((u0 - us + cost - 1) / cost, (long)a.p.T);
                t1 = u1 <= us ? 0 : (int)min((u1 - us + cost - 1) / cost, (long)a.p.T);
            }
            if (t0 >= t1) continue;
            t0 = __builtin_amdgcn_readfirstlane(t0);
            t1 = __builtin_amdgcn_readfirstlane(t1);
            const long nch = cpt * (t1 - t0);
            const int r0 = bi * GB, c0 = bj * GB;
            // a wavefront's 32 x 32 pairs; on the diagonal the ten tiles with
            // pairs k <= j go to wavefronts 0 .. 9, spread over the SIMDs
            int tr = wv >> 2, tc = wv & 3;
            const bool active = bi != bj || wv < 10;
            if (bi == bj) {
                tr = wv < 4 ? 0 : wv < 7 ? 1 : wv < 9 ? 2 : 3;
                tc = wv < 4 ? wv : wv < 7 ? wv - 3 : wv < 9 ? wv - 5 : 3;
            }
            const int wr = 32 * tr, wc = 32 * tc;
            // rows past K read the last trajectory instead: their pairs are
            // never used
            const float* const rowa = a.frames + (long)min(r0 + srow, K - 1) * TP;
            const float* const rowb = a.frames + (long)min(c0 + srow, K - 1) * TP;
            float4 ra, rb, rc;
            // chunk pc of frame t0 + f
            const long first = (long)t0 * a.P + 4 * quad;
            const float *pa = rowa + first, *pb = rowb + first, *ps = a.frames + first;
            auto fetch = [&](int f, long pc) {
                if (LOAD == 2) {
                    ra = *reinterpret_cast<const float4*>(pa);
                    rb = *reinterpret_cast<const float4*>(pb);
                    rc = *reinterpret_cast<const float4*>(ps);   // the shift: trajectory 0
                    return;
                }
                const long off = (long)(t0 + f) * a.P, p0 = pc * GPC + 4 * quad;
                if (LOAD == 1) {
                    // past the row's end: its last vector, then zeros
                    const long q = off + min(p0, a.P - 4);
                    ra = *reinterpret_cast<const float4*>(rowa + q);
                    rb = *reinterpret_cast<const float4*>(rowb + q);
                    rc = *reinterpret_cast<const float4*>(a.frames + q);
                    if (p0 >= a.P) ra = rb = rc = make_float4(0.f, 0.f, 0.f, 0.f);
                } else {
                    ra = load4<false>(rowa + off, p0, a.P);
                    rb = load4<false>(rowb + off, p0, a.P);
                    rc = load4<false>(a.frames + off, p0, a.P);
                }
            };
            dbl4 g[2][2];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int n = 0; n < 2; ++n) g[m][n] = dbl4{0.0, 0.0, 0.0, 0.0};
            double na = 0.0, nbv = 0.0;
            // a row's norm over the frame: its GQ quad lanes (adjacent lanes)
            // combined by a butterfly, the same bits in each, into the
            // frame's half of nrm (halves alternate with the frame, so that a
            // wavefront still in the previous frame's end reads its own half)
            auto frame_norms = [&](int f) {
                double* nf = nrm + (f & 1) * 2 * GB;
                double x = na, y = nbv;
#pragma unroll
                for (int s = 1; s < GQ; s <<= 1) {
                    x += __shfl_xor(x, s);
                    y += __shfl_xor(y, s);
                }
                if (quad == 0) {
                    nf[srow] = x;
                    nf[GB + srow] = y;
                }
                na = 0.0;
                nbv = 0.0;
            };
            // the staged values as FP64 x = rho - c (exact), into LDS, with
            // their squares added to the rows' partial norms; in slices
            double xc[4], x[4];
            auto slice = [&](int s, int buf) {
                double2* const da = sa + buf * (BUF / 2);
                double2* const db = sb + buf * (BUF / 2);
                switch (s) {
                    case 0: xc[0] = (double)rc.x; xc[1] = (double)rc.y; break;
                    case 1: xc[2] = (double)rc.z; xc[3] = (double)rc.w; break;
                    case 2: x[0] = (double)ra.x - xc[0]; x[1] = (double)ra.y - xc[1]; break;
                    case 3: x[2] = (double)ra.z - xc[2]; x[3] = (double)ra.w - xc[3]; break;
                    case 4: da[0] = make_double2(x[0], x[1]); da[1] = make_double2(x[2], x[3]); break;
                    case 5: na = __builtin_fma(x[1], x[1], __builtin_fma(x[0], x[0], na)); break;
                    case 6: na = __builtin_fma(x[3], x[3], __builtin_fma(x[2], x[2], na)); break;
                    case 7: x[0] = (double)rb.x - xc[0]; x[1] = (double)rb.y - xc[1]; break;
                    case 8: x[2] = (double)rb.z - xc[2]; x[3] = (double)rb.w - xc[3]; break;
                    case 9: db[0] = make_double2(x[0], x[1]); db[1] = make_double2(x[2], x[3]); break;
                    case 10: nbv = __builtin_fma(x[1], x[1], __builtin_fma(x[0], x[0], nbv)); break;
                    default: nbv = __builtin_fma(x[3], x[3], __builtin_fma(x[2], x[2], nbv)); break;
                }
            };
            constexpr int SLICES = 12;
            // fragments of one matrix step
            const double* const fa = As + (wr + li) * GLS + lk;
            const double* const fb = Bs + (wc + li) * GLS + lk;
            struct Frag {
                double a[2], b[2];
            };
            auto frag = [&](int buf, int kk) {
                Frag f;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    f.a[m] = fa[buf * BUF + 16 * m * GLS + 4 * kk];
                    f.b[m] = fb[buf * BUF + 16 * m * GLS + 4 * kk];
                }
                return f;
            };
            auto mac = [&](const Frag& f, int m, int n) {
                g[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[m], f.b[n], g[m][n], 0, 0, 0);
            };
            auto mac4 = [&](const Frag& f) {
                mac(f, 0, 0);
                mac(f, 0, 1);
                mac(f, 1, 0);
                mac(f, 1, 1);
            };
            int fc = 0, fn = 0;     // frame of the current chunk and of the next one to fetch
            long pcc = 0, pn = 0;   // their chunks within the frame
            auto advance = [&](int& f, long& pc) {
                if (++pc == cpt) {
                    pc = 0;
                    ++f;
                }
            };
            // past the last chunk the last one again: staged, never read
            auto next = [&]() {
                if (LOAD == 2) {
                    const long step = ++pn < nch ? GPC : 0;   // pn: chunks of the segment
                    pa += step;
                    pb += step;
                    ps += step;
                } else if (fn < t1 - t0 - 1 || pn < cpt - 1) {
                    advance(fn, pn);
                }
            };
            const long slot = a.p.tpc ? blockIdx.x / a.p.npb : (long)blockIdx.x - span_of(a.p, us);
            const int ld = slab_ld(a.p);
            double* const out = a.part + slab_at(a.p, slot, bi, bj);

            __syncthreads();   // the previous block's LDS reads are done
            fetch(0, 0);
#pragma unroll
            for (int s = 0; s < SLICES; ++s) slice(s, 0);
            next();
            fetch(fn, pn);
            next();
            __syncthreads();
            Frag f0 = frag(0, 0);
            // two LDS buffers: chunk c + 1 is staged into the other one while
            // chunk c is contracted, one barrier per chunk
            for (long c = 0; c < nch; ++c) {
                const int cur = (int)(c & 1);
                const bool frame_done = pcc == cpt - 1;
                // the staged norms so far cover the frame's chunks up to c
                if (frame_done) frame_norms(fc);
                Frag last;
                if (active) {
#pragma unroll
                    for (int kk = 0; kk < GSTEPS - 2; ++kk) {
                        const Frag f1 = frag(cur, kk + 1);
                        mac(f0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (2 * kk < SLICES) slice(2 * kk, cur ^ 1);
                        mac(f0, 0, 1);
                        __builtin_amdgcn_sched_barrier(0);
                        if (2 * kk + 1 < SLICES) slice(2 * kk + 1, cur ^ 1);
                        mac(f0, 1, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (kk == GSTEPS - 3 && LOAD == 2) fetch(fn, pn);
                        mac(f0, 1, 1);
                        __builtin_amdgcn_sched_barrier(0);
                        f0 = f1;
                    }
                    if (LOAD != 2) fetch(fn, pn);
                    last = frag(cur, GSTEPS - 1);
                } else {
#pragma unroll
                    for (int s = 0; s < SLICES; ++s) slice(s, cur ^ 1);
                    fetch(fn, pn);
                }
                if (LOAD != 2) next();
                // behind the barrier the other buffer is staged, and this
                // one, whose last two steps are in registers, may be
                __syncthreads();
                if (active) {
                    mac4(f0);
                    f0 = frag(cur ^ 1, 0);
                    mac4(last);
                }
                if (LOAD == 2) next();
                if (frame_done && active) {
                    const double wt = a.w[t0 + fc];
                    const double* nf = nrm + (fc & 1) * 2 * GB;
                    // element r of a lane's accumulator is pair (4 r + lk, li) of the 16 x 16 tile
#pragma unroll
                    for (int m = 0; m < 2; ++m)
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int row = wr + 16 * m + 4 * r + lk, col = wc + 16 * n + li;
                                const double ns = nf[row] + nf[GB + col];
                                const double d2 = ns - 2.0 * g[m][n][r];
                                const double v = wt * sqrt(a.dA * fmax(d2, 0.0));
                                g[m][n][r] = 0.0;
                                // a d^2 this small against the norms may be
                                // mostly the expansion's rounding: the
                                // partial turns negative (no contribution
                                // is) and stays so, and the pair goes to the
                                // direct form
                                const int k = r0 + row, j = c0 + col;
                                if (k < j && j < K) {
                                    double* o = out + (long)row * ld + col;
                                    const double prev = fc == 0 ? 0.0 : *o;
                                    *o = (d2 < a.tau * ns || prev < 0.0) ? -1.0 : prev + v;
                                }
                            }
                    // nothing of the frame's epilogue stays in flight: the
                    // loop's wait bookkeeping then never holds the next
                    // chunk's LDS reads or the prefetch behind these accesses
                    __builtin_amdgcn_s_waitcnt(0);
                }
                advance(fc, pcc);
            }
        }
    }
}

// Adds a pair's time sums over its block's slabs in order, for k <= j, and
// writes both (k, j) and (j, k): the result is exactly symmetric; d_kk = 0.
// A pair with a negative partial (marked by the Gram kernel) is appended to
// list (the order of the list does not matter, each entry is evaluated on
// its own) and its entries are left for dissim_pairs_kernel.
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double* part, GramPlan p, double* out, int2* list,
                                                          unsigned* count) {
    const int K = p.K;
    const int j = blockIdx.x * 256 + threadIdx.x;
    for (int k = blockIdx.y; k <= j && j < K; k += gridDim.y) {
        if (j == k) {
            out[(long)k * K + k] = 0.0;
            continue;
        }
        const int bi = k / GB, bj = j / GB;
        const double* src = part + slab_at(p, 0, bi, bj) + (long)(k - bi * GB) * slab_ld(p) + (j - bj * GB);
        const long step = slab_step(p);
        const int n = block_slots(p, bi, bj);
        double s = 0.0;
        bool marked = false;
        for (int c = 0; c < n; ++c) {
            const double v = src[c * step];
            marked |= v < 0.0;
            s += v;
        }
        out[(long)k * K + j] = marked ? 0.0 : s;
        out[(long)j * K + k] = marked ? 0.0 : s;
        if (marked) list[atomicAdd(count, 1u)] = make_int2(k, j);
    }
}

// Adds the partial time sums of FP64 frames in a fixed order.
__global__ __launch_bounds__(256) void dissim_reduce_kernel(const double* part, int ntc, int K, double* out) {
    const long kk = (long)K * K;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < kk; i += (long)gridDim.x * 256) {
        double s = 0.0;
        bool negative = false;
        for (int c = 0; c < ntc; ++c) {
            const double v = part[(long)c * kk + i];
            negative |= v < 0.0;
            s += v;
        }
        out[i] = negative ? 0.0 : s;
    }
}

// The marked pairs in the direct form of eq. (16): per frame the sum over
// pixels of (rho_k - rho_j)^2, the differences of the FP32 values exact in
// FP64, fused multiply-adds.  A workgroup per pair of the list (a strided
// loop over the list), pixels strided over its threads, then a butterfly in
// each wavefront and the four wavefronts in order: the same bits on every
// run.  Writes d_kj and d_jk.
__global__ __launch_bounds__(256) void dissim_pairs_kernel(const float* frames, const double* w, double dA,
                                                           int K, int T, long P, const int2* list,
                                                           const unsigned* count, double* out) {
    __shared__ double red[4];
    const unsigned n = *count;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long TP = (long)T * P;
    for (unsigned it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 kj = list[it];
        const float* fa = frames + (long)kj.x * TP;
        const float* fb = frames + (long)kj.y * TP;
        double acc = 0.0;
        for (int t = 0; t < T; ++t) {
            double s = 0.0;
            for (long p = threadIdx.x; p < P; p += 256) {
                const double e = (double)fa[(long)t * P + p] - (double)fb[(long)t * P + p];
                s = __builtin_fma(e, e, s);
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
            if (lane == 0) red[wv] = s;
            __syncthreads();
            if (threadIdx.x == 0) acc += w[t] * sqrt(dA * (((red[0] + red[1]) + red[2]) + red[3]));
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            out[(long)kj.x * K + kj.y] = acc;
            out[(long)kj.y * K + kj.x] = acc;
        }
    }
}

struct Plan {
    int nb, npb, tpc, ntc;
};

Plan plan_of(int K, int T) {
    Plan p;
    p.nb = (K + BK - 1) / BK;
    p.npb = p.nb * (p.nb + 1) / 2;
    // enough workgroups to fill the chip: split the frames into chunks
    const int want = std::max(1, (2048 + p.npb - 1) / p.npb);
    p.ntc = std::min(T, want);
    p.tpc = (T + p.ntc - 1) / p.ntc;
    p.ntc = (T + p.tpc - 1) / p.tpc;
    return p;
}

constexpr long GCUS = 256;   // compute units, one Gram workgroup on each

size_t slab_bytes(const GramPlan& p) {
    return (size_t)(p.tpc ? p.ntc : p.slots) * (size_t)slab_step(p) * sizeof(double);
}

// Chunks of as many frames that the last round of workgroups over the
// compute units is as full as possible (cost = rounds x frames per
// workgroup; ties to more frames, less workspace), or one round of equal
// spans where their longest is shorter than those rounds and their slabs
// take no more workspace.  879 trajectories x 77 frames: 252 workgroups of
// nine frames, 36 units, against spans of at most 33.
GramPlan plan_gram(int K, int T) {
    GramPlan p{};
    p.K = K;
    p.T = T;
    p.nb = (K + GB - 1) / GB;
    p.npb = p.nb * (p.nb + 1) / 2;
    long best = -1;
    p.tpc = 1;
    for (int tpc = 1; tpc <= T; ++tpc) {
        const long ntc = (T + tpc - 1) / tpc;
        const long cost = (p.npb * ntc + GCUS - 1) / GCUS * tpc;
        if (best < 0 || cost <= best) {
            best = cost;
            p.tpc = tpc;
        }
    }
    p.ntc = (T + p.tpc - 1) / p.tpc;
    p.spans = (long)p.npb * p.ntc;

    GramPlan q = p;
    q.tpc = q.ntc = 0;
    q.spans = GCUS;
    q.units = block_start(q, q.nb, q.nb);
    // a span holds a frame at least, so that every workgroup between a
    // block's first and last has a slab of it
    const long len = (q.units + GCUS - 1) / GCUS;
    if (q.units < GCUS * GFULL) return p;
    const long longest = std::max((len + GFULL - 1) / GFULL * GFULL, (len + GDIAG - 1) / GDIAG * GDIAG);
    if (longest >= best * GFULL) return p;
    for (int bi = 0; bi < q.nb; ++bi)
        for (int bj = bi; bj < q.nb; ++bj) q.slots = std::max(q.slots, block_slots(q, bi, bj));
    return slab_bytes(q) <= slab_bytes(p) ? q : p;
}

// Workspace of a call: the partial sums, and for FP32 frames behind them the
// count and list of the pairs marked for the direct form (room for every
// pair k < j).
constexpr size_t kListHead = 256;
size_t list_bytes(int K) { return kListHead + (size_t)K * (K - 1) / 2 * sizeof(int2); }
size_t need_bytes(int32_t precision, int K, int T) {
    if (precision == TDSE_F32) return slab_bytes(plan_gram(K, T)) + list_bytes(K);
    return (size_t)plan_of(K, T).ntc * K * K * sizeof(double);
}

}  // namespace

extern "C" tdse_status tdse_dissimilarity_workspace_size(int32_t K, int32_t T, size_t* bytes) {
    if (!bytes || K < 1 || T < 1) return TDSE_ERR_ARG;
    // the larger of the two precisions' needs
    *bytes = std::max(need_bytes(TDSE_F32, K, T), need_bytes(TDSE_F64, K, T));
    return TDSE_OK;
}

namespace {

// The launches of tdse_dissimilarity with its workspace at `ws` (laid out
// as need_bytes says; every entry a kernel reads is written first by an
// earlier one on the stream, so stale contents do no harm).
tdse_status dissim_launch(int32_t precision, const void* frames, int32_t K, int32_t T, int64_t P,
                          const double* weights, double dA, double* out, void* ws, hipStream_t st) {
    double* part = static_cast<double*>(ws);
    if (precision == TDSE_F64) {
        const Plan p = plan_of(K, T);
        DissimArgs a;
        a.frames = frames;
        a.w = weights;
        a.dA = dA;
        a.K = K;
        a.T = T;
        a.P = P;
        a.nb = p.nb;
        a.npb = p.npb;
        a.tpc = p.tpc;
        a.part = part;
        hipLaunchKernelGGL(dissim_kernel<double>, dim3((unsigned)(p.npb * p.ntc)), dim3(256), 0, st, a);
        if (hipGetLastError() != hipSuccess) return TDSE_ERR_DEVICE;
        const unsigned g = (unsigned)std::min<long>(((long)K * K + 255) / 256, 4096);
        hipLaunchKernelGGL(dissim_reduce_kernel, dim3(g), dim3(256), 0, st, static_cast<const double*>(part), p.ntc,
                           (int)K, out);
        return hipGetLastError() == hipSuccess ? TDSE_OK : TDSE_ERR_DEVICE;
    }
    const GramPlan p = plan_gram(K, T);
    char* tail = static_cast<char*>(ws) + slab_bytes(p);
    unsigned* count = reinterpret_cast<unsigned*>(tail);
    int2* list = reinterpret_cast<int2*>(tail + kListHead);
    GramArgs g;
    g.frames = static_cast<const float*>(frames);
    g.w = weights;
    g.dA = dA;
    g.P = P;
    g.p = p;
    // The expansion's rounding error in a frame's d^2 is below about
    // 0.4 P eps64 (|x_k|^2 + |x_j|^2) (sequential sums of P / 8 pixels
    // per lane for the norms, P / 4 matrix steps for the cross term), so
    // an unmarked d^2 is good to 0.4 eps64 / 2^-30 = 5e-8 of itself.
    g.tau = std::ldexp((double)P, -30);
    g.part = part;
    g.count = count;
    const bool vec = P % 4 == 0 && (reinterpret_cast<uintptr_t>(frames) & 15) == 0;
    const dim3 grid((unsigned)p.spans);
    if (vec && P % GPC == 0)
        hipLaunchKernelGGL(dissim_gram_kernel<2>, grid, dim3(GTHREADS), 0, st, g);
    else if (vec)
        hipLaunchKernelGGL(dissim_gram_kernel<1>, grid, dim3(GTHREADS), 0, st, g);
    else
        hipLaunchKernelGGL(dissim_gram_kernel<0>, grid, dim3(GTHREADS), 0, st, g);
    if (hipGetLastError() != hipSuccess) return TDSE_ERR_DEVICE;
    hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)((K + 255) / 256), (unsigned)std::min(K, 65535)),
                       dim3(256), 0, st,
                       static_cast<const double*>(part), p, out, list, count);
    if (hipGetLastError() != hipSuccess) return TDSE_ERR_DEVICE;
    if (K > 1) {
        // usually an empty list: every workgroup reads the count and ends
        const unsigned gp = (unsigned)std::min<long>((long)K * (K - 1) / 2, 1024);
        hipLaunchKernelGGL(dissim_pairs_kernel, dim3(gp), dim3(256), 0, st,
                           static_cast<const float*>(frames), weights, dA, (int)K, (int)T, (long)P,
                           static_cast<const int2*>(list), static_cast<const unsigned*>(count), out);
    }
    return hipGetLastError() == hipSuccess ? TDSE_OK : TDSE_ERR_DEVICE;
}

// Checks shared by both entry points; *need = bytes of partial sums.
tdse_status dissim_check(int32_t precision, const void* frames, int32_t K, int32_t T, int64_t P,
                         const double* weights, double dA, const double* out, size_t* need) {
    if (!frames || !weights || !out || K < 1 || T < 1 || P < 1) return TDSE_ERR_ARG;
    if (precision != TDSE_F32 && precision != TDSE_F64) return TDSE_ERR_ARG;
    if (!(dA > 0)) return TDSE_ERR_ARG;
    const long nwg = precision == TDSE_F32 ? plan_gram(K, T).spans : (long)plan_of(K, T).npb * plan_of(K, T).ntc;
    if (nwg > (1L << 31) - 1) return TDSE_ERR_ARG;
    *need = need_bytes(precision, K, T);
    return TDSE_OK;
}

// Partial sums of tdse_dissimilarity_noalloc: one fixed array per GPU,
// allocated with the code object, never by a call.  Host code must not use
// this name as a device address (on the host it names a stand-in); it uses
// the address hipGetSymbolAddress returns for the current device.
constexpr size_t kNoallocScratchBytes = (size_t)TDSE_DISSIM_NOALLOC_MAX_BYTES;
static __device__ __align__(256) double scratch[kNoallocScratchBytes / sizeof(double)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device.
tdse_status scratch_on_current_device(double** ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return TDSE_ERR_DEVICE;
    if (dev >= kMaxDevices) return TDSE_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TDSE_ERR_DEVICE;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return TDSE_OK;
}

}  // namespace

extern "C" tdse_status tdse_dissimilarity(int32_t precision, const void* frames, int32_t K, int32_t T,
                                          int64_t P, const double* weights, double dA, double* out,
                                          void* workspace, size_t workspace_bytes, void* stream) {
    size_t need = 0;
    const tdse_status st = dissim_check(precision, frames, K, T, P, weights, dA, out, &need);
    if (st != TDSE_OK) return st;
    if (!workspace || workspace_bytes < need) return TDSE_ERR_ARG;
    return dissim_launch(precision, frames, K, T, P, weights, dA, out, workspace,
                         static_cast<hipStream_t>(stream));
}

extern "C" tdse_status tdse_dissimilarity_noalloc(int32_t precision, const void* frames, int32_t K,
                                                  int32_t T, int64_t P, const double* weights, double dA,
                                                  double* out, void* stream) {
    size_t need = 0;
    tdse_status st = dissim_check(precision, frames, K, T, P, weights, dA, out, &need);
    if (st != TDSE_OK) return st;
    if (need > kNoallocScratchBytes) return TDSE_ERR_CAPACITY;
    double* part = nullptr;
    st = scratch_on_current_device(&part);
    if (st != TDSE_OK) return st;
    return dissim_launch(precision, frames, K, T, P, weights, dA, out, part,
                         static_cast<hipStream_t>(stream));
}
