// poisson.hip -- elliptic solver of the pressure projection and of the
// potential (Sec. II): Fourier transform in the two periodic directions,
// then one tridiagonal (Thomas) system across the gap per Fourier mode,
// with zero-flux walls (pressure) or zero wall value (potential).
//
// Data flow for one solve, all FP64:
//   real [j][k][i]  --x R2C-->  half spectrum [j][kx][k] (kx < nx/2+1)
//   --z C2C--> [j][kx][kz]  --Thomas in j per (kx,kz)-->  --z C2C^-1-->
//   --x C2R--> real [j][k][i]
// The x transforms stage their output / input through LDS so that the
// spectrum is written and read in runs of consecutive z lines, and every z
// line is one contiguous run of nz values.
// The FFTs are self-sorting (Stockham) in LDS with radix 8, 4, 2 and 3 stages;
// two real x-lines share one complex transform.
#include <algorithm>
#include <mutex>
#include <set>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace nspnp {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// multiply by -i (forward) or +i (inverse)
__device__ __forceinline__ double2 rot(double2 a, bool inv) {
    return inv ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// In-place length-R DFT of v with kernel exp(-+ 2 pi i / R).
template <int R>
__device__ __forceinline__ void dft_small(double2 *v, bool inv);

template <>
__device__ __forceinline__ void dft_small<2>(double2 *v, bool) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <>
__device__ __forceinline__ void dft_small<4>(double2 *v, bool inv) {
    const double2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const double2 s13 = cadd(v[1], v[3]), d13 = rot(csub(v[1], v[3]), inv);
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
}

// radix 8 as two radix-4 DFTs of the even and odd inputs joined by the
// eighth roots of unity: X_k = E_k + w^k O_k, X_{k+4} = E_k - w^k O_k
template <>
__device__ __forceinline__ void dft_small<8>(double2 *v, bool inv) {
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft_small<4>(e, inv);
    dft_small<4>(o, inv);
    const double c = 0.70710678118654752440;  // cos(pi / 4)
    const double2 w1 = make_double2(c, inv ? c : -c), w3 = make_double2(-c, inv ? c : -c);
    const double2 t1 = cmul(o[1], w1), t2 = rot(o[2], inv), t3 = cmul(o[3], w3);
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], t1);
    v[5] = csub(e[1], t1);
    v[2] = cadd(e[2], t2);
    v[6] = csub(e[2], t2);
    v[3] = cadd(e[3], t3);
    v[7] = csub(e[3], t3);
}

// kOwn: the products with sin(2 pi / 3) are rounded on their own (where the
// direction is a run-time value the compiler cannot fuse them into the sums;
// a kernel with a fixed direction that has to agree with that asks for it).
__device__ __forceinline__ double2 scale_own(double s, double2 a) {
#pragma clang fp contract(off)
    return make_double2(s * a.x, s * a.y);
}
template <bool kOwn>
__device__ __forceinline__ void dft3(double2 *v, bool inv) {
    const double s3 = 0.86602540378443864676;  // sin(2 pi / 3)
    const double2 t1 = cadd(v[1], v[2]);
    const double2 t2 = csub(v[1], v[2]);
    const double2 m = make_double2(v[0].x - 0.5 * t1.x, v[0].y - 0.5 * t1.y);
    const double2 p = kOwn ? scale_own(s3, t2) : make_double2(s3 * t2.x, s3 * t2.y);
    // -i s3 t2 (forward) / +i s3 t2 (inverse)
    const double2 r = rot(p, inv);
    v[0] = cadd(v[0], t1);
    v[1] = cadd(m, r);
    v[2] = csub(m, r);
}
template <>
__device__ __forceinline__ void dft_small<3>(double2 *v, bool inv) {
    dft3<false>(v, inv);
}

// q = e / d and r = e % d for 0 <= e, d < 2^22 from a float reciprocal
// rd = 1/d (to one unit in the last place): the product is within a unit of
// the true quotient, so one correction step makes the result exact (integer division has no hardware
// instruction on the GPU).
__device__ __forceinline__ void divmod(int e, int d, float rd, int &q, int &r) {
    q = (int)((float)e * rd);
    r = e - q * d;
    if (r < 0) {
        --q;
        r += d;
    } else if (r >= d) {
        ++q;
        r -= d;
    }
}

// Quotient and remainder by a block-uniform divisor: shifts and a mask when
// it is a power of two, else the float-reciprocal divmod (same range).
struct Div {
    int d, sh;
    float rd;
    __device__ explicit Div(int dd) : d(dd), sh(((dd & (dd - 1)) == 0) ? __builtin_ctz((unsigned)dd) : -1),
                                      rd(__builtin_amdgcn_rcpf((float)dd)) {}
    __device__ __forceinline__ void split(int e, int &q, int &r) const {
        if (sh >= 0) {
            q = e >> sh;
            r = e & (d - 1);
        } else {
            divmod(e, d, rd, q, r);
        }
    }
};

// One radix-R Stockham pass over nl lines of length N in LDS; tw holds this
// pass's twiddles exp(-2 pi i r k ts / N) as [r - 1][k] (k < Ns), staged in
// LDS, so the lanes of a wave (consecutive k) read consecutive entries.
template <int R>
__device__ __forceinline__ void stage_pass(const double2 *__restrict__ src, double2 *__restrict__ dst, int N,
                                           int nl, int Ns, const double2 *__restrict__ tw, bool inv, int tid,
                                           int nth) {
    const int NR = N / R;
    const float rNR = 1.0f / (float)NR, rNs = 1.0f / (float)Ns;
    // powers of two (every pass of a 2^a line): shifts and masks instead of
    // the float-reciprocal divmod (block-uniform choice)
    const bool p2 = ((NR & (NR - 1)) | (Ns & (Ns - 1))) == 0;
    const int lNR = __builtin_ctz((unsigned)NR), lNs = __builtin_ctz((unsigned)Ns);
    for (int e = tid; e < nl * NR; e += nth) {
        int line, jb, blk, k;
        if (p2) {
            line = e >> lNR;
            jb = e & (NR - 1);
            blk = jb >> lNs;
            k = jb & (Ns - 1);
        } else {
            divmod(e, NR, rNR, line, jb);
            divmod(jb, Ns, rNs, blk, k);
        }
        const double2 *in = src + line * N;
        double2 *out = dst + line * N;
        double2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = in[jb + r * NR];
#pragma unroll
        for (int r = 1; r < R; ++r) {
            double2 w = tw[(r - 1) * Ns + k];
            if (inv) w.y = -w.y;
            v[r] = cmul(v[r], w);
        }
        dft_small<R>(v, inv);
        const int base = blk * Ns * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r) out[base + r * Ns] = v[r];
    }
}

// nl lines of length N in b0; returns the buffer (0 or 1) holding the result.
// kR8: the plan may hold radix-8 passes (instantiated only for such plans:
// the radix-8 pass's registers would otherwise bound every transform's
// occupancy).
template <bool kR8>
__device__ int lds_fft(double2 *b0, double2 *b1, int N, int nl, const FftPlan &pl, const double2 *tw, bool inv) {
    double2 *src = b0, *dst = b1;
    int which = 0;
    int Ns = 1, off = 0;  // off: this pass's twiddles in the staged table
    for (int s = 0; s < pl.nstages; ++s) {
        const int R = pl.radix[s];
        const double2 *twp = tw + off;
        if (kR8 && R == 8) stage_pass<kR8 ? 8 : 4>(src, dst, N, nl, Ns, twp, inv, threadIdx.x, blockDim.x);
        else if (R == 4) stage_pass<4>(src, dst, N, nl, Ns, twp, inv, threadIdx.x, blockDim.x);
        else if (R == 2) stage_pass<2>(src, dst, N, nl, Ns, twp, inv, threadIdx.x, blockDim.x);
        else stage_pass<3>(src, dst, N, nl, Ns, twp, inv, threadIdx.x, blockDim.x);
        off += Ns * (R - 1);
        __syncthreads();
        double2 *t = src;
        src = dst;
        dst = t;
        which ^= 1;
        Ns *= R;
    }
    return which;
}

// The twiddle table to LDS (before the caller's first barrier).  The table
// is laid out in pass order at init (pass after pass, [r - 1][k]).
__device__ __forceinline__ void stage_twiddles(double2 *s_tw, const double2 *tw, int N) {
    for (int e = threadIdx.x; e < N; e += blockDim.x) s_tw[e] = tw[e];
}

// ---- x direction: real lines <-> half spectra, two lines per transform ----
// The right-hand side of each line is produced while it is loaded: a plain
// FP64 array, the divergence of the staggered velocity (pressure), or the
// charge -(c+ - c-)/(2 lam^2) (potential).
// The line pairs of an x-transform block into LDS (pair p from buf + p ld), as
// (line 2p, line 2p+1) complex values, for one source type S (block-uniform).  Each batch of kXB
// elements per thread issues all of its loads before any value is formed
// (elements past the block or lines past the grid read element 0 of line 0
// and are dropped), so a thread waits for memory once per batch.  Offsets
// within one field fit in 32 bits.
constexpr int kXB = 2;

template <typename T, int S>
__device__ __forceinline__ void r2c_stage(const PoissonSrc &src, const Dims &d, const Tables &tb, double ch,
                                          double sc, double idx, double idz, int64_t pair0, int ppb, double2 *buf,
                                          int ld) {
    const int nx = d.nx, nz = d.nz, M = d.M, n = ppb * nx, bd = (int)blockDim.x;
    const int64_t nlines = (int64_t)M * nz;
    const unsigned upl = (unsigned)d.plane;
    // (line = j nz + k < 512 * 1024 and e < ppb nx: the float-reciprocal
    // divmod is exact for both)
    const Div dnx(nx), dnz(nz);
    for (int e0 = threadIdx.x; e0 < n; e0 += kXB * bd) {
        unsigned q[kXB][2];
        bool ok[kXB][2];
        int jr[kXB][2], kr[kXB][2], ir[kXB];
#pragma unroll
        for (int u = 0; u < kXB; ++u) {
            const int e = e0 + u * bd;
            int p, i;
            dnx.split(e < n ? e : 0, p, i);
            ir[u] = i;
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                const int64_t line = 2 * (pair0 + p) + l;
                ok[u][l] = e < n && line < nlines;
                const int li = ok[u][l] ? (int)line : 0;
                int j, k;
                dnz.split(li, j, k);
                q[u][l] = (unsigned)li * (unsigned)nx + (unsigned)i;
                jr[u][l] = j;
                kr[u][l] = k;
            }
        }
        double val[kXB][2];
        if constexpr (S == SRC_REAL) {
            const double *a = (const double *)src.a;
            double x[kXB][2];
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) x[u][l] = a[q[u][l]];
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) val[u][l] = x[u][l];
        } else if constexpr (S == SRC_CHARGE) {
            const T *cp = (const T *)src.a, *cm = (const T *)src.b;
            T xp[kXB][2], xm[kXB][2];
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) {
                    xp[u][l] = ld_once(cp + q[u][l]);
                    xm[u][l] = ld_once(cm + q[u][l]);
                }
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) val[u][l] = ch * ((double)xp[u][l] - (double)xm[u][l]);
            // wall values g of phi (inhomogeneous Dirichlet data): L_y at the
            // first / last row carries + g / (dn dc), moved to the right side
            if (src.wall) {
#pragma unroll
                for (int u = 0; u < kXB; ++u)
#pragma unroll
                    for (int l = 0; l < 2; ++l) {
                        const int j = jr[u][l];
                        if (j == 0 || j == M - 1) {
                            const unsigned in_plane = q[u][l] - (unsigned)j * upl;
                            const double g = src.wall[(j == 0 ? 0u : upl) + in_plane];
                            val[u][l] -= (j == 0 ? tb.lyc_lo[0] : tb.lyc_up[M - 1]) * g;
                        }
                    }
            }
        } else {
            // divergence: (u_{i+1} - u_i)/dx + (v_{j+1} - v_j)/dy_j + (w_{k+1} - w_k)/dz, times sc
            const T *uu = (const T *)src.a, *vv = (const T *)src.b, *ww = (const T *)src.c;
            T ux[kXB][2], u0[kXB][2], vt[kXB][2], vb[kXB][2], wz[kXB][2], w0[kXB][2];
            double idn[kXB][2];
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) {
                    const unsigned qq = q[u][l];
                    const int j = jr[u][l];
                    const unsigned i = (unsigned)ir[u], k = (unsigned)kr[u][l];
                    const unsigned xp = qq - i + ((i + 1 == (unsigned)nx) ? 0u : i + 1);
                    const unsigned zp = qq + ((k + 1 == (unsigned)nz) ? 0u : k + 1) * (unsigned)nx - k * (unsigned)nx;
                    ux[u][l] = uu[xp];
                    u0[u][l] = uu[qq];
                    vt[u][l] = vv[(j + 1 < M) ? qq + upl : qq];
                    vb[u][l] = vv[qq];
                    wz[u][l] = ww[zp];
                    w0[u][l] = ww[qq];
                    idn[u][l] = tb.idn[j];
                }
#pragma unroll
            for (int u = 0; u < kXB; ++u)
#pragma unroll
                for (int l = 0; l < 2; ++l) {
                    const int j = jr[u][l];
                    const double t = (j + 1 < M) ? (double)vt[u][l] : 0.0;
                    const double b = (j > 0) ? (double)vb[u][l] : 0.0;
                    const double div = ((double)ux[u][l] - (double)u0[u][l]) * idx + (t - b) * idn[u][l] +
                                       ((double)wz[u][l] - (double)w0[u][l]) * idz;
                    val[u][l] = div * sc;
                }
        }
#pragma unroll
        for (int u = 0; u < kXB; ++u) {
            const int e = e0 + u * bd;
            if (e < n) {
                int p, i;
                dnx.split(e, p, i);
                buf[p * ld + i] = make_double2(ok[u][0] ? val[u][0] : 0.0, ok[u][1] ? val[u][1] : 0.0);
            }
        }
    }
}

// Slots of each of the two FFT buffers of an x-transform block; the [kx][line]
// staging of the transposed spectrum stores / loads fits one of them.
__host__ __device__ inline int x_buffer_slots(int nx, int ppb) { return ppb * (nx + 2); }

template <typename T, bool kR8>
__global__ void __launch_bounds__(256) k_fft_x_r2c(Dims d, Tables tb, FftPlan pl, PoissonBatch b,
                                                   const double *clock, double2 *spec, int64_t nspec, int ppb) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y;
    PoissonSrc src = b.src[prob];
    src.a = member_ptr(src.a, b.ms);
    src.b = member_ptr(src.b, b.ms);
    src.c = member_ptr(src.c, b.ms);
    if (src.wall) src.wall = member_ptr(src.wall, b.ms);
    clock = member_ptr(clock, b.ms);
    const double ch = member_ptr(b.phys, b.ms)->ch;
    double2 *out = member_ptr(spec, b.ms) + prob * nspec;
    const int nx = d.nx, nxh = d.nxh;
    const int64_t nlines = (int64_t)d.M * d.nz;
    const int bs = x_buffer_slots(nx, ppb);
    double2 *bf[2] = {sm, sm + bs};
    double2 *s_tw = sm + 2 * bs;
    stage_twiddles(s_tw, tb.twx, nx);
    const double sc = (src.type == SRC_DIV) ? ((src.alp > 0.0) ? 1.0 / (src.alp * clock[1]) : src.fixed) : 0.0;
    const double idx = 1.0 / d.dx, idz = 1.0 / d.dz;
    // XCD-aware block order: the pairs whose spectra share 128-byte lines of a
    // [j][kx][kz] row run on one XCD, so their partial-line stores merge in
    // that XCD's L2 before they reach memory
    const int64_t pair0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * ppb;
    if (src.type == SRC_DIV) r2c_stage<T, SRC_DIV>(src, d, tb, ch, sc, idx, idz, pair0, ppb, bf[0], nx);
    else if (src.type == SRC_CHARGE) r2c_stage<T, SRC_CHARGE>(src, d, tb, ch, sc, idx, idz, pair0, ppb, bf[0], nx);
    else r2c_stage<T, SRC_REAL>(src, d, tb, ch, sc, idx, idz, pair0, ppb, bf[0], nx);
    __syncthreads();
    const int w = lds_fft<kR8>(bf[0], bf[1], nx, ppb, pl, s_tw, false);
    // (offsets from the LDS base rather than bf[w]: a pointer picked from an
    // array at run time loses its address space and becomes a flat access,
    // which would also wait for every vector load in flight)
    const double2 *z = sm + w * bs;
    double2 *o = sm + (1 - w) * bs;  // [kk][line] staging for the transposed store
    const int nl2 = 2 * ppb;
    const Div dnxh(nxh), dnl2(nl2), dnz(d.nz);
    for (int e = threadIdx.x; e < ppb * nxh; e += blockDim.x) {
        int p, kk;
        dnxh.split(e, p, kk);
        const double2 zk = z[p * nx + kk];
        const double2 zc = z[p * nx + (kk == 0 ? 0 : nx - kk)];
        // A = (Z_k + conj(Z_{N-k}))/2, B = (Z_k - conj(Z_{N-k}))/(2i)
        o[kk * nl2 + 2 * p] = make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y - zc.y));
        o[kk * nl2 + 2 * p + 1] = make_double2(0.5 * (zk.y + zc.y), -0.5 * (zk.x - zc.x));
    }
    __syncthreads();
    // spectrum layout [j][kx][kz]: consecutive lines (k) of one kx are contiguous
    for (int e = threadIdx.x; e < nl2 * nxh; e += blockDim.x) {
        int kk, l;
        dnl2.split(e, kk, l);
        const int64_t line = 2 * pair0 + l;
        if (line < nlines) {
            int j, k;
            dnz.split((int)line, j, k);
            out[((int64_t)j * nxh + kk) * d.nz + k] = o[e];
        }
    }
}

// Persistent blocks over tiles of ppb line pairs: the next tile's spectrum
// values (transposed load, whole runs of consecutive lines per kx) are loaded
// into registers while the current tile is transformed in LDS.
constexpr int kCPer = 12;  // prefetched values per thread: 2 ppb (nx/2+1) <= kCPer * 256

template <typename T, bool kR8>
__global__ void __launch_bounds__(256) k_fft_x_c2r(Dims d, Tables tb, FftPlan pl, PoissonBatch b,
                                                   const double2 *spec, int64_t nspec, int ppb) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y;
    const double2 *in = member_ptr(spec, b.ms) + prob * nspec;
    const int nx = d.nx, nxh = d.nxh, nz = d.nz;
    const int64_t nlines = (int64_t)d.M * d.nz;
    const int ntiles = (int)(((nlines + 1) / 2 + ppb - 1) / ppb);
    const int bs = x_buffer_slots(nx, ppb);
    double2 *bf[2] = {sm, sm + bs};
    double2 *s_tw = sm + 2 * bs;
    stage_twiddles(s_tw, tb.twx, nx);
    const int nl2 = 2 * ppb, nst = nl2 * nxh;
    const Div dnl2(nl2), dnz(nz), dnx(nx);
    double2 *o = bf[1];  // [kk][line] staging of the transposed load
    const bool as_state = b.out_state[prob] != 0;
    double *o64 = (double *)member_ptr(b.out[prob], b.ms);
    T *ot = (T *)member_ptr(b.out[prob], b.ms);
    double2 nxt[kCPer];
    auto load = [&](int t) {
        const int64_t l0 = 2 * (int64_t)t * ppb;
#pragma unroll
        for (int q = 0; q < kCPer; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            double2 v = make_double2(0.0, 0.0);
            if (e < nst) {
                int kk, l, j, k;
                dnl2.split(e, kk, l);
                const int64_t line = l0 + l;
                if (line < nlines) {
                    dnz.split((int)line, j, k);
                    v = ld_once(in + ((int64_t)j * nxh + kk) * nz + k);
                }
            }
            nxt[q] = v;
        }
    };
    int t = blockIdx.x;
    if (t < ntiles) load(t);
    for (; t < ntiles; t += gridDim.x) {
        const int64_t pair0 = (int64_t)t * ppb;
#pragma unroll
        for (int q = 0; q < kCPer; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            if (e < nst) o[e] = nxt[q];
        }
        __syncthreads();
        if (t + (int)gridDim.x < ntiles) load(t + gridDim.x);  // lands during the passes
        for (int e = threadIdx.x; e < ppb * nx; e += blockDim.x) {
            int p, kk;
            dnx.split(e, p, kk);
            const bool lower = kk < nxh;
            const int src = lower ? kk : nx - kk;
            double2 A = o[src * nl2 + 2 * p];
            double2 B = o[src * nl2 + 2 * p + 1];
            if (!lower) {  // Hermitian continuation of a real line's spectrum
                A.y = -A.y;
                B.y = -B.y;
            }
            bf[0][e] = make_double2(A.x - B.y, A.y + B.x);  // Z = A + i B
        }
        __syncthreads();
        const double2 *z = sm + lds_fft<kR8>(bf[0], bf[1], nx, ppb, pl, s_tw, true) * bs;  // LDS base offset: no flat access
        for (int e = threadIdx.x; e < ppb * nx; e += blockDim.x) {
            int p, i;
            dnx.split(e, p, i);
            const int64_t la = 2 * (pair0 + p), lb = la + 1;
            const double2 v = z[e];
            if (as_state) {
                if (la < nlines) st_once(ot + la * nx + i, (T)v.x);
                if (lb < nlines) st_once(ot + lb * nx + i, (T)v.y);
            } else {
                if (la < nlines) st_once(o64 + la * nx + i, v.x);
                if (lb < nlines) st_once(o64 + lb * nx + i, v.y);
            }
        }
        __syncthreads();  // o and the result buffer are reused by the next tile
    }
}

// ---- x lines of 64, 128, 256 and 512 points: a wave per line pair, in registers ----
// A block of 4 waves owns 8 consecutive lines (16 of 128 points, 32 of 64); a
// wave transforms one pair (2, 4) with 4 or 8 values per lane, all passes in
// registers (radix 4, for 128 points a last pass of radix 2; radix 8 for 512;
// as make_plan has them) and exchanges within the wave through its own piece
// of LDS, without block barriers.  Each exchange has an index map that keeps
// its writes and reads free of bank conflicts.  The 8 lines make whole
// 128-byte lines of the [j][kx][kz] spectrum.  Butterflies
// and their order are those of the general kernels: the same bit for bit.
// Bound by memory; many independent waves with every load of a line in flight
// beat tiles behind block barriers: 512 x 385 x 512 FP64 forward 1.49 -> 1.03
// ms (5.4 TB/s), inverse 0.95 -> 0.56 ms (5.7 TB/s), mixed 1.14 -> 0.66 and
// 0.93 -> 0.50 ms; 256 x 193 x 256 FP64 165 -> 130 and 106 -> 62 us, 128 x 129
// x 128 36 -> 29 and 30 -> 15 us, 64 x 129 x 256 34 -> 28 and 29 -> 15 us.
// Which product of a complex multiplication is rounded before the fused
// multiply-add is written out, as the general kernels' compilation has it (the
// general kernels leave it to the compiler: one that fuses otherwise there would
// leave the two equal to rounding).
__device__ __forceinline__ double2 twiddle(double2 a, double2 w, bool inv) {
    if (inv) return make_double2(__builtin_fma(a.x, w.x, a.y * w.y), __builtin_fma(a.y, w.x, -(a.x * w.y)));
    return make_double2(__builtin_fma(a.x, w.x, -(a.y * w.y)), __builtin_fma(a.y, w.x, a.x * w.y));
}
// (kZ: the forward z transform's)
template <int R, bool kZ>
__device__ __forceinline__ void wave_dft(double2 *v, bool inv) {
    if constexpr (R == 4) {
        dft_small<4>(v, inv);
    } else {  // as dft_small<8>
        double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft_small<4>(e, inv);
        dft_small<4>(o, inv);
        const double c = 0.70710678118654752440;  // cos(pi / 4)
        double2 t1, t3;
        if (inv) {
            const double m1 = o[1].y * c, m3 = o[3].y * -c;
            t1 = make_double2(__builtin_fma(o[1].x, c, -m1), __builtin_fma(c, o[1].x, m1));
            t3 = make_double2(__builtin_fma(-c, o[3].x, m3), __builtin_fma(c, o[3].x, m3));
        } else {
            const double m1 = (kZ ? o[1].y : o[1].x) * c, m3 = o[3].y * c;
            t1 = kZ ? make_double2(__builtin_fma(o[1].x, c, m1), __builtin_fma(-c, o[1].x, m1))
                    : make_double2(__builtin_fma(c, o[1].y, m1), __builtin_fma(o[1].y, c, -m1));
            t3 = make_double2(__builtin_fma(-c, o[3].x, m3), __builtin_fma(o[3].x, -c, -m3));
        }
        const double2 t2 = rot(o[2], inv);
        v[0] = cadd(e[0], o[0]);
        v[4] = csub(e[0], o[0]);
        v[1] = cadd(e[1], t1);
        v[5] = csub(e[1], t1);
        v[2] = cadd(e[2], t2);
        v[6] = csub(e[2], t2);
        v[3] = cadd(e[3], t3);
        v[7] = csub(e[3], t3);
    }
}

template <int N, bool kZ = false>
struct WaveFft {
    static constexpr int R = N == 512 ? 8 : 4;   // values per lane and radix
    static constexpr int kLanes = N / R;         // lanes of a line or pair
    static constexpr int kPer = 64 / kLanes;     // lines or pairs per wave
    // LDS slots of one pair (64, 128 points: the pairs of a block in different banks)
    static constexpr int kSlots = N == 512 ? 568 : (N == 256 ? 328 : (N == 128 ? 162 : 81));
    // slot of element i on the way from the pass with input stride Ns
    static __device__ __forceinline__ int slot(int i, int Ns) {
        if (Ns == 1) return i + (i >> 4);
        if (R == 4) return Ns == 4 ? i + 4 * (i >> 4) : i;
        return i + 8 * (i >> 6);
    }
    // v[r] holds element lane + kLanes r before and after; z: the pair's slots
    static __device__ __forceinline__ void run(double2 *v, double2 *z, const double2 *__restrict__ tw, int lane,
                                               bool inv) {
        wave_dft<R, kZ>(v, inv);  // (the first pass's twiddles are 1)
        int off = R - 1;
#pragma unroll
        for (int Ns = R; Ns < N; Ns *= R) {
            const bool two = Ns * R > N;  // 128 points: a last pass of radix 2, two butterflies a lane
            const int pNs = Ns / R, blk = lane / pNs, pk = lane % pNs, k = lane % Ns;
            double2 w[R];
#pragma unroll
            for (int r = 1; r < R; ++r) w[r] = two ? tw[off + lane + (r & 1) * kLanes] : tw[off + (r - 1) * Ns + k];
            off += Ns * (R - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) z[slot(blk * Ns + pk + r * pNs, pNs)] = v[r];
            wave_sync();
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = z[slot(lane + kLanes * r, pNs)];
            wave_sync();
            if (two) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const double2 c = twiddle(v[r + 2], w[r + 2], inv);
                    v[r + 2] = csub(v[r], c);
                    v[r] = cadd(v[r], c);
                }
            } else {
#pragma unroll
                for (int r = 1; r < R; ++r) v[r] = twiddle(v[r], w[r], inv);
                wave_dft<R, kZ>(v, inv);
            }
        }
    }
};

// The right-hand side of lines (j, k) and (j, k + 1) at x = lane + 64 r, r in
// [r0, r0 + B), all loads ahead of the arithmetic (that of r2c_stage).  j and
// k are wave-uniform.
template <typename T, int S, int N, int B>
__device__ __forceinline__ void line_rhs(const PoissonSrc &src, const Dims &d, const Tables &tb, double ch, double sc,
                                         double idx, double idz, int j, int k, int lane, int r0, double2 *v) {
    const int M = d.M, nz = d.nz;
    const size_t upl = (size_t)d.plane, q0 = (size_t)j * upl + (size_t)k * N;
    unsigned i[B];
#pragma unroll
    for (int t = 0; t < B; ++t) i[t] = (unsigned)(lane + 64 * (r0 + t));
    double val[B][2];
    if constexpr (S == SRC_REAL) {
        const double *a = (const double *)src.a + q0;
#pragma unroll
        for (int t = 0; t < B; ++t) {
            val[t][0] = a[i[t]];
            val[t][1] = (a + N)[i[t]];
        }
    } else if constexpr (S == SRC_CHARGE) {
        const T *cp = (const T *)src.a + q0, *cm = (const T *)src.b + q0;
        T xp[B][2], xm[B][2];
#pragma unroll
        for (int t = 0; t < B; ++t)
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                xp[t][l] = ld_once(cp + l * N + i[t]);
                xm[t][l] = ld_once(cm + l * N + i[t]);
            }
#pragma unroll
        for (int t = 0; t < B; ++t)
#pragma unroll
            for (int l = 0; l < 2; ++l) val[t][l] = ch * ((double)xp[t][l] - (double)xm[t][l]);
        // wall values g of phi, as in r2c_stage
        if (src.wall && (j == 0 || j == M - 1)) {
            const double *gw = src.wall + (j == 0 ? 0 : upl) + (size_t)k * N;
#pragma unroll
            for (int t = 0; t < B; ++t)
#pragma unroll
                for (int l = 0; l < 2; ++l) {
                    const double g = (gw + l * N)[i[t]];
                    val[t][l] -= (j == 0 ? tb.lyc_lo[0] : tb.lyc_up[M - 1]) * g;
                }
        }
    } else {
        const T *u0 = (const T *)src.a + q0, *v0 = (const T *)src.b + q0, *w0 = (const T *)src.c + q0;
        const T *w2 = (k + 2 == nz) ? (const T *)src.c + (size_t)j * upl : w0 + 2 * N;  // line k + 2
        const bool has_up = j + 1 < M, has_dn = j > 0;
        const T *v1 = has_up ? v0 + upl : v0;
        T ux[B][2], uc[B][2], vt[B][2], vb[B][2], wc[B][3];
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const unsigned ip = (i[t] + 1 == (unsigned)N) ? 0u : i[t] + 1;
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                ux[t][l] = (u0 + l * N)[ip];
                uc[t][l] = (u0 + l * N)[i[t]];
                vt[t][l] = (v1 + l * N)[i[t]];
                vb[t][l] = (v0 + l * N)[i[t]];
                wc[t][l] = (w0 + l * N)[i[t]];
            }
            wc[t][2] = w2[i[t]];
        }
        const double idn = uniform_load(tb.idn, j);
#pragma unroll
        for (int t = 0; t < B; ++t)
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                const double tt = has_up ? (double)vt[t][l] : 0.0;
                const double bb = has_dn ? (double)vb[t][l] : 0.0;
                const double div = ((double)ux[t][l] - (double)uc[t][l]) * idx + (tt - bb) * idn +
                                   ((double)wc[t][l + 1] - (double)wc[t][l]) * idz;
                val[t][l] = div * sc;
            }
    }
#pragma unroll
    for (int t = 0; t < B; ++t) v[r0 + t] = make_double2(val[t][0], val[t][1]);
}

template <typename T, int N>
__global__ void __launch_bounds__(256) k_lines_r2c(Dims d, Tables tb, PoissonBatch b, const double *clock,
                                                   double2 *spec, int64_t nspec) {
    using F = WaveFft<N>;
    constexpr int nxh = N / 2 + 1, kLines = 8 * F::kPer, B = F::kPer == 1 ? 4 : N / 64;
    __shared__ double2 s_z[4 * F::kPer * F::kSlots];
    const int prob = blockIdx.y;
    PoissonSrc src = b.src[prob];
    src.a = member_ptr(src.a, b.ms);
    src.b = member_ptr(src.b, b.ms);
    src.c = member_ptr(src.c, b.ms);
    if (src.wall) src.wall = member_ptr(src.wall, b.ms);
    clock = member_ptr(clock, b.ms);
    const double ch = member_ptr(b.phys, b.ms)->ch;
    double2 *out = member_ptr(spec, b.ms) + prob * nspec;
    const int nz = d.nz, nlines = d.M * nz;
    const int line0 = (int)xcd_tile(blockIdx.x, gridDim.x) * kLines;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const double sc = (src.type == SRC_DIV) ? ((src.alp > 0.0) ? 1.0 / (src.alp * clock[1]) : src.fixed) : 0.0;
    const double idx = 1.0 / d.dx, idz = 1.0 / d.dz;
    // right-hand side of the wave's pair h, elements lane + 64 r
    auto rhs = [&](int h, int r0, double2 *v) {
        // (a pair past the last line repeats the last one and is not stored)
        const int first = line0 + 2 * (wave * F::kPer + h), line = first < nlines ? first : nlines - 2;
        const int j = line / nz, k = line - j * nz;
        if (src.type == SRC_DIV) line_rhs<T, SRC_DIV, N, B>(src, d, tb, ch, sc, idx, idz, j, k, lane, r0, v);
        else if (src.type == SRC_CHARGE) line_rhs<T, SRC_CHARGE, N, B>(src, d, tb, ch, sc, idx, idz, j, k, lane, r0, v);
        else line_rhs<T, SRC_REAL, N, B>(src, d, tb, ch, sc, idx, idz, j, k, lane, r0, v);
    };
    {
        const int l = lane % F::kLanes;
        double2 *zw = s_z + wave * F::kPer * F::kSlots, *z = zw + lane / F::kLanes * F::kSlots;
        double2 v[F::R];
        if constexpr (F::kPer == 1) {
#pragma unroll
            for (int r0 = 0; r0 < F::R; r0 += B) rhs(0, r0, v);
        } else {  // by the whole wave, pair by pair, and through LDS to each pair's lanes
#pragma unroll
            for (int h = 0; h < F::kPer; ++h) rhs(h, 0, v + h * B);
#pragma unroll
            for (int h = 0; h < F::kPer; ++h)
#pragma unroll
                for (int t = 0; t < B; ++t) zw[h * F::kSlots + lane + 64 * t] = v[h * B + t];
            wave_sync();
#pragma unroll
            for (int r = 0; r < F::R; ++r) v[r] = z[l + F::kLanes * r];
            wave_sync();
        }
        F::run(v, z, tb.twx, l, false);
#pragma unroll
        for (int r = 0; r < F::R; ++r) z[l + F::kLanes * r] = v[r];
    }
    __syncthreads();
    // A = (Z_k + conj(Z_{N-k}))/2 for the even lines, B = (Z_k - conj(Z_{N-k}))/(2i)
    // for the odd ones; a thread keeps its line
    const int l = threadIdx.x % kLines, line = line0 + l;
    if (line >= nlines) return;
    const int j = line / nz, k = line - j * nz;
    const double2 *z = s_z + (l >> 1) * F::kSlots;
    double2 *o = out + (int64_t)j * nxh * nz + k;
#pragma unroll 4
    for (int kk = threadIdx.x / kLines; kk < nxh; kk += 256 / kLines) {
        const double2 zk = z[kk], zc = z[kk == 0 ? 0 : N - kk];
        o[(int64_t)kk * nz] = (l & 1) ? make_double2(0.5 * (zk.y + zc.y), -0.5 * (zk.x - zc.x))
                                      : make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y - zc.y));
    }
}

template <typename T, int N>
__global__ void __launch_bounds__(256) k_lines_c2r(Dims d, Tables tb, PoissonBatch b, const double2 *spec,
                                                   int64_t nspec) {
    using F = WaveFft<N>;
    constexpr int nxh = N / 2 + 1, kLines = 8 * F::kPer, kRows = 256 / kLines, kIt = (nxh + kRows - 1) / kRows;
    constexpr int kLine = N == 128 ? 65 : (N == 64 ? 40 : N / 2 + 2);  // (the lines of a pair in different banks)
    __shared__ double2 s_z[4 * F::kPer * F::kSlots];
    const int prob = blockIdx.y;
    const double2 *in = member_ptr(spec, b.ms) + prob * nspec;
    const int nz = d.nz, nlines = d.M * nz;
    const int line0 = (int)xcd_tile(blockIdx.x, gridDim.x) * kLines;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    {
        const int l = threadIdx.x % kLines, line = line0 + l < nlines ? line0 + l : nlines - 1;
        const int j = line / nz, k = line - j * nz, k0 = threadIdx.x / kLines;
        const double2 *p = in + (int64_t)j * nxh * nz + k;
        double2 v[kIt];
#pragma unroll
        for (int t = 0; t < kIt; ++t) v[t] = ld_once(p + (int64_t)(k0 + kRows * t < nxh ? k0 + kRows * t : nxh - 1) * nz);
        double2 *o = s_z + (l >> 1) * F::kSlots + (l & 1) * kLine;
#pragma unroll
        for (int t = 0; t < kIt; ++t)
            if (k0 + kRows * t < nxh) o[k0 + kRows * t] = v[t];
    }
    __syncthreads();
    const int pair = wave * F::kPer + lane / F::kLanes, l = lane % F::kLanes;
    if (line0 + 2 * wave * F::kPer >= nlines) return;
    double2 *z = s_z + pair * F::kSlots;
    double2 v[F::R];
#pragma unroll
    for (int r = 0; r < F::R; ++r) {
        const int kk = l + F::kLanes * r;
        const bool lower = kk < nxh;
        const int src = lower ? kk : N - kk;
        double2 A = z[src], B = z[kLine + src];
        if (!lower) {  // Hermitian continuation of a real line's spectrum
            A.y = -A.y;
            B.y = -B.y;
        }
        v[r] = make_double2(A.x - B.y, A.y + B.x);  // Z = A + i B
    }
    wave_sync();
    F::run(v, z, tb.twx, l, true);
    if (line0 + 2 * pair >= nlines) return;
    const int64_t la = (int64_t)(line0 + 2 * pair) * N;
    const bool as_state = b.out_state[prob] != 0;
    double *o64 = (double *)member_ptr(b.out[prob], b.ms) + la;
    T *ot = (T *)member_ptr(b.out[prob], b.ms) + la;
#pragma unroll
    for (int r = 0; r < F::R; ++r) {
        const int i = l + F::kLanes * r;
        if (as_state) {
            st_once(ot + i, (T)v[r].x);
            st_once(ot + N + i, (T)v[r].y);
        } else {
            st_once(o64 + i, v[r].x);
            st_once(o64 + N + i, v[r].y);
        }
    }
}

// ---- z direction: contiguous complex lines, tiles of tk lines ----
// Lines of 64 to 512 points, powers of two: a wave per line (2, 4 lines of 128,
// 64 points), in registers (WaveFft).
// 256 x 193 x 256 75 -> 62 us (6.5 TB/s, the spectra partly in the last-level
// cache), 512 x 385 x 512 0.69 -> 0.60 ms forward, 0.66 -> 0.59 ms inverse,
// 128 x 129 x 128 20 -> 14 us, 256 x 129 x 64 18 -> 14 us.
template <int N, bool kInv>
__global__ void __launch_bounds__(256) k_lines_z(Dims d, const double2 *__restrict__ tw, double2 *spec, int64_t nspec,
                                                 size_t ms) {
    using F = WaveFft<N, true>;
    __shared__ double2 s_z[4 * F::kPer * F::kSlots];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int mine = wave * F::kPer + lane / F::kLanes, l = lane % F::kLanes;
    const int64_t nlines = (int64_t)d.M * d.nxh, line0 = (int64_t)blockIdx.x * (4 * F::kPer);  // (j, kx)
    if (line0 + wave * F::kPer >= nlines) return;
    const bool in = F::kPer == 1 || line0 + mine < nlines;
    double2 *p = member_ptr(spec, ms) + blockIdx.y * nspec + (in ? line0 + mine : nlines - 1) * N + l;
    double2 v[F::R];
#pragma unroll
    for (int r = 0; r < F::R; ++r) v[r] = p[F::kLanes * r];
    F::run(v, s_z + mine * F::kSlots, tw, l, kInv);
    if (!in) return;
#pragma unroll
    for (int r = 0; r < F::R; ++r) p[F::kLanes * r] = v[r];
}

// Other lengths.
// Persistent blocks: each block loops over tiles (j, kx0..kx0+tk-1) of its
// problem and member; the next tile's values are loaded into registers while
// the current tile is transformed in LDS, so the HBM latency overlaps the
// FFT passes.  kPer values per thread cover tk * nz <= kPer * 256 points.
constexpr int kZPer = 8;

template <bool kR8>
__global__ void __launch_bounds__(256) k_fft_z(Dims d, FftPlan pl, const double2 *tw, double2 *spec, int64_t nspec,
                                               int tk, int inverse, size_t ms) {
    extern __shared__ double2 sm[];
    double2 *data = member_ptr(spec, ms) + blockIdx.y * nspec;
    const int nz = d.nz, nxh = d.nxh;
    const int tiles_x = (nxh + tk - 1) / tk;
    const int ntiles = d.M * tiles_x;
    const int pts = tk * nz;
    double2 *bf[2] = {sm, sm + tk * nz};
    double2 *s_tw = sm + 2 * tk * nz;
    stage_twiddles(s_tw, tw, nz);
    double2 nxt[kZPer];
    auto tile_base = [&](int t, int &nt) -> double2 * {
        const int j = t / tiles_x;
        const int kx0 = (t - j * tiles_x) * tk;
        nt = (nxh - kx0 < tk) ? nxh - kx0 : tk;  // lines in this tile
        // lines (j, kx) are contiguous runs of nz values: the tile is one block of memory
        return data + ((int64_t)j * nxh + kx0) * nz;
    };
    auto load = [&](int t) {
        int nt;
        const double2 *base = tile_base(t, nt);
#pragma unroll
        for (int q = 0; q < kZPer; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            nxt[q] = (e < nt * nz) ? base[e] : make_double2(0.0, 0.0);
        }
    };
    int t = blockIdx.x;
    if (t < ntiles) load(t);
    for (; t < ntiles; t += gridDim.x) {
        int nt;
        double2 *base = tile_base(t, nt);
#pragma unroll
        for (int q = 0; q < kZPer; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            if (e < pts) bf[0][e] = nxt[q];
        }
        __syncthreads();
        if (t + (int)gridDim.x < ntiles) load(t + gridDim.x);  // lands during the passes
        const double2 *z = sm + lds_fft<kR8>(bf[0], bf[1], nz, tk, pl, s_tw, inverse != 0) * (tk * nz);  // no flat access
        for (int e = threadIdx.x; e < nt * nz; e += blockDim.x) base[e] = z[e];
        __syncthreads();  // bf[0] and the result buffer are reused by the next tile
    }
}

// ---- whole planes: x and z transforms of one row in one kernel ----
// A block owns one row j of one problem and member, all of its nx x nz plane:
// forward, the x transforms of the line pairs, the half spectrum and its z
// transforms; inverse, the same backwards.  Each saves a pass over the
// spectrum (read and write) and a launch.  The first and the last pass of the
// spectrum's or the solution's own direction run along the lines and take
// their values from memory or store them there; the half spectrum is split,
// or joined, as the first pass of the second direction reads it: 5 or 6 trips
// through LDS for 64 x 64.  The passes between run across the lines, whose LDS
// stride is odd in 16-byte units: free of bank conflicts, and a wave's
// twiddles are one or two entries.  The butterflies and their order are those of the separate
// kernels, so the results are the same bit for bit.
// 32 members of 64 x 65 x 64 and of 48 x 49 x 48, mixed form: forward 102 and
// 48 us (3.0 TB/s: LDS passes and their latency), inverse 79 and 37; 119 and
// 60, 87 and 43 with every pass through LDS and the right-hand side formed
// element by element; a 32 x 33 x 32 grid in FP64 7.1 and 6.3 us (10.8 and
// 7.3; two kernels each way 12 and 11: latency and launches).
struct PlanePass {
    int N, nl, Ns;     // points per line, lines, product of the radices before
    bool first, last;
};

// ld(line, jb, NR, v) and st(line, base, Ns, v) move elements jb + r NR and
// base + r Ns of a line.  kOwn: as k_fft_z, whose direction is a run-time
// value, see dft3.
template <int R, bool kOwn, class Ld, class St>
__device__ __forceinline__ void plane_pass(const PlanePass &p, bool along, const double2 *__restrict__ tw, bool inv,
                                           const Ld &ld, const St &st) {
    const int NR = p.N / R;
    const Div by(along ? NR : p.nl), dNs(p.Ns);
    for (int e = threadIdx.x; e < p.nl * NR; e += blockDim.x) {
        int hi, lo, blk, k;
        by.split(e, hi, lo);
        const int line = along ? hi : lo, jb = along ? lo : hi;
        dNs.split(jb, blk, k);
        double2 v[R];
        ld(line, jb, NR, v);
        if (!p.first) {  // (the first pass's twiddles are 1)
#pragma unroll
            for (int r = 1; r < R; ++r) v[r] = twiddle(v[r], tw[(r - 1) * p.Ns + k], inv);
        }
        if constexpr (R == 3) dft3<kOwn>(v, inv);
        else dft_small<R>(v, inv);
        st(line, __mul24(blk, p.Ns * R) + k, p.Ns, v);
    }
}

// Position of element i of a line between the first pass and the second: the
// first pass of radix 4, along the line, writes every fourth element.
__device__ __forceinline__ int plane_slot(int i, int sw) { return i ^ ((i >> 4) & sw); }

// nl lines of length N (LDS stride ld), buffers b0 and b1 in turn, the first
// pass writes b0; returns the buffer (0 or 1) of the last pass.
// kIn: the first pass runs along the lines, kOut: the last, and stores through
// fst instead of LDS (no barrier after it).
template <bool kOwn, bool kIn, bool kOut, class Ld, class St>
__device__ __forceinline__ int plane_fft(double2 *b0, double2 *b1, int N, int nl, int ld, const FftPlan &pl,
                                         const double2 *tw, bool inv, const Ld &fld, const St &fst) {
    double2 *dst = b0, *src = b1;
    int which = 0, off = 0;
    const int sw = (kIn && pl.nstages > 1 && pl.radix[0] == 4) ? 3 : 0;
    PlanePass p{N, nl, 1, true, false};
    for (int s = 0; s < pl.nstages; ++s) {
        const int R = pl.radix[s];
        p.first = s == 0;
        p.last = s + 1 == pl.nstages;
        const int swl = s == 1 ? sw : 0, sws = s == 0 ? sw : 0;
        auto go = [&](auto rr) {
            constexpr int RR = decltype(rr)::value;
            plane_pass<RR, kOwn>(
                p, (kIn && p.first) || (kOut && p.last), tw + off, inv,
                [&](int line, int jb, int NR, double2(&v)[RR]) {
                    if (p.first) {
                        fld(line, jb, NR, v);
                    } else {
                        const double2 *in = src + __mul24(line, ld);
#pragma unroll
                        for (int r = 0; r < RR; ++r) v[r] = in[plane_slot(jb + r * NR, swl)];
                    }
                },
                [&](int line, int base, int Ns, const double2(&v)[RR]) {
                    if (kOut && p.last) {
                        fst(line, base, Ns, v);
                    } else {
                        double2 *out = dst + __mul24(line, ld);
#pragma unroll
                        for (int r = 0; r < RR; ++r) out[plane_slot(base + r * Ns, sws)] = v[r];
                    }
                });
        };
        if (R == 4) go(std::integral_constant<int, 4>{});
        else if (R == 2) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 3>{});
        off += p.Ns * (R - 1);
        p.Ns *= R;
        if (kOut && p.last) break;
        __syncthreads();
        double2 *t = src;
        src = dst;
        dst = t;
        which ^= 1;
    }
    return which ^ 1;
}

// An element of a plane: a block-uniform base and an offset of 32 bits in
// bytes, which the loads and stores take as they are.
template <typename P>
__device__ __forceinline__ P *in_plane(P *base, unsigned i) {
    using C = std::conditional_t<std::is_const_v<P>, const char, char>;
    return (P *)((C *)base + (size_t)(i * (unsigned)sizeof(P)));
}

// The right-hand side of row j (that of r2c_stage) into LDS as line pairs, V
// neighbouring elements of both lines of a pair per thread and load (the
// state's fields and, nx being even, their lines are aligned to 2 elements,
// and to 4 where nx is a multiple of 4).
template <typename T, int S, int V>
__device__ __forceinline__ void plane_rhs(const PoissonSrc &src, const Dims &d, const Tables &tb, double ch, double sc,
                                          double idx, double idz, int j, double2 *buf, int ld) {
    using TV = T __attribute__((ext_vector_type(V)));
    const int M = d.M, nz = d.nz;
    const unsigned un = (unsigned)d.nx;
    const size_t upl = (size_t)d.plane, row = (size_t)j * upl;
    const Div dv(d.nx / V);
    for (int e = threadIdx.x; e < nz / 2 * (d.nx / V); e += blockDim.x) {
        int p, i;
        dv.split(e, p, i);
        i *= V;
        const unsigned o0 = 2u * (unsigned)__mul24(p, d.nx) + (unsigned)i, o[2] = {o0, o0 + un};
        double val[V][2];
        if constexpr (S == SRC_REAL) {
            const double *a = (const double *)src.a + row;
#pragma unroll
            for (int l = 0; l < 2; ++l)
#pragma unroll
                for (int t = 0; t < V; ++t) val[t][l] = *in_plane(a, o[l] + t);
        } else if constexpr (S == SRC_CHARGE) {
            const T *cp = (const T *)src.a + row, *cm = (const T *)src.b + row;
            TV xp[2], xm[2];
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                xp[l] = ld_once((const TV *)in_plane(cp, o[l]));
                xm[l] = ld_once((const TV *)in_plane(cm, o[l]));
            }
#pragma unroll
            for (int l = 0; l < 2; ++l)
#pragma unroll
                for (int t = 0; t < V; ++t) val[t][l] = ch * ((double)xp[l][t] - (double)xm[l][t]);
            if (src.wall && (j == 0 || j == M - 1)) {  // wall values g of phi
                const double *gw = src.wall + (j == 0 ? 0 : upl);
#pragma unroll
                for (int l = 0; l < 2; ++l)
#pragma unroll
                    for (int t = 0; t < V; ++t) {
                        const double g = *in_plane(gw, o[l] + t);
                        val[t][l] -= (j == 0 ? tb.lyc_lo[0] : tb.lyc_up[M - 1]) * g;
                    }
            }
        } else {
            const T *u0 = (const T *)src.a + row, *v0 = (const T *)src.b + row, *w0 = (const T *)src.c + row;
            const bool has_up = j + 1 < M, has_dn = j > 0;
            const T *v1 = has_up ? v0 + upl : v0;
            const unsigned ip = (unsigned)i + V == un ? 0u : (unsigned)i + V;  // the element after the last
            const unsigned o2 = (2 * p + 2 == nz) ? (unsigned)i : o[1] + un;   // line 2p + 2
            TV uc[2], vt[2], vb[2], wc[3];
            T un1[2];
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                uc[l] = *(const TV *)in_plane(u0, o[l]);
                un1[l] = *in_plane(u0, o[l] - (unsigned)i + ip);
                vt[l] = *(const TV *)in_plane(v1, o[l]);
                vb[l] = *(const TV *)in_plane(v0, o[l]);
                wc[l] = *(const TV *)in_plane(w0, o[l]);
            }
            wc[2] = *(const TV *)in_plane(w0, o2);
            const double idn = uniform_load(tb.idn, j);
#pragma unroll
            for (int l = 0; l < 2; ++l)
#pragma unroll
                for (int t = 0; t < V; ++t) {
                    const T ux = t + 1 < V ? uc[l][t + 1 < V ? t + 1 : 0] : un1[l];
                    const double tt = has_up ? (double)vt[l][t] : 0.0;
                    const double bb = has_dn ? (double)vb[l][t] : 0.0;
                    const double div = ((double)ux - (double)uc[l][t]) * idx + (tt - bb) * idn +
                                       ((double)wc[l + 1][t] - (double)wc[l][t]) * idz;
                    val[t][l] = div * sc;
                }
        }
#pragma unroll
        for (int t = 0; t < V; ++t) buf[__mul24(p, ld) + i + t] = make_double2(val[t][0], val[t][1]);
    }
}

// LDS slots of one of the two buffers: the line pairs or the half spectrum.
__host__ __device__ inline int plane_slots(int nx, int nz) {
    const int a = nz / 2 * (nx + 1), b = (nx / 2 + 1) * (nz + 1);
    return a > b ? a : b;
}
inline size_t plane_lds(int nx, int nz) { return (2 * (size_t)plane_slots(nx, nz) + nx + nz) * sizeof(double2); }

template <typename T>
__global__ void __launch_bounds__(1024) k_plane_fwd(Dims d, Tables tb, FftPlan plx, FftPlan plz, PoissonBatch b,
                                                    const double *clock, double2 *spec, int64_t nspec) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y;
    PoissonSrc src = b.src[prob];
    src.a = member_ptr(src.a, b.ms);
    src.b = member_ptr(src.b, b.ms);
    src.c = member_ptr(src.c, b.ms);
    if (src.wall) src.wall = member_ptr(src.wall, b.ms);
    clock = member_ptr(clock, b.ms);
    const double ch = member_ptr(b.phys, b.ms)->ch;
    const int nx = d.nx, nz = d.nz, nxh = d.nxh, np = nz / 2, ldx = nx + 1, ldz = nz + 1;
    const int j = (int)xcd_tile(blockIdx.x, gridDim.x);  // neighbouring rows share an L2
    double2 *out = member_ptr(spec, b.ms) + prob * nspec + (int64_t)j * nxh * nz;
    const int bs = plane_slots(nx, nz);
    double2 *s_twx = sm + 2 * bs, *s_twz = s_twx + nx;
    stage_twiddles(s_twx, tb.twx, nx);
    stage_twiddles(s_twz, tb.twz, nz);
    const double sc = (src.type == SRC_DIV) ? ((src.alp > 0.0) ? 1.0 / (src.alp * clock[1]) : src.fixed) : 0.0;
    const double idx = 1.0 / d.dx, idz = 1.0 / d.dz;
    if (src.type == SRC_REAL) plane_rhs<T, SRC_REAL, 1>(src, d, tb, ch, sc, idx, idz, j, sm + bs, ldx);
    else if (sizeof(T) == 4 && (nx & 3) == 0) {
        if (src.type == SRC_DIV) plane_rhs<T, SRC_DIV, 4>(src, d, tb, ch, sc, idx, idz, j, sm + bs, ldx);
        else plane_rhs<T, SRC_CHARGE, 4>(src, d, tb, ch, sc, idx, idz, j, sm + bs, ldx);
    } else {
        if (src.type == SRC_DIV) plane_rhs<T, SRC_DIV, 2>(src, d, tb, ch, sc, idx, idz, j, sm + bs, ldx);
        else plane_rhs<T, SRC_CHARGE, 2>(src, d, tb, ch, sc, idx, idz, j, sm + bs, ldx);
    }
    __syncthreads();
    const double2 *f = sm + bs;
    const int w = plane_fft<false, false, false>(
        sm, sm + bs, nx, np, ldx, plx, s_twx, false,
        [&](int p, int jb, int NR, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = f[__mul24(p, ldx) + jb + r * NR];
        },
        [](int, int, int, auto &) {});
    const double2 *z = sm + w * bs;
    plane_fft<true, false, true>(
        sm + (1 - w) * bs, sm + w * bs, nz, nxh, ldz, plz, s_twz, false,
        [&](int kk, int jb, int NR, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
            const int kc = kk == 0 ? 0 : nx - kk;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // A = (Z_k + conj(Z_{N-k}))/2 for the even lines, B = (Z_k - conj(Z_{N-k}))/(2i)
                // for the odd ones
                const int k = jb + r * NR;
                const double2 zk = z[__mul24(k >> 1, ldx) + kk], zc = z[__mul24(k >> 1, ldx) + kc];
                v[r] = (k & 1) ? make_double2(0.5 * (zk.y + zc.y), -0.5 * (zk.x - zc.x))
                               : make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y - zc.y));
            }
        },
        [&](int kk, int base, int Ns, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
#pragma unroll
            for (int r = 0; r < R; ++r) *in_plane(out, (unsigned)(__mul24(kk, nz) + base + r * Ns)) = v[r];
        });
}

template <typename T>
__global__ void __launch_bounds__(1024) k_plane_inv(Dims d, Tables tb, FftPlan plx, FftPlan plz, PoissonBatch b,
                                                    const double2 *spec, int64_t nspec) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y;
    const int nx = d.nx, nz = d.nz, nxh = d.nxh, np = nz / 2, ldx = nx + 1, ldz = nz + 1;
    const int j = (int)xcd_tile(blockIdx.x, gridDim.x);
    const double2 *in = member_ptr(spec, b.ms) + prob * nspec + (int64_t)j * nxh * nz;
    const int bs = plane_slots(nx, nz);
    double2 *s_twx = sm + 2 * bs, *s_twz = s_twx + nx;
    stage_twiddles(s_twx, tb.twx, nx);
    stage_twiddles(s_twz, tb.twz, nz);
    const int w = plane_fft<true, true, false>(
        sm, sm + bs, nz, nxh, ldz, plz, s_twz, true,
        [&](int kk, int jb, int NR, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = ld_once(in_plane(in, (unsigned)(__mul24(kk, nz) + jb + r * NR)));
        },
        [](int, int, int, auto &) {});
    const double2 *o = sm + w * bs;
    const bool as_state = b.out_state[prob] != 0;
    double *o64 = (double *)member_ptr(b.out[prob], b.ms) + (int64_t)j * d.plane;
    T *ot = (T *)member_ptr(b.out[prob], b.ms) + (int64_t)j * d.plane;
    plane_fft<false, false, true>(
        sm + (1 - w) * bs, sm + w * bs, nx, np, ldx, plx, s_twx, true,
        [&](int p, int jb, int NR, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int kk = jb + r * NR;
                const bool lower = kk < nxh;
                const double2 *q = o + __mul24(lower ? kk : nx - kk, ldz) + 2 * p;
                double2 A = q[0], B = q[1];
                if (!lower) {  // Hermitian continuation of a real line's spectrum
                    A.y = -A.y;
                    B.y = -B.y;
                }
                v[r] = make_double2(A.x - B.y, A.y + B.x);  // Z = A + i B
            }
        },
        [&](int p, int base, int Ns, auto &v) {
            constexpr int R = (int)(sizeof(v) / sizeof(v[0]));
            const unsigned q = 2u * (unsigned)__mul24(p, nx) + (unsigned)base;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned qa = q + (unsigned)(r * Ns), qb = qa + (unsigned)nx;
                if (as_state) {
                    st_once(in_plane(ot, qa), (T)v[r].x);
                    st_once(in_plane(ot, qb), (T)v[r].y);
                } else {
                    st_once(in_plane(o64, qa), v[r].x);
                    st_once(in_plane(o64, qb), v[r].y);
                }
            }
        });
}

// Whole planes where two blocks fit a CU's LDS (64 x 64: 70 KB a block).
inline bool plane_fits(const nspnp_state *s) {
    return plane_lds(s->d.nx, s->d.nz) <= std::min((size_t)80 << 10, (size_t)s->lds_max);
}
// One butterfly per thread of the pass that has the most of them.
inline unsigned plane_threads(const nspnp_state *s) {
    int work = 64;
    for (int q = 0; q < s->planx.nstages; ++q) work = std::max(work, s->d.nz / 2 * (s->d.nx / s->planx.radix[q]));
    for (int q = 0; q < s->planz.nstages; ++q) work = std::max(work, s->d.nxh * (s->d.nz / s->planz.radix[q]));
    return (unsigned)std::min(1024, (work + 63) / 64 * 64);
}

// ---- y direction: one tridiagonal solve per (kx, kz) mode ----
// (lo_j psi_{j-1} + (di_j - kx^2 - kz^2) psi_j + up_j psi_{j+1}) = rhs_j / (nx nz)
// kind 0: zero-flux walls, mode (0,0) pinned at row 0 then shifted to zero
// volume mean; kind 1: zero wall value at the half-cell distance.
//
// The matrices do not change in time, so the Thomas pivots of every mode are
// computed once (k_thomas_factors) and stored as fac[kind][mode][row] =
// (g, c') with g = 1/den.  Each solve is then two linear recurrences
//   d'_j = g_j r_j + m_j d'_{j-1}  (m_j = -lo_j g_j),   x_j = d'_j - c'_j x_{j+1}.

// One thread per (kind, mode): the forward pass of Thomas' algorithm on the
// matrix only.
// Also g alone in row order, gv[kind][row][mode], for the row-slab solve and
// the fused y-march.  (fac_all may be NULL: not kept.)
__global__ void __launch_bounds__(256) k_thomas_factors(Dims d, Tables tb, double2 *fac_all, double *gv_all,
                                                        size_t ms) {
    const int kind = blockIdx.y;
    const int64_t nmodes = (int64_t)d.nxh * d.nz;
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= nmodes) return;
    const int M = d.M;
    double2 *fac = fac_all ? member_ptr(fac_all, ms) + ((int64_t)kind * nmodes + m) * M : nullptr;
    double *gv = member_ptr(gv_all, ms) + (int64_t)kind * M * nmodes + m;
    const int kx = (int)(m / d.nz), kz = (int)(m % d.nz);  // spectrum layout [j][kx][kz]
    const double k2 = tb.kx2[kx] + tb.kz2[kz];
    const bool pin = (kind == 0 && m == 0);
    double cprev = 0.0;
    for (int j = 0; j < M; ++j) {
        const double aa = tb.lyc_lo[j], cc = tb.lyc_up[j];
        const double lo = (j > 0) ? aa : 0.0;
        double up = (j < M - 1) ? cc : 0.0;
        double di = -(lo + up);
        if (kind == 1) {
            if (j == 0) di -= aa;
            if (j == M - 1) di -= cc;
        }
        double B = di - k2;
        if (pin && j == 0) {
            B = 1.0;
            up = 0.0;
        }
        const double den = B - lo * cprev;
        const double cj = up / den, g = 1.0 / den;
        if (fac) fac[j] = make_double2(g, cj);
        gv[(int64_t)j * nmodes] = g;
        cprev = cj;
    }
}

// ---- y solve over slabs of rows in registers ----
// A block owns kModes neighbouring modes of one problem over all rows; its
// threads split the rows into slabs of L, as the Crank-Nicolson solve does
// (k_cn_rows), with the recurrence coefficients of each mode from its g,
//   m_j = -lo_j g_j,   c'_j = up_j g_j:
// the forward sweep with a zero input, the slabs' inputs from their exits and
// the products of m through LDS, the input times the running product; then
// the backward sweep the same way.  Every access is a run of 512 bytes.
// Reads the spectrum and g once and writes the spectrum once, 40 bytes per
// mode and row against 48 and two dozen shuffles per mode for the lane-split
// solve below: bound by memory, 0.86 ms at 512 x 385 x 512 (4.7 TB/s; 1.13 ms
// lane-split, 0.94 with tiles of 8 modes), one problem of 256 x 193 x 256 in
// 45 us (63).  1024 threads leave 128 VGPRs: slabs of 16 rows spill 40 bytes a
// lane (also at 193 to 256 rows, whose blocks have 512 threads at most).  A
// run's own solves on up to kLaneRows rows stay lane-split, 0.111 against 0.087
// ms at 256 x 193 x 256: that keeps FP64 results bit for bit, down to plane means
// that are zero but for rounding; the mixed form shares the rule.
constexpr int kModes = 32;

template <int L>
__global__ void __launch_bounds__(1024) k_mode_rows(Dims d, Tables tb, PoissonBatch b, double2 *spec_all,
                                                    const double *gv_all, int64_t nspec) {
    extern __shared__ double2 s_m[];  // exits up, exits down [slab][kModes], products up, down, then lo, up
    const uint3 blk = xcd_block3();
    const int prob = (int)blk.y, kind = b.kind[prob];
    const int M = d.M, S = (int)blockDim.x / kModes;
    const int c = (int)threadIdx.x % kModes, slab = (int)threadIdx.x / kModes, j0 = slab * L;
    const unsigned nm = (unsigned)d.nxh * (unsigned)d.nz;
    const unsigned m = blk.x * (unsigned)kModes + (unsigned)c;
    const bool in = m < nm;
    const unsigned um = in ? m : nm - 1;  // (past the last mode: it again, not stored)
    double2 *spec = member_ptr_at(spec_all, b.ms, blk.z) + prob * nspec;
    const double *gv = gv_all + (int64_t)kind * M * nm;
    // offsets within one spectrum: rows * modes < 2^32 for every supported
    // grid; rows past the last repeat it (their g is taken as zero)
    auto off = [&](int t) { return (unsigned)(j0 + t < M ? j0 + t : M - 1) * nm + um; };
    double2 x[L];
    double g[L];
#pragma unroll
    for (int t = 0; t < L; ++t) x[t] = spec[off(t)];
#pragma unroll
    for (int t = 0; t < L; ++t) g[t] = gv[off(t)];
    double2 *s_f = s_m, *s_b = s_f + S * kModes;
    double *s_pf = (double *)(s_b + S * kModes), *s_pb = s_pf + S * kModes;
    double *s_lo = s_pb + S * kModes, *s_up = s_lo + S * L;
    for (int j = threadIdx.x; j < S * L; j += blockDim.x) {
        s_lo[j] = (j > 0 && j < M) ? tb.lyc_lo[j] : 0.0;
        s_up[j] = (j < M - 1) ? tb.lyc_up[j] : 0.0;
    }
    __syncthreads();
    const bool pin = kind == 0 && um == 0;  // the pressure's (0, 0) mode: row 0 holds 0
    const double scale = 1.0 / ((double)d.nx * (double)d.nz);
    double P = 1.0, dx_ = 0.0, dy_ = 0.0;
#pragma unroll
    for (int t = 0; t < L; ++t) {
        if (j0 + t >= M) g[t] = 0.0;
        const double mm = -s_lo[j0 + t] * g[t];
        const double gs = (pin && j0 + t == 0) ? 0.0 : g[t] * scale;
        dx_ = gs * x[t].x + mm * dx_;
        dy_ = gs * x[t].y + mm * dy_;
        x[t] = make_double2(dx_, dy_);
        P *= mm;
    }
    const int at = slab * kModes + c;
    s_f[at] = make_double2(dx_, dy_);
    s_pf[at] = P;
    __syncthreads();
    double vx = 0.0, vy = 0.0;
    for (int t = 0; t < slab; ++t) {
        const double2 e = s_f[t * kModes + c];
        const double p = s_pf[t * kModes + c];
        vx = e.x + p * vx;
        vy = e.y + p * vy;
    }
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const double mm = -s_lo[j0 + t] * g[t];
        vx *= mm;
        vy *= mm;
        x[t].x += vx;
        x[t].y += vy;
    }
    if (pin && j0 == 0) g[0] = 0.0;  // (its row does not couple upwards)
    P = 1.0;
    dx_ = dy_ = 0.0;
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        const double nn = -s_up[j0 + t] * g[t];
        dx_ = x[t].x + nn * dx_;
        dy_ = x[t].y + nn * dy_;
        x[t] = make_double2(dx_, dy_);
        P *= nn;
    }
    s_b[at] = make_double2(dx_, dy_);
    s_pb[at] = P;
    __syncthreads();
    vx = vy = 0.0;
    for (int t = S - 1; t > slab; --t) {
        const double2 e = s_b[t * kModes + c];
        const double p = s_pb[t * kModes + c];
        vx = e.x + p * vx;
        vy = e.y + p * vy;
    }
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        const double nn = -s_up[j0 + t] * g[t];
        vx *= nn;
        vy *= nn;
        x[t].x += vx;
        x[t].y += vy;
    }
    if (kind == 0 && blk.x == 0) {  // zero volume mean of the pressure-type solution
        double sx = 0.0, sy = 0.0, vol = 0.0;
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const double h = (j0 + t < M) ? tb.dn[j0 + t] : 0.0;
            sx += x[t].x * h;
            sy += x[t].y * h;
            vol += h;
        }
        if (c == 0) {
            s_f[slab] = make_double2(sx, sy);
            s_pf[slab] = vol;
        }
        __syncthreads();
        if (pin) {
            sx = sy = vol = 0.0;
            for (int t = 0; t < S; ++t) {
                sx += s_f[t].x;
                sy += s_f[t].y;
                vol += s_pf[t];
            }
            const double mx = sx / vol, my = sy / vol;
#pragma unroll
            for (int t = 0; t < L; ++t) x[t] = make_double2(x[t].x - mx, x[t].y - my);
        }
    }
    if (!in) return;
#pragma unroll
    for (int t = 0; t < L; ++t)
        if (j0 + t < M) spec[off(t)] = x[t];
}

// ---- y solve of ensembles: a mode's column in the registers of two lanes ----
// A wave owns kColModes neighbouring modes of one problem and member, all
// rows; a lane holds the real or the imaginary parts of the lower or the upper
// L rows of one mode, every load of them in flight at once (runs of 256
// bytes).  The scans of the lane-split solve below become loops over the rows
// in place, the same operations in the same order on up to 64 rows, so the
// results are its bit for bit, without its 80 moves through LDS per mode.  The
// four waves of a block solve four members, which share the modes' pivots
// (staged in LDS).
// 32 members of 64 x 65 x 64 and of 48 x 49 x 48: 72 and 36 us (3.8 TB/s)
// against 137 and 58 lane-split, which is bound by those moves.
constexpr int kColModes = 16;
constexpr int kColRows = 64;

// The other half's value, lane for lane: the lower half's in the upper one
// (kDown: the upper half's in the lower one), and `own` in the half itself.
template <bool kDown>
__device__ __forceinline__ double other_half(double v, double own) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v), w = __builtin_bit_cast(uint64_t, own);
    // the upper half of the first and the lower half of the second change places
    unsigned r[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned x = (unsigned)(u >> (32 * i)), o = (unsigned)(w >> (32 * i));
        r[i] = kDown ? __builtin_amdgcn_permlane32_swap(x, o, false, false)[1]
                     : __builtin_amdgcn_permlane32_swap(o, x, false, false)[0];
    }
    return __builtin_bit_cast(double, (uint64_t)r[1] << 32 | (uint64_t)r[0]);
}

template <int L>
__global__ void __launch_bounds__(256, 2) k_mode_columns(Dims d, Tables tb, PoissonBatch b, double2 *spec_all,
                                                         const double2 *fac_all, int64_t nspec, int nmem) {
    constexpr int NR = 2 * L, LD = NR + 1;
    __shared__ double s_g[kColModes * LD], s_c[kColModes * LD];  // pivots [mode][row]
    __shared__ double s_lo[NR], s_v[4][2][64];
    const int prob = (int)blockIdx.y, kind = b.kind[prob];
    const int M = d.M;
    const unsigned nm = (unsigned)d.nxh * (unsigned)d.nz, m0 = blockIdx.x * (unsigned)kColModes;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int mem = (int)blockIdx.z * 4 + wave;
    const double2 *fac = fac_all + ((int64_t)kind * nm + m0) * M;
    const int nc = (int)(nm - m0 < (unsigned)kColModes ? nm - m0 : (unsigned)kColModes);
    constexpr int kF = kColModes * NR / 256;  // pivots per thread
    double2 f[kF];
#pragma unroll
    for (int u = 0; u < kF; ++u) {
        const int e = (int)threadIdx.x + 256 * u, c = e / NR, j = e % NR;
        f[u] = fac[(c < nc && j < M) ? c * M + j : 0];
    }
    const int half = lane >> 5, r0 = half * L, cm = (lane & 31) >> 1;
    // lanes past the last mode work on it again and do not store
    const unsigned um = m0 + (unsigned)(cm < nc ? cm : nc - 1);
    // row t of the lower half is wave-uniform (the spectrum of up to 64 rows has
    // less than 2^32 bytes); rows past the last read the lower half's
    char *base = (char *)(member_ptr_at(spec_all, b.ms, mem < nmem ? mem : 0) + prob * nspec);
    const size_t row = (size_t)nm * sizeof(double2);
    const unsigned at_lo = um * 16u + (lane & 1) * 8u, at = at_lo + (unsigned)r0 * (unsigned)row;
    double x[L];
#pragma unroll
    for (int t = 0; t < L; ++t)
        x[t] = *(const double *)(base + (size_t)(t < M ? t : M - 1) * row + (r0 + t < M ? at : at_lo));
#pragma unroll
    for (int u = 0; u < kF; ++u) {  // (rows past the last: zero)
        const int e = (int)threadIdx.x + 256 * u, c = e / NR, j = e % NR;
        s_g[c * LD + j] = j < M ? f[u].x : 0.0;
        s_c[c * LD + j] = j < M ? f[u].y : 0.0;
    }
    if (threadIdx.x < NR) s_lo[threadIdx.x] = (threadIdx.x > 0 && (int)threadIdx.x < M) ? tb.lyc_lo[threadIdx.x] : 0.0;
    __syncthreads();
    if (mem >= nmem) return;
    const double *pg = s_g + (int)(um - m0) * LD + r0, *pc = s_c + (int)(um - m0) * LD + r0, *lo = s_lo + r0;
    const bool pin = kind == 0 && um == 0;
    const double scale = 1.0 / ((double)d.nx * (double)d.nz);
    // keeps the scheduler from running steps into each other (registers)
    auto hold = [] { __builtin_amdgcn_sched_barrier(0); };
    // d'_j = g_j r_j + m_j d'_{j-1}
    double q[L], y[L];
#pragma unroll
    for (int t = 0; t < L; ++t) {
        if (t % 8 == 0) hold();
        const double g = pg[t], r = x[t] * scale;
        q[t] = -lo[t] * g;
        x[t] = y[t] = g * ((t == 0 && pin && half == 0) ? 0.0 : r);
    }
#pragma unroll
    for (int s = 1; s < NR; s *= 2) {
        if (s >= L) {  // (the last one: the lower half's rows do not change)
#pragma unroll
            for (int t0 = s - L; t0 < L; t0 += 8) {
                double c[8];
                hold();
#pragma unroll
                for (int t = 0; t < 8; ++t) c[t] = other_half<false>(y[t0 + t + L - s], 0.0);
#pragma unroll
                for (int t = 0; t < 8; ++t) y[t0 + t] = __builtin_fma(q[t0 + t], c[t], y[t0 + t]);
            }
            break;
        }
        double c[L];
        hold();
#pragma unroll
        for (int t = 0; t < s; ++t) c[t] = other_half<false>(y[L + t - s], 0.0);
#pragma unroll
        for (int t = L - 1; t >= s; --t) y[t] = __builtin_fma(q[t], y[t - s], y[t]);
#pragma unroll
        for (int t = 0; t < s; ++t) y[t] = __builtin_fma(q[t], c[t], y[t]);
        hold();
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t < s) c[t] = other_half<false>(q[L + t - s], 1.0);
#pragma unroll
        for (int t = L - 1; t >= s; --t) q[t] *= q[t - s];
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t < s) q[t] *= c[t];
    }
    wave_sync();  // (the pivots are read again, not kept)
    {
        const double in = other_half<false>(y[L - 1], 0.0);
#pragma unroll
        for (int t = 0; t < L; ++t) {
            const double mm = -lo[t] * pg[t];
            x[t] = __builtin_fma(mm, t ? y[t ? t - 1 : 0] : in, x[t]);
        }
    }
    // x_j = d'_j - c'_j x_{j+1}
#pragma unroll
    for (int t = 0; t < L; ++t) {
        y[t] = x[t];
        q[t] = -pc[t];
    }
#pragma unroll
    for (int s = 1; s < NR; s *= 2) {
        if (s >= L) {  // (the last one)
#pragma unroll
            for (int t0 = 0; t0 < NR - s; t0 += 8) {
                double c[8];
                hold();
#pragma unroll
                for (int t = 0; t < 8; ++t) c[t] = other_half<true>(y[t0 + t + s - L], 0.0);
#pragma unroll
                for (int t = 0; t < 8; ++t) y[t0 + t] = __builtin_fma(q[t0 + t], c[t], y[t0 + t]);
            }
            break;
        }
        double c[L];
        hold();
#pragma unroll
        for (int t = L - s; t < L; ++t) c[t] = other_half<true>(y[t + s - L], 0.0);
#pragma unroll
        for (int t = 0; t + s < L; ++t) y[t] = __builtin_fma(q[t], y[t + s], y[t]);
#pragma unroll
        for (int t = L - s; t < L; ++t) y[t] = __builtin_fma(q[t], c[t], y[t]);
        hold();
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t + s >= L) c[t] = other_half<true>(q[t + s - L], 1.0);
#pragma unroll
        for (int t = 0; t + s < L; ++t) q[t] *= q[t + s];
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (t + s >= L) q[t] *= c[t];
    }
    wave_sync();
    {
        const double in = other_half<true>(y[0], 0.0);
#pragma unroll
        for (int t = 0; t < L; ++t)
            x[t] = __builtin_fma(-pc[t], t + 1 < L ? y[t + 1 < L ? t + 1 : 0] : in, x[t]);
    }
    if (kind == 0 && m0 == 0) {  // zero volume mean of the pressure-type solution
        double(&v)[2][64] = s_v[wave];
        if (pin) {
#pragma unroll
            for (int t = 0; t < L; ++t) v[lane & 1][r0 + t] = x[t];
        }
        wave_sync();
        const bool in = lane < M;
        double vol = in ? tb.dn[lane] : 0.0, sx = in ? v[0][lane] * vol : 0.0, sy = in ? v[1][lane] * vol : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            sx += __shfl_xor(sx, o, 64);
            sy += __shfl_xor(sy, o, 64);
            vol += __shfl_xor(vol, o, 64);
        }
        const double mean = ((lane & 1) ? sy : sx) / vol;
        if (pin) {
#pragma unroll
            for (int t = 0; t < L; ++t) x[t] -= mean;
        }
    }
    if (cm >= nc) return;
#pragma unroll
    for (int t = 0; t < L; ++t)
        if (r0 + t < M) *(double *)(base + (size_t)t * row + at) = x[t];
}

// Solve of one tile of tm consecutive modes of one problem: the tile's rows
// are staged in LDS with coalesced loads; each group of W lanes then solves
// one mode at a time with its rows split into W contiguous lane segments of R
// rows (the mode's pivots are one contiguous read per group; 16 or 32 lanes
// where they hold all rows, with R 1: the idle lanes of a whole wave would
// only pass values through, so the result is the same).  Each recurrence is
// a local sweep per lane, a scan of affine maps across the group and a second
// sweep from the correct incoming value.  The tile is written back with
// coalesced stores.  The members of a batch share one grid, so all of them
// read member 0's pivots, which then stay in the caches: 32 instead of 48
// bytes of memory traffic per mode and row.
// Loads per thread and wait of the staging: a whole 16-mode tile up to 192 rows.
constexpr int thomas_batch(int R) { return R == 1 ? 4 : 12; }

template <int R, int W>
__global__ void __launch_bounds__(256) k_thomas_tile(Dims d, Tables tb, PoissonBatch b, double2 *spec_all,
                                                     const double2 *fac_all, int64_t nspec, int tm) {
    constexpr int kThBatch = thomas_batch(R);
    extern __shared__ double2 s_x[];
    const uint3 blk = xcd_block3();
    const int prob = (int)blk.y;
    const int kind = b.kind[prob];
    const int64_t nmodes = (int64_t)d.nxh * d.nz;
    const int M = d.M;
    double2 *spec = member_ptr_at(spec_all, b.ms, blk.z) + prob * nspec;
    const double2 *fac = fac_all + (int64_t)kind * nmodes * M;
    const int64_t m0 = (int64_t)blk.x * tm;
    const int ncol = (int)((nmodes - m0) < tm ? (nmodes - m0) : tm);
    const int LD = tm + 1;
    const int lane = (int)threadIdx.x % W, wave = (int)threadIdx.x / W, nwave = (int)blockDim.x / W;  // (groups)
    const int js = lane * R;
    // Pivots (1/den, c') of a column: unconditional loads (padding rows read
    // the last row and ignore it); the next column's are fetched while the
    // current one is solved, unconditionally (the wave's last column re-reads
    // its own) so that the wait for the current pivots stays partial
    double2 fnext[R];
    auto load_pivots = [&](int c, double2 *f) {
        const double2 *fm = fac + (m0 + c) * M;
#pragma unroll
        for (int t = 0; t < R; ++t) f[t] = fm[(js + t < M) ? js + t : M - 1];
    };
    // one row per lane: with the tile's loads (latency; with more rows their
    // registers cost more: 256 x 193 x 256 111 against 115 us)
    if (R == 1 && wave < ncol) load_pivots(wave, fnext);
    // Staging in batches of kThBatch unconditional loads per thread (lanes
    // past the tile read its first mode and discard it): one wait per batch.
    // Offsets within one spectrum: rows * modes < 2^32 for every supported grid.
    const unsigned unm = (unsigned)nmodes, um0 = (unsigned)m0;
    const int ntile = M * tm, bd = (int)blockDim.x;
    const Div dtm(tm);  // (e < 2^22: the float-reciprocal divmod is exact)
    for (int e0 = threadIdx.x; e0 < ntile; e0 += kThBatch * bd) {
        double2 v[kThBatch];
#pragma unroll
        for (int u = 0; u < kThBatch; ++u) {
            const int e = e0 + u * bd;
            int j, c;
            dtm.split(e, j, c);
            v[u] = spec[(e < ntile && c < ncol) ? (unsigned)j * unm + um0 + (unsigned)c : um0];
        }
#pragma unroll
        for (int u = 0; u < kThBatch; ++u) {
            const int e = e0 + u * bd;
            int j, c;
            dtm.split(e, j, c);
            if (e < ntile) s_x[j * LD + c] = (c < ncol) ? v[u] : make_double2(0.0, 0.0);
        }
    }
    __syncthreads();
    constexpr int kSteps = W == 64 ? 6 : (W == 32 ? 5 : 4);
    const double scale = 1.0 / ((double)d.nx * (double)d.nz);
    double lo[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int j = js + t;
        lo[t] = (j > 0 && j < M) ? tb.lyc_lo[j] : 0.0;
    }
    if (R > 1 && wave < ncol) load_pivots(wave, fnext);
    for (int c = wave; c < ncol; c += nwave) {
        const int64_t m = m0 + c;
        const bool pin = (kind == 0 && m == 0);
        double2 fcur[R];
#pragma unroll
        for (int t = 0; t < R; ++t) fcur[t] = fnext[t];
        load_pivots(c + nwave < ncol ? c + nwave : c, fnext);
        double g[R], mm[R], nn[R];
        double2 x[R];
        double Qs = 1.0, Ss = 1.0;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int j = js + t;
            if (j < M) {
                const double2 f = fcur[t];
                g[t] = f.x;
                mm[t] = -lo[t] * f.x;
                nn[t] = -f.y;
                const double2 r = s_x[j * LD + c];
                x[t] = (pin && j == 0) ? make_double2(0.0, 0.0) : make_double2(r.x * scale, r.y * scale);
            } else {  // padding rows pass values through
                g[t] = 0.0;
                mm[t] = 1.0;
                nn[t] = 1.0;
                x[t] = make_double2(0.0, 0.0);
            }
            Qs *= mm[t];
            Ss *= nn[t];
        }
        // multipliers of the scans of x -> T + Q x (forward, from lane 0 up)
        // and x -> U + S x (backward, from the last lane down)
        double qm[kSteps], sm[kSteps];
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const int sft = 1 << st;
            qm[st] = Qs;
            sm[st] = Ss;
            const double Qp = __shfl_up(Qs, sft, W), Sp = __shfl_down(Ss, sft, W);
            if (lane >= sft) Qs *= Qp;
            if (lane + sft < W) Ss *= Sp;
        }
        // forward sweep
        double tx = 0.0, ty = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            tx = g[t] * x[t].x + mm[t] * tx;
            ty = g[t] * x[t].y + mm[t] * ty;
        }
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const double px = __shfl_up(tx, 1 << st, W), py = __shfl_up(ty, 1 << st, W);
            if (lane >= (1 << st)) {
                tx += qm[st] * px;
                ty += qm[st] * py;
            }
        }
        double dx_ = __shfl_up(tx, 1, W), dy_ = __shfl_up(ty, 1, W);
        if (lane == 0) dx_ = dy_ = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            dx_ = g[t] * x[t].x + mm[t] * dx_;
            dy_ = g[t] * x[t].y + mm[t] * dy_;
            x[t] = make_double2(dx_, dy_);
        }
        // backward sweep
        double ux = 0.0, uy = 0.0;
#pragma unroll
        for (int t = R - 1; t >= 0; --t) {
            const bool in = g[t] != 0.0;
            ux = (in ? x[t].x : 0.0) + nn[t] * ux;
            uy = (in ? x[t].y : 0.0) + nn[t] * uy;
        }
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const double px = __shfl_down(ux, 1 << st, W), py = __shfl_down(uy, 1 << st, W);
            if (lane + (1 << st) < W) {
                ux += sm[st] * px;
                uy += sm[st] * py;
            }
        }
        double xx = __shfl_down(ux, 1, W), xy = __shfl_down(uy, 1, W);
        if (lane == W - 1) xx = xy = 0.0;
#pragma unroll
        for (int t = R - 1; t >= 0; --t) {
            const bool in = g[t] != 0.0;
            xx = (in ? x[t].x : 0.0) + nn[t] * xx;
            xy = (in ? x[t].y : 0.0) + nn[t] * xy;
            x[t] = make_double2(xx, xy);
        }
        if (pin) {  // zero volume mean of the pressure-type solution
            double sx = 0.0, sy = 0.0, vol = 0.0;
#pragma unroll
            for (int t = 0; t < R; ++t) {
                const int j = js + t;
                if (j < M) {
                    const double h = tb.dn[j];
                    sx += x[t].x * h;
                    sy += x[t].y * h;
                    vol += h;
                }
            }
#pragma unroll
            for (int o = W / 2; o > 0; o >>= 1) {
                sx += __shfl_xor(sx, o, W);
                sy += __shfl_xor(sy, o, W);
                vol += __shfl_xor(vol, o, W);
            }
            const double mx = sx / vol, my = sy / vol;
#pragma unroll
            for (int t = 0; t < R; ++t) x[t] = make_double2(x[t].x - mx, x[t].y - my);
        }
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int j = js + t;
            if (j < M) s_x[j * LD + c] = x[t];
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < ntile; e += bd) {
        int j, c;
        dtm.split(e, j, c);
        if (c < ncol) spec[(unsigned)j * unm + um0 + (unsigned)c] = s_x[j * LD + c];
    }
}

// ---- the elliptic chain fused along y (mode-solve method 0) ----
// One block per tile of tk x-modes (every kz) and problem.  The forward
// kernel marches the rows upward: the row's z transform in LDS, then one
// forward-elimination step of every (kx, kz) mode's tridiagonal system with
// the pivot formed on the way, den_j = B_j - lo_j c'_{j-1}, c'_j = up_j / den_j
// (the arithmetic of k_thomas_factors), and d'_j = (r_j - lo_j d'_{j-1}) /
// den_j stored in place.  The backward kernel marches down: x_j = d'_j -
// c'_j x_{j+1} with c' = up g from the precomputed row-order table, then the row's
// inverse z transform.  Each solve thus reads and writes the spectrum twice
// (plus c'), against three times for separate z transforms and mode solves.
// The pressure problem's (0, 0) mode is pinned at row 0; its volume mean
// sum_j w_j x_j / sum_j w_j (w = cell height) is known after the forward
// march as sum_k a_k d'_k with a_k = w_k - c'_{k-1} a_{k-1} (a_0 = w_0),
// and the backward march removes it.
constexpr int kZtQ = 4;  // modes per thread (tk nz <= 1024)

// one row's (j) wall-normal operator terms of mode kind, as k_thomas_factors
__device__ __forceinline__ void ythomas_row(const Tables &tb, int kind, int M, int j, double &lo, double &up,
                                            double &di) {
    const double aa = uniform_load(tb.lyc_lo, j), cc = uniform_load(tb.lyc_up, j);
    lo = (j > 0) ? aa : 0.0;
    up = (j < M - 1) ? cc : 0.0;
    di = -(lo + up);
    if (kind == 1) {
        if (j == 0) di -= aa;
        if (j == M - 1) di -= cc;
    }
}

template <bool kR8>
__global__ void __launch_bounds__(256) k_zthomas_fwd(Dims d, Tables tb, FftPlan pl, PoissonBatch b,
                                                     double2 *spec_all, double2 *mu_all, int64_t nspec, int tk) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y, kind = b.kind[prob];
    const int nz = d.nz, nxh = d.nxh, M = d.M;
    double2 *spec = member_ptr(spec_all, b.ms) + prob * nspec;
    const int kx0 = (int)blockIdx.x * tk;
    const int nt = (nxh - kx0 < tk) ? nxh - kx0 : tk;
    const int pts = nt * nz;
    const int bs = tk * nz;
    double2 *s_tw = sm + 2 * bs;
    stage_twiddles(s_tw, tb.twz, nz);
    const double scale = 1.0 / ((double)d.nx * (double)d.nz);
    double k2[kZtQ], cprev[kZtQ];
    double2 dprev[kZtQ];
    double nre[kZtQ], nim[kZtQ];  // the next row (two arrays of doubles stay in registers)
#pragma unroll
    for (int q = 0; q < kZtQ; ++q) {
        const int e = (int)threadIdx.x + q * (int)blockDim.x;
        const int ee = e < pts ? e : 0;
        k2[q] = tb.kx2[kx0 + ee / nz] + tb.kz2[ee % nz];
        cprev[q] = 0.0;
        dprev[q] = make_double2(0.0, 0.0);
    }
    const bool pin = (kind == 0 && kx0 == 0 && threadIdx.x == 0);  // mode (0, 0) of the pressure problem
    double a = 0.0, vol = 0.0, sx = 0.0, sy = 0.0;
    auto row_ptr = [&](int j) { return spec + ((int64_t)j * nxh + kx0) * nz; };
    {
        const double2 *r0 = row_ptr(0);
#pragma unroll
        for (int q = 0; q < kZtQ; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            const double2 v = r0[e < pts ? e : 0];
            nre[q] = v.x;
            nim[q] = v.y;
        }
    }
    for (int j = 0; j < M; ++j) {
#pragma unroll
        for (int q = 0; q < kZtQ; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            if (e < pts) sm[e] = make_double2(nre[q], nim[q]);
        }
        __syncthreads();
        if (j + 1 < M) {  // the next row's loads land during this row's passes
            const double2 *rn = row_ptr(j + 1);
#pragma unroll
            for (int q = 0; q < kZtQ; ++q) {
                const int e = (int)threadIdx.x + q * (int)blockDim.x;
                const double2 v = rn[e < pts ? e : 0];
                nre[q] = v.x;
                nim[q] = v.y;
            }
        }
        const int w = lds_fft<kR8>(sm, sm + bs, nz, nt, pl, s_tw, false);
        const double2 *z = sm + w * bs;  // (offset from the LDS base: no flat access)
        double lo, up0, di;
        ythomas_row(tb, kind, M, j, lo, up0, di);
        const double wj = tb.dn[j];
        double2 *out = row_ptr(j);
#pragma unroll
        for (int q = 0; q < kZtQ; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            if (e < pts) {
                double2 r = z[e];
                r.x *= scale;
                r.y *= scale;
                double B = di - k2[q], up = up0;
                if (pin && q == 0 && j == 0) {
                    B = 1.0;
                    up = 0.0;
                    r = make_double2(0.0, 0.0);
                }
                const double den = B - lo * cprev[q];
                const double g = 1.0 / den, mm = -lo * g;
                const double2 dn_ = make_double2(g * r.x + mm * dprev[q].x, g * r.y + mm * dprev[q].y);
                if (pin && q == 0) {  // volume-mean weights of the pinned mode
                    a = (j == 0) ? wj : wj - cprev[q] * a;
                    sx += a * dn_.x;
                    sy += a * dn_.y;
                    vol += wj;
                }
                cprev[q] = up / den;
                dprev[q] = dn_;
                out[e] = dn_;
            }
        }
        __syncthreads();  // the staging buffer is refilled next row
    }
    if (pin) member_ptr(mu_all, b.ms)[prob] = make_double2(sx / vol, sy / vol);
}

template <bool kR8>
__global__ void __launch_bounds__(256) k_zthomas_bwd(Dims d, Tables tb, FftPlan pl, PoissonBatch b,
                                                     double2 *spec_all, const double *gv_all, const double2 *mu_all,
                                                     int64_t nspec, int tk) {
    extern __shared__ double2 sm[];
    const int prob = blockIdx.y, kind = b.kind[prob];
    const int nz = d.nz, nxh = d.nxh, M = d.M;
    const int64_t nmodes = (int64_t)nxh * nz;
    double2 *spec = member_ptr(spec_all, b.ms) + prob * nspec;
    const double *gv = gv_all + (int64_t)kind * M * nmodes;  // (one grid: member 0's)
    const int kx0 = (int)blockIdx.x * tk;
    const int nt = (nxh - kx0 < tk) ? nxh - kx0 : tk;
    const int pts = nt * nz;
    const int bs = tk * nz;
    double2 *s_tw = sm + 2 * bs;
    stage_twiddles(s_tw, tb.twz, nz);
    const bool pin = (kind == 0 && kx0 == 0 && threadIdx.x == 0);
    const double2 mu = pin ? member_ptr(mu_all, b.ms)[prob] : make_double2(0.0, 0.0);
    double2 xprev[kZtQ], nd[kZtQ];
    double nc[kZtQ];
    auto row_ptr = [&](int j) { return spec + ((int64_t)j * nxh + kx0) * nz; };
    auto cp_ptr = [&](int j) { return gv + (int64_t)j * nmodes + (int64_t)kx0 * nz; };
    {
        const double2 *r0 = row_ptr(M - 1);
        const double *c0 = cp_ptr(M - 1);
#pragma unroll
        for (int q = 0; q < kZtQ; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            nd[q] = r0[e < pts ? e : 0];
            nc[q] = c0[e < pts ? e : 0];
            xprev[q] = make_double2(0.0, 0.0);
        }
    }
    for (int j = M - 1; j >= 0; --j) {
        const double up = (j < M - 1) ? uniform_load(tb.lyc_up, j) : 0.0;
#pragma unroll
        for (int q = 0; q < kZtQ; ++q) {
            const int e = (int)threadIdx.x + q * (int)blockDim.x;
            if (e < pts) {
                const double cj = (pin && q == 0 && j == 0) ? 0.0 : up * nc[q];
                const double2 x = make_double2(nd[q].x - cj * xprev[q].x, nd[q].y - cj * xprev[q].y);
                xprev[q] = x;
                sm[e] = (pin && q == 0) ? make_double2(x.x - mu.x, x.y - mu.y) : x;
            }
        }
        __syncthreads();
        if (j > 0) {  // the next row's d' and g land during this row's passes
            const double2 *rn = row_ptr(j - 1);
            const double *cn = cp_ptr(j - 1);
#pragma unroll
            for (int q = 0; q < kZtQ; ++q) {
                const int e = (int)threadIdx.x + q * (int)blockDim.x;
                nd[q] = rn[e < pts ? e : 0];
                nc[q] = cn[e < pts ? e : 0];
            }
        }
        const int w = lds_fft<kR8>(sm, sm + bs, nz, nt, pl, s_tw, true);
        const double2 *z = sm + w * bs;
        double2 *out = row_ptr(j);
        for (int e = threadIdx.x; e < pts; e += blockDim.x) out[e] = z[e];
        __syncthreads();
    }
}

// modes per tile of the y solve: at most `want`, within 64 KB of LDS
inline int thomas_tile_modes(int M, int want) {
    int tm = 65536 / (M * (int)sizeof(double2)) - 1;
    if (tm > want) tm = want;
    return tm < 1 ? 1 : tm;
}

// line pairs per block of the x transforms: about `points` complex values,
// within 64 KB of LDS for the two staging buffers
inline int pairs_per_block(int nx, int points, int lds_bytes = 65536) {
    int p = nx >= points ? 1 : points / nx;
    // two buffers of x_buffer_slots(nx, p) plus the twiddle table
    const int lds_max = (lds_bytes - nx * (int)sizeof(double2)) / (2 * (nx + 2) * (int)sizeof(double2));
    if (p > lds_max) p = lds_max;
    return p < 1 ? 1 : p;
}
inline int modes_per_tile(int nz, int nxh, int points) {
    int t = nz >= points ? 1 : points / nz;
    if (t > 32) t = 32;
    if (t > nxh) t = nxh;
    // two staging buffers plus the twiddle table within 64 KB of LDS
    const int lds_max = (65536 - nz * (int)sizeof(double2)) / (2 * nz * (int)sizeof(double2));
    if (t > lds_max) t = lds_max;
    return t < 1 ? 1 : t;
}

}  // namespace

// Kernels that need more than 64 KB of dynamic LDS ask for the device's
// larger per-workgroup limit, once per (device, kernel); the record is
// shared by every handle and guarded for callers on several host threads.
hipError_t lds_opt_in(const void *fn, size_t bytes, int lds_max) {
    if (bytes <= 65536) return hipSuccess;
    if (bytes > (size_t)lds_max) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    static std::mutex mu;
    static std::set<std::pair<int, const void *>> opted;
    std::lock_guard<std::mutex> lock(mu);
    if (opted.count({dev, fn})) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds_max);
    if (e == hipSuccess) opted.insert({dev, fn});
    return e;
}

namespace {
// The forms of the elliptic chain, by the handle's sizes and shapes.
bool has_r8(const FftPlan &p) {
    for (int q = 0; q < p.nstages; ++q)
        if (p.radix[q] == 8) return true;
    return false;
}
bool march_form(const nspnp_state *s) { return s->tiles.thomas == 0 && s->mu; }  // z transforms fused with the y solve
// (the plane kernels' passes: radix 4, 2 and 3)
bool planes_form(const nspnp_state *s) {
    return !march_form(s) && !has_r8(s->planx) && !has_r8(s->planz) && plane_fits(s);
}
// 64 to 512 points, powers of two: a wave per line pair, or per 2 or 4
bool wave_line(int n) { return n == 64 || n == 128 || n == 256 || n == 512; }
// Members that share the pivots, and two waves for every SIMD: fewer waves
// would leave the chip waiting for single columns.
bool columns_form(const nspnp_state *s, int nprob, int nmem) {
    const int64_t nmodes = (int64_t)s->d.nxh * s->d.nz;
    return s->d.M <= kColRows && nmem >= 4 && (nmodes + kColModes - 1) / kColModes * nprob * nmem >= 2048;
}
}  // namespace

unsigned elliptic_tiles_read(const nspnp_state *s) {
    const bool planes = planes_form(s);
    unsigned r = 0;
    if (!planes && !wave_line(s->d.nx)) r |= kReadFftx;
    if (!planes && !march_form(s) && !wave_line(s->d.nz)) r |= kReadFftz;
    if (s->d.M <= kLaneRows && !columns_form(s, 2, s->nmem)) r |= kReadThomas;
    return r;
}

// All members of the handle are solved when b.ms is the member stride;
// caller-owned arrays (b.ms = 0) are solved for member 0 only.
hipError_t launch_poisson_batch(nspnp_state *s, const PoissonBatch &b) {
    const Dims &d = s->d;
    const int nmem = b.ms ? s->nmem : 1;
    const int64_t nlines = (int64_t)d.M * d.nz;
    const int64_t nspec = (int64_t)d.nxh * d.nz * d.M;
    const int ppb = pairs_per_block(d.nx, s->tiles.fftx);
    const int64_t npairs = (nlines + 1) / 2;
    const bool r8x = has_r8(s->planx), r8z = has_r8(s->planz);
    const bool march = march_form(s), planes = planes_form(s);
    const dim3 gp((unsigned)d.M, (unsigned)b.nprob, (unsigned)nmem);
    const size_t ldsp = plane_lds(d.nx, d.nz);
    const unsigned tp = plane_threads(s);
    const bool lines = !planes && wave_line(d.nx);
    const int lpb = d.nx == 64 ? 32 : (d.nx == 128 ? 16 : 8);  // lines per block
    const dim3 gl((unsigned)((nlines + lpb - 1) / lpb), (unsigned)b.nprob, (unsigned)nmem);
    if (lines) {
        ProfScope prof_(s, K_FFTX_FWD);
#define NSPNP_LR(TT, NN) k_lines_r2c<TT, NN><<<gl, 256, 0, s->stream>>>(d, s->tb, b, s->clock, s->spec, nspec)
        if (s->fp64) {
            if (d.nx == 64) NSPNP_LR(double, 64);
            else if (d.nx == 128) NSPNP_LR(double, 128);
            else if (d.nx == 256) NSPNP_LR(double, 256);
            else NSPNP_LR(double, 512);
        } else {
            if (d.nx == 64) NSPNP_LR(float, 64);
            else if (d.nx == 128) NSPNP_LR(float, 128);
            else if (d.nx == 256) NSPNP_LR(float, 256);
            else NSPNP_LR(float, 512);
        }
#undef NSPNP_LR
    } else if (planes) {
        ProfScope prof_(s, K_FFTX_FWD);
        const hipError_t e = lds_opt_in(s->fp64 ? (const void *)k_plane_fwd<double> : (const void *)k_plane_fwd<float>,
                                        ldsp, s->lds_max);
        if (e != hipSuccess) return e;
        if (s->fp64) k_plane_fwd<double><<<gp, tp, ldsp, s->stream>>>(d, s->tb, s->planx, s->planz, b, s->clock, s->spec, nspec);
        else k_plane_fwd<float><<<gp, tp, ldsp, s->stream>>>(d, s->tb, s->planx, s->planz, b, s->clock, s->spec, nspec);
    } else {
        ProfScope prof_(s, K_FFTX_FWD);
        const dim3 gx((unsigned)((npairs + ppb - 1) / ppb), (unsigned)b.nprob, (unsigned)nmem);
        const size_t ldsx = (2 * (size_t)x_buffer_slots(d.nx, ppb) + d.nx) * sizeof(double2);
        const void *fn = s->fp64 ? (r8x ? (const void *)k_fft_x_r2c<double, true> : (const void *)k_fft_x_r2c<double, false>)
                                 : (r8x ? (const void *)k_fft_x_r2c<float, true> : (const void *)k_fft_x_r2c<float, false>);
        const hipError_t e = lds_opt_in(fn, ldsx, s->lds_max);
        if (e != hipSuccess) return e;
#define NSPNP_R2C(TT, RR) k_fft_x_r2c<TT, RR><<<gx, 256, ldsx, s->stream>>>(d, s->tb, s->planx, b, s->clock, s->spec, nspec, ppb)
        if (s->fp64) {
            if (r8x) NSPNP_R2C(double, true);
            else NSPNP_R2C(double, false);
        } else {
            if (r8x) NSPNP_R2C(float, true);
            else NSPNP_R2C(float, false);
        }
#undef NSPNP_R2C
    }
    if (march) {
        // z transforms and mode solves fused into two row marches: tiles of
        // tk x-modes, about one mode of a row per thread (the marches are
        // serial in y, so the most tiles give the most parallelism)
        const int tk = std::max(1, std::min(d.nxh, 256 / d.nz));
        if (tk * d.nz > kZtQ * 256) return hipErrorInvalidValue;
        const dim3 gy((unsigned)((d.nxh + tk - 1) / tk), (unsigned)b.nprob, (unsigned)nmem);
        const size_t lds = (2 * (size_t)tk * d.nz + d.nz) * sizeof(double2);
        {
            ProfScope prof_(s, K_FFTZ_FWD);
            if (r8z) k_zthomas_fwd<true><<<gy, 256, lds, s->stream>>>(d, s->tb, s->planz, b, s->spec, s->mu, nspec, tk);
            else k_zthomas_fwd<false><<<gy, 256, lds, s->stream>>>(d, s->tb, s->planz, b, s->spec, s->mu, nspec, tk);
        }
        {
            ProfScope prof_(s, K_FFTZ_INV);
            if (r8z)
                k_zthomas_bwd<true><<<gy, 256, lds, s->stream>>>(d, s->tb, s->planz, b, s->spec, s->gv, s->mu, nspec, tk);
            else
                k_zthomas_bwd<false><<<gy, 256, lds, s->stream>>>(d, s->tb, s->planz, b, s->spec, s->gv, s->mu, nspec,
                                                                 tk);
        }
    } else {
        int tk = modes_per_tile(d.nz, d.nxh, s->tiles.fftz);
        if (tk * d.nz > kZPer * 256) tk = std::max(1, kZPer * 256 / d.nz);
        const int ztiles = d.M * ((d.nxh + tk - 1) / tk);
        // persistent blocks: about 8 per CU over all problems and members
        const int zblocks = std::max(1, std::min(ztiles, 2048 / std::max(1, b.nprob * nmem)));
        const dim3 gz((unsigned)zblocks, (unsigned)b.nprob, (unsigned)nmem);
        const size_t ldsz = (2 * (size_t)tk * d.nz + d.nz) * sizeof(double2);
        const bool zlines = !planes && wave_line(d.nz);
        auto z_lines = [&](auto inv) {
            constexpr bool kInv = decltype(inv)::value;
            const int lb = d.nz == 64 ? 16 : (d.nz == 128 ? 8 : 4);  // lines per block
            const dim3 g((unsigned)(((int64_t)d.M * d.nxh + lb - 1) / lb), (unsigned)b.nprob, (unsigned)nmem);
#define NSPNP_LZ(NN) k_lines_z<NN, kInv><<<g, 256, 0, s->stream>>>(d, s->tb.twz, s->spec, nspec, b.ms)
            if (d.nz == 64) NSPNP_LZ(64);
            else if (d.nz == 128) NSPNP_LZ(128);
            else if (d.nz == 256) NSPNP_LZ(256);
            else NSPNP_LZ(512);
#undef NSPNP_LZ
        };
        if (zlines) {
            ProfScope prof_(s, K_FFTZ_FWD);
            z_lines(std::false_type{});
        } else if (!planes) {
            ProfScope prof_(s, K_FFTZ_FWD);
            if (r8z) k_fft_z<true><<<gz, 256, ldsz, s->stream>>>(d, s->planz, s->tb.twz, s->spec, nspec, tk, 0, b.ms);
            else k_fft_z<false><<<gz, 256, ldsz, s->stream>>>(d, s->planz, s->tb.twz, s->spec, nspec, tk, 0, b.ms);
        }
        const int64_t nmodes = (int64_t)d.nxh * d.nz;
        // (caller-owned right-hand sides take the row-slab solve in FP64 too)
        if (d.M > kLaneRows || !s->fac || b.src[0].type == SRC_REAL) {
            ProfScope prof_(s, K_THOMAS);
            // 8 to 32 slabs (256 to 1024 threads a block)
            const int L = d.M <= 32 ? 4 : (d.M <= 128 ? 8 : ((d.M <= 192 || (d.M > 256 && d.M <= 384)) ? 12 : 16));
            const int S = (d.M + L - 1) / L;
            const dim3 gm((unsigned)((nmodes + kModes - 1) / kModes), (unsigned)b.nprob, (unsigned)nmem);
            const size_t ldsm = (size_t)S * kModes * 48 + 2 * (size_t)S * L * sizeof(double);
#define NSPNP_MR(LL) k_mode_rows<LL><<<gm, S * kModes, ldsm, s->stream>>>(d, s->tb, b, s->spec, s->gv, nspec)
            if (L == 4) NSPNP_MR(4);
            else if (L == 8) NSPNP_MR(8);
            else if (L == 12) NSPNP_MR(12);
            else NSPNP_MR(16);
#undef NSPNP_MR
        } else if (columns_form(s, b.nprob, nmem)) {
            ProfScope prof_(s, K_THOMAS);
            const dim3 gm((unsigned)((nmodes + kColModes - 1) / kColModes), (unsigned)b.nprob, (unsigned)((nmem + 3) / 4));
#define NSPNP_MC(LL) k_mode_columns<LL><<<gm, 256, 0, s->stream>>>(d, s->tb, b, s->spec, s->fac, nspec, nmem)
            if (d.M <= 16) NSPNP_MC(8);
            else if (d.M <= 32) NSPNP_MC(16);
            else if (d.M <= 48) NSPNP_MC(24);
            else NSPNP_MC(32);
#undef NSPNP_MC
        } else {
            ProfScope prof_(s, K_THOMAS);
            const int lanes = d.M <= 16 ? 16 : (d.M <= 32 ? 32 : 64);
            int tm = thomas_tile_modes(d.M, s->tiles.thomas);
            // small problems: fewer modes per tile, down to one per group of
            // lanes, until every CU has two blocks (a group solves its modes
            // one after the other, about 1 us each)
            while (tm > 256 / lanes && (nmodes + tm - 1) / tm * b.nprob * nmem < 512) tm = std::max(tm / 2, 256 / lanes);
            const dim3 gt((unsigned)((nmodes + tm - 1) / tm), (unsigned)b.nprob, (unsigned)nmem);
            const size_t ldst = (size_t)d.M * (tm + 1) * sizeof(double2);
            const int rpl = (d.M + 63) / 64;  // rows per lane (up to kLaneRows: at most 5)
#define NSPNP_TH(RR, WW) k_thomas_tile<RR, WW><<<gt, 256, ldst, s->stream>>>(d, s->tb, b, s->spec, s->fac, nspec, tm)
#define NSPNP_TH_CASE(RR)                                                                                \
        case RR:                                                                                             \
            NSPNP_TH(RR, 64);                                                                                \
            break;
            switch (rpl) {
                case 1:
                    if (lanes == 16) NSPNP_TH(1, 16);
                    else if (lanes == 32) NSPNP_TH(1, 32);
                    else NSPNP_TH(1, 64);
                    break;
                NSPNP_TH_CASE(2)
                NSPNP_TH_CASE(3)
                NSPNP_TH_CASE(4)
                NSPNP_TH_CASE(5)
                default:
                    return hipErrorInvalidValue;
            }
#undef NSPNP_TH_CASE
#undef NSPNP_TH
        }
        if (zlines) {
            ProfScope prof_(s, K_FFTZ_INV);
            z_lines(std::true_type{});
        } else if (!planes) {
            ProfScope prof_(s, K_FFTZ_INV);
            if (r8z) k_fft_z<true><<<gz, 256, ldsz, s->stream>>>(d, s->planz, s->tb.twz, s->spec, nspec, tk, 1, b.ms);
            else k_fft_z<false><<<gz, 256, ldsz, s->stream>>>(d, s->planz, s->tb.twz, s->spec, nspec, tk, 1, b.ms);
        }
    }
    if (lines) {
        ProfScope prof_(s, K_FFTX_INV);
#define NSPNP_LC(TT, NN) k_lines_c2r<TT, NN><<<gl, 256, 0, s->stream>>>(d, s->tb, b, s->spec, nspec)
        if (s->fp64) {
            if (d.nx == 64) NSPNP_LC(double, 64);
            else if (d.nx == 128) NSPNP_LC(double, 128);
            else if (d.nx == 256) NSPNP_LC(double, 256);
            else NSPNP_LC(double, 512);
        } else {
            if (d.nx == 64) NSPNP_LC(float, 64);
            else if (d.nx == 128) NSPNP_LC(float, 128);
            else if (d.nx == 256) NSPNP_LC(float, 256);
            else NSPNP_LC(float, 512);
        }
#undef NSPNP_LC
    } else if (planes) {
        ProfScope prof_(s, K_FFTX_INV);
        const hipError_t e = lds_opt_in(s->fp64 ? (const void *)k_plane_inv<double> : (const void *)k_plane_inv<float>,
                                        ldsp, s->lds_max);
        if (e != hipSuccess) return e;
        if (s->fp64) k_plane_inv<double><<<gp, tp, ldsp, s->stream>>>(d, s->tb, s->planx, s->planz, b, s->spec, nspec);
        else k_plane_inv<float><<<gp, tp, ldsp, s->stream>>>(d, s->tb, s->planx, s->planz, b, s->spec, nspec);
    } else {
        ProfScope prof_(s, K_FFTX_INV);
        // at least 8 lines per block, so that every kx of the transposed load
        // reads whole 128-byte lines of the [j][kx][kz] spectrum
        // (the device's whole LDS per workgroup may be used for that)
        int ppbc = std::max(ppb, pairs_per_block(d.nx, 4 * d.nx, s->lds_max));
        ppbc = std::max(1, std::min(ppbc, kCPer * 256 / (2 * d.nxh)));  // prefetch registers
        const int ctiles = (int)((npairs + ppbc - 1) / ppbc);
        const int cblocks = std::max(1, std::min(ctiles, 2048 / std::max(1, b.nprob * nmem)));
        const dim3 gc((unsigned)cblocks, (unsigned)b.nprob, (unsigned)nmem);
        const size_t ldsc = (2 * (size_t)x_buffer_slots(d.nx, ppbc) + d.nx) * sizeof(double2);
        const void *fn = s->fp64 ? (r8x ? (const void *)k_fft_x_c2r<double, true> : (const void *)k_fft_x_c2r<double, false>)
                                 : (r8x ? (const void *)k_fft_x_c2r<float, true> : (const void *)k_fft_x_c2r<float, false>);
        const hipError_t e = lds_opt_in(fn, ldsc, s->lds_max);
        if (e != hipSuccess) return e;
#define NSPNP_C2R(TT, RR) k_fft_x_c2r<TT, RR><<<gc, 256, ldsc, s->stream>>>(d, s->tb, s->planx, b, s->spec, nspec, ppbc)
        if (s->fp64) {
            if (r8x) NSPNP_C2R(double, true);
            else NSPNP_C2R(double, false);
        } else {
            if (r8x) NSPNP_C2R(float, true);
            else NSPNP_C2R(float, false);
        }
#undef NSPNP_C2R
    }
    return hipGetLastError();
}

// Raise the dynamic-LDS limit of the FP64 x transforms ahead of use (their
// blocks may take more than 64 KB), so that later launches find the record.
hipError_t prime_x_transform_lds(int lds_max) {
    const void *fns[6] = {(const void *)k_fft_x_r2c<double, false>, (const void *)k_fft_x_r2c<double, true>,
                          (const void *)k_fft_x_c2r<double, false>, (const void *)k_fft_x_c2r<double, true>,
                          (const void *)k_plane_fwd<double>, (const void *)k_plane_inv<double>};
    for (const void *fn : fns) {
        const hipError_t e = lds_opt_in(fn, (size_t)lds_max, lds_max);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Thomas pivots of both elliptic operators for every member of the handle
// (once, at init: they depend on the grid only).
hipError_t launch_thomas_factors(nspnp_state *s) {
    const int64_t nmodes = (int64_t)s->d.nxh * s->d.nz;
    const dim3 g((unsigned)((nmodes + 255) / 256), 2, (unsigned)s->nmem);
    k_thomas_factors<<<g, 256, 0, s->stream>>>(s->d, s->tb, s->fac, s->gv, s->mstride);
    return hipGetLastError();
}

}  // namespace nspnp
