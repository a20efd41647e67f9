// reduce.hip -- seeded initial state, adaptive time step and the plane
// reductions behind the diagnostics (wall shear stress and friction of
// Sec. II, ion fluxes through the y-faces of Fig. 1, ion contents, kinetic
// energy, divergence).  Every reduction runs in a fixed order (fixed launch
// shape, fixed LDS tree) so results are bitwise reproducible.
#include <algorithm>

#include "internal.h"

namespace nspnp {
namespace {

// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): output n of the generator
// seeded with s is mix(s + n * 0x9E3779B97F4A7C15).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t n) {
    uint64_t z = seed + n * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// uniform on [-1, 1) from stream (field, index)
__device__ __forceinline__ double noise(uint64_t seed, int field, int64_t idx) {
    const uint64_t n = ((uint64_t)field << 40) + (uint64_t)idx + 1ull;
    const double u01 = (double)(splitmix64(seed, n) >> 11) * (1.0 / 9007199254740992.0);
    return 2.0 * u01 - 1.0;
}

template <typename T>
__global__ void __launch_bounds__(256) k_init(Dims d, Tables tb, double u_top, double u_bot, uint64_t seed,
                                              double an, double cn, T *u, T *v, T *w, T *cp, T *cm, T *phi, T *p,
                                              T *h0, T *h1, T *h2, T *h3, T *h4) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= d.n) return;
    const int j = (int)(q / d.plane);
    const double ulin = 0.5 * (u_top + u_bot) + 0.5 * (u_top - u_bot) * tb.yc[j];
    u[q] = (T)(ulin + an * noise(seed, 0, q));
    v[q] = (T)((j > 0) ? an * noise(seed, 1, q) : 0.0);
    w[q] = (T)(an * noise(seed, 2, q));
    cp[q] = (T)(cn * noise(seed, 3, q));
    cm[q] = (T)(cn * noise(seed, 4, q));
    phi[q] = (T)0;
    p[q] = (T)0;
    h0[q] = h1[q] = h2[q] = h3[q] = h4[q] = (T)0;
}

template <typename T>
__global__ void __launch_bounds__(256) k_shift_conc(Dims d, double mp, double mm, T *cp, T *cm) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= d.n) return;
    cp[q] = (T)(1.0 + ((double)cp[q] - mp));
    cm[q] = (T)(1.0 + ((double)cm[q] - mm));
}

constexpr int kRedThreads = 256;

// ---- adaptive time step: max of the advective rate and of c+ + c- ----
// Once per Runge-Kutta step: the quantities of the adaptive dt rule and the
// health check of every cell.  Each thread owns one (x, z) column and marches
// a slab of rows, carrying the next row's v and phi (the top-face values of
// the current row) so that every field is read about once.  Per block:
// [0] max CFL rate, [1] max(c+ + c-), [2] min(c+, c-), [3] 1 if any value is
// not finite, [4] max |dPhi| across the cell's x, z and upper y faces.  All
// five are maxima or minima, so the result does not depend on the order.
constexpr int kDtRows = 4;  // rows per load batch of k_dt_partial

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_dt_partial(Dims d, Tables tb, const Phys *phys, const T *u,
                                                            const T *v, const T *w, const T *cp, const T *cm,
                                                            const T *phi, double *part, int chunks,
                                                            int slab_rows, size_t ms) {
    __shared__ double s[kDtParts][kRedThreads];
    u = member_ptr(u, ms); v = member_ptr(v, ms); w = member_ptr(w, ms);
    cp = member_ptr(cp, ms); cm = member_ptr(cm, ms); phi = member_ptr(phi, ms); part = member_ptr(part, ms);
    const double e0 = member_ptr(phys, ms)->e0;
    double rate = 0.0, cmax = 0.0, cmin = 1e300, pe = 0.0;
    bool bad = false;
    // XCD-aware order: consecutive z-lines (chunks) run on one XCD, so the
    // z-neighbour line each reads comes from that XCD's L2
    const unsigned bt = xcd_tile(blockIdx.x, gridDim.x);
    const int chunk = (int)(bt % (unsigned)chunks), slab = (int)(bt / (unsigned)chunks);
    const int64_t pl = d.plane;
    const int64_t e = (int64_t)chunk * blockDim.x + threadIdx.x;
    const int j0 = slab * slab_rows;
    const int j1 = (j0 + slab_rows < d.M) ? j0 + slab_rows : d.M;
    if (e < pl && j0 < j1) {
        const int i = (int)(e % d.nx), k = (int)(e / d.nx);
        const int64_t exp_ = e - i + ((i + 1 == d.nx) ? 0 : i + 1);
        const int64_t ezp = e + (int64_t)(((k + 1 == d.nz) ? 0 : k + 1) - k) * d.nx;
        double v0 = (double)v[(int64_t)j0 * pl + e], f0 = (double)phi[(int64_t)j0 * pl + e];
        // Rows are reduced in batches of kDtRows: the batch's loads are all
        // issued before any is used (rows past the slab re-read its last row
        // and are ignored), one memory latency per batch.  Offsets within
        // one field fit in 32 bits.
        const unsigned upl = (unsigned)pl, ue = (unsigned)e, uxp = (unsigned)exp_, uzp = (unsigned)ezp;
        struct RowVals {
            T v1, f1, u0, w0, c1, c2, ux, wz, fx, fz;
        };
        auto load_row = [&](int j, RowVals &r) {
            const unsigned row = (unsigned)j * upl, q = row + ue;
            const unsigned qt = (j + 1 < d.M) ? q + upl : q;
            r.v1 = v[qt];
            r.f1 = phi[qt];
            r.u0 = u[q];
            r.w0 = w[q];
            r.c1 = ld_once(cp + q);
            r.c2 = ld_once(cm + q);
            r.ux = u[row + uxp];
            r.wz = w[row + uzp];
            r.fx = phi[row + uxp];
            r.fz = phi[row + uzp];
        };
        for (int jb = j0; jb < j1; jb += kDtRows) {
            RowVals rb[kDtRows];
#pragma unroll
            for (int t = 0; t < kDtRows; ++t) load_row(jb + t < j1 ? jb + t : j1 - 1, rb[t]);
#pragma unroll
            for (int t = 0; t < kDtRows; ++t) {
                const int j = jb + t;
                if (j >= j1) break;
                const RowVals &cur = rb[t];
                const bool top = j + 1 < d.M;
                const double v1 = top ? (double)cur.v1 : 0.0;
                const double f1 = top ? (double)cur.f1 : 0.0;
                const double u0 = (double)cur.u0, w0 = (double)cur.w0;
                const double c1 = (double)cur.c1, c2 = (double)cur.c2;
                const double uc = 0.5 * (u0 + (double)cur.ux);
                const double vc = 0.5 * (v0 + v1);
                const double wc = 0.5 * (w0 + (double)cur.wz);
                rate = fmax(rate, fabs(uc) / d.dx + fabs(vc) / uniform_load(tb.dn, j) + fabs(wc) / d.dz);
                cmax = fmax(cmax, c1 + c2);
                cmin = fmin(cmin, fmin(c1, c2));
                bad = bad || !__builtin_isfinite(u0) || !__builtin_isfinite(v0) || !__builtin_isfinite(w0) ||
                      !__builtin_isfinite(c1) || !__builtin_isfinite(c2) || !__builtin_isfinite(f0);
                double dphi = fmax(fabs((double)cur.fx - f0), fabs((double)cur.fz - f0));
                if (top) dphi = fmax(dphi, fabs(f1 - f0 + e0 * uniform_load(tb.dc, j + 1)));
                pe = fmax(pe, dphi);
                v0 = v1;
                f0 = f1;
            }
        }
    }
    s[0][threadIdx.x] = rate;
    s[1][threadIdx.x] = cmax;
    s[2][threadIdx.x] = cmin;
    s[3][threadIdx.x] = bad ? 1.0 : 0.0;
    s[4][threadIdx.x] = pe;
    __syncthreads();
    for (int o = kRedThreads / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            s[0][threadIdx.x] = fmax(s[0][threadIdx.x], s[0][threadIdx.x + o]);
            s[1][threadIdx.x] = fmax(s[1][threadIdx.x], s[1][threadIdx.x + o]);
            s[2][threadIdx.x] = fmin(s[2][threadIdx.x], s[2][threadIdx.x + o]);
            s[3][threadIdx.x] = fmax(s[3][threadIdx.x], s[3][threadIdx.x + o]);
            s[4][threadIdx.x] = fmax(s[4][threadIdx.x], s[4][threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x < kDtParts) part[kDtParts * blockIdx.x + threadIdx.x] = s[threadIdx.x][0];
}

// ---- per-plane sums for diagnostics ----
// out[j * kPlaneQ + q], q as in PlaneQ: sums of u, c+, c-; total ion fluxes
// at node j; kinetic energy of row j; max |div u|; min c+, min c-,
// max (c+ + c-); max |dPhi| across the x, z and lower y faces of row j.
// Only the quantities of `what` are formed (the others are 0), from the
// fields that they need.
//
// Bound by memory: 2048 blocks or more over the grid (plane_chunks blocks per
// row, each its part of the row), every load of an element issued before its
// arithmetic; the block sums go to part[(j * chunks + chunk) * Q + q] and
// k_plane_close combines a row's in order, so results repeat bit for bit.
// Blocks run through the rows of one part before the next (row_chunk), on one
// XCD: the row above or below comes from its L2 (256 x 193 x 256 FP64: ion
// sums 107 -> 99 us, energies 273 -> 235 us against rows dealt out to all
// XCDs).  With one block a row and every quantity they took 454 and 820 us.
constexpr int kEnergyQ = 3;

__device__ __forceinline__ void row_chunk(int M, int &j, int &chunk) {
    const int t = (int)xcd_tile(blockIdx.x, gridDim.x);
    chunk = t / M;
    j = t - chunk * M;
}

// Combines a value over the block (fixed order: lanes, then waves); valid in thread 0.
enum { OP_SUM = 0, OP_MAX, OP_MIN };
template <int kOp>
__device__ __forceinline__ double combine(double a, double b) {
    return kOp == OP_SUM ? a + b : (kOp == OP_MAX ? fmax(a, b) : fmin(a, b));
}
template <int kOp>
__device__ __forceinline__ double block_reduce(double v, double *s_wave) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = combine<kOp>(v, __shfl_xor(v, o, 64));
    const int wave = threadIdx.x >> 6;
    __syncthreads();  // (the previous quantity's values have been read)
    if ((threadIdx.x & 63) == 0) s_wave[wave] = v;
    __syncthreads();
    for (int w = 1; w < kRedThreads / 64; ++w) v = combine<kOp>(v, s_wave[w]);
    return v;
}
// (max and min of PlaneQ, sums else)
__device__ __forceinline__ int plane_op(int q) {
    return (q == PQ_MAX_DIV || q == PQ_MAX_CSUM || q == PQ_MAX_DPHI) ? OP_MAX
                                                                    : ((q == PQ_MIN_CP || q == PQ_MIN_CM) ? OP_MIN : OP_SUM);
}

template <typename T, int kWhat>
__global__ void __launch_bounds__(kRedThreads) k_plane(Dims d, const Phys *phys, Tables tb, const T *u, const T *v,
                                                       const T *w, const T *cp, const T *cm, const T *phi,
                                                       double *part, int chunks, size_t ms) {
    __shared__ double s_wave[kRedThreads / 64];
    u = member_ptr(u, ms); v = member_ptr(v, ms); w = member_ptr(w, ms);
    cp = member_ptr(cp, ms); cm = member_ptr(cm, ms); phi = member_ptr(phi, ms); part = member_ptr(part, ms);
    const Phys ph = *member_ptr(phys, ms);
    const int M = d.M;
    int j, chunk;
    if (kWhat == PLANE_WALL) {  // the first and the last row
        chunk = (int)blockIdx.x >> 1;
        j = (blockIdx.x & 1) ? M - 1 : 0;
    } else {
        row_chunk(M, j, chunk);
    }
    const unsigned pl = (unsigned)d.plane, nx = (unsigned)d.nx, nz = (unsigned)d.nz;
    const unsigned per = (pl + chunks - 1) / chunks, lo = chunk * per, hi = lo + per < pl ? lo + per : pl;
    const unsigned base = (unsigned)j * pl;
    double *out = part + ((size_t)j * chunks + chunk) * kPlaneQ;
    if constexpr (kWhat == PLANE_WALL) {
        double a = 0.0;
        for (unsigned e = lo + threadIdx.x; e < hi; e += kRedThreads) a += (double)u[base + e];
        a = block_reduce<OP_SUM>(a, s_wave);
        if (threadIdx.x == 0) out[PQ_SUM_U] = a;
        return;
    }
    // rows below and above (the row itself at the walls: loaded, not used)
    const bool has_dn = j > 0, has_up = j + 1 < M;
    const unsigned dn_off = has_dn ? pl : 0u, up_off = has_up ? pl : 0u;
    const double idc = 1.0 / tb.dc[j], dcj = tb.dc[j];
    if constexpr (kWhat == PLANE_IONS) {
        const bool lim = ph.limited != 0.0, hyb = ph.hybrid != 0.0;
        double s1 = 0.0, s2 = 0.0, j1 = 0.0, j2 = 0.0;
        for (unsigned e = lo + threadIdx.x; e < hi; e += kRedThreads) {
            const unsigned q = base + e, qd = q - dn_off;
            const double c1 = (double)cp[q], c2 = (double)cm[q], d1 = (double)cp[qd], d2 = (double)cm[qd];
            const double vv = (double)v[q], dph = (double)phi[q] - (double)phi[qd];
            s1 += c1;
            s2 += c2;
            if (has_dn) {
                const double e_y = ph.e0 + dph * idc;
                const double m1 = 0.5 * (c1 + d1), m2 = 0.5 * (c2 + d2);
                // advective face values: the mean, or the limited upwind value
                double f1 = m1, f2 = m2;
                if (lim) {
                    const bool up = vv >= 0.0, have = up ? (j > 1) : has_up;
                    const unsigned quu = have ? (up ? q - 2 * pl : q + pl) : q;
                    f1 = adv_face(d1, c1, (double)cp[quu], up, have);
                    f2 = adv_face(d2, c2, (double)cm[quu], up, have);
                }
                // migration face values (hybrid rule: upwind where |dPhi| >= 2)
                const double dpy = hyb ? y_dphi(ph.e0, dcj, dph) : 0.0;
                const double g1 = mig_face(hyb, m1, d1, c1, dpy, 1.0);
                const double g2 = mig_face(hyb, m2, d2, c2, dpy, -1.0);
                j1 += vv * f1 - ph.kd * ((c1 - d1) * idc + g1 * e_y);
                j2 += vv * f2 - ph.kd * ((c2 - d2) * idc - g2 * e_y);
            }
        }
        const double r[4] = {block_reduce<OP_SUM>(s1, s_wave), block_reduce<OP_SUM>(s2, s_wave),
                             block_reduce<OP_SUM>(j1, s_wave), block_reduce<OP_SUM>(j2, s_wave)};
        if (threadIdx.x == 0) {
            out[PQ_SUM_CP] = r[0];
            out[PQ_SUM_CM] = r[1];
            out[PQ_FLUX_P] = r[2];
            out[PQ_FLUX_M] = r[3];
        }
        return;
    }
    const double idx = 1.0 / d.dx, idz = 1.0 / d.dz, idn = 1.0 / tb.dn[j];
    const double wu = 0.5 * d.dx * tb.dn[j] * d.dz, wv = 0.5 * d.dx * dcj * d.dz;
    const double ey0 = ph.e0 * dcj;
    double ke = 0.0, dv = 0.0, m1 = 1e300, m2 = 1e300, cs = 0.0, pe = 0.0;
    for (unsigned e = lo + threadIdx.x; e < hi; e += kRedThreads) {
        const unsigned k = e / nx, i = e - k * nx, q = base + e;
        const unsigned xp = (i + 1 == nx) ? q - i : q + 1, zp = (k + 1 == nz) ? q - k * nx : q + nx;
        const double uu = (double)u[q], ww = (double)w[q], vv = (double)v[q], f0 = (double)phi[q];
        const double ux = (double)u[xp], wz = (double)w[zp], va = (double)v[q + up_off];
        const double fx = (double)phi[xp], fz = (double)phi[zp], fd = (double)phi[q - dn_off];
        const double c1 = (double)cp[q], c2 = (double)cm[q];
        ke += wu * (uu * uu + ww * ww);
        if (has_dn) {
            ke += wv * vv * vv;
            pe = fmax(pe, fabs(f0 - fd + ey0));
        }
        pe = fmax(pe, fmax(fabs(fx - f0), fabs(fz - f0)));
        const double vt = has_up ? va : 0.0, vb = has_dn ? vv : 0.0;
        dv = fmax(dv, fabs((ux - uu) * idx + (vt - vb) * idn + (wz - ww) * idz));
        m1 = fmin(m1, c1);
        m2 = fmin(m2, c2);
        cs = fmax(cs, c1 + c2);
    }
    const double r[6] = {block_reduce<OP_SUM>(ke, s_wave), block_reduce<OP_MAX>(dv, s_wave),
                         block_reduce<OP_MIN>(m1, s_wave), block_reduce<OP_MIN>(m2, s_wave),
                         block_reduce<OP_MAX>(cs, s_wave), block_reduce<OP_MAX>(pe, s_wave)};
    if (threadIdx.x == 0) {
        out[PQ_KE] = r[0];
        out[PQ_MAX_DIV] = r[1];
        out[PQ_MIN_CP] = r[2];
        out[PQ_MIN_CM] = r[3];
        out[PQ_MAX_CSUM] = r[4];
        out[PQ_MAX_DPHI] = r[5];
    }
}

// A row's block sums combined in order: one thread per (row, quantity).  The
// rows and quantities that `what` does not form become 0.  (One block per row:
// its sums are the result, and this is not launched.)
__global__ void __launch_bounds__(kRedThreads) k_plane_close(int M, int what, const double *part, double *out,
                                                             int chunks, size_t ms) {
    part = member_ptr(part, ms);
    out = member_ptr(out, ms);
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= M * kPlaneQ) return;
    const int j = t / kPlaneQ, q = t - j * kPlaneQ;
    const bool have = what == PLANE_WALL   ? q == PQ_SUM_U && (j == 0 || j == M - 1)
                      : what == PLANE_IONS ? q >= PQ_SUM_CP && q <= PQ_FLUX_M
                                           : q >= PQ_KE;
    double v = 0.0;
    if (have) {
        const double *p = part + (size_t)j * chunks * kPlaneQ + q;
        const int op = plane_op(q);
        v = p[0];
        for (int c = 1; c < chunks; ++c) {
            const double x = p[(size_t)c * kPlaneQ];
            v = op == OP_SUM ? v + x : (op == OP_MAX ? fmax(v, x) : fmin(v, x));
        }
    }
    out[t] = v;
}

// Kinetic-energy budget terms of one cell row, in the volume-weighted forms
// of the semi-discrete equations:
//   out[4 j + 0]  sum over the row's velocity unknowns of |grad u|^2 times the
//                 control volume of each difference (x, z differences of u, w
//                 and v; y differences of u, w across centre rows and of v
//                 across cell rows; the half cells next to the walls in rows
//                 0 and M-1), so that Re^-1 times its total is the dissipation
//   out[4 j + 1]  sum of u . f Omega, f the Coulomb force at the u, v, w points
//   out[4 j + 2]  row 0: sum of (u - u_bot); row M-1: sum of (u_top - u)
//   out[4 j + 3]  0
// The wall work follows on the host from out[2] of the two wall rows.  Split
// and combined as the plane sums (part: kEnergyQ per block).  A thread marches
// in z over the lines of its block and carries what the next line needs of this
// one: 18 loads a cell instead of 24, and a third less from the L2, which bounds
// it (256 x 193 x 256 FP64 235 -> 182 us, six fields at 3.3 TB/s; 820 us with
// one block a row and divisions per element).
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_energy(Dims d, const Phys *phys, Tables tb, const T *u, const T *v,
                                                        const T *w, const T *cp, const T *cm, const T *phi,
                                                        double *part, int chunks, int stride, size_t ms) {
    __shared__ double s_wave[kRedThreads / 64];
    u = member_ptr(u, ms); v = member_ptr(v, ms); w = member_ptr(w, ms);
    cp = member_ptr(cp, ms); cm = member_ptr(cm, ms); phi = member_ptr(phi, ms); part = member_ptr(part, ms);
    const Phys ph = *member_ptr(phys, ms);
    const int M = d.M;
    int j, chunk;
    row_chunk(M, j, chunk);
    const unsigned pl = (unsigned)d.plane, nx = (unsigned)d.nx, nz = (unsigned)d.nz;
    // the block's z-lines, split over groups of threads of one line's (or 256) columns
    const unsigned cw = nx < (unsigned)kRedThreads ? nx : (unsigned)kRedThreads, groups = kRedThreads / cw;
    const unsigned grp = threadIdx.x / cw, per = (nz + chunks - 1) / chunks, lo = chunk * per;
    const unsigned hi = lo + per < nz ? lo + per : nz, gper = lo < hi ? (hi - lo + groups - 1) / groups : 0;
    const unsigned k0 = lo + grp * gper, k1 = grp < groups ? (k0 + gper < hi ? k0 + gper : hi) : 0;
    const unsigned base = (unsigned)j * pl;
    const bool has_dn = j > 0, has_up = j + 1 < M;
    const unsigned dn_off = has_dn ? pl : 0u, up_off = has_up ? pl : 0u;
    const double dx = d.dx, dz = d.dz, dn = tb.dn[j];
    const double dcj = tb.dc[j], dcu = tb.dc[j + 1];
    // weights of the squared differences and of the force work
    const double area = dx * dz, wxn = dn * dz / dx, wzn = dn * dx / dz, wxc = dcj * dz / dx, wzc = dcj * dx / dz;
    const double wyu = area / dcu, wyb = area / dcj, wyn = area / dn;
    const double idc = 1.0 / dcj;
    const double fxw = ph.kf * 0.5 * dn * dz, fzw = ph.kf * 0.5 * dn * dx, fyw = ph.kf * 0.5 * dcj * area;
    double dis = 0.0, fwk = 0.0, wall = 0.0;
    for (unsigned i = threadIdx.x - grp * cw; i < nx; i += cw) {
        // the values of the line before, and of this line as its neighbour loaded them
        double uu = 0.0, vv = 0.0, ww = 0.0, cz = 0.0, fz = 0.0;
        if (k0 < k1) {
            const unsigned q = base + k0 * nx + i, zm = base + (k0 == 0 ? nz - 1 : k0 - 1) * nx + i;
            uu = (double)u[q], vv = (double)v[q], ww = (double)w[q];
            cz = (double)cp[zm] - (double)cm[zm], fz = (double)phi[zm];
        }
        for (unsigned k = k0; k < k1; ++k) {
            const unsigned q = base + k * nx + i;
            const unsigned xp = (i + 1 == nx) ? q - i : q + 1, xm = (i == 0) ? q + nx - 1 : q - 1;
            const unsigned zp = (k + 1 == nz) ? q - k * nx : q + nx;
            const unsigned qu = q + up_off, qd = q - dn_off;
            const double f0 = (double)phi[q];
            const double ux = (double)u[xp], uz = (double)u[zp], ua = (double)u[qu];
            const double wx = (double)w[xp], wz = (double)w[zp], wa = (double)w[qu];
            const double vx = (double)v[xp], vz = (double)v[zp], va = (double)v[qu];
            const double r0 = (double)cp[q] - (double)cm[q], rx = (double)cp[xm] - (double)cm[xm];
            const double rz = cz, rd = (double)cp[qd] - (double)cm[qd];
            const double fx = (double)phi[xm], fd = (double)phi[qd];
            auto sq = [](double a) { return a * a; };
            dis += (sq(ux - uu) + sq(wx - ww)) * wxn + (sq(uz - uu) + sq(wz - ww)) * wzn;
            if (has_up) dis += (sq(ua - uu) + sq(wa - ww)) * wyu;
            if (has_dn) dis += sq(vx - vv) * wxc + sq(vz - vv) * wzc;
            const double vb = has_dn ? vv : 0.0, vt = has_up ? va : 0.0;
            dis += sq(vt - vb) * wyn;
            if (!has_dn) {
                dis += (sq(uu - ph.u_bot) + sq(ww)) * wyb;
                wall += uu - ph.u_bot;
            }
            if (!has_up) {
                dis += (sq(ph.u_top - uu) + sq(ww)) * wyu;
                wall += ph.u_top - uu;
            }
            // Coulomb force sF K rho_face grad Phi at the u, w and v points
            fwk += uu * (r0 + rx) * (f0 - fx) * fxw + ww * (r0 + rz) * (f0 - fz) * fzw;
            if (has_dn) fwk += vv * (r0 + rd) * (ph.e0 + (f0 - fd) * idc) * fyw;
            uu = uz, vv = vz, ww = wz, cz = r0, fz = f0;
        }
    }
    const double r[kEnergyQ] = {block_reduce<OP_SUM>(dis, s_wave), block_reduce<OP_SUM>(fwk, s_wave),
                                block_reduce<OP_SUM>(wall, s_wave)};
    if (threadIdx.x == 0)
        for (int q = 0; q < kEnergyQ; ++q) part[((size_t)j * chunks + chunk) * stride + q] = r[q];
}

__global__ void __launch_bounds__(kRedThreads) k_energy_close(int M, const double *part, double *out, int chunks,
                                                              size_t ms) {
    part = member_ptr(part, ms);
    out = member_ptr(out, ms);
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= M * 4) return;
    const int j = t >> 2, q = t & 3;
    double v = 0.0;
    if (q < kEnergyQ)
        for (int c = 0; c < chunks; ++c) v += part[((size_t)j * chunks + c) * kEnergyQ + q];
    out[t] = v;
}

// time sums (weight alp dt) of the plane means of u, c+ - c- and phi per row
template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_stats(Dims d, const T *u, const T *cp, const T *cm, const T *phi,
                                                       const double *clock, double *stats, double alp, size_t ms) {
    __shared__ double s[3][kRedThreads];
    u = member_ptr(u, ms); cp = member_ptr(cp, ms); cm = member_ptr(cm, ms); phi = member_ptr(phi, ms);
    clock = member_ptr(clock, ms);
    stats = member_ptr(stats, ms);
    const int j = blockIdx.x;
    const int64_t base = (int64_t)j * d.plane;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int64_t e = threadIdx.x; e < d.plane; e += blockDim.x) {
        const int64_t q = base + e;
        a0 += (double)u[q];
        a1 += (double)cp[q] - (double)cm[q];
        a2 += (double)phi[q];
    }
    s[0][threadIdx.x] = a0;
    s[1][threadIdx.x] = a1;
    s[2][threadIdx.x] = a2;
    __syncthreads();
    for (int o = kRedThreads / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o)
            for (int qq = 0; qq < 3; ++qq) s[qq][threadIdx.x] += s[qq][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double wgt = alp * clock[1];
        const double inv = 1.0 / (double)d.plane;
        for (int qq = 0; qq < 3; ++qq) stats[3 * j + qq] += wgt * s[qq][0] * inv;
        if (j == 0) stats[3 * d.M] += wgt;
    }
}

__global__ void k_fill(double *p, int64_t n, double v, size_t ms) {
    p = member_ptr(p, ms);
    for (int64_t q = threadIdx.x; q < n; q += blockDim.x) p[q] = v;
}

inline dim3 grid1(int64_t n, int b = 256) { return dim3((unsigned)((n + b - 1) / b)); }

}  // namespace

hipError_t launch_init_fields(nspnp_state *s) {
    const nspnp_config &c = s->cfg;
    if (s->fp64) {
        double **f = (double **)s->f;
        double **h = (double **)s->h;
        k_init<double><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d, s->tb, c.u_top, c.u_bot, c.seed, c.u_noise,
                                                            c.c_noise, f[0], f[1], f[2], f[3], f[4], f[5], f[6],
                                                            h[0], h[1], h[2], h[3], h[4]);
    } else {
        float **f = (float **)s->f;
        float **h = (float **)s->h;
        k_init<float><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d, s->tb, c.u_top, c.u_bot, c.seed, c.u_noise,
                                                           c.c_noise, f[0], f[1], f[2], f[3], f[4], f[5], f[6],
                                                           h[0], h[1], h[2], h[3], h[4]);
    }
    return hipGetLastError();
}

hipError_t launch_shift_conc(nspnp_state *s, double mp, double mm) {
    if (s->fp64)
        k_shift_conc<double><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d, mp, mm, (double *)s->f[3], (double *)s->f[4]);
    else
        k_shift_conc<float><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d, mp, mm, (float *)s->f[3], (float *)s->f[4]);
    return hipGetLastError();
}

hipError_t launch_dt(nspnp_state *s, int *nparts) {
    // columns in chunks of one block; rows split into slabs so that the
    // partials fit kDtMaxBlocks per member and the members together have about
    // 4096 blocks (a slab reads one row of v and phi beyond its own and loads
    // kDtRows at a time: 32 members of 64 x 65 x 64 with single rows 92 us, with
    // 8 rows 39; of 48 x 49 x 48 43 and 25)
    static_assert(kDtThreads == kRedThreads, "dt block size");
    const int chunks = dt_chunks(s->d.plane);
    const int slabs = std::max(1, std::min({s->d.M, kDtMaxBlocks / chunks, 4096 / (chunks * s->nmem)}));
    const int slab_rows = (s->d.M + slabs - 1) / slabs;
    const unsigned nb = (unsigned)(chunks * ((s->d.M + slab_rows - 1) / slab_rows));
    if ((int64_t)nb * kDtParts > s->nred) return hipErrorInvalidValue;  // the layout sized red for this
    const dim3 g(nb, 1, (unsigned)s->nmem);
    if (s->fp64)
        k_dt_partial<double><<<g, kRedThreads, 0, s->stream>>>(
            s->d, s->tb, s->d_phys, (const double *)s->f[0], (const double *)s->f[1], (const double *)s->f[2],
            (const double *)s->f[3], (const double *)s->f[4], (const double *)s->f[5], s->red, chunks, slab_rows,
            s->mstride);
    else
        k_dt_partial<float><<<g, kRedThreads, 0, s->stream>>>(
            s->d, s->tb, s->d_phys, (const float *)s->f[0], (const float *)s->f[1], (const float *)s->f[2],
            (const float *)s->f[3], (const float *)s->f[4], (const float *)s->f[5], s->red, chunks, slab_rows,
            s->mstride);
    *nparts = (int)nb;
    return hipGetLastError();
}

// Blocks per row of the plane reductions: about 2048 over the grid, at least
// two rounds of elements per thread.
static int plane_chunks(const nspnp_state *s) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(run_stats_chunks(s->d.M), s->d.plane / (2 * kRedThreads)));
}

// per-plane sums of every member (results in each member's dev_out copy, the
// block sums behind them in the reduction scratch; those that `what` does not
// form are not defined)
hipError_t launch_plane_sums(nspnp_state *s, int what, double *dev_out) {
    const int chunks = plane_chunks(s);
    const int M = s->d.M;
    if (dev_out != s->red || (int64_t)M * kPlaneQ * (chunks + 1) > s->nred) return hipErrorInvalidValue;
    double *part = chunks > 1 ? dev_out + (size_t)M * kPlaneQ : dev_out;
    const dim3 g((unsigned)chunks * (what == PLANE_WALL ? 2u : (unsigned)M), 1, (unsigned)s->nmem);
    auto go = [&](auto zero) {
        using T = decltype(zero);
        const T *f[6];
        for (int q = 0; q < 6; ++q) f[q] = (const T *)s->f[q];
#define NSPNP_PLANE(W)                                                                                            \
    k_plane<T, W><<<g, kRedThreads, 0, s->stream>>>(s->d, s->d_phys, s->tb, f[0], f[1], f[2], f[3], f[4], f[5], part, \
                                                    chunks, s->mstride)
        if (what == PLANE_WALL) NSPNP_PLANE(PLANE_WALL);
        else if (what == PLANE_IONS) NSPNP_PLANE(PLANE_IONS);
        else NSPNP_PLANE(PLANE_DIAG);
#undef NSPNP_PLANE
    };
    if (s->fp64) go(double{});
    else go(float{});
    if (chunks == 1) return hipGetLastError();
    k_plane_close<<<dim3((unsigned)((M * kPlaneQ + kRedThreads - 1) / kRedThreads), 1, (unsigned)s->nmem), kRedThreads,
                    0, s->stream>>>(M, what, part, dev_out, chunks, s->mstride);
    return hipGetLastError();
}

// energy-budget partial sums, 4 per row (k_energy)
hipError_t launch_energy_sums(nspnp_state *s, double *dev_out) {
    const int chunks = plane_chunks(s);
    const int M = s->d.M;
    if (dev_out != s->red || (int64_t)M * (4 + kEnergyQ * chunks) > s->nred) return hipErrorInvalidValue;
    double *part = chunks > 1 ? dev_out + 4 * (size_t)M : dev_out;
    const int stride = chunks > 1 ? kEnergyQ : 4;
    const dim3 g((unsigned)(chunks * M), 1, (unsigned)s->nmem);
    auto go = [&](auto zero) {
        using T = decltype(zero);
        k_energy<T><<<g, kRedThreads, 0, s->stream>>>(s->d, s->d_phys, s->tb, (const T *)s->f[0], (const T *)s->f[1],
                                                      (const T *)s->f[2], (const T *)s->f[3], (const T *)s->f[4],
                                                      (const T *)s->f[5], part, chunks, stride, s->mstride);
    };
    if (s->fp64) go(double{});
    else go(float{});
    if (chunks == 1) return hipGetLastError();
    k_energy_close<<<dim3((unsigned)((4 * M + kRedThreads - 1) / kRedThreads), 1, (unsigned)s->nmem), kRedThreads, 0,
                     s->stream>>>(M, part, dev_out, chunks, s->mstride);
    return hipGetLastError();
}

// n doubles at p (on this handle's device) set to v, on the solver's stream
hipError_t launch_fill(nspnp_state *s, double *p, int64_t n, double v) {
    k_fill<<<dim3(1, 1, 1), 256, 0, s->stream>>>(p, n, v, 0);
    return hipGetLastError();
}

hipError_t launch_stats_reset(nspnp_state *s) {
    k_fill<<<dim3(1, 1, (unsigned)s->nmem), 256, 0, s->stream>>>(s->stats, 3 * (int64_t)s->d.M + 2, 0.0, s->mstride);
    return hipGetLastError();
}

namespace {

// Run statistics (the averages behind mean and RMS profiles, Sec. III).
// k_run_stats: block (chunk, row j) sums q and q^2 for q = u, v, w, c+, c-,
// phi, p over its part of the row, in batches of kStatBatch elements per
// thread whose loads are all issued first, and writes the kRunStatsQ sums to
// the scratch slot (j, chunk).  k_run_stats_close: thread (j, q) adds the chunks
// in order and accumulates w * (plane mean) with w = t - t_last, the time
// since the previous sample (t from the device clock, after this substep's
// advance); k_run_stats_tail then adds w to the accumulated time and sets
// t_last = t.  The
// sums never depend on timing (no atomics), so runs repeat bit for bit.
constexpr int kStatBatch = 4;

template <typename T>
__global__ void __launch_bounds__(kRedThreads) k_run_stats(Dims d, const T *f0, const T *f1, const T *f2, const T *f3,
                                                           const T *f4, const T *f5, const T *f6, double *part,
                                                           int chunks, size_t ms) {
    __shared__ double sm[kRunStatsQ][kRedThreads / 64];
    const T *f[kRunStatsFields] = {member_ptr(f0, ms), member_ptr(f1, ms), member_ptr(f2, ms), member_ptr(f3, ms),
                                   member_ptr(f4, ms), member_ptr(f5, ms), member_ptr(f6, ms)};
    part = member_ptr(part, ms);
    const int chunk = blockIdx.x, j = blockIdx.y;
    const int pl = (int)d.plane;
    const int per = (pl + chunks - 1) / chunks;
    const int e_lo = chunk * per, e_hi = (e_lo + per < pl) ? e_lo + per : pl;
    const unsigned base = (unsigned)j * (unsigned)pl;
    const int bd = (int)blockDim.x;
    double a[kRunStatsQ];
#pragma unroll
    for (int q = 0; q < kRunStatsQ; ++q) a[q] = 0.0;
    for (int e0 = e_lo + (int)threadIdx.x; e0 < e_hi; e0 += kStatBatch * bd) {
        T x[kStatBatch][kRunStatsFields];
#pragma unroll
        for (int u = 0; u < kStatBatch; ++u) {
            const int e = (e0 + u * bd < e_hi) ? e0 + u * bd : e0;  // in range; dropped below
#pragma unroll
            for (int q = 0; q < kRunStatsFields; ++q) x[u][q] = f[q][base + (unsigned)e];
        }
#pragma unroll
        for (int u = 0; u < kStatBatch; ++u) {
            if (e0 + u * bd < e_hi) {
#pragma unroll
                for (int q = 0; q < kRunStatsFields; ++q) {
                    const double v = (double)x[u][q];
                    a[q] += v;
                    a[kRunStatsFields + q] += v * v;
                }
            }
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < kRunStatsQ; ++q) {
        double v = a[q];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) sm[q][wave] = v;
    }
    __syncthreads();
    if (threadIdx.x < kRunStatsQ) {
        const int q = threadIdx.x;
        double v = 0.0;
        for (int w = 0; w < (bd >> 6); ++w) v += sm[q][w];
        part[((size_t)j * chunks + chunk) * kRunStatsQ + q] = v;
    }
}

__global__ void __launch_bounds__(kStatCloseThreads) k_run_stats_close(Dims d, const double *part, int chunks,
                                                                       const double *clock, double *rs, size_t ms) {
    part = member_ptr(part, ms);
    clock = member_ptr(clock, ms);
    rs = member_ptr(rs, ms);
    const int M = d.M;
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= M * kRunStatsQ) return;
    const int j = t / kRunStatsQ, q = t - j * kRunStatsQ;
    const double wgt = clock[0] - rs[kRunStatsQ * M + 1];
    const double *pj = part + (size_t)j * chunks * kRunStatsQ + q;
    double v = 0.0;
    for (int c0 = 0; c0 < chunks; c0 += 8) {  // chunks in order, 8 loads in flight
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = pj[(size_t)(c0 + u < chunks ? c0 + u : c0) * kRunStatsQ];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (c0 + u < chunks) v += x[u];
    }
    rs[q * M + j] += wgt * (v / (double)d.plane);
}

// after k_run_stats_close (which reads t_last): accumulated time, t_last, count
__global__ void k_run_stats_tail(int M, const double *clock, double *rs, size_t ms) {
    clock = member_ptr(clock, ms);
    rs = member_ptr(rs, ms);
    if (threadIdx.x == 0) {
        double *tail = rs + kRunStatsQ * M;
        tail[0] += clock[0] - tail[1];
        tail[1] = clock[0];
        tail[2] += 1.0;
    }
}

// Clear the run statistics and take the current time as the start.
__global__ void k_run_stats_begin(int M, const double *clock, double *rs, size_t ms) {
    clock = member_ptr(clock, ms);
    rs = member_ptr(rs, ms);
    const int n = kRunStatsQ * M + kRunStatsTail;
    for (int e = threadIdx.x; e < n; e += blockDim.x) rs[e] = (e == kRunStatsQ * M + 1) ? clock[0] : 0.0;
}

}  // namespace

hipError_t launch_run_stats_begin(nspnp_state *s) {
    k_run_stats_begin<<<dim3(1, 1, (unsigned)s->nmem), 256, 0, s->stream>>>(s->d.M, s->clock, s->rstats, s->mstride);
    return hipGetLastError();
}

hipError_t launch_run_stats(nspnp_state *s) {
    ProfScope prof_(s, K_STATS);
    const int chunks = run_stats_chunks(s->d.M);
    if ((int64_t)s->d.M * chunks * kRunStatsQ > s->nred) return hipErrorInvalidValue;  // the layout sized red for this
    const dim3 g((unsigned)chunks, (unsigned)s->d.M, (unsigned)s->nmem);
    if (s->fp64)
        k_run_stats<double><<<g, kRedThreads, 0, s->stream>>>(
            s->d, (const double *)s->f[0], (const double *)s->f[1], (const double *)s->f[2], (const double *)s->f[3],
            (const double *)s->f[4], (const double *)s->f[5], (const double *)s->f[6], s->red, chunks, s->mstride);
    else
        k_run_stats<float><<<g, kRedThreads, 0, s->stream>>>(
            s->d, (const float *)s->f[0], (const float *)s->f[1], (const float *)s->f[2], (const float *)s->f[3],
            (const float *)s->f[4], (const float *)s->f[5], (const float *)s->f[6], s->red, chunks, s->mstride);
    const unsigned nclose = (unsigned)((s->d.M * kRunStatsQ + kStatCloseThreads - 1) / kStatCloseThreads);
    k_run_stats_close<<<dim3(nclose, 1, (unsigned)s->nmem), kStatCloseThreads, 0, s->stream>>>(
        s->d, s->red, chunks, s->clock, s->rstats, s->mstride);
    k_run_stats_tail<<<dim3(1, 1, (unsigned)s->nmem), 64, 0, s->stream>>>(s->d.M, s->clock, s->rstats, s->mstride);
    return hipGetLastError();
}

hipError_t launch_stats_accum(nspnp_state *s, double alp) {
    const dim3 g((unsigned)s->d.M, 1, (unsigned)s->nmem);
    if (s->fp64)
        k_stats<double><<<g, kRedThreads, 0, s->stream>>>(s->d, (const double *)s->f[0], (const double *)s->f[3],
                                                          (const double *)s->f[4], (const double *)s->f[5], s->clock,
                                                          s->stats, alp, s->mstride);
    else
        k_stats<float><<<g, kRedThreads, 0, s->stream>>>(s->d, (const float *)s->f[0], (const float *)s->f[3],
                                                         (const float *)s->f[4], (const float *)s->f[5], s->clock,
                                                         s->stats, alp, s->mstride);
    return hipGetLastError();
}

}  // namespace nspnp
