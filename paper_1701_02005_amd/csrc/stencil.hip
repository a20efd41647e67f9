// stencil.hip -- explicit right-hand sides, Crank-Nicolson wall-normal
// solves, divergence and projection correction of one Runge-Kutta substep of
// the NS-PNP scheme (Sec. II, Eqs. (1)-(3), Fig. 1), for gfx950.
//
// Layout: every field is [j][k][i] (i = x fastest, k = z, j = cell row).
// u lives on x-faces, w on z-faces, v on the bottom y-face of each row (row 0
// is the wall), c+-, phi and p at cell centres.  T is the storage and stencil
// type: double for the FP64 form, float for the mixed form.
#include <type_traits>

#include "internal.h"

namespace nspnp {
namespace {

struct Idx {
    int i, j, k, ip, im, kp, km;
    int64_t c0, xp, xm, zp, zm;
};

__device__ __forceinline__ Idx make_idx(const Dims &d, int64_t q) {
    Idx t;
    t.i = (int)(q % d.nx);
    int64_t r = q / d.nx;
    t.k = (int)(r % d.nz);
    t.j = (int)(r / d.nz);
    t.ip = (t.i + 1 == d.nx) ? 0 : t.i + 1;
    t.im = (t.i == 0) ? d.nx - 1 : t.i - 1;
    t.kp = (t.k + 1 == d.nz) ? 0 : t.k + 1;
    t.km = (t.k == 0) ? d.nz - 1 : t.k - 1;
    t.c0 = q;
    t.xp = q - t.i + t.ip;
    t.xm = q - t.i + t.im;
    t.zp = q + (int64_t)(t.kp - t.k) * d.nx;
    t.zm = q + (int64_t)(t.km - t.k) * d.nx;
    return t;
}

struct ExplicitArgs {
    Dims d;
    const Phys *phys;
    size_t ms;
    Tables tb;
    Stage st;
    const void *u, *v, *w, *cp, *cm, *phi, *p;
    void *h[5];
    void *r[5];  // Crank-Nicolson right-hand sides, state type (computed in it)
    double *dbg[5];
    const double *clock;
    int mode;  // 0: substep (H update + CN right-hand sides); 1: H to dbg only
    int tx, tz;     // a block's (x, z) tile: tx columns of tz z-lines
    int ntx;        // tiles across x
    int chunks;     // tiles per (x, z) plane
    int slabs;      // row slabs per member
    int slab_rows;  // rows marched by one block
    int implicit_xz;  // 1: x/z diffusion goes to the implicit (alpha) part of r, not to H
};

__device__ __forceinline__ void shift_explicit(ExplicitArgs &a, unsigned mem) {
    const size_t ms = a.ms;
    a.phys = member_ptr_at(a.phys, ms, mem);
    a.u = member_ptr_at(a.u, ms, mem); a.v = member_ptr_at(a.v, ms, mem); a.w = member_ptr_at(a.w, ms, mem);
    a.cp = member_ptr_at(a.cp, ms, mem); a.cm = member_ptr_at(a.cm, ms, mem);
    a.phi = member_ptr_at(a.phi, ms, mem); a.p = member_ptr_at(a.p, ms, mem);
    for (int f = 0; f < 5; ++f) { a.h[f] = member_ptr_at(a.h[f], ms, mem); a.r[f] = member_ptr_at(a.r[f], ms, mem); }
    a.clock = member_ptr_at(a.clock, ms, mem);
}

// Convection, horizontal diffusion, Coulomb force and ion transport at one
// cell, then the Crank-Nicolson right-hand side
//   r = dt [gam H^k + zet H^{k-1} - alp G p + alp nu L_y q].
//
// Data movement.  A block owns a 2-D tile of (x, z) columns (tx along x, tz
// z-lines) and marches a slab of rows.  Rows j and j+1 of all seven fields,
// each over the tile plus a one-column halo (periodic in x and z), sit in a
// two-slot LDS ring.  The global loads of row j+2 (coalesced, two halo
// positions per thread) and of H^{k-1} at row j+1 are issued before row j is
// computed and land in LDS / registers after it, so the memory latency hides
// behind a whole row of arithmetic and every neighbour value is an LDS read.
// Own-column values of row j-1 and the two row-(j-1) neighbours the v-point
// needs are carried in registers from the previous row.
constexpr int kNF = 7;  // u v w c+ c- phi p

// Minus the divergence of (limited face value - mean) times the face velocity
// of one species: x and z faces right, left, front, back, y faces top and
// bottom.  q: c at x +1 -1 +2 -2, z +1 -1 +2 -2; col: rows j - 2 .. j + 2 of the
// cell's column (rows outside the grid are not used).
template <typename T>
__device__ __forceinline__ T limit_delta(const T *q, const T *col, T uR, T uL, T wF, T wB, T vt, T vb, int j, int M,
                                         T idx, T idz, T idn) {
    const T half = T(0.5);
    const bool ur = uR >= T(0), ul = uL >= T(0), wf = wF >= T(0), wb = wB >= T(0);
    const bool upt = vt >= T(0), upb = vb >= T(0);
    const bool have_t = upt ? (j > 0) : (j + 2 < M), have_b = upb ? (j > 1) : (j + 1 < M);
    const T cc = col[2], cyp = col[3], cym = col[1];
    const T cxp = q[0], cxm = q[1], czp = q[4], czm = q[5];
    const T dR = adv_face(cc, cxp, ur ? cxm : q[2], ur, true) - half * (cxp + cc);
    const T dL = adv_face(cxm, cc, ul ? q[3] : cxp, ul, true) - half * (cc + cxm);
    const T dF = adv_face(cc, czp, wf ? czm : q[6], wf, true) - half * (czp + cc);
    const T dB = adv_face(czm, cc, wb ? q[7] : czp, wb, true) - half * (cc + czm);
    // top face (rows j, j + 1) and bottom face (rows j - 1, j)
    const T dT = (j + 1 < M) ? adv_face(cc, cyp, upt ? cym : col[4], upt, have_t) - half * (cyp + cc) : T(0);
    const T dD = (j > 0) ? adv_face(cym, cc, upb ? col[0] : cyp, upb, have_b) - half * (cc + cym) : T(0);
    return -((uR * dR - uL * dL) * idx + (wF * dF - wB * dB) * idz + (vt * dT - vb * dD) * idn);
}

template <typename T, int kHalo>
struct HaloRegs {
    T v[kNF][kHalo];
};

// kMode (a compile-time copy of ExplicitArgs::mode): the export of H alone
// is its own instantiation, so the substep kernel carries none of its state.
// kTx > 0: the tile is kTx columns by kTz z-lines (a.tx, a.tz ignored), so
// every LDS neighbour offset is a compile-time constant.
// kLim (the mixed form): the limited advective flux of migration_face 2 is
// formed here instead of in a pass of its own, which reads u, v, w, c+- and
// the ions' H and r again and rewrites those: 256 x 193 x 256 277 us against 222
// and 157 (carrying the y faces' values from row to row, a sixth of its
// arithmetic less, changes nothing).  The values two
// columns away come from the caches (the row's own tile loads them), those two
// rows up from memory one row early.  FP64 keeps the pass: its kernel has 147
// of the 168 VGPRs of three waves without the limiter (in it, not measured).
template <typename T, int kHalo, int kWaves, int kMode, int kTx = 0, int kTz = 0, bool kLim = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kWaves))) k_explicit(ExplicitArgs a) {
    extern __shared__ unsigned char s_raw[];
    T *sm = (T *)s_raw;  // [slot 0..1][field 0..6][halo tile]
    const unsigned chunks = (unsigned)a.chunks, slabs = (unsigned)a.slabs;
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);  // x-tiles fastest: z-neighbour tiles share an L2
    const unsigned chunk = tile % chunks;
    const unsigned slab = (tile / chunks) % slabs;
    const unsigned mem = tile / (chunks * slabs);
    shift_explicit(a, mem);
    const Phys ph = *a.phys;
    const Dims &d = a.d;
    const int nx = d.nx, nz = d.nz, M = d.M;
    const int pl = (int)d.plane;
    const int tx = kTx ? kTx : a.tx, tz = kTx ? kTz : a.tz, hx = tx + 2, HS = hx * (tz + 2);
    const int i0 = (int)(chunk % (unsigned)a.ntx) * tx, k0 = (int)(chunk / (unsigned)a.ntx) * tz;
    const int lk = (int)threadIdx.x / tx, li = (int)threadIdx.x - lk * tx;
    const int i = i0 + li, k = k0 + lk;
    const bool active = lk < tz && i < nx && k < nz;
    const int c = (lk + 1) * hx + (li + 1);  // own position in the halo tile

    const T *__restrict__ F[kNF] = {(const T *)a.u, (const T *)a.v, (const T *)a.w, (const T *)a.cp,
                                    (const T *)a.cm, (const T *)a.phi, (const T *)a.p};
    // halo positions this thread loads: in-plane byte offsets, fixed for every
    // row.  Positions past the halo tile load the plane's first element
    // (which exists) and are never stored: the loads are unconditional, so a
    // row's loads go out together.  Every access is a field's base pointer plus
    // a 32-bit byte offset (row offset + in-plane offset; a field of every
    // supported grid is below 2^32 bytes), which the hardware adds itself.
    unsigned off[kHalo];
    int spos[kHalo];
    bool in_tile[kHalo];
#pragma unroll
    for (int q = 0; q < kHalo; ++q) {
        const int sp = (int)threadIdx.x + q * (int)blockDim.x;
        spos[q] = sp;
        in_tile[q] = sp < HS;
        const int hz = sp / hx, hxp = sp - hz * hx;
        int gi = (i0 - 1 + hxp) % nx, gk = (k0 - 1 + hz) % nz;
        if (gi < 0) gi += nx;
        if (gk < 0) gk += nz;
        off[q] = in_tile[q] ? (unsigned)(gk * nx + gi) * (unsigned)sizeof(T) : 0u;
    }
    const unsigned plb = (unsigned)pl * (unsigned)sizeof(T);  // bytes per row of a field
    auto load_rows = [&](int row, HaloRegs<T, kHalo> &r) {
        const unsigned base = (unsigned)row * plb;
#pragma unroll
        for (int f = 0; f < kNF; ++f)
#pragma unroll
            for (int q = 0; q < kHalo; ++q) r.v[f][q] = *byte_at(F[f], base + off[q]);
    };
    auto store_rows = [&](int slot, const HaloRegs<T, kHalo> &r) {
#pragma unroll
        for (int f = 0; f < kNF; ++f)
#pragma unroll
            for (int q = 0; q < kHalo; ++q)
                if (in_tile[q]) sm[(slot * kNF + f) * HS + spos[q]] = r.v[f][q];
    };
    auto X = [&](int slot, int f, int dx, int dz) -> T { return sm[(slot * kNF + f) * HS + c + dz * hx + dx]; };

    const T half = T(0.5), two = T(2);
    const T idx_ = T(1.0 / d.dx), idz_ = T(1.0 / d.dz);
    const T ix2 = idx_ * idx_, iz2 = idz_ * idz_;
    const T kf = T(ph.kf), ire = T(ph.ire), kd = T(ph.kd), e0 = T(ph.e0);
    constexpr int mode = kMode;
    const T dt = T(a.clock[1]);
    const T gam = T(a.st.gam), zet = T(a.st.zet), alp = T(a.st.alp);
    const bool use_old = (a.st.k > 0) && mode == 0;
    const bool keep = (a.st.k < 2) && mode == 0;
    const bool imp = a.implicit_xz != 0;  // x/z diffusion: implicit part of r instead of H
    const int e = active ? k * nx + i : 0;
    const unsigned ueb = (unsigned)e * (unsigned)sizeof(T);  // own column, bytes
    const int ip = (i + 1 >= nx) ? 0 : i + 1;
    const int kp = (k + 1 >= nz) ? 0 : k + 1;
    const int e_xp = k * nx + ip, e_zp = kp * nx + i;
    unsigned two_off[4] = {0, 0, 0, 0};  // x + 2, x - 2, z + 2, z - 2, bytes in the plane
    if constexpr (kLim) {
        if (active) {
            auto wrap = [](int q, int n) { return q < 0 ? q + n : (q >= n ? q - n : q); };  // n >= 4
            two_off[0] = (unsigned)(k * nx + wrap(i + 2, nx)) * (unsigned)sizeof(T);
            two_off[1] = (unsigned)(k * nx + wrap(i - 2, nx)) * (unsigned)sizeof(T);
            two_off[2] = (unsigned)(wrap(k + 2, nz) * nx + i) * (unsigned)sizeof(T);
            two_off[3] = (unsigned)(wrap(k - 2, nz) * nx + i) * (unsigned)sizeof(T);
        }
    }

    const int j0 = (int)slab * a.slab_rows;
    const int j1 = (j0 + a.slab_rows < M) ? j0 + a.slab_rows : M;
    const int jl = (j1 < M - 1) ? j1 : M - 1;  // last row staged in LDS

    // row j0 - 1: own-column values and the two neighbours the v-point needs
    const T zero = T(0);
    T um = zero, vm = zero, wm = zero, am = zero, bm = zero, fm = zero, pm = zero, u_xp_m = zero, w_zp_m = zero;
    if (j0 > 0 && active) {
        const int q = (j0 - 1) * pl;
        um = F[0][q + e]; vm = F[1][q + e]; wm = F[2][q + e]; am = F[3][q + e]; bm = F[4][q + e];
        fm = F[5][q + e]; pm = F[6][q + e];
        u_xp_m = F[0][q + e_xp];
        w_zp_m = F[2][q + e_zp];
    }
    T c_mm[2] = {zero, zero};  // c+- of row j - 2
    if constexpr (kLim) {
        if (j0 > 1)
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) c_mm[sp] = *byte_at(F[3 + sp], (unsigned)(j0 - 2) * plb + ueb);
    }
    T hold_c[5], hold_n[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        hold_c[f] = (use_old && active) ? ld_once(byte_at((const T *)a.h[f], (unsigned)j0 * plb + ueb)) : zero;
        hold_n[f] = zero;
    }
    {
        HaloRegs<T, kHalo> r0, r1;  // both rows in flight together (above the last row: it again, not used)
        load_rows(j0, r0);
        load_rows(j0 + 1 < M ? j0 + 1 : j0, r1);
        store_rows(j0 & 1, r0);
        store_rows((j0 + 1) & 1, r1);
    }
    __syncthreads();

    HaloRegs<T, kHalo> rn;
    for (int j = j0; j < j1; ++j) {
        const int sc = j & 1, sn = sc ^ 1;
        const bool pre = (j + 2 <= jl);
        // FP64: the wave issuing the next row's loads takes issue priority so
        // they leave before the other waves' arithmetic (measured: 0.418 ->
        // 0.415 ms at 256 x 193 x 256; the FP32 form is slower with it)
        if constexpr (sizeof(T) == 8) __builtin_amdgcn_s_setprio(2);
        if (pre) load_rows(j + 2, rn);  // lands in LDS after this row
        if (use_old && active && j + 1 < j1) {
#pragma unroll
            for (int f = 0; f < 5; ++f) hold_n[f] = ld_once(byte_at((const T *)a.h[f], (unsigned)(j + 1) * plb + ueb));
        }
        if constexpr (sizeof(T) == 8) __builtin_amdgcn_s_setprio(0);
        T far[2][5];  // c+- of row j at the four, and of row j + 2
        if constexpr (kLim) {
            const unsigned row = (unsigned)j * plb, up2 = (unsigned)(j + 2 < M ? j + 2 : M - 1) * plb + ueb;
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) {
#pragma unroll
                for (int q = 0; q < 4; ++q) far[sp][q] = *byte_at(F[3 + sp], row + two_off[q]);
                far[sp][4] = *byte_at(F[3 + sp], up2);
            }
        }
        const bool has_up = (j + 1 < M), has_dn = (j > 0);
        const unsigned qb = (unsigned)j * plb + ueb;  // this cell, bytes
        if (active) {
            const T idn = T(uniform_load(a.tb.idn, j));
            const T idcb = T(uniform_load(a.tb.idc, j)), idct = T(uniform_load(a.tb.idc, j + 1));
            const T uc = X(sc, 0, 0, 0), vc = X(sc, 1, 0, 0), wc = X(sc, 2, 0, 0);
            const T ac = X(sc, 3, 0, 0), bc = X(sc, 4, 0, 0), ph0 = X(sc, 5, 0, 0), pc = X(sc, 6, 0, 0);
            const T up_ = has_up ? X(sn, 0, 0, 0) : zero, vp = has_up ? X(sn, 1, 0, 0) : zero;
            const T wp = has_up ? X(sn, 2, 0, 0) : zero, ap = has_up ? X(sn, 3, 0, 0) : zero;
            const T bp = has_up ? X(sn, 4, 0, 0) : zero, fp = has_up ? X(sn, 5, 0, 0) : zero;
            const T rho0 = ac - bc;
            const T uxp = X(sc, 0, 1, 0), wzp = X(sc, 2, 0, 1);

            // (delta: added to H, and dt gam times it to r, each rounded as a pass
            // over the stored values rounds them)
            auto emit = [&](int f, T hval, T gp, T nu_ly, T delta) {
                if constexpr (mode == 1) {
                    a.dbg[f][(size_t)j * (size_t)pl + (unsigned)e] = (double)hval;
                    return;
                }
                T rv = dt * (gam * hval + zet * hold_c[f] - alp * gp + alp * nu_ly);
                if constexpr (kLim) {
                    if (f >= 3) {
                        asm("" : "+v"(rv));  // (not merged into the sums below)
                        asm("" : "+v"(hval));
                        rv = __builtin_fmaf(dt * gam, delta, rv);
                        hval = hval + delta;
                    }
                }
                st_once(byte_at((T *)a.r[f], qb), rv);
                if (keep) st_once(byte_at((T *)a.h[f], qb), hval);
            };

            // ---------------- u on the x-face ----------------
            {
                const T uxm = X(sc, 0, -1, 0), uzp = X(sc, 0, 0, 1), uzm = X(sc, 0, 0, -1);
                const T a1 = half * (uxp + uc), a2 = half * (uc + uxm);
                const T cx = (a1 * a1 - a2 * a2) * idx_;
                T flux_t = T(0), flux_b = T(0), ut = T(ph.u_top), ub = T(ph.u_bot);
                if (has_up) {
                    ut = up_;
                    flux_t = half * (vp + X(sn, 1, -1, 0)) * half * (ut + uc);
                }
                if (has_dn) {
                    ub = um;
                    flux_b = half * (vc + X(sc, 1, -1, 0)) * half * (uc + ub);
                }
                const T cy = (flux_t - flux_b) * idn;
                const T wf = half * (wzp + X(sc, 2, -1, 1));
                const T wb = half * (wc + X(sc, 2, -1, 0));
                const T cz = (wf * half * (uzp + uc) - wb * half * (uc + uzm)) * idz_;
                const T lap = (uxp - two * uc + uxm) * ix2 + (uzp - two * uc + uzm) * iz2;
                const T rhox = X(sc, 3, -1, 0) - X(sc, 4, -1, 0);
                const T f = kf * half * (rho0 + rhox) * (ph0 - X(sc, 5, -1, 0)) * idx_;
                const T ly = ((ut - uc) * idct - (uc - ub) * idcb) * idn;
                const T lapH = imp ? zero : lap, lapI = imp ? lap : zero;
                emit(0, -(cx + cy + cz) + ire * lapH + f, (pc - X(sc, 6, -1, 0)) * idx_, ire * (ly + lapI), zero);
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---------------- w on the z-face ----------------
            {
                const T wzm = X(sc, 2, 0, -1), wxp = X(sc, 2, 1, 0), wxm = X(sc, 2, -1, 0);
                const T a1 = half * (wzp + wc), a2 = half * (wc + wzm);
                const T cz = (a1 * a1 - a2 * a2) * idz_;
                const T ur = half * (uxp + X(sc, 0, 1, -1));
                const T ul = half * (uc + X(sc, 0, 0, -1));
                const T cx = (ur * half * (wxp + wc) - ul * half * (wc + wxm)) * idx_;
                T flux_t = T(0), flux_b = T(0), wt = T(0), wb = T(0);
                if (has_up) {
                    wt = wp;
                    flux_t = half * (vp + X(sn, 1, 0, -1)) * half * (wt + wc);
                }
                if (has_dn) {
                    wb = wm;
                    flux_b = half * (vc + X(sc, 1, 0, -1)) * half * (wc + wb);
                }
                const T cy = (flux_t - flux_b) * idn;
                const T lap = (wxp - two * wc + wxm) * ix2 + (wzp - two * wc + wzm) * iz2;
                const T rhoz = X(sc, 3, 0, -1) - X(sc, 4, 0, -1);
                const T f = kf * half * (rho0 + rhoz) * (ph0 - X(sc, 5, 0, -1)) * idz_;
                const T ly = ((wt - wc) * idct - (wc - wb) * idcb) * idn;
                const T lapH = imp ? zero : lap, lapI = imp ? lap : zero;
                emit(2, -(cx + cy + cz) + ire * lapH + f, (pc - X(sc, 6, 0, -1)) * idz_, ire * (ly + lapI), zero);
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---------------- v on the bottom y-face of row j ----------------
            if (has_dn) {
                const T vwl = T(uniform_load(a.tb.vwl, j)), vwu = T(uniform_load(a.tb.vwu, j));
                const T idn_lo = T(uniform_load(a.tb.idn, j - 1));
                const T vtop = has_up ? vp : T(0);
                const T vbot = (j > 1) ? vm : T(0);
                const T a1 = half * (vtop + vc), a2 = half * (vc + vbot);
                const T cy = (a1 * a1 - a2 * a2) * idcb;
                const T ur = u_xp_m * vwl + uxp * vwu;
                const T ul = um * vwl + uc * vwu;
                const T vxp = X(sc, 1, 1, 0), vxm = X(sc, 1, -1, 0), vzp = X(sc, 1, 0, 1), vzm = X(sc, 1, 0, -1);
                const T cx = (ur * half * (vxp + vc) - ul * half * (vc + vxm)) * idx_;
                const T wf = w_zp_m * vwl + wzp * vwu;
                const T wbk = wm * vwl + wc * vwu;
                const T cz = (wf * half * (vzp + vc) - wbk * half * (vc + vzm)) * idz_;
                const T lap = (vxp - two * vc + vxm) * ix2 + (vzp - two * vc + vzm) * iz2;
                const T rhoy = am - bm;
                const T ey = e0 + (ph0 - fm) * idcb;
                const T f = kf * half * (rho0 + rhoy) * ey;
                const T ly = ((vtop - vc) * idn - (vc - vbot) * idn_lo) * idcb;
                const T lapH = imp ? zero : lap, lapI = imp ? lap : zero;
                emit(1, -(cx + cy + cz) + ire * lapH + f, (pc - pm) * idcb, ire * (ly + lapI), zero);
            } else {
                emit(1, T(0), T(0), T(0), zero);
                if constexpr (mode == 0) st_once(byte_at((T *)a.r[1], qb), T(0));
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---------------- ions at the cell centre ----------------
            {
                const T fxp = X(sc, 5, 1, 0), fxm = X(sc, 5, -1, 0), fzp = X(sc, 5, 0, 1), fzm = X(sc, 5, 0, -1);
                const T gx_r = (fxp - ph0) * idx_, gx_l = (ph0 - fxm) * idx_;
                const T gz_f = (fzp - ph0) * idz_, gz_b = (ph0 - fzm) * idz_;
                const T ey_t = has_up ? e0 + (fp - ph0) * idct : T(0);
                const T ey_b = has_dn ? e0 + (ph0 - fm) * idcb : T(0);
                const T vt = has_up ? vp : T(0);
                // potential differences across the six faces (the hybrid
                // migration rule's switch; block-uniform hyb)
                const bool hyb = ph.hybrid != 0.0;
                const T dpx_r = fxp - ph0, dpx_l = ph0 - fxm, dpz_f = fzp - ph0, dpz_b = ph0 - fzm;
                T dpy_t = T(0), dpy_b = T(0);
                if (hyb) {
                    if (has_up) dpy_t = y_dphi(e0, T(uniform_load(a.tb.dc, j + 1)), fp - ph0);
                    if (has_dn) dpy_b = y_dphi(e0, T(uniform_load(a.tb.dc, j)), ph0 - fm);
                }
#pragma unroll
                for (int sp = 0; sp < 2; ++sp) {
                    const int fi = 3 + sp;
                    const T zs = sp == 0 ? T(1) : T(-1);
                    const T cc = sp == 0 ? ac : bc;
                    const T cu = sp == 0 ? ap : bp;
                    const T cd = sp == 0 ? am : bm;
                    const T cxp = X(sc, fi, 1, 0), cxm = X(sc, fi, -1, 0), czp = X(sc, fi, 0, 1), czm = X(sc, fi, 0, -1);
                    const T fxr = half * (cxp + cc), fxl = half * (cc + cxm);
                    const T fzf = half * (czp + cc), fzb = half * (cc + czm);
                    const T ax = (uxp * fxr - uc * fxl) * idx_;
                    const T az = (wzp * fzf - wc * fzb) * idz_;
                    T at = T(0), ab = T(0), mt = T(0), mb = T(0), dft = T(0), dfb = T(0);
                    if (has_up) {
                        const T fy = half * (cu + cc);
                        at = vt * fy;
                        mt = mig_face(hyb, fy, cc, cu, dpy_t, zs) * ey_t;
                        dft = (cu - cc) * idct;
                    }
                    if (has_dn) {
                        const T fy = half * (cc + cd);
                        ab = vc * fy;
                        mb = mig_face(hyb, fy, cd, cc, dpy_b, zs) * ey_b;
                        dfb = (cc - cd) * idcb;
                    }
                    const T ay = (at - ab) * idn;
                    const T mx = (mig_face(hyb, fxr, cc, cxp, dpx_r, zs) * gx_r -
                                  mig_face(hyb, fxl, cxm, cc, dpx_l, zs) * gx_l) * idx_;
                    const T mz = (mig_face(hyb, fzf, cc, czp, dpz_f, zs) * gz_f -
                                  mig_face(hyb, fzb, czm, cc, dpz_b, zs) * gz_b) * idz_;
                    const T my = (mt - mb) * idn;
                    const T dxx = (cxp - two * cc + cxm) * ix2 + (czp - two * cc + czm) * iz2;
                    const T dxxH = imp ? zero : dxx;
                    const T diffI = imp ? kd * ((dft - dfb) * idn + dxx) : kd * (dft - dfb) * idn;
                    T delta = zero;
                    if constexpr (kLim) {
                        const T q[8] = {cxp, cxm, far[sp][0], far[sp][1], czp, czm, far[sp][2], far[sp][3]};
                        const T col[5] = {c_mm[sp], cd, cc, cu, far[sp][4]};
                        delta = limit_delta(q, col, uxp, uc, wzp, wc, vt, has_dn ? vc : zero, j, M, idx_, idz_, idn);
                    }
                    emit(fi, -(ax + ay + az) + kd * (dxxH + zs * (mx + my + mz)), T(0), diffI, delta);
                }
            }
            // carry row j as row j - 1 of the next step
            if constexpr (kLim) {
                c_mm[0] = am;
                c_mm[1] = bm;
            }
            um = uc; vm = vc; wm = wc; am = ac; bm = bc; fm = ph0; pm = pc;
            u_xp_m = uxp;
            w_zp_m = wzp;
        }
#pragma unroll
        for (int f = 0; f < 5; ++f) hold_c[f] = hold_n[f];
        __syncthreads();  // every wave is done with slot sc (row j)
        if (pre) store_rows(sc, rn);
        __syncthreads();
    }
}

struct CnArgs {
    Dims d;
    size_t ms;
    Stage st;
    void *q[5];
    void *r[5];          // right-hand sides, state type
    const double *coef;  // per stage: [3 systems][g, m, n][cn_rows(M)]
    int out_r;           // 1: the solution replaces r (a factor of the three-direction factorisation)
};

// Row coefficients of the Crank-Nicolson matrix (I - beta L_y) of system
// sys: 0 = cell rows with wall values (u, w), 1 = interior nodes (v),
// 2 = cell rows with zero-flux walls (c+, c-).  lo/up are the L_y
// coefficient tables of the system's rows (node rows for sys 1).
__device__ __forceinline__ void cn_row(const double *lo_tab, const double *up_tab, int sys, int M, int j,
                                       double beta, double &A, double &B, double &C) {
    double lo, up, di;
    const double aa = lo_tab[j], cc = up_tab[j];
    if (sys == 1) {
        lo = (j > 1) ? aa : 0.0;
        up = (j < M - 1) ? cc : 0.0;
        di = -(aa + cc);
    } else {
        lo = (j > 0) ? aa : 0.0;
        up = (j < M - 1) ? cc : 0.0;
        di = -(lo + up);
        if (sys == 0) {
            if (j == 0) di -= aa;
            if (j == M - 1) di -= cc;
        }
    }
    A = -beta * lo;
    B = 1.0 - beta * di;
    C = -beta * up;
}


// The matrix is the same for every (x, z) column, so Thomas elimination
// reduces to two linear recurrences with column-independent coefficients:
//   d'_j = g_j r_j + m_j d'_{j-1},   x_j = d'_j + n_j x_{j+1}
// with g = 1/den, m = -A/den, n = -c' (den, c' of the Thomas forward pass).
// One block per member, Runge-Kutta stage (blockIdx.y) and system
// (blockIdx.x): the matrix rows are formed by all threads into LDS, one
// thread runs the (serial) forward pass from LDS, and the block stores its
// 3 cn_rows(M) coefficients with coalesced writes, zeros past the last row
// and, for the nodes, in row 0 (the wall: no unknown).  Launched once per
// Runge-Kutta step (dt changes only at the first stage).
// It first combines the partials of the step's reductions (nparts of them, 0: dt
// stays): the step dt (adaptive runs only, Sec. II time stepping with the limits
// of include/nspnp.h) and the sticky health word.  Every block forms them, the
// first of a member stores them, without a launch of its own (32 x 33 x 32: 6.3
// us against 3.2 and 4.3; 128 x 129 x 128 14.9 against 4.8 and 11.5).
__device__ __forceinline__ double dt_close(int nparts, const double *part, const Phys &ph, const Dims &d, double *clock,
                                           bool store, double (*s)[4]) {
    double acc[kDtParts] = {0.0, 0.0, 1e300, 0.0, 0.0};
    for (int b = threadIdx.x; b < nparts; b += blockDim.x) {
        acc[0] = fmax(acc[0], part[kDtParts * b + 0]);
        acc[1] = fmax(acc[1], part[kDtParts * b + 1]);
        acc[2] = fmin(acc[2], part[kDtParts * b + 2]);
        acc[3] = fmax(acc[3], part[kDtParts * b + 3]);
        acc[4] = fmax(acc[4], part[kDtParts * b + 4]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int q = 0; q < kDtParts; ++q) {
            const double v = __shfl_xor(acc[q], o, 64);
            acc[q] = q == 2 ? fmin(acc[q], v) : fmax(acc[q], v);
        }
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < kDtParts; ++q) s[q][threadIdx.x >> 6] = acc[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kDtParts; ++q) {
        acc[q] = s[q][0];
        for (int w = 1; w < 4; ++w) acc[q] = q == 2 ? fmin(acc[q], s[q][w]) : fmax(acc[q], s[q][w]);
    }
    const double re = ph.re, rs = 1.0 / ph.kd;
    double dt = 1e30;
    if (acc[0] > 0.0) dt = ph.cfl / acc[0];
    if (acc[1] > 0.0) dt = fmin(dt, 2.0 * ph.debye * ph.debye * rs / acc[1]);
    const double nu_min = re < rs ? re : rs;
    if (ph.implicit_xz == 0.0)  // explicit x/z diffusion limit
        dt = fmin(dt, nu_min / (4.0 / (d.dx * d.dx) + 4.0 / (d.dz * d.dz)));
    const bool adaptive = ph.adaptive != 0.0, good = dt > 0.0 && __builtin_isfinite(dt);
    if (store && threadIdx.x == 0) {
        int bits = (int)clock[2];
        if (acc[3] != 0.0) bits |= kHealthNonFinite;
        if (acc[2] < 0.0) bits |= kHealthNegative;
        if (adaptive) {
            if (!good) bits |= kHealthNonFinite;
            else clock[1] = dt;
        }
        clock[2] = (double)bits;
        clock[3] = acc[4];
    }
    // (clock[1] is not stored to in the cases in which it is read)
    return adaptive && good ? dt : clock[1];
}

struct CnStages {
    double alp[3];
};

__global__ void __launch_bounds__(256) k_cn_coef(Dims d, Tables tb, const Phys *phys, double *clock, double *coef,
                                                 CnStages stages, int nparts, const double *part, size_t ms) {
    __shared__ double s_dt[kDtParts][4];
    __shared__ double s_a[kMaxRows + kCnPad], s_b[kMaxRows + kCnPad], s_c[kMaxRows + kCnPad];
    phys = member_ptr(phys, ms);
    clock = member_ptr(clock, ms);
    const int M = d.M, Mp = cn_rows(M);
    const int stage = blockIdx.y, sys = blockIdx.x;
    coef = member_ptr(coef, ms) + (size_t)stage * cn_stage_stride(M) + (size_t)sys * 3 * Mp;
    const double nu = (sys == 2) ? phys->kd : phys->ire;
    const double dt =
        nparts ? dt_close(nparts, member_ptr(part, ms), *phys, d, clock, stage == 0 && sys == 0, s_dt) : clock[1];
    const double beta = 0.5 * stages.alp[stage] * dt * nu;
    const double *lo_tab = sys == 1 ? tb.lyn_lo : tb.lyc_lo, *up_tab = sys == 1 ? tb.lyn_up : tb.lyc_up;
    const int j0 = (sys == 1) ? 1 : 0;
    for (int j = threadIdx.x; j < Mp; j += blockDim.x) {
        double A = 0.0, B = 1.0, C = 0.0;
        if (j >= j0 && j < M) cn_row(lo_tab, up_tab, sys, M, j, beta, A, B, C);
        s_a[j] = A;
        s_b[j] = B;
        s_c[j] = C;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // batches of kB rows, loaded together ahead of the dependent chain
        // (padding rows: A = C = 0)
        constexpr int kB = 8;
        static_assert(kCnPad % kB == 0, "whole batches");
        double cprev = 0.0;
        for (int jb = 0; jb < M; jb += kB) {
            double A[kB], B[kB], C[kB];
#pragma unroll
            for (int t = 0; t < kB; ++t) {
                A[t] = s_a[jb + t];
                B[t] = s_b[jb + t];
                C[t] = s_c[jb + t];
            }
#pragma unroll
            for (int t = 0; t < kB; ++t) {
                const double rden = 1.0 / (B[t] - A[t] * cprev);
                cprev = C[t] * rden;
                s_a[jb + t] = rden;
                s_b[jb + t] = -A[t] * rden;
                s_c[jb + t] = -cprev;
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < Mp; j += blockDim.x) {
        const bool in = j >= j0 && j < M;
        coef[j] = in ? s_a[j] : 0.0;
        coef[Mp + j] = in ? s_b[j] : 0.0;
        coef[2 * Mp + j] = in ? s_c[j] : 0.0;
    }
}

// ---- FP64, up to kCnLaneRows rows ----
// Columns staged per block: 16 (one 128-byte line per row) for blocks of up
// to 256 threads, 32 for 512-thread blocks.
inline int cn_tile_cols(int threads) { return threads > 256 ? 32 : 16; }

// Crank-Nicolson solve of one tile of kCnTx columns: the rows of r are staged
// in LDS with coalesced loads; each wave then solves one column at a time
// with its rows split into 64 contiguous lane segments.  Each recurrence is
// a local sweep per lane followed by a 6-step scan of affine maps across the
// wave (x -> T + Q x composed lane by lane) and a second local sweep from the
// correct incoming value.  Finally q += x with coalesced stores.
// Staging in batches of kCnBatch loads per thread in flight per wait: 6,
// measured best (more registers cost occupancy), or all of up to 64 rows.
// Bound by memory: 0.273 ms at 256 x 193 x 256 (5.5 TB/s).
constexpr int kCnLaneRows = 320;

template <int kCnTx, int kCnMaxR, int W>
__global__ void __launch_bounds__(512) k_cn_scan(CnArgs a) {
    using T = double;
    constexpr int kCnBatch = kCnMaxR == 1 ? 4 : 6, kSteps = W == 64 ? 6 : (W == 32 ? 5 : 4);
    constexpr bool kAhead = kCnMaxR == 1;
    extern __shared__ double s_r[];
    const uint3 blk = xcd_block3();  // adjacent column tiles share an L2
    const int f = (int)blk.y;
    const size_t ms = a.ms;
    const int sys = (f == 1) ? 1 : (f >= 3 ? 2 : 0);
    const int j0 = (sys == 1) ? 1 : 0;
    const int M = a.d.M;
    const int64_t pl = a.d.plane;
    const int64_t c0 = (int64_t)blk.x * kCnTx;
    const int ncol = (int)((pl - c0) < kCnTx ? (pl - c0) : kCnTx);
    const T *r = (const T *)member_ptr_at(a.r[f], ms, blk.z);  // may be rewritten in place (out_r)
    T *__restrict__ q = (T *)member_ptr_at(a.q[f], ms, blk.z);
    const double *__restrict__ coef =
        member_ptr_at(a.coef, ms, blk.z) + (size_t)a.st.k * cn_stage_stride(M) + (size_t)sys * 3 * cn_rows(M);
    const double *__restrict__ cg = coef, *__restrict__ cm = coef + cn_rows(M), *__restrict__ cn = coef + 2 * cn_rows(M);
    constexpr int LD = kCnTx + 1;
    const int nrow = M - j0;
    const int ntile = nrow * kCnTx, bd = (int)blockDim.x;
    const int lane = threadIdx.x % W, wave = threadIdx.x / W, nwave = blockDim.x / W;  // (groups of W lanes)
    const int R = kCnMaxR;  // rows per lane (the launcher picks ceil(rows / 64))
    const int js = j0 + lane * R;
    // this lane's recurrence coefficients (the same for every column)
    double g[kCnMaxR], mm[kCnMaxR], nn[kCnMaxR];
    auto load_coef = [&] {
#pragma unroll
        for (int t = 0; t < kCnMaxR; ++t) {
            const int j = js + t < M ? js + t : M - 1;
            g[t] = cg[j];
            mm[t] = cm[j];
            nn[t] = cn[j];
        }
    };
    // One row per lane: the coefficients, and below the first values of q, go
    // out with the loads of r (latency; with more rows their registers cost
    // more: 256 x 193 x 256 279 against 287 us)
    if (kAhead) load_coef();
    // Staging in batches of kCnBatch unconditional loads per thread (lanes
    // past the tile read its first element, which exists, and discard it), so
    // that a thread waits for memory once per batch, not once per element.
    // (offsets within one field: rows * plane < 2^32 for every supported grid)
    const unsigned upl = (unsigned)pl, uc0 = (unsigned)c0;
    const unsigned o_safe = (unsigned)j0 * upl + uc0;
    for (int e0 = threadIdx.x; e0 < ntile; e0 += kCnBatch * bd) {
        T v[kCnBatch];
#pragma unroll
        for (int u = 0; u < kCnBatch; ++u) {
            const int e = e0 + u * bd, jj = j0 + e / kCnTx, c = e % kCnTx;
            v[u] = ld_once(r + ((e < ntile && c < ncol) ? (unsigned)jj * upl + uc0 + (unsigned)c : o_safe));
        }
#pragma unroll
        for (int u = 0; u < kCnBatch; ++u) {
            const int e = e0 + u * bd, jj = j0 + e / kCnTx, c = e % kCnTx;
            if (e < ntile) s_r[jj * LD + c] = (c < ncol) ? (double)v[u] : 0.0;
        }
    }
    T qv[kCnBatch];
    auto load_q = [&](int e0) {
#pragma unroll
        for (int u = 0; u < kCnBatch; ++u) {
            const int e = e0 + u * bd, jj = j0 + e / kCnTx, c = e % kCnTx;
            qv[u] = ld_once(q + ((e < ntile && c < ncol) ? (unsigned)jj * upl + uc0 + (unsigned)c : o_safe));
        }
    };
    if (kAhead && !a.out_r) load_q((int)threadIdx.x);
    __syncthreads();
    if (!kAhead) load_coef();
    double Qs = 1.0, Ss = 1.0;
#pragma unroll
    for (int t = 0; t < kCnMaxR; ++t) {
        const bool in = js + t < M;
        g[t] = in ? g[t] : 0.0;
        mm[t] = in ? mm[t] : 1.0;
        nn[t] = in ? nn[t] : 1.0;
        Qs *= mm[t];
        Ss *= nn[t];
    }
    // multipliers of the scans of the affine maps x -> T + Q x across lanes
    // (forward, from lane 0 up) and x -> U + S x (backward, from lane 63 down)
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
    for (int c = wave; c < ncol; c += nwave) {
        double *col = s_r + c;
        double x[kCnMaxR];
#pragma unroll
        for (int t = 0; t < kCnMaxR; ++t) {
            const int j = js + t;
            x[t] = (t < R && j < M) ? col[j * LD] : 0.0;
        }
        // forward d'_j = g_j r_j + m_j d'_{j-1}: local sweep, scan, sweep
        double Tf = 0.0;
#pragma unroll
        for (int t = 0; t < kCnMaxR; ++t) Tf = g[t] * x[t] + mm[t] * Tf;
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const double Tp = __shfl_up(Tf, 1 << st, W);
            if (lane >= (1 << st)) Tf += qm[st] * Tp;
        }
        double din = __shfl_up(Tf, 1, W);
        if (lane == 0) din = 0.0;
#pragma unroll
        for (int t = 0; t < kCnMaxR; ++t) {
            din = g[t] * x[t] + mm[t] * din;
            x[t] = din;
        }
        // backward x_j = d'_j + n_j x_{j+1}
        double U = 0.0;
#pragma unroll
        for (int t = kCnMaxR - 1; t >= 0; --t) U = (g[t] != 0.0 ? x[t] : 0.0) + nn[t] * U;
#pragma unroll
        for (int st = 0; st < kSteps; ++st) {
            const double Up = __shfl_down(U, 1 << st, W);
            if (lane + (1 << st) < W) U += sm[st] * Up;
        }
        double xin = __shfl_down(U, 1, W);
        if (lane == W - 1) xin = 0.0;
#pragma unroll
        for (int t = kCnMaxR - 1; t >= 0; --t) {
            xin = (g[t] != 0.0 ? x[t] : 0.0) + nn[t] * xin;
            x[t] = xin;
        }
#pragma unroll
        for (int t = 0; t < kCnMaxR; ++t) {
            const int j = js + t;
            if (t < R && j < M) col[j * LD] = x[t];
        }
    }
    __syncthreads();
    if (a.out_r) {  // a factor of the three-direction factorisation: the solution replaces r
        T *rw = (T *)member_ptr_at(a.r[f], ms, blk.z);  // r was read before the barrier
        for (int e = threadIdx.x; e < ntile; e += bd) {
            const int jj = j0 + e / kCnTx, c = e % kCnTx;
            if (c < ncol) st_once(rw + ((unsigned)jj * upl + uc0 + (unsigned)c), (T)s_r[jj * LD + c]);
        }
        return;
    }
    for (int e0 = threadIdx.x; e0 < ntile; e0 += kCnBatch * bd) {
        if (!kAhead || e0 != (int)threadIdx.x) load_q(e0);
#pragma unroll
        for (int u = 0; u < kCnBatch; ++u) {
            const int e = e0 + u * bd, jj = j0 + e / kCnTx, c = e % kCnTx;
            if (e < ntile && c < ncol) st_once(q + ((unsigned)jj * upl + uc0 + (unsigned)c), (T)((double)qv[u] + s_r[jj * LD + c]));
        }
    }
}

// ---- the mixed form, and FP64 above kCnLaneRows rows ----
// Crank-Nicolson solve of the five fields in one pass.  A block owns kCx
// neighbouring columns of one field over all rows; its threads split the rows
// into slabs of L.  Each thread holds its L rows in registers: the forward
// sweep with a zero input, l; the inputs of the slabs from their exits and
// the products of m (a scan over the slabs below, through LDS); l plus the
// input times the running product of m; then the backward sweep the same way.
// r and q are read once and q written once (kOut: the solution replaces r,
// a factor of the three-direction factorisation), every access a run of kCx
// neighbouring values.  64 columns: a wave is one slab, its recurrence
// coefficients wave-uniform (scalar loads); 32 columns (more than 16 slabs of
// 16 rows): two slabs a wave, the coefficients from LDS.
// Bound by memory (15 values a cell): 512 x 385 x 512 FP64 2.34 ms (5.2 TB/s),
// mixed 1.11 ms (5.4 TB/s); 256 x 193 x 256 mixed 0.130 ms.  The lane scans
// took 3.65, 2.37 and 0.191 ms (short runs of a row, and shuffles); a
// three-pass form, its first pass in the explicit kernel, 2.29 ms and 0.15 ms
// more in that kernel.  Not by default for FP64 columns of up to kCnLaneRows
// rows, though it is faster there too (0.256 against 0.273 ms at 256 x 193 x
// 256, 48 against 51 us at 128 x 129 x 128): the lane scans keep the results of
// such runs bit for bit, down to plane means that are zero but for rounding.
// cnslab 16 or 32 asks for it.
template <typename T, int L, int kCx, bool kOut>
__global__ void __launch_bounds__(1024) k_cn_rows(CnArgs a) {
    extern __shared__ double s_x[];  // exits [slab][kCx], the slabs' products, (kCx 32) the coefficients
    const uint3 blk = xcd_block3();  // adjacent column tiles share an L2
    const int f = (int)blk.y;
    const int sys = (f == 1) ? 1 : (f >= 3 ? 2 : 0);
    const int M = a.d.M, Mp = cn_rows(M);
    const int S = (int)blockDim.x / kCx;
    const int col = (int)threadIdx.x % kCx;
    int slab = (int)threadIdx.x / kCx;
    if constexpr (kCx == 64) slab = __builtin_amdgcn_readfirstlane(slab);
    const unsigned upl = (unsigned)a.d.plane;
    const unsigned c = blk.x * (unsigned)kCx + (unsigned)col;
    const bool in = c < upl;
    const unsigned uc = in ? c : upl - 1;  // (columns past the plane repeat its last one and store nothing)
    T *r = (T *)member_ptr_at(a.r[f], a.ms, blk.z);
    T *q = (T *)member_ptr_at(a.q[f], a.ms, blk.z);
    const int j0 = slab * L;
    // row t of the slab at this column (64 columns: a wave-uniform row base and
    // the column's 32-bit offset); rows past the last repeat it (their
    // coefficients are zero)
    auto at = [&](T *p, int t) -> T * {
        const int j = j0 + t < M ? j0 + t : M - 1;
        if constexpr (kCx == 64) return byte_at(p + (size_t)j * upl, uc * (unsigned)sizeof(T));
        else return p + ((unsigned)j * upl + uc);
    };
    T rv[L];
#pragma unroll
    for (int t = 0; t < L; ++t) rv[t] = ld_once(at(r, t));
    const double *coef = member_ptr_at(a.coef, a.ms, blk.z) + (size_t)a.st.k * cn_stage_stride(M) + (size_t)sys * 3 * Mp;
    double *s_p = s_x + S * kCx, *s_c = s_p + S;
    typedef const __attribute__((address_space(4))) double cdouble;
    cdouble *ug = (cdouble *)(coef + (kCx == 64 ? j0 : 0));
    if constexpr (kCx != 64) {
        for (int e = threadIdx.x; e < 3 * Mp; e += blockDim.x) s_c[e] = coef[e];
        __syncthreads();
    }
    auto cg = [&](int t) { return kCx == 64 ? ug[t] : s_c[j0 + t]; };
    auto cm = [&](int t) { return kCx == 64 ? ug[Mp + t] : s_c[Mp + j0 + t]; };
    auto cn = [&](int t) { return kCx == 64 ? ug[2 * Mp + t] : s_c[2 * Mp + j0 + t]; };
    double x[L];
    double P = 1.0, d = 0.0;
#pragma unroll
    for (int t = 0; t < L; ++t) {
        d = cg(t) * (double)rv[t] + cm(t) * d;
        x[t] = d;
        P *= cm(t);
    }
    s_x[slab * kCx + col] = d;
    if (col == 0) s_p[slab] = P;
    // q is loaded while the exits travel; FP64 slabs of 24 rows load its second
    // half after the first has been stored (all of it early would spill: 2.47
    // against 2.34 ms at 512 x 385 x 512)
    constexpr int QE = (sizeof(T) == 8 && L == 24) ? 12 : L;
    T qv[QE];
    if constexpr (!kOut) {
#pragma unroll
        for (int t = 0; t < QE; ++t) qv[t] = ld_once(at(q, t));
    }
    __syncthreads();
    double v = 0.0;
    for (int t = 0; t < slab; ++t) v = s_x[t * kCx + col] + s_p[t] * v;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < L; ++t) {
        v *= cm(t);
        x[t] += v;
    }
    P = 1.0;
    d = 0.0;
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        d = x[t] + cn(t) * d;
        x[t] = d;
        P *= cn(t);
    }
    s_x[slab * kCx + col] = d;
    if (col == 0) s_p[slab] = P;
    __syncthreads();
    v = 0.0;
    for (int t = S - 1; t > slab; --t) v = s_x[t * kCx + col] + s_p[t] * v;
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        v *= cn(t);
        x[t] += v;
    }
    if (!in) return;
    // (the wall row of the nodes is no unknown: it keeps its value, also where
    // the rows above are not finite)
    const int jlo = sys == 1 ? 1 : 0;
    if constexpr (kOut) {
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (j0 + t < M && (t > 0 || j0 >= jlo)) st_once(at(r, t), (T)x[t]);
    } else {
#pragma unroll
        for (int t = 0; t < QE; ++t)
            if (j0 + t < M && (t > 0 || j0 >= jlo)) st_once(at(q, t), (T)((double)qv[t] + x[t]));
        if constexpr (QE < L) {
#pragma unroll
            for (int t = QE; t < L; ++t) qv[t - QE] = ld_once(at(q, t));
#pragma unroll
            for (int t = QE; t < L; ++t)
                if (j0 + t < M) st_once(at(q, t), (T)((double)qv[t - QE] + x[t]));
        }
    }
}

// ---- implicit x/z diffusion (three-direction approximate factorisation) ----
// (I - b L) x = r along a periodic line of N points, L = (x_{+1} - 2 x + x_{-1}) / h^2,
// is a cyclic tridiagonal system with constant diagonal d = 1 + 2 b / h^2 and
// off-diagonal e = -b / h^2.  With gamma = -d, the corners move into a rank-one
// term (Sherman-Morrison): the tridiagonal B (first diagonal d - gamma, last
// d - e^2 / gamma) is solved for y = B^-1 r, and x = y - ((y_0 + (e/gamma) y_{N-1})
// / (1 + z_0 + (e/gamma) z_{N-1})) z with z = B^-1 (gamma, 0, .., 0, e).  B and z
// are the same for every line of a field, stage and direction: k_cyc_coef makes
// B's elimination recurrences (d'_i = g_i r_i + m_i d'_{i-1}, x_i = d'_i + n_i
// x_{i+1}) and z once per Runge-Kutta step.
struct CycArgs {
    Dims d;
    size_t ms;
    Stage st;
    void *q[5];
    void *r[5];
    const double *cyc;
    int lines;  // x-lines: lines per wave
};

// One block per stage, diffusivity and direction; one thread runs the serial
// recurrences in LDS, elimination and forward sweep of z together (the
// division of a row is what the chain waits for), and the block stores them.
constexpr int kMaxLine = 1024;

__global__ void __launch_bounds__(64) k_cyc_coef(Dims d, const Phys *phys, const double *clock, double *cyc,
                                                 CnStages stages, size_t ms) {
    __shared__ double s_t[4][kMaxLine];  // g, m, n, z
    phys = member_ptr(phys, ms);
    clock = member_ptr(clock, ms);
    cyc = member_ptr(cyc, ms);
    const int stage = blockIdx.y, sys = blockIdx.x;
    const int ty = sys >> 1, dir = sys & 1;  // diffusivity (velocity, ions), direction
    const int N = dir == 0 ? d.nx : d.nz;
    const double h = dir == 0 ? d.dx : d.dz;
    const double nu = ty == 0 ? phys->ire : phys->kd;
    const double b = 0.5 * stages.alp[stage] * clock[1] * nu;
    const double dg = 1.0 + 2.0 * b / (h * h), e = -b / (h * h), gam = -dg;
    const int64_t nb = cyc_block_doubles(d.nx, d.nz), Nmax = (nb - 4) / 4;
    double *blk = cyc + ((int64_t)(stage * 2 + ty) * 2 + dir) * nb;
    double *g = s_t[0], *m = s_t[1], *n = s_t[2], *z = s_t[3];
    if (threadIdx.x == 0) {
        double cprev = 0.0, dp = 0.0;
        for (int i = 0; i < N; ++i) {
            const double bi = (i == 0) ? dg - gam : (i == N - 1 ? dg - e * e / gam : dg);
            const double ai = (i == 0) ? 0.0 : e;
            const double rden = 1.0 / (bi - ai * cprev);
            const double ci = (i == N - 1) ? 0.0 : e * rden;
            const double mi = -ai * rden;
            g[i] = rden;
            m[i] = mi;
            n[i] = -ci;
            cprev = ci;
            // z = B^-1 u, u = (gamma, 0, ..., 0, e)
            const double ui = (i == 0) ? gam : (i == N - 1 ? e : 0.0);
            dp = rden * ui + mi * dp;
            z[i] = dp;
        }
        for (int i = N - 2; i >= 0; --i) {
            dp = z[i] + n[i] * dp;
            z[i] = dp;
        }
        const double vf = e / gam;
        blk[4 * Nmax] = vf;
        blk[4 * Nmax + 1] = 1.0 / (1.0 + z[0] + vf * z[N - 1]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += 64)
#pragma unroll
        for (int q = 0; q < 4; ++q) blk[q * Nmax + i] = s_t[q][i];
}

// One line over the lanes of a wave, R contiguous points per lane: affine-map
// scans across the wave, then the periodic correction (the line's end values
// y_0, y_{N-1} broadcast from their lanes).  The recurrences' coefficients and
// the scans' multipliers are the same for every line.
template <int R>
struct CycWave {
    double g[R], mm[R], nn[R], zz[R], qm[6], sm[6], vf, sf;
    int lane, last_lane, last_t;
    __device__ __forceinline__ void load(const CycArgs &a, int ty, int dir, unsigned mem, int N) {
        const int64_t nb = cyc_block_doubles(a.d.nx, a.d.nz), Nmax = (nb - 4) / 4;
        const double *cb = member_ptr_at(a.cyc, a.ms, mem) + ((int64_t)(a.st.k * 2 + ty) * 2 + dir) * nb;
        const double *cg = cb, *cm = cb + Nmax, *cn = cb + 2 * Nmax, *cz = cb + 3 * Nmax;
        vf = cb[4 * Nmax];
        sf = cb[4 * Nmax + 1];
        lane = threadIdx.x & 63;
        last_lane = (N - 1) / R;
        last_t = (N - 1) - last_lane * R;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const int i = lane * R + t;
            const bool in = i < N;
            g[t] = in ? cg[i] : 0.0;
            mm[t] = in ? cm[i] : 1.0;
            nn[t] = in ? cn[i] : 1.0;
            zz[t] = in ? cz[i] : 0.0;
        }
    }
    __device__ __forceinline__ void products() {
        double Qs = 1.0, Ss = 1.0;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            Qs *= mm[t];
            Ss *= nn[t];
        }
#pragma unroll
        for (int st = 0; st < 6; ++st) {
            const int sft = 1 << st;
            qm[st] = Qs;
            sm[st] = Ss;
            const double Qp = __shfl_up(Qs, sft, 64), Sp = __shfl_down(Ss, sft, 64);
            if (lane >= sft) Qs *= Qp;
            if (lane + sft < 64) Ss *= Sp;
        }
    }
    // the solution of a line (points past its end: 0 in)
    __device__ __forceinline__ void solve(double *x) const {
        double Tf = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t) Tf = g[t] * x[t] + mm[t] * Tf;
#pragma unroll
        for (int st = 0; st < 6; ++st) {
            const double Tp = __shfl_up(Tf, 1 << st, 64);
            if (lane >= (1 << st)) Tf += qm[st] * Tp;
        }
        double din = __shfl_up(Tf, 1, 64);
        if (lane == 0) din = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t) {
            din = g[t] * x[t] + mm[t] * din;
            x[t] = din;
        }
        double U = 0.0;
#pragma unroll
        for (int t = R - 1; t >= 0; --t) U = (g[t] != 0.0 ? x[t] : 0.0) + nn[t] * U;
#pragma unroll
        for (int st = 0; st < 6; ++st) {
            const double Up = __shfl_down(U, 1 << st, 64);
            if (lane + (1 << st) < 64) U += sm[st] * Up;
        }
        double xin = __shfl_down(U, 1, 64);
        if (lane == 63) xin = 0.0;
#pragma unroll
        for (int t = R - 1; t >= 0; --t) {
            xin = (g[t] != 0.0 ? x[t] : 0.0) + nn[t] * xin;
            x[t] = xin;
        }
        // periodic correction from the line's end values
        double ylast = 0.0;
#pragma unroll
        for (int t = 0; t < R; ++t)
            if (t == last_t) ylast = x[t];
        const double y0 = __shfl(x[0], 0, 64);
        const double yl = __shfl(ylast, last_lane, 64);
        const double wcor = (y0 + vf * yl) * sf;
#pragma unroll
        for (int t = 0; t < R; ++t) x[t] = x[t] - wcor * zz[t];
    }
};

// x-lines, the solution in place of r: contiguous, so each wave takes its
// lines straight from memory, cyc_lines(R) at a time, the next ones' loads in
// flight while these are solved, without block barriers.  Lines whose lanes
// hold more than 16 bytes apiece (R > 2 in FP64, R > 3 in FP32) are loaded and
// stored along the line, whole runs of memory, and turned into the lanes'
// contiguous points in the wave's own piece of LDS: a lane's points taken from
// memory one by one are a part of each 128-byte line R times over.  The three
// solves of the implicit form together (k_cyc_x, the wall-normal solve,
// k_cyc_z), points one by one, turned, and through tiles of 16 lines in LDS:
//   128 x 129 x 128 FP64 (R 2)       149 / -   / 162 us (this kernel 45, 57 in tiles)
//   192 x 129 x 128 FP64 (R 3)       248 / 202 / 221
//   256 x 129 x 128 FP64, mixed      385, 225 / 252, 171 / 284, 248
//   1024 x 129 x 128 FP64, mixed     5705, 2101 / 956, 657 / 1651, 1604
//   144 x 129 x 128 mixed (R 3)      114 / 125 / 164
// Bound by the scans' moves between lanes on short lines (128 points 3.7 TB/s).
constexpr int cyc_lines(int R) { return R <= 2 ? 4 : (R <= 4 ? 2 : 1); }

template <typename T, int R>
__global__ void __launch_bounds__(256) k_cyc_x(CycArgs a) {
    constexpr int kB = cyc_lines(R);
    constexpr bool kTurn = R > (sizeof(T) == 8 ? 2 : 3);
    // (R + 1 slots for each lane's R points: reads along t are free of bank conflicts)
    __shared__ double s_z[kTurn ? 4 * kB * 64 * (R + 1) : 1];
    const int f = (int)blockIdx.y, N = a.d.nx;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nlines = a.d.M * a.d.nz;
    T *rr = (T *)member_ptr_at(a.r[f], a.ms, blockIdx.z);
    CycWave<R> s;
    s.load(a, f < 3 ? 0 : 1, 0, blockIdx.z, N);
    const int js = s.lane * R;
    const int l0 = ((int)blockIdx.x * 4 + wave) * a.lines, l1 = l0 + a.lines < nlines ? l0 + a.lines : nlines;
    if (l0 >= l1) return;
    // point of the line that this lane moves as its t-th
    auto pt = [&](int t) { return kTurn ? s.lane + 64 * t : js + t; };
    double *z = s_z + (kTurn ? wave * kB * 64 * (R + 1) : 0);
    auto slot = [](int b, int i) { return b * 64 * (R + 1) + i + i / R; };
    T v[kB][R];
    // points past the line and lines past the last one read what exists
    auto load = [&](int l) {
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const T *p = rr + (int64_t)(l + b < l1 ? l + b : l1 - 1) * N;
#pragma unroll
            for (int t = 0; t < R; ++t) v[b][t] = ld_once(p + (pt(t) < N ? pt(t) : 0));
        }
    };
    load(l0);
    s.products();
    for (int l = l0; l < l1; l += kB) {
        double x[kB][R];
        if constexpr (kTurn) {
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int t = 0; t < R; ++t) z[slot(b, pt(t))] = pt(t) < N ? (double)v[b][t] : 0.0;
            wave_sync();
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int t = 0; t < R; ++t) x[b][t] = z[slot(b, js) + t];
        } else {
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int t = 0; t < R; ++t) x[b][t] = js + t < N ? (double)v[b][t] : 0.0;
        }
        if (l + kB < l1) load(l + kB);  // lands while these are solved
#pragma unroll
        for (int b = 0; b < kB; ++b) s.solve(x[b]);
        if constexpr (kTurn) {
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int t = 0; t < R; ++t) z[slot(b, js) + t] = x[b][t];
            wave_sync();
#pragma unroll
            for (int b = 0; b < kB; ++b)
#pragma unroll
                for (int t = 0; t < R; ++t) x[b][t] = z[slot(b, pt(t))];
            wave_sync();  // (the slots are written again for the next lines)
        }
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            T *p = rr + (int64_t)(l + b) * N;
#pragma unroll
            for (int t = 0; t < R; ++t)
                if (l + b < l1 && pt(t) < N) st_once(p + pt(t), (T)x[b][t]);
        }
    }
}

// z-lines, added to the fields: one tile of kCycTx neighbouring columns of one
// field per block, staged in LDS in 128-byte runs (FP64), a wave per line.
constexpr int kCycTx = 16;

constexpr int kCycBatch = 8;  // loads per thread per wait

template <typename T, int R>
__global__ void __launch_bounds__(256) k_cyc_z(CycArgs a) {
    extern __shared__ double s_l[];
    const uint3 blk = xcd_block3();
    const int f = (int)blk.y;
    const int nx = a.d.nx, N = a.d.nz;
    const int ntl = (nx + kCycTx - 1) / kCycTx;
    const int j = (int)blk.x / ntl, l0 = ((int)blk.x - j * ntl) * kCycTx;
    const int nl = (nx - l0) < kCycTx ? (nx - l0) : kCycTx;
    const unsigned row = (unsigned)j * (unsigned)a.d.plane;
    const T *rr = (const T *)member_ptr_at(a.r[f], a.ms, blk.z);
    T *qq = (T *)member_ptr_at(a.q[f], a.ms, blk.z);
    constexpr int LD = kCycTx + 1;
    const int ntile = N * kCycTx, bd = (int)blockDim.x;
    // element e of the tile: point i = e / kCycTx of line c = e % kCycTx
    auto addr = [&](int e) -> unsigned { return row + (unsigned)(e / kCycTx) * (unsigned)nx + (unsigned)(l0 + e % kCycTx); };
    for (int e0 = threadIdx.x; e0 < ntile; e0 += kCycBatch * bd) {
        T v[kCycBatch];
#pragma unroll
        for (int u = 0; u < kCycBatch; ++u) {
            const int e = e0 + u * bd;
            v[u] = ld_once(rr + ((e < ntile && e % kCycTx < nl) ? addr(e) : row));
        }
#pragma unroll
        for (int u = 0; u < kCycBatch; ++u) {
            const int e = e0 + u * bd;
            if (e < ntile) s_l[e / kCycTx * LD + e % kCycTx] = (e % kCycTx < nl) ? (double)v[u] : 0.0;
        }
    }
    __syncthreads();
    CycWave<R> s;
    s.load(a, f < 3 ? 0 : 1, 1, blk.z, N);
    s.products();
    const int js = s.lane * R, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    for (int c = wave; c < nl; c += nwave) {
        double *col = s_l + c;
        double x[R];
#pragma unroll
        for (int t = 0; t < R; ++t) x[t] = (js + t < N) ? col[(js + t) * LD] : 0.0;
        s.solve(x);
#pragma unroll
        for (int t = 0; t < R; ++t)
            if (js + t < N) col[(js + t) * LD] = x[t];
    }
    __syncthreads();
    for (int e0 = threadIdx.x; e0 < ntile; e0 += kCycBatch * bd) {
        T v[kCycBatch];
#pragma unroll
        for (int u = 0; u < kCycBatch; ++u) {
            const int e = e0 + u * bd;
            v[u] = ld_once(qq + ((e < ntile && e % kCycTx < nl) ? addr(e) : row));
        }
#pragma unroll
        for (int u = 0; u < kCycBatch; ++u) {
            const int e = e0 + u * bd;
            if (e < ntile && e % kCycTx < nl) st_once(qq + addr(e), (T)((double)v[u] + s_l[e / kCycTx * LD + e % kCycTx]));
        }
    }
}

// projection correction: u -= a G psi;  p += psi - (a / (2 Re)) L_y psi.
// Each thread owns one (x, z) column of a 2-D tile and marches a slab of
// rows, carrying psi of rows j-1 and j, so psi is read about once; its x-
// and z-neighbours in row j come from the caches (mostly the block's own
// loads).
struct CorrArgs {
    Dims d;
    const Phys *phys;
    size_t ms;
    Tables tb;
    void *u, *v, *w, *p;
    const double *psi;
    double *clock;
    double alp;
    double fixed;
    int update_p;
    int advance_clock;
    int tx, tz, ntx, chunks, slabs, slab_rows;
};

constexpr int kCorrRows = 4;  // rows per load batch of k_correct

// kImp: the pressure update takes the full Laplacian of psi (x/z diffusion
// implicit too), p += psi - (a / (2 Re)) (L_x + L_y + L_z) psi.
template <typename T, bool kImp>
__global__ void __launch_bounds__(256) k_correct(CorrArgs a) {
    const Dims &d = a.d;
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);
    const unsigned chunks = (unsigned)a.chunks, slabs = (unsigned)a.slabs;
    const unsigned chunk = tile % chunks;
    const unsigned slab = (tile / chunks) % slabs;
    const unsigned mem = tile / (chunks * slabs);
    const int nx = d.nx, nz = d.nz, M = d.M;
    const int lk = (int)threadIdx.x / a.tx;
    const int i = (int)(chunk % (unsigned)a.ntx) * a.tx + ((int)threadIdx.x - lk * a.tx);
    const int k = (int)(chunk / (unsigned)a.ntx) * a.tz + lk;
    if (lk >= a.tz || i >= nx || k >= nz) return;
    const int64_t pl = d.plane;
    const int e = k * nx + i;
    const int exm = e - i + ((i == 0) ? nx - 1 : i - 1);
    const int ezm = ((k == 0) ? nz - 1 : k - 1) * nx + i;
    const size_t ms = a.ms;
    double *clock = member_ptr_at(a.clock, ms, mem);
    const Phys *ph = member_ptr_at(a.phys, ms, mem);
    const int j0 = (int)slab * a.slab_rows;
    const int j1 = (j0 + a.slab_rows < M) ? j0 + a.slab_rows : M;
    // substep time t += alp dt (dt is read, never written, by this kernel)
    if (a.advance_clock && e == 0 && j0 == 0) clock[0] += a.alp * clock[1];
    T *u = (T *)member_ptr_at(a.u, ms, mem), *v = (T *)member_ptr_at(a.v, ms, mem);
    T *w = (T *)member_ptr_at(a.w, ms, mem), *p = (T *)member_ptr_at(a.p, ms, mem);
    const double *psi = member_ptr_at(a.psi, ms, mem);
    const double sc = (a.alp > 0.0) ? a.alp * clock[1] : a.fixed;
    const double ire = ph->ire;
    const double idx = 1.0 / d.dx, idz = 1.0 / d.dz;
    double s_dn = (j0 > 0) ? psi[(int64_t)(j0 - 1) * pl + e] : 0.0;  // psi of row j - 1
    double s0 = psi[(int64_t)j0 * pl + e];
    // Rows are corrected in batches of kCorrRows: the batch's loads are all
    // issued before any result is stored (rows past the slab re-read its last
    // row and are ignored), one memory latency per batch.  Offsets within one
    // field fit in 32 bits.
    const unsigned upl = (unsigned)pl;
    struct RowVals {
        double s_up, sxm, szm, sxp, szp;
        T u, v, w, p;
    };
    const int exp_ = e - i + ((i + 1 == nx) ? 0 : i + 1);
    const int ezp = ((k + 1 == nz) ? 0 : k + 1) * nx + i;
    auto load_row = [&](int j, RowVals &r) {
        const unsigned row = (unsigned)j * upl, q = row + (unsigned)e;
        r.s_up = psi[(j + 1 < M) ? q + upl : q];
        r.sxm = psi[row + (unsigned)exm];
        r.szm = psi[row + (unsigned)ezm];
        if (kImp) {
            r.sxp = psi[row + (unsigned)exp_];
            r.szp = psi[row + (unsigned)ezp];
        }
        r.u = ld_once(u + q);
        r.w = ld_once(w + q);
        r.v = ld_once(v + q);
        r.p = ld_once(p + q);  // unconditional (p is always allocated): no branch in the batch
    };
    for (int jb = j0; jb < j1; jb += kCorrRows) {
        RowVals rb[kCorrRows];
#pragma unroll
        for (int t = 0; t < kCorrRows; ++t) load_row(jb + t < j1 ? jb + t : j1 - 1, rb[t]);
#pragma unroll
        for (int t = 0; t < kCorrRows; ++t) {
            const int j = jb + t;
            if (j >= j1) break;
            const RowVals &cur = rb[t];
            const unsigned q = (unsigned)j * upl + (unsigned)e;
            const double s_up = (j + 1 < M) ? cur.s_up : 0.0;
            st_once(u + q, (T)((double)cur.u - sc * (s0 - cur.sxm) * idx));
            st_once(w + q, (T)((double)cur.w - sc * (s0 - cur.szm) * idz));
            const double idcb = uniform_load(a.tb.idc, j);
            if (j > 0) st_once(v + q, (T)((double)cur.v - sc * (s0 - s_dn) * idcb));
            if (a.update_p) {
                const double ft = (j + 1 < M) ? (s_up - s0) * uniform_load(a.tb.idc, j + 1) : 0.0;
                const double fb = (j > 0) ? (s0 - s_dn) * idcb : 0.0;
                double ly = (ft - fb) * uniform_load(a.tb.idn, j);
                if (kImp)
                    ly += (cur.sxp - 2.0 * s0 + cur.sxm) * (idx * idx) + (cur.szp - 2.0 * s0 + cur.szm) * (idz * idz);
                st_once(p + q, (T)((double)cur.p + s0 - 0.5 * sc * ire * ly));
            }
            s_dn = s0;
            s0 = s_up;
        }
    }
}

template <typename Src, typename Dst>
__global__ void __launch_bounds__(256) k_copy_convert(int64_t n, const Src *in, Dst *out) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    out[q] = (Dst)in[q];
}

inline dim3 grid1(int64_t n, int b = 256) { return dim3((unsigned)((n + b - 1) / b)); }

}  // namespace

// Rows that one block of a row march takes: `rows`, halved while it is above
// `least` and leaves the chip with fewer than two blocks per CU.  A march is
// serial in its rows, about 2.7 us a row in the explicit kernel: with 16 rows
// a 32 x 33 x 32 grid has 8 blocks and takes 44 us, with 1 row 128 blocks.
// The results do not depend on it.
static int march_rows(int M, int rows, int64_t columns, int least) {
    while (rows > least && columns * ((M + rows - 1) / rows) < 512) rows = (rows + 1) / 2;
    return rows;
}

// Column tiles of the explicit kernel: up to 64 columns along x in the mixed
// form, 32 in FP64 (whole x-lines when nx is smaller), times as many z-lines
// as the block has room for.  The FP64 32 x 8 tile loads 1.33 halo values
// per cell against 1.55 for 64 x 4 (256 bytes of a row per access run);
// the FP32 form keeps 64 columns, a whole 256-byte run of a row.
// Lines of a multiple of 48 but not of that width take 48 x 4 tiles on 192
// threads of the 256: no lane idle (32 members of 48 x 49 x 48, mixed, 71.5 ->
// 67.6 us; FP64 48 x 97 x 96 and 144 x 97 x 96, mean,
// 57.9 -> 39.7 us with 32 x 8 tiles before).
// slab_rows is what a block marches at most (march_rows).
static void explicit_tiling(const Dims &d, bool fp64, int &threads, int slab_rows, int nmem, ExplicitArgs &a) {
    const int wx = fp64 ? 32 : 64;
    a.tx = d.nx < wx ? d.nx : wx;
    if (a.tx > threads) a.tx = threads;
    if (threads == 256 && d.nx % 48 == 0 && d.nx % wx != 0) {
        a.tx = 48;
        threads = 192;
    }
    a.tz = threads / a.tx;
    a.ntx = (d.nx + a.tx - 1) / a.tx;
    a.chunks = a.ntx * ((d.nz + a.tz - 1) / a.tz);
    a.slab_rows = march_rows(d.M, slab_rows, (int64_t)a.chunks * nmem, 1);
    a.slabs = (d.M + a.slab_rows - 1) / a.slab_rows;
}

// Launch of the explicit kernel with its halo-tile LDS ring; kHalo halo
// positions per thread cover the tile plus halo ((tx+2)(tz+2) <= kHalo * threads).
// The limited advective flux where that is a form of this kernel.
static bool explicit_limits(const nspnp_state *s, const ExplicitArgs &a, int threads) {
    return s->cfg.migration_face == 2 && !s->fp64 && a.mode == 0 && (a.tx + 2) * (a.tz + 2) <= 2 * threads;
}
static hipError_t explicit_launch(nspnp_state *s, const ExplicitArgs &a, int threads, unsigned blocks) {
    const int hs = (a.tx + 2) * (a.tz + 2);
    const size_t lds = 2 * (size_t)kNF * hs * s->wsize;
    const bool dbg = a.mode == 1;
    if (explicit_limits(s, a, threads)) {
        if (threads == 256 && a.tx == 64 && a.tz == 4) k_explicit<float, 2, 3, 0, 64, 4, true><<<blocks, threads, lds, s->stream>>>(a);
        else if (threads == 192 && a.tx == 48 && a.tz == 4) k_explicit<float, 2, 3, 0, 48, 4, true><<<blocks, threads, lds, s->stream>>>(a);
        else k_explicit<float, 2, 3, 0, 0, 0, true><<<blocks, threads, lds, s->stream>>>(a);
        return hipGetLastError();
    }
    if (!dbg && threads == 256 && s->fp64 && a.tx == 32 && a.tz == 8) {  // the common tiles
        // three waves per SIMD: 147 VGPRs, no spill; asking for two gives the
        // same registers and time (0.415 ms at 256 x 193 x 256, 3.32 ms at 512 x
        // 385 x 512)
        k_explicit<double, 2, 3, 0, 32, 8><<<blocks, threads, lds, s->stream>>>(a);
    } else if (!dbg && threads == 256 && !s->fp64 && a.tx == 64 && a.tz == 4) {
        k_explicit<float, 2, 3, 0, 64, 4><<<blocks, threads, lds, s->stream>>>(a);
    } else if (!dbg && threads == 192 && a.tx == 48 && a.tz == 4) {
        if (s->fp64) k_explicit<double, 2, 3, 0, 48, 4><<<blocks, threads, lds, s->stream>>>(a);
        else k_explicit<float, 2, 3, 0, 48, 4><<<blocks, threads, lds, s->stream>>>(a);
    } else if (hs <= 2 * threads) {
        if (s->fp64) {
            if (dbg) k_explicit<double, 2, 2, 1><<<blocks, threads, lds, s->stream>>>(a);
            else k_explicit<double, 2, 2, 0><<<blocks, threads, lds, s->stream>>>(a);
        } else {
            if (dbg) k_explicit<float, 2, 3, 1><<<blocks, threads, lds, s->stream>>>(a);
            else k_explicit<float, 2, 3, 0><<<blocks, threads, lds, s->stream>>>(a);
        }
    } else if (hs <= 4 * threads) {
        if (s->fp64) {
            if (dbg) k_explicit<double, 4, 2, 1><<<blocks, threads, lds, s->stream>>>(a);
            else k_explicit<double, 4, 2, 0><<<blocks, threads, lds, s->stream>>>(a);
        } else {
            if (dbg) k_explicit<float, 4, 3, 1><<<blocks, threads, lds, s->stream>>>(a);
            else k_explicit<float, 4, 3, 0><<<blocks, threads, lds, s->stream>>>(a);
        }
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Crank-Nicolson recurrence coefficients of the three stages: computed on
// the device once per Runge-Kutta step, after the step's dt.
hipError_t launch_step_coef(nspnp_state *s, int nparts) {
    CnStages cs;
    for (int q = 0; q < 3; ++q) cs.alp[q] = kRkAlp[q];
    k_cn_coef<<<dim3(3, 3, (unsigned)s->nmem), 256, 0, s->stream>>>(s->d, s->tb, s->d_phys, s->clock, s->cn_coef, cs,
                                                                   nparts, s->red, s->mstride);
    if (s->cfg.implicit_xz)
        k_cyc_coef<<<dim3(4, 3, (unsigned)s->nmem), 64, 0, s->stream>>>(s->d, s->d_phys, s->clock, s->cyc, cs,
                                                                        s->mstride);
    s->cn_fresh = true;
    return hipGetLastError();
}

namespace {

// Limited advective face values of the ions (migration_face 2).  The explicit
// kernel forms the central advective flux; this pass adds, cell by cell, the
// difference between the limited flux's divergence and the central one to
// the ions' H (when the stage keeps it) and to their Crank-Nicolson
// right-hand side (dt gam times the difference), or, in mode 1, to the
// exported H.  The face values reach two cells upwind (periodic in x and z;
// the upwind cell alone where it is a wall row).
//
// One thread per (x, z) column marches a slab of rows with rows j-2 .. j+2
// of c+- of its own column in registers (the next row loaded one step
// ahead); x and z neighbours come from the same row, which the neighbouring
// columns' threads read at the same time.
struct AdvArgs {
    Dims d;
    size_t ms;
    Tables tb;
    Stage st;
    const void *u, *v, *w, *c[2];
    void *h[2], *r[2];
    double *dbg[2];
    const double *clock;
    int mode;            // 0: substep (H, r of this stage); 1: dbg only
    int ntiles;          // 256-column tiles per plane
    int slabs, slab_rows;
};

template <typename T>
__global__ void __launch_bounds__(256) k_adv_limit(AdvArgs a) {
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x);  // column tiles fastest: z-neighbours share an L2
    const unsigned ct = tile % (unsigned)a.ntiles;
    const unsigned slab = (tile / (unsigned)a.ntiles) % (unsigned)a.slabs;
    const unsigned mem = tile / ((unsigned)a.ntiles * (unsigned)a.slabs);
    const int pl = (int)a.d.plane;
    const int e = (int)(ct * blockDim.x + threadIdx.x);
    if (e >= pl) return;
    const int M = a.d.M, nx = a.d.nx, nz = a.d.nz;
    const size_t ms = a.ms;
    const int i = e % nx, k = e / nx;
    auto wrap = [](int q, int n) { return q < 0 ? q + n : (q >= n ? q - n : q); };  // n >= 4
    // a field's base plus a 32-bit byte offset (a field of every supported
    // grid is below 2^32 bytes); rows outside the grid are clamped to an
    // existing row and their values not used
    const unsigned W = (unsigned)sizeof(T), P = (unsigned)pl * W;
    const unsigned kx = (unsigned)(k * nx) * W;
    const unsigned ex = (unsigned)e * W;
    const unsigned dxp = kx + (unsigned)wrap(i + 1, nx) * W, dxm = kx + (unsigned)wrap(i - 1, nx) * W;
    const unsigned dxp2 = kx + (unsigned)wrap(i + 2, nx) * W, dxm2 = kx + (unsigned)wrap(i - 2, nx) * W;
    const unsigned dzp = (unsigned)(wrap(k + 1, nz) * nx + i) * W, dzm = (unsigned)(wrap(k - 1, nz) * nx + i) * W;
    const unsigned dzp2 = (unsigned)(wrap(k + 2, nz) * nx + i) * W, dzm2 = (unsigned)(wrap(k - 2, nz) * nx + i) * W;
    auto rowb = [&](int jj) { return (unsigned)(jj < 0 ? 0 : (jj >= M ? M - 1 : jj)) * P; };
    const T *u = member_ptr_at((const T *)a.u, ms, mem), *v = member_ptr_at((const T *)a.v, ms, mem);
    const T *w = member_ptr_at((const T *)a.w, ms, mem);
    const T *cf[2] = {member_ptr_at((const T *)a.c[0], ms, mem), member_ptr_at((const T *)a.c[1], ms, mem)};
    T *hf[2] = {member_ptr_at((T *)a.h[0], ms, mem), member_ptr_at((T *)a.h[1], ms, mem)};
    T *rf[2] = {member_ptr_at((T *)a.r[0], ms, mem), member_ptr_at((T *)a.r[1], ms, mem)};
    const T idx_ = T(1.0 / a.d.dx), idz_ = T(1.0 / a.d.dz);
    const T dtg = T(member_ptr_at(a.clock, ms, mem)[1]) * T(a.st.gam);
    const bool keep = a.st.k < 2;
    const int j0 = (int)slab * a.slab_rows;
    const int j1 = (j0 + a.slab_rows < M) ? j0 + a.slab_rows : M;
    // own-column window rows j-2 .. j+2 of both species, and v at row j
    T win[2][5];
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int q = 0; q < 5; ++q) win[sp][q] = *byte_at(cf[sp], rowb(j0 - 2 + q) + ex);
    T vj = *byte_at(v, rowb(j0) + ex);
    for (int j = j0; j < j1; ++j) {
        const unsigned rb = rowb(j);
        // this row's loads, then the next row's window entry (one step ahead)
        const T uL = *byte_at(u, rb + ex), uR = *byte_at(u, rb + dxp);
        const T wB = *byte_at(w, rb + ex), wF = *byte_at(w, rb + dzp);
        const T vn = *byte_at(v, rowb(j + 1) + ex);
        T nb[2][8];  // x +1 -1 +2 -2, z +1 -1 +2 -2
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            const unsigned off[8] = {dxp, dxm, dxp2, dxm2, dzp, dzm, dzp2, dzm2};
#pragma unroll
            for (int q = 0; q < 8; ++q) nb[sp][q] = *byte_at(cf[sp], rb + off[q]);
        }
        T hv[2], rv[2];
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            hv[sp] = *byte_at((const T *)hf[sp], rb + ex);  // (read in every mode and stage: unconditional)
            rv[sp] = *byte_at((const T *)rf[sp], rb + ex);
        }
        T nxt[2];
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) nxt[sp] = *byte_at(cf[sp], rowb(j + 3) + ex);
        const T vb = (j > 0) ? vj : T(0), vt = (j + 1 < M) ? vn : T(0);
        const T idn = T(uniform_load(a.tb.idn, j));
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
            const T delta = limit_delta(nb[sp], win[sp], uR, uL, wF, wB, vt, vb, j, M, idx_, idz_, idn);
            if (a.mode == 1) {
                a.dbg[sp][(size_t)j * (size_t)pl + (size_t)e] += (double)delta;
            } else {
                if (keep) *byte_at(hf[sp], rb + ex) = hv[sp] + delta;
                *byte_at(rf[sp], rb + ex) = rv[sp] + dtg * delta;
            }
        }
        // advance the window
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
#pragma unroll
            for (int q = 0; q < 4; ++q) win[sp][q] = win[sp][q + 1];
            win[sp][4] = nxt[sp];
        }
        vj = vn;
    }
}

}  // namespace

hipError_t launch_adv_limit(nspnp_state *s, const Stage &st, double *const out[5]) {
    AdvArgs a{};
    a.d = s->d;
    a.ms = out ? 0 : s->mstride;
    a.tb = s->tb;
    a.st = st;
    a.u = s->f[0]; a.v = s->f[1]; a.w = s->f[2];
    for (int q = 0; q < 2; ++q) {
        a.c[q] = s->f[3 + q];
        a.h[q] = s->h[3 + q];
        a.r[q] = s->r[3 + q];
        a.dbg[q] = out ? out[3 + q] : nullptr;
    }
    a.clock = s->clock;
    a.mode = out ? 1 : 0;
    a.ntiles = (int)((s->d.plane + 255) / 256);
    a.slab_rows = march_rows(s->d.M, 32, (int64_t)a.ntiles * (out ? 1 : s->nmem), 1);
    a.slabs = (s->d.M + a.slab_rows - 1) / a.slab_rows;
    const int nm = out ? 1 : s->nmem;
    const unsigned blocks = (unsigned)((int64_t)a.ntiles * a.slabs * nm);
    if (s->fp64) k_adv_limit<double><<<blocks, 256, 0, s->stream>>>(a);
    else k_adv_limit<float><<<blocks, 256, 0, s->stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_explicit(nspnp_state *s, const Stage &st, bool /*write_r*/) {
    ExplicitArgs a{};
    a.d = s->d;
    a.phys = s->d_phys;
    a.ms = s->mstride;
    a.tb = s->tb;
    a.st = st;
    a.u = s->f[0]; a.v = s->f[1]; a.w = s->f[2]; a.cp = s->f[3]; a.cm = s->f[4]; a.phi = s->f[5]; a.p = s->f[6];
    for (int q = 0; q < 5; ++q) { a.h[q] = s->h[q]; a.r[q] = s->r[q]; a.dbg[q] = nullptr; }
    a.clock = s->clock;
    a.mode = 0;
    a.implicit_xz = s->cfg.implicit_xz;
    ProfScope prof_(s, K_EXPLICIT);
    int tb = s->tiles.expl;
    explicit_tiling(s->d, s->fp64, tb, s->tiles.slab, s->nmem, a);
    const hipError_t e2 = explicit_launch(s, a, tb, (unsigned)((int64_t)a.chunks * a.slabs * s->nmem));
    if (e2 != hipSuccess || s->cfg.migration_face != 2 || explicit_limits(s, a, tb)) return e2;
    return launch_adv_limit(s, st, nullptr);
}

hipError_t launch_explicit_debug(nspnp_state *s, double *const out[5]) {
    ExplicitArgs a{};
    a.d = s->d;
    a.phys = s->d_phys;
    a.ms = 0;
    a.tb = s->tb;
    a.st = Stage{0, 0, 0, 0};
    a.u = s->f[0]; a.v = s->f[1]; a.w = s->f[2]; a.cp = s->f[3]; a.cm = s->f[4]; a.phi = s->f[5]; a.p = s->f[6];
    for (int q = 0; q < 5; ++q) { a.h[q] = s->h[q]; a.r[q] = s->r[q]; a.dbg[q] = out[q]; }
    a.clock = s->clock;
    a.mode = 1;
    a.implicit_xz = s->cfg.implicit_xz;
    int tb = 256;
    explicit_tiling(s->d, s->fp64, tb, s->tiles.slab, 1, a);
    const hipError_t e = explicit_launch(s, a, tb, (unsigned)((int64_t)a.chunks * a.slabs));
    if (e != hipSuccess || s->cfg.migration_face != 2) return e;
    return launch_adv_limit(s, a.st, out);
}

// Periodic-line solves of the five fields along x (into r) or z (added to q).
static hipError_t launch_cyc(nspnp_state *s, const Stage &st, bool along_z) {
    CycArgs c{};
    c.d = s->d;
    c.ms = s->mstride;
    c.st = st;
    for (int q = 0; q < 5; ++q) { c.q[q] = s->f[q]; c.r[q] = s->r[q]; }
    c.cyc = s->cyc;
    const int N = along_z ? s->d.nz : s->d.nx;
    int rpl = (N + 63) / 64;  // points per lane, rounded up to an instantiated count
    const int have[] = {1, 2, 3, 4, 6, 8, 12, 16};
    int R = 0;
    for (int h : have)
        if (!R && h >= rpl) R = h;
    if (!R) return hipErrorInvalidValue;
    // x: up to 16 lines a wave, fewer while that leaves the chip with fewer
    // than four blocks per CU
    const int64_t nlines = (int64_t)s->d.M * s->d.nz;
    c.lines = 16;
    while (c.lines > 1 && (nlines + 4 * c.lines - 1) / (4 * c.lines) * 5 * s->nmem < 1024) c.lines /= 2;
    const dim3 gx((unsigned)((nlines + 4 * c.lines - 1) / (4 * c.lines)), 5, (unsigned)s->nmem);
    const dim3 gz((unsigned)(s->d.M * ((s->d.nx + kCycTx - 1) / kCycTx)), 5, (unsigned)s->nmem);
    const size_t lds = (size_t)N * (kCycTx + 1) * sizeof(double);
    if (along_z && lds > (size_t)s->lds_max) return hipErrorInvalidValue;
    auto go_z = [&](const void *fn, auto kernel) -> hipError_t {
        const hipError_t e = lds_opt_in(fn, lds, s->lds_max);
        if (e != hipSuccess) return e;
        kernel<<<gz, 256, lds, s->stream>>>(c);
        return hipGetLastError();
    };
    auto go_x = [&](auto kernel) -> hipError_t {
        kernel<<<gx, 256, 0, s->stream>>>(c);
        return hipGetLastError();
    };
#define NSPNP_CYC_CASE(RR)                                                                             \
    case RR:                                                                                           \
        if (!along_z) return s->fp64 ? go_x(k_cyc_x<double, RR>) : go_x(k_cyc_x<float, RR>);           \
        return s->fp64 ? go_z((const void *)k_cyc_z<double, RR>, k_cyc_z<double, RR>)                  \
                       : go_z((const void *)k_cyc_z<float, RR>, k_cyc_z<float, RR>);
    switch (R) {
        NSPNP_CYC_CASE(1)
        NSPNP_CYC_CASE(2)
        NSPNP_CYC_CASE(3)
        NSPNP_CYC_CASE(4)
        NSPNP_CYC_CASE(6)
        NSPNP_CYC_CASE(8)
        NSPNP_CYC_CASE(12)
        NSPNP_CYC_CASE(16)
        default:
            return hipErrorInvalidValue;
    }
#undef NSPNP_CYC_CASE
}

// Planes on which the lane scans take 8 waves on 16 columns whatever Tiles::cn:
// up to two such blocks per CU.
static bool cn_small(const nspnp_state *s) { return (s->d.plane + 15) / 16 * 5 * s->nmem <= 512; }

// Lane-scan Crank-Nicolson solve of the five fields (tiles of 16 or 32 columns).
static hipError_t launch_cn_lane(nspnp_state *s, const CnArgs &a) {
    // up to 32 rows: groups of 16 or 32 lanes a column, which hold all of its
    // rows (a whole wave's idle lanes would only pass values through: the result
    // is the same); small planes: 8 waves on 16 columns (32 x 33 x 32 8.6 us with
    // one column a wave, 6.5 so; latency)
    const int lanes = s->d.M <= 16 ? 16 : (s->d.M <= 32 ? 32 : 64);
    const bool small = cn_small(s);
    const int tb = small ? (lanes == 16 ? 256 : 512) : s->tiles.cn;
    const int tcols = small ? 16 : cn_tile_cols(tb);
    const dim3 g((unsigned)((s->d.plane + tcols - 1) / tcols), 5, (unsigned)s->nmem);
    const size_t lds = (size_t)s->d.M * (tcols + 1) * sizeof(double);
    if (lds > (size_t)s->lds_max) return hipErrorInvalidValue;
    const int rpl = (s->d.M + 63) / 64;  // rows per lane (M <= kCnLaneRows: at most 5)
    // tiles above 64 KB of LDS (tall columns) use the device's larger limit
    auto launch = [&](const void *fn, auto kernel) -> hipError_t {
        const hipError_t e = lds_opt_in(fn, lds, s->lds_max);
        if (e != hipSuccess) return e;
        kernel<<<g, tb, lds, s->stream>>>(a);
        return hipGetLastError();
    };
#define NSPNP_CN_CASE(RR, WW)                                                                          \
    if (tcols == 32) return launch((const void *)k_cn_scan<32, RR, WW>, k_cn_scan<32, RR, WW>);        \
    return launch((const void *)k_cn_scan<16, RR, WW>, k_cn_scan<16, RR, WW>);
    switch (rpl) {
        case 1:
            if (lanes == 16) { NSPNP_CN_CASE(1, 16) }
            if (lanes == 32) { NSPNP_CN_CASE(1, 32) }
            NSPNP_CN_CASE(1, 64)
        case 2: NSPNP_CN_CASE(2, 64)
        case 3: NSPNP_CN_CASE(3, 64)
        case 4: NSPNP_CN_CASE(4, 64)
        case 5: NSPNP_CN_CASE(5, 64)
        default: return hipErrorInvalidValue;
    }
#undef NSPNP_CN_CASE
}

// Rows a thread holds in the Crank-Nicolson solve; 0: lane scans.  The result's
// rounding depends on it, so with cnslab 0, the default, it follows from the
// type and the rows alone; cnslab 16 and 32 ask for another.  24 rows where they make
// 8 or 16 whole slabs: 0.130 ms (mixed) against 0.145 for 12 and 0.136 for
// 16 at 256 x 193 x 256; 16 at up to 128 (28.9 against 30.8 us for 24, 33.4
// for 8 at 128 x 129 x 128); short columns split into at least 8 slabs, which
// fill the chip on small planes.
int cn_slab_rows(const nspnp_state *s) {
    const int M = s->d.M;
    if (s->fp64 && s->tiles.cnslab == 0 && M <= kCnLaneRows) return 0;
    if (s->tiles.cnslab == 16 || M > 384) return 16;
    if (s->tiles.cnslab == 32) return 24;
    if (M <= 32) return 4;
    if (M <= 64) return 8;
    return (M <= 128 || (M > 192 && M <= 256)) ? 16 : 24;
}

bool cn_tile_read(const nspnp_state *s) { return cn_slab_rows(s) == 0 && !cn_small(s); }

// out_r: the solution replaces r, else it is added to the fields
static hipError_t launch_cn_y(nspnp_state *s, const Stage &st, bool out_r) {
    CnArgs a{};
    a.d = s->d;
    a.ms = s->mstride;
    a.st = st;
    for (int q = 0; q < 5; ++q) { a.q[q] = s->f[q]; a.r[q] = s->r[q]; }
    a.coef = s->cn_coef;
    a.out_r = out_r ? 1 : 0;
    if (!cn_slab_rows(s)) return launch_cn_lane(s, a);
    const int L = cn_slab_rows(s), S = (s->d.M + L - 1) / L;
    const int cx = S <= 16 ? 64 : 32;  // a block has at most 1024 threads
    if (S * cx > 1024) return hipErrorInvalidValue;
    const dim3 g((unsigned)((s->d.plane + cx - 1) / cx), 5, (unsigned)s->nmem);
    const size_t lds = ((size_t)S * (cx + 1) + (cx == 64 ? 0 : 3 * cn_rows(s->d.M))) * sizeof(double);
    auto go = [&](auto rows, auto cols) {
        constexpr int R = decltype(rows)::value, C = decltype(cols)::value;
        if (s->fp64) {
            if (out_r) k_cn_rows<double, R, C, true><<<g, S * C, lds, s->stream>>>(a);
            else k_cn_rows<double, R, C, false><<<g, S * C, lds, s->stream>>>(a);
        } else {
            if (out_r) k_cn_rows<float, R, C, true><<<g, S * C, lds, s->stream>>>(a);
            else k_cn_rows<float, R, C, false><<<g, S * C, lds, s->stream>>>(a);
        }
        return hipGetLastError();
    };
    using std::integral_constant;
    if (L == 4) return go(integral_constant<int, 4>{}, integral_constant<int, 64>{});
    if (L == 8) return go(integral_constant<int, 8>{}, integral_constant<int, 64>{});
    if (L == 24) return go(integral_constant<int, 24>{}, integral_constant<int, 64>{});
    if (cx == 64) return go(integral_constant<int, 16>{}, integral_constant<int, 64>{});
    return go(integral_constant<int, 16>{}, integral_constant<int, 32>{});
}

hipError_t launch_cn_solve(nspnp_state *s, const Stage &st) {
    ProfScope prof_(s, K_CN);
    hipError_t e = hipSuccess;
    // (a step's first stage has made them; after a restart within a step, or a new dt)
    if (!s->cn_fresh && (e = launch_step_coef(s, 0)) != hipSuccess) return e;
    if (!s->cfg.implicit_xz) return launch_cn_y(s, st, false);
    // three-direction factorisation: x-lines into r, y (this solve) into r, then z-lines with q += solution
    if ((e = launch_cyc(s, st, false)) != hipSuccess) return e;
    if ((e = launch_cn_y(s, st, true)) != hipSuccess) return e;
    return launch_cyc(s, st, true);
}

hipError_t launch_correct(nspnp_state *s, const Stage &st, bool update_p, double fixed, bool advance_clock) {
    ProfScope prof_(s, K_CORRECT);
    CorrArgs a{};
    a.d = s->d;
    a.phys = s->d_phys;
    a.ms = s->mstride;
    a.tb = s->tb;
    a.u = s->f[0]; a.v = s->f[1]; a.w = s->f[2]; a.p = s->f[6];
    a.psi = s->psi;
    a.clock = s->clock;
    a.alp = st.alp;
    a.fixed = fixed;
    a.update_p = update_p ? 1 : 0;
    a.advance_clock = advance_clock ? 1 : 0;
    const int tb = s->tiles.corr < 256 ? s->tiles.corr : 256;
    a.tx = s->d.nx < 64 ? s->d.nx : 64;
    if (a.tx > tb) a.tx = tb;
    a.tz = tb / a.tx;
    a.ntx = (s->d.nx + a.tx - 1) / a.tx;
    a.chunks = a.ntx * ((s->d.nz + a.tz - 1) / a.tz);
    a.slab_rows = march_rows(s->d.M, s->tiles.slab, (int64_t)a.chunks * s->nmem, kCorrRows);
    a.slabs = (s->d.M + a.slab_rows - 1) / a.slab_rows;
    const dim3 g((unsigned)((int64_t)a.chunks * a.slabs * s->nmem));
    if (s->cfg.implicit_xz) {
        if (s->fp64) k_correct<double, true><<<g, tb, 0, s->stream>>>(a);
        else k_correct<float, true><<<g, tb, 0, s->stream>>>(a);
    } else {
        if (s->fp64) k_correct<double, false><<<g, tb, 0, s->stream>>>(a);
        else k_correct<float, false><<<g, tb, 0, s->stream>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_convert(nspnp_state *s, int field, const double *in, double *out, bool to_state) {
    if (to_state) {
        if (s->fp64)
            k_copy_convert<double, double><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d.n, in, (double *)s->f[field]);
        else
            k_copy_convert<double, float><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d.n, in, (float *)s->f[field]);
    } else {
        if (s->fp64)
            k_copy_convert<double, double><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d.n, (const double *)s->f[field], out);
        else
            k_copy_convert<float, double><<<grid1(s->d.n), 256, 0, s->stream>>>(s->d.n, (const float *)s->f[field], out);
    }
    return hipGetLastError();
}

}  // namespace nspnp
