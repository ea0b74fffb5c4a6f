// Matrix-free Q2 operators of the pressure (Eq. 3) and heat (Eq. 4) equations on
// rectilinear meshes (27-node cells, 3-point Gauss rules), one wave per strip of
// cell columns.
//
// Layout: a lane is one cell column x and carries its nodes 2x and 2x + 1 on the
// three node rows of one cell row; node 2x + 2 is the next lane's (DPP wave shift).
// The waves of a block sit side by side along y and march upward one cell layer
// (two node planes) at a time.  The cell columns of all y bands are laid end to
// end, each band followed by the lane of its last node column and an empty one,
// and a block takes 64 consecutive columns (62 owned).  A band owns the node rows
// above its first cell row (the first wave's, which is halo; W - 1 cell rows of W waves).  The node row that
// two waves share passes through LDS with one barrier per layer.  Every node value
// is produced by exactly one lane, as a fixed expression.
//
// Cells are evaluated in the Legendre modes of an axis: for node values
// (v0, v1, v2) the functionals
//   c = v0 + 4 v1 + v2,  e = v0 - 2 v1 + v2,  d = v0 - v2
// make the 1D mass h/30 [4 2 -1; 2 16 2; -1 2 4] and stiffness
// 1/(3h) [7 -8 1; -8 16 -8; 1 -8 7] diagonal, M = h (1/36, 1/45, 1/12),
// K = M (0, 60, 12) / h^2, with the same three patterns on the way back.  Mass and
// stiffness of a cell are one scaling of its 27 modes (about 250 operations for a
// cell where the sum-factorised products of op_q2.hip take 650); the modes of a
// node column along z and of a row along y are formed once for the cells that
// share them.  The convection term is evaluated at the 27 Gauss points from the
// same modes: value c/6 + 2/15 e +- sqrt(3/20) d (middle c/6 - e/6), derivative
// -d -+ 2 sqrt(3/5) e (middle -d), and projected back onto the modes.
//
// What bounds it: the pressure kernels (650 instructions for a cell layer, 93 or 160
// registers) are issue bound, FP64 at 4.3 clocks each; the heat kernels (1300 to 1400)
// are bound by dependent chains at one (FP64) or two (FP32) waves per SIMD.  FP64 heat
// keeps both fields' 27 modes, the result's and the next layer's nodes in 390 registers:
// with eight waves (256 each) it spilled and took 314 us where four waves take 157, for
// a third of halo rows instead of a seventh; the pressure's modes in LDS, read again
// for every plane of points, 188.  Kernel times against the tile kernels of op_q2.hip,
// us, at 128 x 128 x 64 cells | 101 x 77 x 33 graded | 24^3:
//   FP64 pressure  141.7 -> 58.1 | 48.0 -> 20.2 | 18.1 -> 11.9
//   FP32 pressure   89.5 -> 36.8 | 35.1 -> 17.7 | 17.3 -> 10.7
//   FP64 heat      410.7 -> 157  | 117.4 -> 53.8 | 33.8 -> 15.1
//   FP32 heat      216.6 -> 74.5 | 70.2 -> 33.7 | 30.1 -> 17.7
#include "strip.h"

namespace hts {

namespace {

#pragma clang fp contract(off)

template <typename T>
struct Modes {
    T c, e, d;
};
template <typename T>
__device__ __forceinline__ Modes<T> to_modes(T v0, T v1, T v2)
{
    const T s = v0 + v2;
    return {fma_(T(4), v1, s), fma_(T(-2), v1, s), v0 - v2};
}
// weights of the modes on the way back relative to the first (masses 1/36, 1/45, 1/12)
template <typename T>
__device__ __forceinline__ void from_modes(const Modes<T> &m, T &v0, T &v1, T &v2)
{
    const T t = fma_(T(0.8), m.e, m.c);
    v0 = fma_(T(3), m.d, t);
    v1 = fma_(T(-1.6), m.e, T(4) * m.c);
    v2 = fma_(T(-3), m.d, t);
}
constexpr double GV = 2.3237900077244501;   // 6 sqrt(3/20)
constexpr double GD = 1.5491933384829668;   // 2 sqrt(3/5)
// 6 times the value, and the derivative, at Gauss point q
template <typename T>
__device__ __forceinline__ T gauss_value(const Modes<T> &m, int q)
{
    if (q == 1) return m.c - m.e;
    return fma_(T(q == 0 ? GV : -GV), m.d, fma_(T(0.8), m.e, m.c));
}
template <typename T>
__device__ __forceinline__ T gauss_deriv(const Modes<T> &m, int q)
{
    if (q == 1) return -m.d;
    return fma_(T(q == 0 ? -GD : GD), m.e, -m.d);
}
// integrals of the mode functions with values t0, t1, t2 at the Gauss points,
// weights 5 : 8 : 5, in the scale of from_modes (times 18/5 6)
template <typename T>
__device__ __forceinline__ Modes<T> project(T t0, T t1, T t2)
{
    const T s = t0 + t2;
    return {fma_(T(1.6), t1, s), fma_(T(-2), t1, s), T(0.77459666924148338) * (t0 - t2)};
}

// injection-line rows of node column col at plane k (r: the column's first row at
// or above the planes seen so far)
template <typename T, bool MASKED>
__device__ __forceinline__ T line_rows(const OpDev &o, int &r, int col, int k, const T *Xi)
{
    const LineRow HTS_GLOBAL *rows = gptr<LineRow>(o.lrows);
    const LineEnt HTS_GLOBAL *ents = gptr<LineEnt>(o.lents);
    const double HTS_GLOBAL *lco = gptr<double>(o.lcoef);
    while (rows[r].col == col && rows[r].k < k) r++;
    if (rows[r].col != col || rows[r].k != k || (MASKED && rows[r].row_constrained)) return T(0);
    T la = T(0);
    for (int e = rows[r].beg; e < rows[r].end; e++) {
        if (MASKED && ents[e].col_constrained) continue;
        la = fma_(T(lco[ents[e].src] * ents[e].w), Xi[ents[e].col], la);
    }
    return la;
}

template <typename T, int FIELD, int EPI, bool MASKED, bool GRADED, bool SOLO>
__global__ __launch_bounds__(64 * q2s_waves(FIELD, sizeof(T) == 8))
void k_q2_strip(const typename std::conditional<SOLO, Solo, Tabled>::type at, const T *__restrict__ X,
                T *__restrict__ Y, EpiArgs<T> ep)
{
    constexpr int W2 = q2s_waves(FIELD, sizeof(T) == 8);
    __shared__ double red[W2];
    __shared__ T xch[2][W2][6][64];                          // top-row sums of a wave's cells
    const WorkItem wi = at.item();
    if (SOLO ? wi.inst < 0 : (ep.active && !ep.active[wi.inst])) return;
    const OpDev &o = at.op(wi.inst);
    constexpr bool PIEZO = SOLO && FIELD == 1 && sizeof(T) == 4;
    using PT = typename std::conditional<PIEZO, double, T>::type;
    const int nx = o.nx, ny = o.ny, nz = o.nz, NX = o.NX, NY = o.NY, NZ = o.NZ, m = o.dmask;
    constexpr bool CHEB = EPI == EPI_CHEB;
    constexpr bool HASB = EPI == EPI_RESID || EPI == EPI_RESID_NORM || CHEB;
    const T *Xi = X + o.off;
    T *Yi = Y + o.off;
    const T *Bi = HASB ? ep.b + o.off : nullptr;
    T *Di = CHEB ? ep.d + o.off : nullptr;
    const T *Ii = CHEB ? ep.invd + o.off : nullptr;
    const PT *Pi = static_cast<const PT *>(o.P);
    const T *kk = static_cast<const T *>(o.k), *lam = static_cast<const T *>(o.lam), *cT = static_cast<const T *>(o.cT);
    const int64_t plane = (int64_t)NX * NY, cplane = (int64_t)nx * ny;
    const uint32_t pbytes = (uint32_t)(plane * sizeof(T)), cbytes = (uint32_t)(cplane * sizeof(T));
    constexpr uint32_t SZ = sizeof(T), PW = sizeof(PT) / sizeof(T);
    const bool adv = FIELD == 1 && o.cadv != 0.0;

    // ---- the lane's cell column (x = nx: the last node column, nx + 1: empty)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tot = ((NY + 2 * W2 - 3) / (2 * W2 - 2)) * (nx + 2);
    const int pos = wi.tx * Q2S_OWNED + lane - 1;
    const bool pin = pos >= 0 && pos < tot;
    const int band = (pin ? pos : 0) / (nx + 2), x = (pin ? pos : 0) - band * (nx + 2);
    const int J = band * (W2 - 1) - 1 + wave;                 // cell row; its node rows 2 J .. 2 J + 2
    const bool xin = pin && x <= nx, xin1 = pin && x < nx;    // nodes 2x and 2x + 1 in the mesh
    const bool mine = xin && lane >= 1 && lane <= Q2S_OWNED && wave > 0;
    // node (r, a) of the lane, r = 0 .. 2: byte offset base + r rowb + a SZ in a
    // node plane; bit 2 r + a of in, con: in the mesh, constrained by an x/y face
    const uint32_t base = (uint32_t)((2 * x + NX * 2 * J) * (int)SZ), rowb = (uint32_t)(NX * (int)SZ);
    uint32_t in = 0, con = 0;
    bool special = false, cols = false;
#pragma unroll
    for (int q = 0; q < 6; q++) {
        const int i = 2 * x + (q & 1), j = 2 * J + (q >> 1);
        const bool here = ((q & 1) ? xin1 : xin) && j >= 0 && j < NY;
        if (here) in |= 1u << q;
        if (MASKED && here) {
            if (((m & 1) && i == 0) || ((m & 2) && i == NX - 1) || ((m & 4) && j == 0) || ((m & 8) && j == NY - 1))
                con |= 1u << q;
            if (o.dcol) cols |= gptr<int32_t>(o.dcol)[i + NX * j] != DCOL_NONE;
        }
    }
    const uint32_t xbits = in & ~con, obits = mine ? in & 15u : 0u;
    auto node = [&](int q) { return base + (uint32_t)(q >> 1) * rowb + (uint32_t)(q & 1) * SZ; };
    auto off_x = [&](int q) { return (xbits >> q) & 1u ? node(q) : OOB; };          // operand
    auto off_p = [&](int q) { return (in >> q) & 1u ? node(q) * PW : OOB; };        // pressure
    auto off_o = [&](int q) { return (obits >> q) & 1u ? node(q) : OOB; };          // owned, rows 0 and 1
    // Dirichlet columns: whether plane k of node q lies in its constrained z-range
    auto in_col = [&](int q, int k) {
        int d = DCOL_NONE;
        if ((in >> q) & 1u) d = gptr<int32_t>(o.dcol)[node(q) / SZ];
        return k >= (d & 0xFFFF) && k <= ((d >> 16) & 0xFFFF);
    };
    const uint32_t co = xin1 && J >= 0 && J < ny ? (uint32_t)((x + nx * J) * (int)SZ) : OOB;
    if (MASKED) {
        cols = __any(cols);
        special = cols || __any(con != 0);
    }
    int lr[FIELD ? 4 : 1];
    bool lines = false;
    if (FIELD == 1 && o.lcol) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            lr[FIELD ? q : 0] = -1;
            if ((obits >> q) & 1u) lr[FIELD ? q : 0] = gptr<int32_t>(o.lcol)[node(q) / SZ];
            lines |= lr[FIELD ? q : 0] >= 0;
        }
        lines = __any(lines);
    }

    // ---- cell factors: 1/36 per axis of the modes, 60 / h^2 and 12 / h^2
    const bool graded = GRADED && o.hzs != nullptr;
    double hx = o.hx, hy = o.hy;
    if (graded) {
        hx = o.hxs[x < nx ? x : nx - 1];
        hy = o.hys[J < 0 ? 0 : (J < ny ? J : ny - 1)];
    }
    const T ihx2 = T(1.0 / (hx * hx)), ihy2 = T(1.0 / (hy * hy)), hxy = T(hx * hy);
    T c1 = T(0), c2 = T(0);
    if (CHEB) {
        const double *Sc = ep.S + (int64_t)wi.inst * NSLOT;
        c1 = T(Sc[ep.s1]);
        c2 = T(Sc[ep.s2]);
    }

    // ---- the march: owned planes kb .. ke - 1 (kb even), cell layers La .. Lb
    const int kb = wi.z0, ke = wi.z1;
    const int La = kb > 0 ? kb / 2 - 1 : 0;
    const int Lb = (ke - 1) / 2 < nz ? (ke - 1) / 2 : nz - 1;
    double acc = 0.0;
    auto zface = [&](int k) { return MASKED && (((m & 16) && k == 0) || ((m & 32) && k == NZ - 1)); };
    auto load_x = [&](int k, T u[3][2]) {
        const Rsrc rx = rsrc(Xi + k * plane, zface(k) ? 0u : pbytes);
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int a = 0; a < 2; a++) u[r][a] = bld<T>(rx, off_x(2 * r + a));
    };
    auto mask_cols = [&](int k, T u[3][2]) {
        if (MASKED && cols) {
#pragma unroll
            for (int r = 0; r < 3; r++)
#pragma unroll
                for (int a = 0; a < 2; a++)
                    if (in_col(2 * r + a, k)) u[r][a] = T(0);
        }
    };
    auto load_p = [&](int k, PT u[3][2]) {
        const Rsrc rp = rsrc(Pi + k * plane, pbytes * PW);
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int a = 0; a < 2; a++) u[r][a] = bld<PT>(rp, off_p(2 * r + a));
    };
    // The pressure of plane k less c_k, so that the sums of the modes do not cancel
    // against its hydrostatic part c_k = P_0 - rho_g z_k (FP64: what c + rho_g z has
    // left through the rounding of c_k goes into the z modes).  FP32: the piezometric
    // pressure as k_piezo32 forms it, P + rho_g z, less the cell's own value at its
    // left middle node (both in FP32, so the differences stay exact)
    const double pref = adv ? (double)Pi[0] : 0.0;
    auto height = [&](int k) { return graded ? o.zn[k] - o.zn[0] : k * (0.5 * o.hz); };
    auto hyd = [&](int k) { return fma_(-o.rho_g, height(k), pref); };
    auto use_p = [&](int k, const PT u[3][2], T p[3][2]) {
        const double zk = height(k);
        const T ck = PIEZO ? T(0) : T(hyd(k));
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int a = 0; a < 2; a++) {
                if (PIEZO) p[r][a] = T(fma_(o.rho_g, zk, (double)u[r][a] - pref));
                else p[r][a] = T(u[r][a]) - ck;
            }
    };
    // the epilogue of the owned nodes of plane k: v = A u
    auto epilogue = [&](int k, T v[2][2]) {
        const Rsrc ry = rsrc(Yi + k * plane, pbytes), rb = rsrc(HASB ? Bi + k * plane : Xi, pbytes),
                   rd = rsrc(CHEB ? Di + k * plane : Yi, pbytes), ri = rsrc(CHEB ? Ii + k * plane : Xi, pbytes),
                   rx = rsrc(Xi + k * plane, pbytes);
        const bool zf = zface(k), sp = MASKED && (special || zf);
        T eb[4], ed[4], ei[4], ex[4] = {T(0), T(0), T(0), T(0)};
        uint32_t same = 0;                                    // constrained: rows of the identity
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint32_t off = off_o(q);
            if (HASB) eb[q] = bld<T>(rb, off);
            if (CHEB) { ed[q] = bld<T>(rd, off); ei[q] = bld<T>(ri, off); }
        }
        if (CHEB || EPI == EPI_DOT || sp) {
#pragma unroll
            for (int q = 0; q < 4; q++) ex[q] = bld<T>(rx, off_o(q));
        }
        if (sp) {
            same = zf ? 15u : con;
            if (cols) {
#pragma unroll
                for (int q = 0; q < 4; q++) same |= in_col(q, k) ? 1u << q : 0u;
            }
        }
        if (FIELD == 1 && lines) {
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (lr[FIELD ? q : 0] >= 0)
                    v[q >> 1][q & 1] += line_rows<T, MASKED>(o, lr[FIELD ? q : 0], (int)(node(q) / SZ), k, Xi);
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int r = q >> 1, a = q & 1;
            const uint32_t off = off_o(q);
            const T xq = ex[q];
            if (MASKED) v[r][a] = (same >> q) & 1u ? xq : v[r][a];
            if (EPI == EPI_STORE) {
                bst<T>(ry, off, v[r][a]);
            } else if (EPI == EPI_RESID) {
                bst<T>(ry, off, eb[q] - v[r][a]);
            } else if (EPI == EPI_RESID_NORM) {
                const T d = eb[q] - v[r][a];
                bst<T>(ry, off, d);
                if (off < pbytes) acc = fma_((double)d, (double)d, acc);
            } else if (EPI == EPI_DOT) {
                bst<T>(ry, off, v[r][a]);
                if (off < pbytes) acc = fma_((double)xq, (double)v[r][a], acc);
            } else if (CHEB) {
                const T d = fma_(c1, ed[q], c2 * ei[q] * (eb[q] - v[r][a]));
                bst<T>(rd, off, d);
                bst<T>(ry, off, xq + d);
            }
        }
    };

    auto march = [&](auto adv_) {
        constexpr bool ADV = decltype(adv_)::value;
        T u0[3][2], u1[3][2], u2[3][2];
        PT p0[3][2], p1[3][2], p2[3][2];
        T tc[2][2] = {{T(0), T(0)}, {T(0), T(0)}};            // sums of the cells below, at plane 2 L
        T ck = T(0), cl = T(0), cc = T(0);
        auto load_c = [&](int L) {
            ck = bld<T>(rsrc(kk + L * cplane, cbytes), co);
            if (FIELD == 1) {
                cl = bld<T>(rsrc(lam + L * cplane, cbytes), co);
                cc = bld<T>(rsrc(cT + L * cplane, cbytes), co);
            }
        };
        load_x(2 * La, u0);
        load_x(2 * La + 1, u1);
        load_x(2 * La + 2, u2);
        if (ADV) {
            load_p(2 * La, p0);
            load_p(2 * La + 1, p1);
            load_p(2 * La + 2, p2);
        }
        load_c(La);
        // the next layer's planes, loaded as soon as this one's are in modes
        auto next = [&](int L) {
#pragma unroll
            for (int r = 0; r < 3; r++)
#pragma unroll
                for (int a = 0; a < 2; a++) {
                    u0[r][a] = u2[r][a];
                    if (ADV) p0[r][a] = p2[r][a];
                }
            if (L == Lb) return;
            load_x(2 * L + 3, u1);
            load_x(2 * L + 4, u2);
            if (ADV) {
                load_p(2 * L + 3, p1);
                load_p(2 * L + 4, p2);
            }
        };
        for (int L = La; L <= Lb; L++) {
            if (L == La) mask_cols(2 * L, u0);
            mask_cols(2 * L + 1, u1);
            mask_cols(2 * L + 2, u2);
            const double hz = graded ? o.hzs[L] : o.hz;
            const T vol = hxy * T(hz / 46656.0);
            const T mass = (FIELD == 0 ? (co < cbytes ? T(o.cm) : T(0)) : cc) * vol;
            // modes of the cell, index i + 3 j + 9 k (c, e, d along x, y, z); shift: added
            // to the mean of the right neighbour's values
            auto modes27 = [&](const T w0[3][2], const T w1[3][2], const T w2[3][2], T U[27], T shift) {
                Modes<T> z[3][2];
#pragma unroll
                for (int r = 0; r < 3; r++)
#pragma unroll
                    for (int a = 0; a < 2; a++) z[r][a] = to_modes(w0[r][a], w1[r][a], w2[r][a]);
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    Modes<T> y[2];
#pragma unroll
                    for (int a = 0; a < 2; a++)
                        y[a] = k == 0 ? to_modes(z[0][a].c, z[1][a].c, z[2][a].c)
                                      : (k == 1 ? to_modes(z[0][a].e, z[1][a].e, z[2][a].e)
                                                : to_modes(z[0][a].d, z[1][a].d, z[2][a].d));
                    const T lft[3] = {y[0].c, y[0].e, y[0].d}, mid[3] = {y[1].c, y[1].e, y[1].d};
#pragma unroll
                    for (int j = 0; j < 3; j++) {
                        const Modes<T> q = to_modes(lft[j], mid[j], j + k == 0 ? from_right(lft[j]) + shift : from_right(lft[j]));
                        U[3 * j + 9 * k] = q.c;
                        U[1 + 3 * j + 9 * k] = q.e;
                        U[2 + 3 * j + 9 * k] = q.d;
                    }
                }
            };
            T U[27], R[27];
            if (ADV) {
                T Q[27];
                {
                    T a0[3][2], a1[3][2], a2[3][2];
                    use_p(2 * L, p0, a0);
                    use_p(2 * L + 1, p1, a1);
                    use_p(2 * L + 2, p2, a2);
                    T shift = T(0);
                    if (PIEZO) {
                        const T own = a1[1][0];
#pragma unroll
                        for (int r = 0; r < 3; r++)
#pragma unroll
                            for (int a = 0; a < 2; a++) {
                                a0[r][a] -= own;
                                a1[r][a] -= own;
                                a2[r][a] -= own;
                            }
                        shift = T(36) * (from_right(own) - own);
                    }
                    modes27(a0, a1, a2, Q, shift);
                    if (!PIEZO) {
                        const double h0 = hyd(2 * L), h1 = hyd(2 * L + 1), h2 = hyd(2 * L + 2);
                        Q[9] += T(36.0 * ((h0 - h1) - (h1 - h2)));
                        Q[18] += T(36.0 * ((h0 - h2) - o.rho_g * hz));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                modes27(u0, u1, u2, U, T(0));
                __builtin_amdgcn_sched_barrier(0);
                next(L);
                __builtin_amdgcn_sched_barrier(0);
                // common factor of the two fields' values and the weights: 5/18 per
                // axis, 1/6 per value (two fields, two cross axes), and 1/6 per axis
                // of the projection's scale
                const T f = ck * T((5.0 / 18.0) * (5.0 / 18.0) * (5.0 / 18.0) / (36.0 * 36.0 * 216.0));
                const T fv = f * (hxy * T(-o.cadv * hz));
                const T fx = fv * ihx2, fy = fv * ihy2, fz = fv * T(1.0 / (hz * hz));
#pragma unroll
                for (int i = 0; i < 27; i++) R[i] = T(0);
#pragma unroll 1
                for (int qz = 0; qz < 3; qz++) {
                    // weights of the z modes in value, derivative and projection
                    const T ze = qz == 1 ? T(-1) : T(0.8), zv = T(GV) * T(1 - qz), zd = T(-GD) * T(1 - qz);
                    const T rc = qz == 1 ? T(1.6) : T(1), re = qz == 1 ? T(-2) : T(1), rd = T(0.77459666924148338) * T(1 - qz);
                    // the products at the 9 points: first the x and y components,
                    // from the values along z, then the z component, from the
                    // derivatives; one row of points at a time (the barriers keep
                    // the scheduler from holding several)
                    T t[3][3], pw[9], uw[9];
#pragma unroll
                    for (int i = 0; i < 9; i++) {
                        pw[i] = fma_(zv, Q[i + 18], fma_(ze, Q[i + 9], Q[i]));
                        uw[i] = fma_(zv, U[i + 18], fma_(ze, U[i + 9], U[i]));
                    }
#pragma unroll
                    for (int qy = 0; qy < 3; qy++) {
                        __builtin_amdgcn_sched_barrier(0);
                        auto row = [&](const T *w, int i) { return Modes<T>{w[i], w[i + 3], w[i + 6]}; };
                        const Modes<T> a{gauss_value(row(pw, 0), qy), fx * gauss_value(row(pw, 1), qy), fx * gauss_value(row(pw, 2), qy)};
                        const Modes<T> b{fy * gauss_deriv(row(pw, 0), qy), fy * gauss_deriv(row(pw, 1), qy), fy * gauss_deriv(row(pw, 2), qy)};
                        const Modes<T> d{gauss_value(row(uw, 0), qy), gauss_value(row(uw, 1), qy), gauss_value(row(uw, 2), qy)};
                        const Modes<T> e{gauss_deriv(row(uw, 0), qy), gauss_deriv(row(uw, 1), qy), gauss_deriv(row(uw, 2), qy)};
#pragma unroll
                        for (int qx = 0; qx < 3; qx++)
                            t[qy][qx] = fma_(gauss_deriv(a, qx), gauss_deriv(d, qx), gauss_value(b, qx) * gauss_value(e, qx));
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 9; i++) {
                        pw[i] = fz * fma_(zd, Q[i + 9], -Q[i + 18]);
                        uw[i] = fma_(zd, U[i + 9], -U[i + 18]);
                    }
                    Modes<T> xs[3];
#pragma unroll
                    for (int qy = 0; qy < 3; qy++) {
                        __builtin_amdgcn_sched_barrier(0);
                        auto row = [&](const T *w, int i) { return Modes<T>{w[i], w[i + 3], w[i + 6]}; };
                        const Modes<T> c{gauss_value(row(pw, 0), qy), gauss_value(row(pw, 1), qy), gauss_value(row(pw, 2), qy)};
                        const Modes<T> h{gauss_value(row(uw, 0), qy), gauss_value(row(uw, 1), qy), gauss_value(row(uw, 2), qy)};
#pragma unroll
                        for (int qx = 0; qx < 3; qx++)
                            t[qy][qx] = fma_(gauss_value(c, qx), gauss_value(h, qx), t[qy][qx]);
                        xs[qy] = project(t[qy][0], t[qy][1], t[qy][2]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // modes along x and y of the plane of points
                    const Modes<T> yc = project(xs[0].c, xs[1].c, xs[2].c), yv = project(xs[0].e, xs[1].e, xs[2].e),
                                   yd = project(xs[0].d, xs[1].d, xs[2].d);
                    const T gq[9] = {yc.c, yv.c, yd.c, yc.e, yv.e, yd.e, yc.d, yv.d, yd.d};
#pragma unroll
                    for (int i = 0; i < 9; i++) {
                        R[i] = fma_(rc, gq[i], R[i]);
                        R[i + 9] = fma_(re, gq[i], R[i + 9]);
                        R[i + 18] = fma_(rd, gq[i], R[i + 18]);
                    }
                }
            } else {
                modes27(u0, u1, u2, U, T(0));
#pragma unroll
                for (int i = 0; i < 27; i++) R[i] = T(0);
            }
            __builtin_amdgcn_sched_barrier(0);
            // mass and stiffness: eigenvalues 0, 5, 1 times 12 / h^2 per axis
            {
                const T stiff = (FIELD == 0 ? ck : cl) * (hxy * T(o.cs * 12.0 * hz / 46656.0));
                const T ax = ihx2 * stiff, ay = ihy2 * stiff, az = T(1.0 / (hz * hz)) * stiff;
                const T sx[3] = {mass, fma_(T(5), ax, mass), ax + mass};
                const T sy[3] = {T(0), T(5) * ay, ay}, sz[3] = {T(0), T(5) * az, az};
#pragma unroll
                for (int j = 0; j < 3; j++)
#pragma unroll
                    for (int i = 0; i < 3; i++) {
                        const T a = j == 0 ? sx[i] : sx[i] + sy[j];
#pragma unroll
                        for (int k = 0; k < 3; k++) {
                            const int n = i + 3 * j + 9 * k;
                            R[n] = fma_(k == 0 ? a : a + sz[k], U[n], R[n]);
                        }
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!ADV) next(L);
            if (L < Lb) load_c(L + 1);
            // back along x (the right node's part goes to the next lane), then y
            T rows[3][2][3];                                  // [row][column][z mode]
#pragma unroll
            for (int k = 0; k < 3; k++) {
                T l[3], c[3];
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    T x0, x1, x2;
                    from_modes(Modes<T>{R[3 * j + 9 * k], R[1 + 3 * j + 9 * k], R[2 + 3 * j + 9 * k]}, x0, x1, x2);
                    l[j] = x0 + from_left(x2);
                    c[j] = x1;
                }
                from_modes(Modes<T>{l[0], l[1], l[2]}, rows[0][0][k], rows[1][0][k], rows[2][0][k]);
                from_modes(Modes<T>{c[0], c[1], c[2]}, rows[0][1][k], rows[1][1][k], rows[2][1][k]);
            }
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int k = 0; k < 3; k++) xch[L & 1][wave][3 * a + k][lane] = rows[2][a][k];
            __syncthreads();
            {
                const int below = wave > 0 ? wave - 1 : 0;
#pragma unroll
                for (int a = 0; a < 2; a++)
#pragma unroll
                    for (int k = 0; k < 3; k++) rows[0][a][k] += xch[L & 1][below][3 * a + k][lane];
            }
            T v0[2][2], v1[2][2];
#pragma unroll
            for (int r = 0; r < 2; r++)
#pragma unroll
                for (int a = 0; a < 2; a++) {
                    T z0, z1, z2;
                    from_modes(Modes<T>{rows[r][a][0], rows[r][a][1], rows[r][a][2]}, z0, z1, z2);
                    v0[r][a] = tc[r][a] + z0;
                    v1[r][a] = z1;
                    tc[r][a] = z2;
                }
            if (2 * L >= kb) {
                epilogue(2 * L, v0);
                if (2 * L + 1 < ke) epilogue(2 * L + 1, v1);
            }
        }
        // the top plane of the mesh has no cells above it
        if (ke == NZ) epilogue(NZ - 1, tc);
    };
    if (adv) march(std::integral_constant<bool, FIELD == 1>{});
    else march(std::false_type{});
    if (EPI == EPI_RESID_NORM || EPI == EPI_DOT) {
        const double s = wave_sum(acc);
        if (lane == 0) red[wave] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double p = red[0];
#pragma unroll
            for (int w = 1; w < W2; w++) p += red[w];
            ep.partial[wi.slot] = p;
        }
    }
}

template <int FIELD, bool MASKED, bool G>
void launch_epi(int epi, int nwork, const Tabled &at, const double *x, double *y, const EpiArgs<double> &ep, hipStream_t s)
{
    const dim3 grid((unsigned)nwork), block(64 * q2s_waves(FIELD, true));
    switch (epi) {
    case EPI_STORE: k_q2_strip<double, FIELD, EPI_STORE, MASKED, G, false><<<grid, block, 0, s>>>(at, x, y, ep); break;
    case EPI_RESID: k_q2_strip<double, FIELD, EPI_RESID, MASKED, G, false><<<grid, block, 0, s>>>(at, x, y, ep); break;
    case EPI_RESID_NORM:
        k_q2_strip<double, FIELD, EPI_RESID_NORM, MASKED, G, false><<<grid, block, 0, s>>>(at, x, y, ep);
        break;
    case EPI_DOT: k_q2_strip<double, FIELD, EPI_DOT, MASKED, G, false><<<grid, block, 0, s>>>(at, x, y, ep); break;
    case EPI_CHEB: k_q2_strip<double, FIELD, EPI_CHEB, MASKED, G, false><<<grid, block, 0, s>>>(at, x, y, ep); break;
    default: throw Error(-1, "bad epilogue");
    }
}

}  // namespace

// FP64 only: the solvers' FP32 operators are those of the refined mode, which keeps
// the tile kernels
void launch_q2s(int field, int epi, bool masked, bool graded, const OpDev *ops, const WorkItem *work, int nwork,
                const double *x, double *y, const EpiArgs<double> &ep, hipStream_t s)
{
    if (nwork <= 0) return;
    const Tabled at{ops, work};
    if (field == 0) {
        if (masked) graded ? launch_epi<0, true, true>(epi, nwork, at, x, y, ep, s) : launch_epi<0, true, false>(epi, nwork, at, x, y, ep, s);
        else graded ? launch_epi<0, false, true>(epi, nwork, at, x, y, ep, s) : launch_epi<0, false, false>(epi, nwork, at, x, y, ep, s);
    } else {
        if (masked) graded ? launch_epi<1, true, true>(epi, nwork, at, x, y, ep, s) : launch_epi<1, true, false>(epi, nwork, at, x, y, ep, s);
        else graded ? launch_epi<1, false, true>(epi, nwork, at, x, y, ep, s) : launch_epi<1, false, false>(epi, nwork, at, x, y, ep, s);
    }
    HTS_LAUNCH_CHECK();
}

// y = A x (masked) of one mesh, as launch_q1s_solo
template <typename T>
void launch_q2s_solo(int field, bool graded, const OpDev &op, int ntx, int zc, const T *x, T *y, hipStream_t s)
{
    const Solo a = solo_work(op, ntx, zc);
    const dim3 grid((unsigned)(8 * a.per)), block(64 * q2s_waves(field, sizeof(T) == 8));
    EpiArgs<T> ep{};
    if (field == 0 && !graded) k_q2_strip<T, 0, EPI_STORE, true, false, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else if (field == 0) k_q2_strip<T, 0, EPI_STORE, true, true, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else if (!graded) k_q2_strip<T, 1, EPI_STORE, true, false, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else k_q2_strip<T, 1, EPI_STORE, true, true, true><<<grid, block, 0, s>>>(a, x, y, ep);
    HTS_LAUNCH_CHECK();
}
template void launch_q2s_solo<double>(int, bool, const OpDev &, int, int, const double *, double *, hipStream_t);
template void launch_q2s_solo<float>(int, bool, const OpDev &, int, int, const float *, float *, hipStream_t);

}  // namespace hts
