// Matrix-free Q1 operators of the pressure (Eq. 3) and heat (Eq. 4)
// equations on rectilinear meshes, one wave per strip of node columns.
//
// Layout: a lane is one node column x and carries R + 1 consecutive node rows
// along y (R cell rows, the cells to the right of the column); the four waves of
// a block sit side by side along y and march upward through its range of node
// planes.  The node columns of all y bands are laid end to end with one empty
// column after each band, and a block takes 64 consecutive ones (62 owned, one
// halo on either side), so rows of any length fill the lanes.  A band owns
// 4 R - 1 node rows.  Neighbours along x are the neighbouring lanes (DPP wave
// shifts), along y registers, along z the previous iteration; only the node row
// that two waves share passes through LDS, with one barrier per cell layer.
// Every node value is produced by exactly one lane, as a fixed expression: no
// atomics, bitwise reproducible, independent of the chunk depth.
//
// Cells are evaluated in Haar coordinates: along one axis the pair of node values
// (v0, v1) becomes (s, d) = (v0 + v1, v0 - v1), and results go back as (s + d, s - d);
// there the unscaled 1D mass [2 1; 1 2] and stiffness [1 -1; -1 1] are diagonal, (3, 1)
// and (0, 2), and the interpolation to the two Gauss points is (1, 1 / sqrt 3).  Mass
// and stiffness are one scaling of the 8 coefficients of a cell, a product at the Gauss
// points weighs pairs of d with 1/3.  The z pair of a node column is formed once for the
// four cells around it, the y pairs once for the two cells beside it, and the same on
// the way back, by sums and differences alone: with d / sqrt 3, where all those weights
// are 1, each pair is rounded once more on either way, and the error against 64 bits
// was up to 1.6 (FP64 pressure), 1.9 (FP32) and 1.2 (FP32 heat) times the tiles'.
//
// What bounds it: on large grids the streaming of the planes (with the cell
// arithmetic taken out a 256 x 256 x 128 apply takes 50 us for pressure FP64 and
// 55 us for heat FP32), on small ones the
// march of a wave.  Against the LDS tiles of op_q1.hip on 256 x 256 x 128 cells
// (four rotating buffer pairs, events around each launch): pressure FP64 78.3 ->
// 54.5 us, FP32 50.6 -> 34.4, heat FP64 153 -> 117, FP32 89.9 -> 70.0; on
// 128 x 128 x 64: 17.3 -> 13.0, 14.0 -> 10.3, 28.3 -> 22.1, 21.0 -> 17.3; on
// 256 x 200 x 128 graded: 68.0 -> 51.6, 44.5 -> 33.4, 135 -> 113, 82.3 -> 68.2.  Two
// cell rows per wave: with four (as scaled pairs) the same at 256 x 256 x 128
// and slower on small grids (48^3 heat FP32 9.5 -> 11.7 us); with one, 8 to 40 %
// slower on the large grid.  Waves side by side share a halo row; on their own
// (four rows each) heat FP32 takes 80 us.  A block's layer costs the same however few of
// its columns the mesh has: heat on columns of at most 8 x 8 cells and 8000 or more
// layers takes 1.05 to 1.6 times the tiles (2 x 2 x 30000: FP64 70 -> 109 us).
//
// One apply of one mesh (SOLO) takes its descriptor by value, finds its work from
// the block index and reads the pressure state itself: 32^3 pressure FP32 8.5 ->
// 4.7 us a call, 128 x 128 x 64 heat FP64 31.7 -> 18.6 (flag, slot and pressure
// copies before it), 256 x 256 x 128 heat FP32 113 -> 68 (and no FP32 copy of the
// pressure).  A SOLO kernel for graded meshes never sees a uniform one, whose factors
// would take 9 to 26 registers from it and spill scalar ones: 256 x 200 x 128 heat FP64
// 120 -> 108 us, FP32 74.9 -> 62.6.
//
// Fused multiply-adds are written out and contraction is off, so that every
// instance of the kernel (graded or not, each epilogue) rounds alike.
//
// Loads and stores are raw buffer accesses on the current plane: a lane whose
// value has to read as zero (outside the mesh, constrained) or that stores
// nothing gets an offset past the end, which the hardware turns into a zero or
// drops, so the march needs no selects or branches for them.
#include <type_traits>

#include "strip.h"

namespace hts {

namespace {

#pragma clang fp contract(off)

// differences among the axes of Haar coefficient i (index x + 2y + 4z)
constexpr int haar_order(int i) { return (i & 1) + (i >> 1 & 1) + (i >> 2); }

// o += 3^n times the Gauss-point product of A and v projected back (2D Haar
// coordinates: 0 ss, 1 ds, 2 sd, 3 dd; n differences of the result's), t = v / 3,
// n3 = v[3] / 9
template <typename T>
__device__ __forceinline__ void haar_prod2(const T A[4], const T v[4], T t1, T t2, T t3, T n3, T &o0, T &o1, T &o2, T &o3)
{
    o0 = fma_(A[0], v[0], fma_(A[1], t1, fma_(A[2], t2, fma_(A[3], n3, o0))));
    o1 = fma_(A[0], v[1], fma_(A[1], v[0], fma_(A[2], t3, fma_(A[3], t2, o1))));
    o2 = fma_(A[0], v[2], fma_(A[2], v[0], fma_(A[1], t3, fma_(A[3], t1, o2))));
    o3 = fma_(A[0], v[3], fma_(A[1], v[2], fma_(A[2], v[1], fma_(A[3], v[0], o3))));
}

// Mass and stiffness on the Haar coefficients, with the weight 3^-n of a coefficient of
// n differences.  Of a uniform mesh: factors for unit coefficients, m by n, k by
// coefficient, each rounded once
template <typename T>
struct HaarDiag {
    T m[4], k[8];
    __device__ __forceinline__ explicit HaarDiag(const OpDev &o)
    {
#pragma unroll
        for (int n = 0; n < 4; n++) m[n] = T(o.hm[n]);
#pragma unroll
        for (int i = 0; i < 8; i++) k[i] = T(o.hk[i]);
    }
    // D: the diagonal of a cell of mass a and stiffness coefficient c
    __device__ __forceinline__ void of_cell(T a, T c, T D[8]) const
    {
        D[0] = a * m[0];
#pragma unroll
        for (int i = 1; i < 8; i++) D[i] = fma_(c, k[i], a * m[haar_order(i)]);
    }
};
// The same of a graded cell from the parts of its column and of its layer: m0, m1, m2 the
// mass by n (a third taken once per column in FP64: fl(1/3) is off by half a unit in the
// last place in every cell), x, y, z a third of the stiffnesses for unit coefficient, c
// the coefficient
template <typename T>
__device__ __forceinline__ void haar_diag_graded(T m0, T m1, T m2, T x, T y, T z, T c, T D[8])
{
    const T third = T(1.0 / 3.0), ct = third * c, xy = x + y;
    D[0] = m0;
    D[1] = fma_(c, x, m1);
    D[2] = fma_(c, y, m1);
    D[4] = fma_(c, z, m1);
    D[3] = fma_(ct, xy, m2);
    D[5] = fma_(ct, x + z, m2);
    D[6] = fma_(ct, y + z, m2);
    D[7] = third * fma_(ct, xy + z, m2);
}

// sum_q N_a(q) (q_h . grad u)(q) dt c_w V / 8 at the 2 x 2 x 2 Gauss points,
// q_h = -k (grad P + rho_g e_z): per axis the product of two bilinear
// fields on the cell's cross-section, both given by Haar coefficients (Q: of P,
// with the gravity part in the z difference), constant along the axis.  ax, ay,
// az: -k dt c_w V / (8 h_d^2) times 1 / 16.  C: 3^n times the result (that of index 7 is 0).
template <typename T>
__device__ __forceinline__ void haar_convect(const T U[8], const T Q[8], T ax, T ay, T az, T C[7])
{
    const T third = T(1.0 / 3.0), ninth = T(1.0 / 9.0);
    const T t3 = U[3] * third, t5 = U[5] * third, t6 = U[6] * third, t7 = U[7] * third, n7 = U[7] * ninth;
#pragma unroll
    for (int i = 0; i < 7; i++) C[i] = T(0);
    const T Ax[4] = {ax * Q[1], ax * Q[3], ax * Q[5], ax * Q[7]}, vx[4] = {U[1], U[3], U[5], U[7]};
    haar_prod2(Ax, vx, t3, t5, t7, n7, C[0], C[2], C[4], C[6]);
    const T Ay[4] = {ay * Q[2], ay * Q[3], ay * Q[6], ay * Q[7]}, vy[4] = {U[2], U[3], U[6], U[7]};
    haar_prod2(Ay, vy, t3, t6, t7, n7, C[0], C[1], C[4], C[5]);
    const T Az[4] = {az * Q[4], az * Q[5], az * Q[6], az * Q[7]}, vz[4] = {U[4], U[5], U[6], U[7]};
    haar_prod2(Az, vz, t5, t6, t7, n7, C[0], C[1], C[2], C[3]);
}

// the 8 Haar coefficients of the cell right of this lane's column from the z
// pairs (s, d) of its two node rows
template <typename T>
__device__ __forceinline__ void haar_cell(T s0, T d0, T s1, T d1, T U[8])
{
    const T y[4] = {s0 + s1, s0 - s1, d0 + d1, d0 - d1};
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const T r = from_right(y[i]);
        U[2 * i] = y[i] + r;
        U[2 * i + 1] = y[i] - r;
    }
}

// The pressure's Haar coefficients 1 .. 7 of a cell, from differences of
// neighbouring nodes (formed first, so that they do not cancel against the
// magnitude of P).  Of a node row: the z pair of the x differences and the z
// difference; set() turns xl, the lower plane's x difference, into the upper one's.
template <typename T>
struct FluxRow {
    T xs, xd, z;
    __device__ __forceinline__ void set(T pl, T pu, T &xl)
    {
        const T xu = pu - from_right(pu);
        xs = xl + xu;
        xd = xl - xu;
        z = pl - pu;
        xl = xu;
    }
};
// yl, yu: the y differences of the two planes
template <typename T>
__device__ __forceinline__ void flux_cell(const FluxRow<T> &f0, const FluxRow<T> &f1, T yl, T yu, T Q[8])
{
    Q[0] = T(0);
    Q[1] = f0.xs + f1.xs;
    Q[3] = f0.xs - f1.xs;
    Q[5] = f0.xd + f1.xd;
    Q[7] = f0.xd - f1.xd;
    const T ys = yl + yu, yd = yl - yu, z = f0.z + f1.z;
    Q[2] = ys + from_right(ys);
    Q[6] = yd + from_right(yd);
    Q[4] = z + from_right(z);
}

// W += the injection lines of a cell (layer L of the blocks from b on): the
// operand's z pair at the line, through the line integrals of the layer, and back
template <typename T>
__device__ __forceinline__ void line_cell(const OpDev &o, int b, int L, const T U[8], T W[8])
{
    const double HTS_GLOBAL *lco = gptr<double>(o.lcoef);
    while (b >= 0) {
        const LineCell HTS_GLOBAL *e = gptr<LineCell>(o.lcell) + ((int64_t)b * o.nz + L);
        const double c = lco[e->src];
        const T px = T(e->px), py = T(e->py), pxy = px * py;
        const T s = fma_(px, U[1], U[0]) + fma_(pxy, U[3], py * U[2]);
        const T d = fma_(px, U[5], U[4]) + fma_(pxy, U[7], py * U[6]);
        const T ga = T(c * e->a), gb = T(c * e->b), gd = T(c * e->d);
        const T ws = fma_(gb, d, ga * s), wd = fma_(gd, d, gb * s);
        W[0] += ws; W[1] = fma_(px, ws, W[1]); W[2] = fma_(py, ws, W[2]); W[3] = fma_(pxy, ws, W[3]);
        W[4] += wd; W[5] = fma_(px, wd, W[5]); W[6] = fma_(py, wd, W[6]); W[7] = fma_(pxy, wd, W[7]);
        b = e->next;
    }
}

// SOLO: descriptor and work in the arguments; its FP32 heat operator reads the
// FP64 pressure state and forms the piezometric pressure as k_piezo32 does.  FP32 heat
// has to fit four waves on a SIMD (at 131 registers, three, a graded 256 x 200 x 128
// apply took 76.7 us, at 128 72.6)
template <typename T, int FIELD, int EPI, bool MASKED, bool GRADED, bool SOLO>
__global__ __launch_bounds__(64 * Q1S_WAVES, FIELD == 1 && sizeof(T) == 4 ? 4 : 1) void k_q1_strip(const typename std::conditional<SOLO, Solo, Tabled>::type at,
                                                  const T *__restrict__ X, T *__restrict__ Y, EpiArgs<T> ep)
{
    constexpr int R = Q1S_ROWS;                               // cell rows of a wave
    constexpr int OWNB = Q1S_WAVES * R - 1;                   // node rows a block owns
    __shared__ double red[Q1S_WAVES];
    __shared__ T xch[2][Q1S_WAVES][2][64];                    // upper-row sums of a wave's last cell row

    const WorkItem wi = at.item();
    if (SOLO ? wi.inst < 0 : (ep.active && !ep.active[wi.inst])) return;
    const OpDev &o = at.op(wi.inst);
    constexpr bool PIEZO = SOLO && FIELD == 1 && sizeof(T) == 4;
    using PT = typename std::conditional<PIEZO, double, T>::type;   // the pressure as stored
    const int nx = o.nx, ny = o.ny, nz = o.nz, NX = o.NX, NY = o.NY, NZ = o.NZ, m = o.dmask;
    constexpr bool CHEB = EPI == EPI_CHEB || EPI == EPI_CHEB0;
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
    const uint32_t rowb = (uint32_t)(NX * sizeof(T));

    // ---- the lane's node column: band and x (x = NX: the empty column)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tot = ((NY + OWNB - 1) / OWNB) * (NX + 1);
    const int pos = wi.tx * Q1S_OWNED + lane - 1;
    const bool pin = pos >= 0 && pos < tot;
    const int band = (pin ? pos : 0) / (NX + 1), x = (pin ? pos : 0) - band * (NX + 1), J0 = band * OWNB - 1 + wave * R;
    const bool xin = pin && x < NX, mine = xin && lane >= 1 && lane <= Q1S_OWNED;
    // byte offsets in a node plane of row 0 of the strip (row r: + r rowb; rows
    // above the mesh run past the end of the plane)
    const uint32_t nbase = (uint32_t)((x + NX * J0) * (int)sizeof(T));
    // owned rows 0 .. R - 1 of owned columns (row 0 of wave 0 is halo)
    const uint32_t own = mine ? nbase : OOB, own0 = mine && wave > 0 ? nbase : OOB;
    auto own_off = [&](int r) { return r == 0 ? own0 : own + r * rowb; };
    uint32_t xo[R + 1];                                       // operand: in the mesh, not on a constrained x/y face
    uint32_t co[R];                                           // cells
    uint32_t cmask = 0;                                       // bit r: row r constrained by an x/y face
    int32_t dl[MASKED ? R + 1 : 1];                           // constrained z-range of row r
    bool special = false, cols = false;
    {
        const bool xface = MASKED && (((m & 1) && x == 0) || ((m & 2) && x == NX - 1));
#pragma unroll
        for (int r = 0; r <= R; r++) {
            const int J = J0 + r;
            const bool in = xin && J >= 0 && J < NY;
            const bool con = MASKED && in && (xface || ((m & 4) && J == 0) || ((m & 8) && J == NY - 1));
            xo[r] = in && !con ? nbase + r * rowb : OOB;
            if (con) cmask |= 1u << r;
            if (MASKED) {
                dl[r] = DCOL_NONE;
                if (o.dcol && in) dl[r] = gptr<int32_t>(o.dcol)[x + NX * J];
                cols |= dl[r] != DCOL_NONE;
            }
            if (r < R) co[r] = xin && x < nx && J >= 0 && J < ny ? (uint32_t)((x + nx * J) * (int)sizeof(T)) : OOB;
        }
    }
    if (MASKED) {
        cols = __any(cols);
        special = cols || __any(cmask != 0);
    }
    int lb[FIELD ? R : 1];                                    // injection lines of the cells
    bool lines = false;
    if (FIELD == 1 && o.lccol) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            lb[FIELD ? r : 0] = -1;
            if (co[r] < cbytes) lb[FIELD ? r : 0] = gptr<int32_t>(o.lccol)[co[r] / sizeof(T)];
            lines |= lb[FIELD ? r : 0] >= 0;
        }
        lines = __any(lines);
    }

    // ---- factors of the unscaled 1D products (formed in double on the host)
    const HaarDiag<T> fd(o);
    const T vx = T(0.0625 * o.q1vx), vy = T(0.0625 * o.q1vy), vz = T(0.0625 * o.q1vz);
    const double rho_g = PIEZO ? 0.0 : o.rho_g;               // 0 where the pressure is piezometric
    const T pz = T(4.0 * rho_g * o.hz);
    // graded meshes (in a batch some may be uniform): parts of the cell column's hx, hy
    // per row (times a factor of the layer)
    const bool graded = GRADED && (SOLO || o.hzs != nullptr);
    T gx[GRADED ? R : 1], gy[GRADED ? R : 1], gm[GRADED ? R : 1], gm1[GRADED ? R : 1], gm2[GRADED ? R : 1];
    if (graded) {
        const double hx = o.hxs[x < nx ? x : nx - 1];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int J = J0 + r;
            const double hy = o.hys[J < 0 ? 0 : (J < ny ? J : ny - 1)];
            gx[r] = T(hy / hx);
            gy[r] = T(hx / hy);
            gm[r] = T(hx * hy * 0.015625);
            gm1[r] = T(hx * hy / 192.0);
            gm2[r] = T(hx * hy / 576.0);
        }
    }
    T c0 = T(0), c1 = T(0), c2 = T(0);
    if (CHEB) {
        const double *Sc = ep.S + (int64_t)wi.inst * NSLOT;
        c1 = T(Sc[ep.s1]);
        c2 = T(Sc[ep.s2]);
        if (EPI == EPI_CHEB0) c0 = T(Sc[ep.s0]);
    }

    // ---- the march
    const int kb = wi.z0, ke = wi.z1;                         // owned node planes
    const int La = kb > 0 ? kb - 1 : 0;                       // cell layers La .. Lb
    const int Lb = ke - 1 < nz ? ke - 1 : nz - 1;
    double acc = 0.0;

    auto zface = [&](int k) { return MASKED && (((m & 16) && k == 0) || ((m & 32) && k == NZ - 1)); };
    auto load_x = [&](int k, T *u) {
        const uint32_t n = zface(k) ? 0u : pbytes;
        if (EPI == EPI_CHEB0) {
            // operand x0 = c0 D^-1 b, in the order of the separate first
            // Chebyshev kernel
            const Rsrc rb = rsrc(Bi + k * plane, n), ri = rsrc(Ii + k * plane, n);
#pragma unroll
            for (int r = 0; r <= R; r++) u[r] = c0 * bld<T>(ri, xo[r]) * bld<T>(rb, xo[r]);
        } else {
            const Rsrc rx = rsrc(Xi + k * plane, n);
#pragma unroll
            for (int r = 0; r <= R; r++) u[r] = bld<T>(rx, xo[r]);
        }
    };
    // Dirichlet columns: rows whose z-range holds plane k read as zero
    auto mask_cols = [&](int k, T *u) {
        if (MASKED && cols) {
#pragma unroll
            for (int r = 0; r <= R; r++) {
                const int lo = dl[r] & 0xFFFF, hi = (dl[r] >> 16) & 0xFFFF;
                if (k >= lo && k <= hi) u[r] = T(0);
            }
        }
    };
    constexpr uint32_t PW = sizeof(PT) / sizeof(T);
    const uint32_t pb0 = xin ? nbase * PW : OOB, pbr0 = xin && J0 >= 0 ? nbase * PW : OOB;
    auto load_p = [&](int k, PT *u) {
        const Rsrc rp = rsrc(Pi + k * plane, pbytes * PW);
#pragma unroll
        for (int r = 0; r <= R; r++) u[r] = bld<PT>(rp, r == 0 ? pbr0 : pb0 + r * rowb * PW);
    };
    const double pref = PIEZO && o.cadv != 0.0 ? (double)Pi[0] : 0.0;
    // loaded pressure of plane k -> the operator's
    auto use_p = [&](int k, const PT *u, T *p) {
        if (PIEZO) {
            const double zk = graded ? o.zn[k] - o.zn[0] : k * o.hz;
#pragma unroll
            for (int r = 0; r <= R; r++) p[r] = T(fma_(o.rho_g, zk, (double)u[r] - pref));
        } else {
#pragma unroll
            for (int r = 0; r <= R; r++) p[r] = T(u[r]);
        }
    };
    auto load_c = [&](int L, T *ck, T *cl, T *cc) {
        const Rsrc rk = rsrc(kk + L * cplane, cbytes);
#pragma unroll
        for (int r = 0; r < R; r++) ck[r] = bld<T>(rk, co[r]);
        if (FIELD == 1) {
            const Rsrc rl = rsrc(lam + L * cplane, cbytes), rc = rsrc(cT + L * cplane, cbytes);
#pragma unroll
            for (int r = 0; r < R; r++) {
                cl[r] = bld<T>(rl, co[r]);
                cc[r] = bld<T>(rc, co[r]);
            }
        }
    };
    T eb[R], ed[R], ei[R], ex[R];
    // epilogue operands of plane k
    auto load_e = [&](int k) {
        const Rsrc rb = rsrc(HASB ? Bi + k * plane : Xi, pbytes), rd = rsrc(CHEB ? Di + k * plane : Xi, pbytes),
                   ri = rsrc(CHEB ? Ii + k * plane : Xi, pbytes);
#pragma unroll
        for (int q = 0; q < R; q++) {
            if (HASB) eb[q] = bld<T>(rb, own_off(q));
            if (EPI == EPI_CHEB) ed[q] = bld<T>(rd, own_off(q));
            if (CHEB) ei[q] = bld<T>(ri, own_off(q));
        }
        if (MASKED && EPI != EPI_CHEB0 && (special || zface(k))) {
            const Rsrc rx = rsrc(Xi + k * plane, pbytes);
#pragma unroll
            for (int q = 0; q < R; q++) ex[q] = bld<T>(rx, own_off(q));
        }
    };
    // v: A u at the owned rows of plane k, u: the plane's operand
    auto epilogue = [&](int k, T *v, const T *u) {
        const Rsrc ry = rsrc(Yi + k * plane, pbytes), rd = rsrc(CHEB ? Di + k * plane : Yi, pbytes);
        const bool zf = zface(k), sp = MASKED && (special || zf);
#pragma unroll
        for (int q = 0; q < R; q++) {
            T xq = u[q];
            if (EPI == EPI_CHEB0) xq = c0 * ei[q] * eb[q];
            if (sp) {
                if (EPI != EPI_CHEB0) xq = ex[q];
                const int lo = dl[MASKED ? q : 0] & 0xFFFF, hi = (dl[MASKED ? q : 0] >> 16) & 0xFFFF;
                if (zf || ((cmask >> q) & 1u) || (k >= lo && k <= hi)) v[q] = xq;
            }
            const uint32_t off = own_off(q);
            if (EPI == EPI_STORE) {
                bst<T>(ry, off, v[q]);
            } else if (EPI == EPI_RESID) {
                bst<T>(ry, off, eb[q] - v[q]);
            } else if (EPI == EPI_RESID_NORM) {
                const T r = eb[q] - v[q];
                bst<T>(ry, off, r);
                if (off < pbytes) acc = fma_((double)r, (double)r, acc);
            } else if (EPI == EPI_DOT) {
                bst<T>(ry, off, v[q]);
                if (off < pbytes) acc = fma_((double)xq, (double)v[q], acc);
            } else if (CHEB) {
                const T r = eb[q] - v[q];
                const T d = fma_(c1, EPI == EPI_CHEB0 ? xq : ed[q], c2 * ei[q] * r);
                bst<T>(rd, off, d);
                bst<T>(ry, off, xq + d);
            }
        }
    };

    auto march = [&](auto adv_) {
        constexpr bool ADV = decltype(adv_)::value;
        T lo[R + 1], up[R + 1], pl[ADV ? R + 1 : 1], pu[ADV ? R + 1 : 1];
        T ck[R], cl[R], cc[R];
        T tc[R];                                              // sums of the cells below, at the plane of `lo`
#pragma unroll
        for (int q = 0; q < R; q++) tc[q] = T(0);
        load_x(La, lo);
        load_x(La + 1, up);
        PT pa[ADV ? R + 1 : 1], pb[ADV ? R + 1 : 1];
        if (ADV) { load_p(La, pa); load_p(La + 1, pb); }
        load_c(La, ck, cl, cc);
        mask_cols(La, lo);
        T xl[ADV ? R + 1 : 1];                                // x differences of the lower plane's pressure
        if (ADV) {
            use_p(La, pa, pl);
#pragma unroll
            for (int r = 0; r <= R; r++) xl[ADV ? r : 0] = pl[ADV ? r : 0] - from_right(pl[ADV ? r : 0]);
        }
        for (int L = La; L <= Lb; L++) {
            T xn[R + 1], kn[R], ln[R], cn[R];
            if (ADV) use_p(L + 1, pb, pu);
            // loads of this layer's epilogue, then of the next layer
            if (L >= kb) load_e(L);
            if (L < Lb) {
                load_x(L + 2, xn);
                if (ADV) load_p(L + 2, pb);
                load_c(L + 1, kn, ln, cn);
            }
            mask_cols(L + 1, up);
            T um = T(0), ux = T(0), uz = T(0), uv = T(0), uw = T(0), g = pz;
            if (graded) {
                const double hz = o.hzs[L], ihz = o.ihzs[L];
                um = T(FIELD == 0 ? o.cm * hz : hz);
                ux = T(o.cs * 0.0625 * hz);
                uz = T(o.cs * 12.0 * ihz);
                uv = T(o.cadv * -0.0078125 * hz);
                uw = T(o.cadv * -0.5 * ihz);
                g = T(4.0 * rho_g * hz);
            }
            T v[R];
            T zs0 = lo[0] + up[0], zd0 = lo[0] - up[0];
            FluxRow<T> f0;
            if (ADV) f0.set(pl[0], pu[0], xl[0]);
            T s0 = T(0), d0 = T(0), us = T(0), ud = T(0);
#pragma unroll
            for (int r = 0; r < R; r++) {
                const T zs1 = lo[r + 1] + up[r + 1], zd1 = lo[r + 1] - up[r + 1];
                T U[8], W[8];
                haar_cell(zs0, zd0, zs1, zd1, U);
                zs0 = zs1;
                zd0 = zd1;
                if (ADV) {
                    T Q[8], lvx = vx, lvy = vy, lvz = vz;
                    if (graded) {
                        lvx = gx[GRADED ? r : 0] * uv;
                        lvy = gy[GRADED ? r : 0] * uv;
                        lvz = gm[GRADED ? r : 0] * uw;
                    }
                    FluxRow<T> f1;
                    f1.set(pl[ADV ? r + 1 : 0], pu[ADV ? r + 1 : 0], xl[ADV ? r + 1 : 0]);
                    flux_cell(f0, f1, pl[ADV ? r : 0] - pl[ADV ? r + 1 : 0], pu[ADV ? r : 0] - pu[ADV ? r + 1 : 0], Q);
                    Q[4] -= g;
                    f0 = f1;
                    T C[7];
                    haar_convect(U, Q, ck[r] * lvx, ck[r] * lvy, ck[r] * lvz, C);
                    W[0] = C[0];
#pragma unroll
                    for (int i = 1; i < 7; i++) W[i] = T(haar_order(i) == 1 ? 1.0 / 3.0 : 1.0 / 9.0) * C[i];
                    W[7] = T(0);
                } else {
#pragma unroll
                    for (int i = 0; i < 8; i++) W[i] = T(0);
                }
                if (FIELD == 1 && lines) line_cell(o, lb[FIELD ? r : 0], L, U, W);
                const T ma = FIELD == 0 ? T(co[r] < cbytes ? 1 : 0) : cc[r], st = FIELD == 0 ? ck[r] : cl[r];
                T D[8];
                if (graded) {
                    const int q = GRADED ? r : 0;
                    haar_diag_graded(ma * (gm[q] * um), ma * (gm1[q] * um), ma * (gm2[q] * um), gx[q] * ux, gy[q] * ux,
                                     gm1[q] * uz, st, D);
                } else {
                    fd.of_cell(ma, st, D);
                }
                // back along x (the right-hand part goes to the next lane), then y, z
                T c[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const int a = 2 * i, b = a + 1;
                    if (FIELD == 0) {
                        const T t = D[b] * U[b];
                        c[i] = fma_(D[a], U[a], t) + from_left(fma_(D[a], U[a], -t));
                    } else {
                        const T s = fma_(D[a], U[a], W[a]), t = fma_(D[b], U[b], W[b]);
                        c[i] = (s + t) + from_left(s - t);
                    }
                }
                const T sl = c[0] + c[1], dw = c[2] + c[3];
                if (r > 0) {
                    const T s = us + sl, d = ud + dw;
                    v[r] = tc[r] + (s + d);
                    tc[r] = s - d;
                } else {
                    s0 = sl;
                    d0 = dw;
                }
                us = c[0] - c[1];
                ud = c[2] - c[3];
            }
            // row 0 is the last wave's row R: the two exchange through LDS (two
            // buffers: a wave is at most one barrier ahead)
            xch[L & 1][wave][0][lane] = us;
            xch[L & 1][wave][1][lane] = ud;
            __syncthreads();
            {
                const int below = wave > 0 ? wave - 1 : 0;
                const T s = xch[L & 1][below][0][lane] + s0, d = xch[L & 1][below][1][lane] + d0;
                v[0] = tc[0] + (s + d);
                tc[0] = s - d;
            }
            if (L >= kb) epilogue(L, v, lo);
#pragma unroll
            for (int r = 0; r <= R; r++) {
                lo[r] = up[r];
                up[r] = xn[r];
                if (ADV) pl[ADV ? r : 0] = pu[ADV ? r : 0];
                if (r < R) { ck[r] = kn[r]; cl[r] = ln[r]; cc[r] = cn[r]; }
            }
        }
        // the top plane of the mesh has no cells above it
        if (ke == NZ) {
            load_e(NZ - 1);
            epilogue(NZ - 1, tc, lo);
        }
    };
    if (FIELD == 1 && o.cadv != 0.0) march(std::integral_constant<bool, FIELD == 1>{});
    else march(std::false_type{});
    if (EPI == EPI_RESID_NORM || EPI == EPI_DOT) {
        const double s = wave_sum(acc);
        if (lane == 0) red[wave] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double p = red[0];
#pragma unroll
            for (int w = 1; w < Q1S_WAVES; w++) p += red[w];
            ep.partial[wi.slot] = p;
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- launchers
template <typename T, int FIELD, int EPI, bool MASKED, bool G>
static void launch_k(int nwork, const OpDev *ops, const WorkItem *work, const T *x, T *y, const EpiArgs<T> &ep,
                     hipStream_t s)
{
    k_q1_strip<T, FIELD, EPI, MASKED, G, false><<<dim3(nwork), dim3(64 * Q1S_WAVES), 0, s>>>(Tabled{ops, work}, x, y,
                                                                                           ep);
}

template <typename T, int FIELD, bool MASKED, bool G>
static void dispatch_epi(int epi, const OpDev *ops, const WorkItem *work, int nwork, const T *x, T *y,
                         const EpiArgs<T> &ep, hipStream_t s)
{
    switch (epi) {
    case EPI_STORE: launch_k<T, FIELD, EPI_STORE, MASKED, G>(nwork, ops, work, x, y, ep, s); break;
    case EPI_RESID: launch_k<T, FIELD, EPI_RESID, MASKED, G>(nwork, ops, work, x, y, ep, s); break;
    case EPI_RESID_NORM: launch_k<T, FIELD, EPI_RESID_NORM, MASKED, G>(nwork, ops, work, x, y, ep, s); break;
    case EPI_DOT: launch_k<T, FIELD, EPI_DOT, MASKED, G>(nwork, ops, work, x, y, ep, s); break;
    case EPI_CHEB: launch_k<T, FIELD, EPI_CHEB, MASKED, G>(nwork, ops, work, x, y, ep, s); break;
    case EPI_CHEB0:
        if (!MASKED) throw Error(-1, "EPI_CHEB0 is for masked operators");
        launch_k<T, FIELD, EPI_CHEB0, true, G>(nwork, ops, work, x, y, ep, s);
        break;
    default: throw Error(-1, "bad epilogue");
    }
}

template <bool G>
static void launch_q1s_g(int field, int epi, bool masked, const OpDev *ops, const WorkItem *work, int nwork,
                         const double *x, double *y, const EpiArgs<double> &ep, hipStream_t s)
{
    if (field == 0) {
        if (masked) dispatch_epi<double, 0, true, G>(epi, ops, work, nwork, x, y, ep, s);
        else dispatch_epi<double, 0, false, G>(epi, ops, work, nwork, x, y, ep, s);
    } else {
        if (masked) dispatch_epi<double, 1, true, G>(epi, ops, work, nwork, x, y, ep, s);
        else dispatch_epi<double, 1, false, G>(epi, ops, work, nwork, x, y, ep, s);
    }
}

// FP64 only: the solvers' FP32 operators are those of the refined mode, which keeps
// the tile kernels.  graded: some instance has a graded mesh; those kernels form
// the per-cell factors per layer, the uniform ones keep them in registers
void launch_q1s(int field, int epi, bool masked, bool graded, const OpDev *ops, const WorkItem *work, int nwork,
                const double *x, double *y, const EpiArgs<double> &ep, hipStream_t s)
{
    if (nwork <= 0) return;
    if (graded) launch_q1s_g<true>(field, epi, masked, ops, work, nwork, x, y, ep, s);
    else launch_q1s_g<false>(field, epi, masked, ops, work, nwork, x, y, ep, s);
    HTS_LAUNCH_CHECK();
}

// y = A x (masked) of one mesh: op by value (off 0), the heat operator's P the FP64
// pressure state, tiles of ntx blocks and planes of zc
template <typename T>
void launch_q1s_solo(int field, bool graded, const OpDev &op, int ntx, int zc, const T *x, T *y, hipStream_t s)
{
    const Solo a = solo_work(op, ntx, zc);
    const dim3 grid((unsigned)(8 * a.per)), block(64 * Q1S_WAVES);
    EpiArgs<T> ep{};
    if (field == 0 && !graded) k_q1_strip<T, 0, EPI_STORE, true, false, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else if (field == 0) k_q1_strip<T, 0, EPI_STORE, true, true, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else if (!graded) k_q1_strip<T, 1, EPI_STORE, true, false, true><<<grid, block, 0, s>>>(a, x, y, ep);
    else k_q1_strip<T, 1, EPI_STORE, true, true, true><<<grid, block, 0, s>>>(a, x, y, ep);
    HTS_LAUNCH_CHECK();
}
template void launch_q1s_solo<double>(int, bool, const OpDev &, int, int, const double *, double *, hipStream_t);
template void launch_q1s_solo<float>(int, bool, const OpDev &, int, int, const float *, float *, hipStream_t);

}  // namespace hts
