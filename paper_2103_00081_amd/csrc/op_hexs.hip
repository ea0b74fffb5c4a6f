// One application of the matrix-free Q1 operators on general hexahedra (op_hex.hip)
// for a single mesh, one wave per strip of cell columns.
//
// Layout: as op_q2s.hip with one node per cell column.  A lane is a node column x on
// two node rows, the lower and upper ones of its cell row; the right neighbours are
// the next lane's (DPP wave shift).  The waves of a block sit side by side along y and
// march upward one cell layer at a time; the node columns of all y bands are laid end
// to end with an empty one after each, a block takes 64 consecutive ones (62 owned),
// and a band owns the node rows above its first wave's (which is halo).  The node row
// that two waves share passes through LDS with one barrier per layer.  Every node value
// is produced by exactly one lane, as a fixed expression.
//
// A trilinear field of a cell is held in Haar modes: along an axis the pair (v0, v1)
// becomes s = v0 + v1 and t = v1 - v0, so the value at the two Gauss points is
// (s -+ t / sqrt 3) / 2 and the derivative t.  The modes along z and y are formed
// once for the cells beside a column, and values, derivatives and their transposes are
// sums of the 8 modes with weights 1 / sqrt 3 per t of a value.  With g, J, C the sums
// without their factors 1/2, every term of a cell has the common factor kappa = 1 / 512:
// stiffness kappa s, mass kappa m / 64, convection kappa c_adv k / 8.  (With t / sqrt 3 as
// the mode the weights are signs, but each mode is rounded once more on either way and
// the error of fl(1 / sqrt 3) enters every entry of J: FP32 pressure was off by 1.3 times
// as much against 64 bits.)  The modes of the coordinates are formed in FP64 against the
// lane's own lower node, so that the FP32 operator rounds sums of a cell's size once
// (formed in FP32 they cost 8 % more error and save 1 us of 44); the FP32 pressure is the
// piezometric one that k_piezo32 forms, against the same node.  Cells outside the mesh are
// computed on whatever their lanes hold and dropped.
//
// What bounds it: the issue of its instructions (a vector instruction in 93 to 100 % of the
// busy time in FP32, 74 % in FP64), 815 for a cell layer of the FP32 heat
// operator (720 pressure) where the tile kernel has 2600, most of them for the Jacobian at
// 8 points.  Four waves per block: eight have a seventh of halo rows instead of a third,
// and take 50.6 us against 52.2 (FP32 heat, 128 x 128 x 64), but 11.9 against 9.0 on
// 40 x 33 x 21, where a block's layer is a wave's; two cell rows per wave (197 registers,
// a seventh of halo rows) 51.0 and 12.2.  Kernel times against k_hex_apply, us,
// at 128 x 128 x 64 cells | 40 x 33 x 21 | 12 x 10 x 8 (there besides a copy, the forming
// of the FP32 pressure and a write of flags before each apply, 5 to 15 us):
//   FP64 pressure   87.7 -> 61.4 | 15.3 -> 8.8 | 14.3 -> 8.3
//   FP32 pressure   61.7 -> 43.6 | 15.1 -> 8.5 | 14.2 -> 8.2
//   FP64 heat      142.9 -> 70.6 | 20.0 -> 10.0 | 18.8 -> 9.1
//   FP32 heat       81.3 -> 50.5 | 19.0 -> 9.1 | 17.0 -> 8.9
// The solves on hexahedra keep the tile kernel: this one has the store epilogue alone, and
// no form over device tables.
#include "strip.h"

namespace hts {

namespace {

constexpr double I3 = 0.57735026918962576451;   // 1 / sqrt 3
constexpr double KAPPA = 1.0 / 512.0;

__device__ __forceinline__ float recip(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fma_(fma_(-x, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma_(fma_(-x, r, 1.0), r, r);
    return fma_(fma_(-x, r, 1.0), r, r);
}

// a / x: as many operations as a recip(x), one rounding less
__device__ __forceinline__ float quot(float a, float x)
{
    const float r = __builtin_amdgcn_rcpf(x), q = a * r;
    return fma_(fma_(-x, q, a), r, q);
}
__device__ __forceinline__ double quot(double a, double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma_(fma_(-x, r, 1.0), r, r);
    const double q = a * r;
    return fma_(fma_(-x, q, a), r, q);
}

// modes of a trilinear field, index x + 2 y + 4 z (0: s, 1: t), from the node pairs
// (lower, upper) of the two rows of this lane and of the next; shift: what the next
// lane's values are to be raised by
template <typename T>
__device__ __forceinline__ void modes8(T a0, T a1, T b0, T b1, T shift, T (&F)[8])
{
    const T as = a0 + a1, at = a1 - a0, bs = b0 + b1, bt = b1 - b0;
    const T l[4] = {as + bs, bs - as, at + bt, bt - at};
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const T r = e == 0 ? from_right(l[e]) + shift : from_right(l[e]);
        F[2 * e] = l[e] + r;
        F[1 + 2 * e] = r - l[e];
    }
}

// derivatives along z at the points (qx, qy), the same on both planes of points
template <typename T>
__device__ __forceinline__ void deriv_z(const T (&F)[8], T (&z)[4])
{
    const T i3 = T(I3);
    const T a = fma_(-i3, F[5], F[4]), b = fma_(i3, F[5], F[4]), c = fma_(-i3, F[7], F[6]), d = fma_(i3, F[7], F[6]);
    z[0] = fma_(-i3, c, a);
    z[1] = fma_(-i3, d, b);
    z[2] = fma_(i3, c, a);
    z[3] = fma_(i3, d, b);
}
// derivatives along x at qy and along y at qx, on one plane of points
template <typename T>
__device__ __forceinline__ void deriv_xy(const T (&F)[8], int qz, T (&x)[2], T (&y)[2])
{
    const T i3 = T(I3), w = qz ? i3 : -i3;
    const T ts = fma_(w, F[5], F[1]), st = fma_(w, F[6], F[2]), tt = fma_(w, F[7], F[3]);
    x[0] = fma_(-i3, tt, ts);
    x[1] = fma_(i3, tt, ts);
    y[0] = fma_(-i3, tt, st);
    y[1] = fma_(i3, tt, st);
}

template <typename T, int FIELD>
__global__ __launch_bounds__(64 * HEXS_WAVES) void k_hex_strip(const Solo at, const T *__restrict__ X, T *__restrict__ Y)
{
    constexpr int W = HEXS_WAVES;
    constexpr bool HEAT = FIELD == 1, PIEZO = HEAT && sizeof(T) == 4;
    __shared__ T xch[2][W][2][64];                            // upper-row sums of a wave's cells
    const WorkItem wi = at.item();
    if (wi.inst < 0) return;
    const OpDev &o = at.op(0);
    const int nx = o.nx, ny = o.ny, nz = o.nz, NX = o.NX, NY = o.NY, NZ = o.NZ, m = o.dmask;
    const int64_t plane = (int64_t)NX * NY, cplane = (int64_t)nx * ny;
    constexpr uint32_t SZ = sizeof(T);
    const uint32_t pbytes = (uint32_t)(plane * SZ), cbytes = (uint32_t)(cplane * SZ), dbytes = (uint32_t)(plane * 8);
    const T *kk = static_cast<const T *>(o.k), *lam = static_cast<const T *>(o.lam), *cT = static_cast<const T *>(o.cT);
    const double *Pi = static_cast<const double *>(o.P);

    // ---- the lane's node column (x = nx: the last, nx + 1: empty) and cell row
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tot = ((NY + W - 2) / (W - 1)) * (nx + 2);
    const int pos = wi.tx * HEXS_OWNED + lane - 1;
    const bool pin = pos >= 0 && pos < tot;
    const int band = (pin ? pos : 0) / (nx + 2), x = (pin ? pos : 0) - band * (nx + 2);
    const int J = band * (W - 1) - 1 + wave;
    const bool xin = pin && x <= nx;
    const bool mine = xin && lane >= 1 && lane <= HEXS_OWNED && wave > 0 && J < NY;
    const bool cell = pin && x < nx && J >= 0 && J < ny;
    uint32_t offx[2], offp[2];
    const double HTS_GLOBAL *cp[2];
    bool con[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const int j = J + r;
        const bool here = xin && j >= 0 && j < NY;
        const uint32_t n = here ? (uint32_t)(x + NX * j) : 0u;
        con[r] = here && (((m & 1) && x == 0) || ((m & 2) && x == NX - 1) || ((m & 4) && j == 0) || ((m & 8) && j == NY - 1));
        offx[r] = here && !con[r] ? n * SZ : OOB;
        offp[r] = here ? n * 8u : OOB;
        cp[r] = gptr<double>(o.xyz) + 3 * (size_t)n;
    }
    const uint32_t offo = mine ? (uint32_t)(x + NX * J) * SZ : OOB;
    const uint32_t co = cell ? (uint32_t)(x + nx * J) * SZ : OOB;
    const bool faces = __any(con[0]);
    const bool adv = HEAT && o.cadv != 0.0;
    const double pref = PIEZO && adv ? Pi[0] : 0.0, zref = PIEZO && adv ? o.xyz[2] : 0.0;

    const int kb = wi.z0, ke = wi.z1;
    const int La = kb > 0 ? kb - 1 : 0, Lb = ke - 1 < nz ? ke - 1 : nz - 1;
    auto zface = [&](int k) { return ((m & 16) && k == 0) || ((m & 32) && k == NZ - 1); };
    struct Plane {
        T u[2];
        double p[2], c[2][3];
    };
    auto load = [&](int k, Plane &a, auto adv_) {
        const Rsrc rx = rsrc(X + k * plane, zface(k) ? 0u : pbytes), rp = rsrc(Pi + (HEAT ? k * plane : 0), dbytes);
#pragma unroll
        for (int r = 0; r < 2; r++) {
            a.u[r] = bld<T>(rx, offx[r]);
            if (decltype(adv_)::value) a.p[r] = bld<double>(rp, offp[r]);
            const double HTS_GLOBAL *c = cp[r] + 3 * (k * plane);
#pragma unroll
            for (int d = 0; d < 3; d++) a.c[r][d] = c[d];
        }
    };
    // one node plane of the result: v = A u
    auto store = [&](int k, T v) {
        const Rsrc ry = rsrc(Y + k * plane, pbytes);
        const bool zf = zface(k);
        if (zf || faces) {
            const T xv = bld<T>(rsrc(X + k * plane, pbytes), offo);
            v = zf || con[0] ? xv : v;
        }
        bst<T>(ry, offo, v);
    };

    auto march = [&](auto adv_) {
        constexpr bool ADV = decltype(adv_)::value;
        Plane lo, hi;
        T mass, stiff, conv, tc = T(0);
        auto load_c = [&](int L) {
            const Rsrc rk = rsrc(kk + L * cplane, cbytes);
            if (HEAT) {
                mass = bld<T>(rsrc(cT + L * cplane, cbytes), co) * T(KAPPA / 64.0);
                stiff = bld<T>(rsrc(lam + L * cplane, cbytes), co) * T(KAPPA * o.cs);
                conv = ADV ? bld<T>(rk, co) * T(KAPPA / 8.0 * o.cadv) : T(0);
            } else {
                mass = T(o.cm * (KAPPA / 64.0));
                stiff = bld<T>(rk, co) * T(KAPPA * o.cs);
                conv = T(0);
            }
        };
        load(La, lo, adv_);
        load(La + 1, hi, adv_);
        load_c(La);
        for (int L = La; L <= Lb; L++) {
            // ---- modes of the coordinates, the operand and the pressure
            T G[3][8], U[8], P[8];
#pragma unroll
            for (int d = 0; d < 3; d++) {
                const double own = lo.c[0][d];
                double g8[8];
                modes8(0.0, hi.c[0][d] - own, lo.c[1][d] - own, hi.c[1][d] - own, 4.0 * (from_right(own) - own), g8);
#pragma unroll
                for (int i = 0; i < 8; i++) G[d][i] = T(g8[i]);
            }
            modes8(lo.u[0], hi.u[0], lo.u[1], hi.u[1], T(0), U);
            if (ADV) {
                if (PIEZO) {
                    auto phi = [&](const Plane &a, int r) {
                        return T(fma_(o.rho_g, a.c[r][2] - zref, a.p[r] - pref));
                    };
                    const T own = phi(lo, 0);
                    modes8(T(0), phi(hi, 0) - own, phi(lo, 1) - own, phi(hi, 1) - own, T(4) * (from_right(own) - own), P);
                } else {
                    const double own = lo.p[0];
                    modes8(T(0), T(hi.p[0] - own), T(lo.p[1] - own), T(hi.p[1] - own), T(4) * T(from_right(own) - own), P);
                }
            }
            const T ms = mass, st = stiff, cv = conv;
            // the next layer's upper plane, while this one is worked on
            lo = hi;
            if (L < Lb) {
                load(L + 2, hi, adv_);
                load_c(L + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            // ---- the 8 Gauss points, one plane at a time
            const T i3 = T(I3);
            T jz[3][4], gz[4], pz[4];
#pragma unroll
            for (int d = 0; d < 3; d++) deriv_z(G[d], jz[d]);
            deriv_z(U, gz);
            if (ADV) deriv_z(P, pz);
            T R[8] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0), T(0)}, fz[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int qz = 0; qz < 2; qz++) {
                T jx[3][2], jy[3][2], gx[2], gy[2], px[2], py[2], uq[4];
#pragma unroll
                for (int d = 0; d < 3; d++) deriv_xy(G[d], qz, jx[d], jy[d]);
                deriv_xy(U, qz, gx, gy);
                if (ADV) deriv_xy(P, qz, px, py);
                {
                    const T w = qz ? i3 : -i3;
                    const T ss = fma_(w, U[4], U[0]), ts = fma_(w, U[5], U[1]), s2 = fma_(w, U[6], U[2]), t2 = fma_(w, U[7], U[3]);
                    const T a = fma_(-i3, ts, ss), b = fma_(i3, ts, ss), c = fma_(-i3, t2, s2), d = fma_(i3, t2, s2);
                    uq[0] = fma_(-i3, c, a);
                    uq[1] = fma_(-i3, d, b);
                    uq[2] = fma_(i3, c, a);
                    uq[3] = fma_(i3, d, b);
                }
                T fx[2] = {T(0), T(0)}, fy[2] = {T(0), T(0)}, mq[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int qx = q & 1, qy = q >> 1;
                    const T J[3][3] = {{jx[0][qy], jy[0][qx], jz[0][q]}, {jx[1][qy], jy[1][qx], jz[1][q]}, {jx[2][qy], jy[2][qx], jz[2][q]}};
                    T C[3][3];                                // cofactors: J^-1 = C^T / det
                    C[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
                    C[0][1] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
                    C[0][2] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
                    C[1][0] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
                    C[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
                    C[1][2] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
                    C[2][0] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
                    C[2][1] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
                    C[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
                    const T det = J[0][0] * C[0][0] + J[0][1] * C[0][1] + J[0][2] * C[0][2];
                    const T idet = ADV ? recip(det) : T(0), sc = ADV ? st * idet : quot(st, det);
                    T cg[3];
#pragma unroll
                    for (int i = 0; i < 3; i++) cg[i] = C[i][0] * gx[qy] + C[i][1] * gy[qx] + C[i][2] * gz[q];
                    // h = C^T C g: the flux, and (C g_P) . (C g) = g_P . h
                    T h[3];
#pragma unroll
                    for (int j = 0; j < 3; j++) h[j] = C[0][j] * cg[0] + C[1][j] * cg[1] + C[2][j] * cg[2];
                    mq[q] = ms * uq[q] * det;
                    if (ADV) {
                        T w;
                        if (PIEZO) {
                            w = px[qy] * h[0] + py[qx] * h[1] + pz[q] * h[2];
                        } else {
                            // the hydrostatic part cancels in the flux itself, before
                            // products that round it differently (with g_P . h as above
                            // 58.4 us instead of 62.4 on 128 x 128 x 64, and up to 1.2
                            // times the tile kernel's error, now 1.0 to 1.1)
                            T cp[3];
#pragma unroll
                            for (int i = 0; i < 3; i++) cp[i] = C[i][0] * px[qy] + C[i][1] * py[qx] + C[i][2] * pz[q];
                            cp[2] = fma_(T(o.rho_g), det, cp[2]);
                            w = cp[0] * cg[0] + cp[1] * cg[1] + cp[2] * cg[2];
                        }
                        mq[q] -= cv * idet * w;
                    }
                    fx[qy] += sc * h[0];
                    fy[qx] += sc * h[1];
                    fz[q] += sc * h[2];
                }
                // onto the modes of the test functions
                const T a = mq[0] + mq[1], b = mq[1] - mq[0], c = mq[2] + mq[3], d = mq[3] - mq[2];
                const T v[4] = {a + c, fma_(i3, b + d, fx[0] + fx[1]), fma_(i3, c - a, fy[0] + fy[1]),
                                fma_(T(1.0 / 3.0), d - b, i3 * ((fx[1] - fx[0]) + (fy[1] - fy[0])))};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    R[i] += v[i];
                    R[i + 4] += qz ? v[i] : -v[i];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            {
                const T a = fz[0] + fz[1], b = fz[1] - fz[0], c = fz[2] + fz[3], d = fz[3] - fz[2];
                R[4] = fma_(i3, R[4], a + c);
                R[5] = i3 * (R[5] + (b + d));
                R[6] = i3 * (R[6] + (c - a));
                R[7] = i3 * fma_(i3, d - b, R[7]);
            }
#pragma unroll
            for (int i = 0; i < 8; i++) R[i] = cell ? R[i] : T(0);
            // ---- back along x (the right node's part goes to the next lane), then y
            T row[2][2];                                      // [row][z mode]
#pragma unroll
            for (int z = 0; z < 2; z++) {
                T l[2];
#pragma unroll
                for (int y = 0; y < 2; y++) {
                    const T s = R[2 * y + 4 * z], t = R[1 + 2 * y + 4 * z];
                    l[y] = (s - t) + from_left(s + t);
                }
                row[0][z] = l[0] - l[1];
                row[1][z] = l[0] + l[1];
                xch[L & 1][wave][z][lane] = row[1][z];
            }
            __syncthreads();
            const int below = wave > 0 ? wave - 1 : 0;
            const T zs = row[0][0] + xch[L & 1][below][0][lane], zt = row[0][1] + xch[L & 1][below][1][lane];
            if (L >= kb) store(L, tc + (zs - zt));
            tc = zs + zt;
        }
        // the top plane of the mesh has no cells above it
        if (ke == NZ) store(NZ - 1, tc);
    };
    if (adv) march(std::integral_constant<bool, HEAT>{});
    else march(std::false_type{});
}

}  // namespace

// y = A x (masked) of one mesh, as launch_q1s_solo
template <typename T>
void launch_hexs_solo(int field, const OpDev &op, int ntx, int zc, const T *x, T *y, hipStream_t s)
{
    const Solo a = solo_work(op, ntx, zc);
    const dim3 grid((unsigned)(8 * a.per)), block(64 * HEXS_WAVES);
    if (field == 0) k_hex_strip<T, 0><<<grid, block, 0, s>>>(a, x, y);
    else k_hex_strip<T, 1><<<grid, block, 0, s>>>(a, x, y);
    HTS_LAUNCH_CHECK();
}
template void launch_hexs_solo<double>(int, const OpDev &, int, int, const double *, double *, hipStream_t);
template void launch_hexs_solo<float>(int, const OpDev &, int, int, const float *, float *, hipStream_t);

}  // namespace hts
