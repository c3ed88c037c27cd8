// GSIS-II macroscopic synthetic solve (Sec. 3.3), point-Jacobi iteration on
// the GPU: on the box one launch per inner iteration (k_mac_iter), on an
// unstructured mesh per-cell and per-face kernels.
//
// Unknowns per fluid cell W = (rho, rho u, E, Er) with E = rho |u|^2 + 1.5 rho Tt + Er,
// Er = (dr/2) rho Tr (monatomic: Er = 0) -- the moments 1, xi, |xi|^2 (+ 1 on
// f1) of the kinetic equation, so the face fluxes are mass rho u_n; momentum
// rho u u_n + (p n + sigma.n)/2; energy (E + p) u_n + (sigma.n).u + q.n + qr.n;
// Er u_n + qr.n, p = rho Tt.
// Stress and heat flux follow Eq. (full_constitutive): the NSF laws of
// Eq. (NSF_constitutive) at the iterate plus the high-order terms frozen at
// each face, HoT = (K_i + K_j)/2 - NSF_face(W^{n+1/2}).  In these units
// sigma_NSF = -(Tt^omega/delta)(grad u + grad u^T - (2/3) div u I),
// q_NSF = -(k_t Tt^omega/delta) grad Tt, qr_NSF = -(k_r Tt^omega/delta) grad Tr,
// [k_t; k_r] = A^{-1}[5; dr]/4 (Eq. mu_kappa), k_t = 15/8 for Pr = 2/3.
// Face gradients: normal difference, tangential = mean of the cells' central
// (one-sided at non-fluid neighbours) gradients.  Convective flux: Rusanov.
// Boundary faces: F_kin + F_eq(W^m) - F_eq(W^{n+1/2}) -- the kinetic flux of
// f^{n+1/2} keeps its non-equilibrium part while the equilibrium part
// follows the iterate -- or, with the Grad-13 wall flux, the same with the
// flux of the Grad-13 distributions of Eq. (G13_VDF) in place of F_eq, built
// from the iterate and the stress and heat fluxes of Eq. (full_constitutive)
// at the cell (NSF from its central gradients plus HoT_c, the kinetic values
// of f^{n+1/2} minus the NSF values at W^{n+1/2}).  Pseudo time: the diagonal of Eq. (res_macro),
// D_i = 1/dtau_i + (1/2) sum_faces Gamma / h, Gamma = s + C_d Tt^omega/(delta rho h),
// with one global step D* = max_i D_i per iteration so the update is exactly
// conservative, and the rotational relaxation 1/(Z tau) on the Er row.
#include "gsis_common.h"
#include "gsis_launch.h"

#include <algorithm>

namespace gsis {

// prims per cell: rho, ux, uy, uz, Tt, Tr, E, Er, c_s, Tt^omega / delta, 1/tau, (unused)
constexpr int NP = 12;

// The per-cell (per-face) arrays of the macroscopic solve are structures of
// arrays: field k of item i at buf[k * n + i], so the lanes of a wave, which
// take consecutive cells, read consecutive words.  Soa is one item's view.
// Every buffer is read and written through global-address-space pointers
// (gptr), so the loads and stores are global rather than flat instructions.
template <typename T> struct Soa {
    gptr<T> p;
    size_t n;
    __device__ __forceinline__ GSIS_GLOBAL_AS T &operator[](int k) const { return p[(size_t)k * n]; }
};
template <typename T> __device__ __forceinline__ Soa<T> soa(T *buf, size_t n, int i) { return Soa<T>{(gptr<T>)buf + i, n}; }
template <typename T> __device__ __forceinline__ Soa<T> soa(gptr<T> buf, size_t n, int i) { return Soa<T>{buf + i, n}; }
template <typename T> __device__ __forceinline__ gptr<T> G(T *p) { return (gptr<T>)p; }

template <class PV>
__device__ __forceinline__ void prim_from_W(const Geo &g, const double *W, PV P)
{
    double rho = W[0], irho = 1.0 / rho;
    double u0 = W[1] * irho, u1 = W[2] * irho, u2 = W[3] * irho;
    double E = W[4];
    double Er = g.species == 1 ? W[5] : 0.0;
    double uu = u0 * u0 + u1 * u1 + u2 * u2;
    double Tt = (2.0 / 3.0) * (E - Er - rho * uu) * irho;
    double Tr = g.species == 1 ? 2.0 * Er / (g.dr * rho) : Tt;
    P[0] = rho; P[1] = u0; P[2] = u1; P[3] = u2; P[4] = Tt; P[5] = Tr; P[6] = E; P[7] = Er;
    P[8] = sqrt(g.gam * Tt / 2.0);
    const double tw = pow_pos(Tt, g.omega);
    P[9] = tw / g.delta;
    P[10] = g.delta * rho * Tt / tw;
    P[11] = 0.0;
}

template <class PV, class GV>
__device__ __forceinline__ void nsf_face(const Geo &g, const PV &L, const PV &R, const GV &gL, const GV &gR, int a,
                                         double ih, double mu, double sigN[3], double *qN, double *qrN)
{
    double G[9];
    for (int b = 0; b < 3; ++b)
        for (int c = 0; c < 3; ++c)
            G[b * 3 + c] = (c == a) ? (R[1 + b] - L[1 + b]) * ih : 0.5 * (gL[b * 3 + c] + gR[b * 3 + c]);
    double div = G[0] + G[4] + G[8];
    for (int b = 0; b < 3; ++b)
        sigN[b] = -mu * (G[b * 3 + a] + G[a * 3 + b] - (b == a ? (2.0 / 3.0) * div : 0.0));
    *qN = -g.kt * mu * (R[4] - L[4]) * ih;
    *qrN = g.species == 1 ? -g.kr * mu * (R[5] - L[5]) * ih : 0.0;
}

// convective flux vector Phi(W).n and the state vector of one side
template <class PV>
__device__ __forceinline__ void side(const PV &P, int a, double Phi[6], double Wv[6])
{
    double rho = P[0], un = P[1 + a], p = P[0] * P[4];
    Phi[0] = rho * un;
#pragma unroll
    for (int b = 0; b < 3; ++b) Phi[1 + b] = rho * P[1 + b] * un + (b == a ? 0.5 * p : 0.0);
    Phi[4] = (P[6] + p) * un;
    Phi[5] = P[7] * un;
    Wv[0] = rho;
#pragma unroll
    for (int b = 0; b < 3; ++b) Wv[1 + b] = rho * P[1 + b];
    Wv[4] = P[6];
    Wv[5] = P[7];
}

// Macroscopic flux (Rusanov + NSF, no high-order terms) across the face from
// L to R = L + e_a.
template <class PV, class GV>
__device__ __forceinline__ void face_flux(const Geo &g, const PV &L, const PV &R, const GV &gL, const GV &gR, int a,
                                          double ih, bool euler, double F[6], double *Gam)
{
    const double TF = 0.5 * (L[4] + R[4]), rF = 0.5 * (L[0] + R[0]);
    // Euler constitutive relations: no stress or heat flux, no diffusive part in Gamma
    const double mu = euler ? 0.0 : pow_pos(TF, g.omega) / g.delta;
    double sigN[3] = {0.0, 0.0, 0.0}, qN = 0.0, qrN = 0.0;
    if (!euler) nsf_face(g, L, R, gL, gR, a, ih, mu, sigN, &qN, &qrN);
    double PhiL[6], WL[6], PhiR[6], WR[6];
    side(L, a, PhiL, WL);
    side(R, a, PhiR, WR);
    double sL = fabs(L[1 + a]) + L[8], sR = fabs(R[1 + a]) + R[8];
    double smax = sL > sR ? sL : sR;
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] = 0.5 * (PhiL[k] + PhiR[k]) - 0.5 * smax * (WR[k] - WL[k]);
    double uF[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) uF[b] = 0.5 * (L[1 + b] + R[1 + b]);
    const double qrn = g.species == 1 ? qrN : 0.0;
#pragma unroll
    for (int b = 0; b < 3; ++b) F[1 + b] += 0.5 * sigN[b];
    F[4] += sigN[0] * uF[0] + sigN[1] * uF[1] + sigN[2] * uF[2] + qN + qrn;
    F[5] += qrn;
    *Gam = euler ? smax : smax + g.Cd * mu * ih / rF;
}

// Outgoing half-range psi-moments of M(rho, u, Tt) through face dir (sum over
// nodes with xi.n > 0 of w (xi.n) psi M), separable on the tensor grid and
// summed node by node on a node list, and the face flux of the equilibrium
// state with the face's boundary rule.  A group of GW adjacent lanes evaluates
// one face: the lanes share the nodes (of each axis) and a butterfly inside
// the group combines them, so every lane of the group ends with the result.
constexpr int FG = 8;    // lanes per face of the set-up kernel (k_mac_fbfix)

// gradient blocks of k_mac_grad: one (cell, axis) per thread, 256 threads,
// axis-major (a block holds one axis of 256 cells), so a wave's neighbour
// reads are coalesced and its work is uniform
__host__ __device__ inline int grad_axis_blocks(const Geo &g) { return (g.ncell + 255) / 256; }
__host__ __device__ inline int grad_blocks(const Geo &g) { return 3 * grad_axis_blocks(g); }
__host__ __device__ inline int face_blocks(const Geo &g) { return (g.nface * FG + 255) / 256; }

// v of the lane that the row permutation CTRL names (data-parallel primitive:
// no trip through LDS as a general shuffle takes)
template <int CTRL> __device__ __forceinline__ double row_perm(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Sum over a group of GW (8, 16 or 64) lanes, the same bits in every lane:
// quad swaps, then the mirrored half row and row (whose other half holds equal
// values in all its lanes).
template <int GW>
__device__ __forceinline__ double group_sum(double v)
{
    static_assert(GW == 8 || GW == 16 || GW == 64, "8, 16 or 64 lanes");
    v += row_perm<0xB1>(v);    // lane ^ 1
    v += row_perm<0x4E>(v);    // lane ^ 2
    v += row_perm<0x141>(v);   // half-row mirror
    if (GW > 8) v += row_perm<0x140>(v);   // row mirror
    if (GW > 16) {
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
    }
    return v;
}

// LIST: the velocity set is a node list.
template <int GW, bool LIST, class PV>
__device__ __forceinline__ void group_equilibrium_flux(const Geo &g, const BcInfo &bc, const Dev &d, const PV &P, int dir, int b,
                                       int sub, double F[6])
{
    const int a = dir / 2;
    const double sg = (dir & 1) ? 1.0 : -1.0;
    const double T = P[4], iT = 1.0 / T;
    const double piT = PI * T;
    const double K = P[0] / (piT * sqrt(piT)) * sg;
    const double h1 = g.species == 1 ? 0.5 * g.dr * P[5] : 0.0;
    const gptr<const double> in = G((const double *)d.inpsi) + (b * 6 + dir) * 6;
    double out[6];
    if constexpr (LIST) {
        // the half-range sums over the outgoing nodes directly
        double s0 = 0.0, s1[3] = {0.0, 0.0, 0.0}, s4 = 0.0;
        const gptr<const double> nt = G((const double *)d.nt64);
        for (int k = sub; k < g.nv; k += GW) {
            const double x = nt[4 * (size_t)k + a];
            if (!(sg * x > 0.0)) continue;
            const double v0 = nt[4 * (size_t)k], v1 = nt[4 * (size_t)k + 1], v2 = nt[4 * (size_t)k + 2];
            const double cx = v0 - P[1], cy = v1 - P[2], cz = v2 - P[3];
            const double ex = nt[4 * (size_t)k + 3] * exp_core(fmax(-(cx * cx + cy * cy + cz * cz) * iT, -745.0)) * x;
            s0 += ex;
            s1[0] += ex * v0;
            s1[1] += ex * v1;
            s1[2] += ex * v2;
            s4 += ex * (v0 * v0 + v1 * v1 + v2 * v2);
        }
        s0 = group_sum<GW>(s0);
#pragma unroll
        for (int q = 0; q < 3; ++q) s1[q] = group_sum<GW>(s1[q]);
        s4 = group_sum<GW>(s4);
        out[0] = K * s0;
#pragma unroll
        for (int q = 0; q < 3; ++q) out[1 + q] = K * s1[q];
        out[4] = K * s4 + h1 * out[0];
        out[5] = h1 * out[0];
        const double sc = bc.kind[b] == 1 ? bc.rho[b] : out[0] / (-in[0]);
#pragma unroll
        for (int k = 0; k < 6; ++k) F[k] = out[k] + sc * in[k];
        return;
    }
    const int b1 = (a + 1) % 3, b2 = (a + 2) % 3;
    double H1 = 0, H2 = 0, H3 = 0;
    for (int k = sub; k < g.n1[a]; k += GW) {
        const double x = G(d.xi64[a])[k];
        if (!(sg * x > 0.0)) continue;
        const double c = x - P[1 + a];
        const double e = G(d.w64[a])[k] * exp_core(fmax(-c * c * iT, -745.0));
        H1 += e * x;
        H2 += e * x * x;
        H3 += e * x * x * x;
    }
    double S[2][3] = {{0, 0, 0}, {0, 0, 0}};
    const int ax2[2] = {b1, b2};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int ax = ax2[q];
        for (int k = sub; k < g.n1[ax]; k += GW) {
            const double x = G(d.xi64[ax])[k], c = x - P[1 + ax];
            const double e = G(d.w64[ax])[k] * exp_core(fmax(-c * c * iT, -745.0));
            S[q][0] += e;
            S[q][1] += e * x;
            S[q][2] += e * x * x;
        }
    }
    H1 = group_sum<GW>(H1);
    H2 = group_sum<GW>(H2);
    H3 = group_sum<GW>(H3);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int p = 0; p < 3; ++p) S[q][p] = group_sum<GW>(S[q][p]);
    out[0] = K * H1 * S[0][0] * S[1][0];
    out[1 + a] = K * H2 * S[0][0] * S[1][0];
    out[1 + b1] = K * H1 * S[0][1] * S[1][0];
    out[1 + b2] = K * H1 * S[0][0] * S[1][1];
    out[4] = K * (H3 * S[0][0] * S[1][0] + H1 * S[0][2] * S[1][0] + H1 * S[0][0] * S[1][2]) + h1 * out[0];
    out[5] = h1 * out[0];
    const double sc = bc.kind[b] == 1 ? bc.rho[b] : out[0] / (-in[0]);
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] = out[k] + sc * in[k];
}

// Stress and heat fluxes of Eq. (NSF_constitutive) at a cell from its central
// gradients (one-sided next to a non-fluid neighbour, zero with none):
// dv[a] = (v(+a) - v(-a)) of v = (ux, uy, uz, Tt, Tr) along axis a, the cell's
// own value standing in for a side that is not a fluid cell, hm / hp whether
// the sides are; mu = Tt^omega / delta of the cell.  sq = (sigma xx yy zz xy
// xz yz, q, qr).
__device__ __forceinline__ void cell_nsf(const Geo &g, const double dv[3][5], const bool hm[3], const bool hp[3],
                                         double mu, double sq[12])
{
    double Gu[9], gt[3], gr[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double iden = (hm[a] && hp[a]) ? 0.5 * g.invh[a] : g.invh[a];
        const bool none = !hm[a] && !hp[a];
#pragma unroll
        for (int b = 0; b < 3; ++b) Gu[b * 3 + a] = none ? 0.0 : dv[a][b] * iden;
        gt[a] = none ? 0.0 : dv[a][3] * iden;
        gr[a] = none ? 0.0 : dv[a][4] * iden;
    }
    const double div = Gu[0] + Gu[4] + Gu[8];
    sq[0] = -mu * (2.0 * Gu[0] - (2.0 / 3.0) * div);
    sq[1] = -mu * (2.0 * Gu[4] - (2.0 / 3.0) * div);
    sq[2] = -mu * (2.0 * Gu[8] - (2.0 / 3.0) * div);
    sq[3] = -mu * (Gu[1] + Gu[3]);
    sq[4] = -mu * (Gu[2] + Gu[6]);
    sq[5] = -mu * (Gu[5] + Gu[7]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        sq[6 + a] = -g.kt * mu * gt[a];
        sq[9 + a] = g.species == 1 ? -g.kr * mu * gr[a] : 0.0;
    }
}

// The same for a group of at least 8 lanes on one cell: lane sub of the group
// holds v of the cell's neighbour across direction sub (0..5; the cell's own
// state, with has = false, where that is not a fluid cell), the other lanes
// the cell's own; the result is the same in every lane of the group.
template <int GW>
__device__ __forceinline__ void group_cell_nsf(const Geo &g, const double v[5], bool has, double mu, double sq[12])
{
    const int base = (int)(threadIdx.x & 63) & ~(GW - 1);
    double dv[3][5];
    bool hm[3], hp[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        hm[a] = __shfl((int)has, base + 2 * a, 64) != 0;
        hp[a] = __shfl((int)has, base + 2 * a + 1, 64) != 0;
#pragma unroll
        for (int k = 0; k < 5; ++k) dv[a][k] = __shfl(v[k], base + 2 * a + 1, 64) - __shfl(v[k], base + 2 * a, 64);
    }
    cell_nsf(g, dv, hm, hp, mu, sq);
}

// sum over the outgoing half of w xi_n c^e B(c) M(c) / (rho (pi T)^{-3/2}) on
// the tensor grid, c in the face's axes (normal, t1, t2), B the Grad-13
// bracket 1 + cs sigma:cc + cq (q.c)(c5 |c|^2 - 1): products of the 1-D sums
// N[i] = sum_{out} w e xi_n c_n^i and S1[j], S2[k] = sum w e c_t^j over the
// tangential axes (e the 1-D Gaussian factor), each given from its power in
// c^e on.  sl = sigma nn, 11, 22, n1, n2, 12.
template <class SV>
__device__ __forceinline__ double g13_bsum(const SV &N, const SV &S1, const SV &S2, const double sl[6],
                                           const double ql[3], double cs, double cq, double c5)
{
#define GSIS_A3(i, j, k) (N[i] * S1[j] * S2[k])
    double r = GSIS_A3(0, 0, 0);
    r += cs * (sl[0] * GSIS_A3(2, 0, 0) + sl[1] * GSIS_A3(0, 2, 0) + sl[2] * GSIS_A3(0, 0, 2)
               + 2.0 * (sl[3] * GSIS_A3(1, 1, 0) + sl[4] * GSIS_A3(1, 0, 1) + sl[5] * GSIS_A3(0, 1, 1)));
    const double t = ql[0] * (c5 * (GSIS_A3(3, 0, 0) + GSIS_A3(1, 2, 0) + GSIS_A3(1, 0, 2)) - GSIS_A3(1, 0, 0))
                   + ql[1] * (c5 * (GSIS_A3(2, 1, 0) + GSIS_A3(0, 3, 0) + GSIS_A3(0, 1, 2)) - GSIS_A3(0, 1, 0))
                   + ql[2] * (c5 * (GSIS_A3(2, 0, 1) + GSIS_A3(0, 2, 1) + GSIS_A3(0, 0, 3)) - GSIS_A3(0, 0, 1));
#undef GSIS_A3
    return r + cq * t;
}

// The Grad-13 half-range sums of group_g13_flux on the tensor grid for a face
// normal to axis A (a compile-time constant, so that every stress and heat-flux
// component is picked by a constant index): out[6] before the boundary rule.
template <int GW, int A>
__device__ __forceinline__ void g13_tensor_flux(const Geo &g, const Dev &d, const double u[3], const double sq[12],
                                                double sg, double iT, double K, double cs, double cq, double c5,
                                                double cr, double h1, bool dia, int sub, double out[6])
{
    constexpr int T1 = (A + 1) % 3, T2 = (A + 2) % 3;
    constexpr int ax[3] = {A, T1, T2};
    // sq slot of sigma_{pq}, p != q: xy 3, xz 4, yz 5
    auto sslot = [](int x, int y) constexpr { return 2 + x + y; };
    double N[6] = {0, 0, 0, 0, 0, 0}, S1[6] = {0, 0, 0, 0, 0, 0}, S2[6] = {0, 0, 0, 0, 0, 0};
    for (int k = sub; k < g.n1[A]; k += GW) {
        const double x = G(d.xi64[A])[k];
        if (!(sg * x > 0.0)) continue;
        const double c = x - u[A];
        double e = G(d.w64[A])[k] * exp_core(fmax(-c * c * iT, -745.0)) * x;
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            N[p] += e;
            e *= c;
        }
    }
    for (int k = sub; k < g.n1[T1]; k += GW) {
        const double c = G(d.xi64[T1])[k] - u[T1];
        double e = G(d.w64[T1])[k] * exp_core(fmax(-c * c * iT, -745.0));
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            S1[p] += e;
            e *= c;
        }
    }
    for (int k = sub; k < g.n1[T2]; k += GW) {
        const double c = G(d.xi64[T2])[k] - u[T2];
        double e = G(d.w64[T2])[k] * exp_core(fmax(-c * c * iT, -745.0));
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            S2[p] += e;
            e *= c;
        }
    }
#pragma unroll
    for (int p = 0; p < 6; ++p) {
        N[p] = group_sum<GW>(N[p]);
        S1[p] = group_sum<GW>(S1[p]);
        S2[p] = group_sum<GW>(S2[p]);
    }
    const double sl[6] = {sq[ax[0]], sq[ax[1]], sq[ax[2]], sq[sslot(A, T1)], sq[sslot(A, T2)], sq[sslot(T1, T2)]};
    double ql[3], rl[3], ul[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        ql[p] = sq[6 + ax[p]];
        rl[p] = sq[9 + ax[p]];
        ul[p] = u[ax[p]];
    }
    const double b0 = g13_bsum((const double *)N, (const double *)S1, (const double *)S2, sl, ql, cs, cq, c5);
    const double bn = g13_bsum((const double *)N + 1, (const double *)S1, (const double *)S2, sl, ql, cs, cq, c5);
    const double b1 = g13_bsum((const double *)N, (const double *)S1 + 1, (const double *)S2, sl, ql, cs, cq, c5);
    const double b2 = g13_bsum((const double *)N, (const double *)S1, (const double *)S2 + 1, sl, ql, cs, cq, c5);
    const double bnn = g13_bsum((const double *)N + 2, (const double *)S1, (const double *)S2, sl, ql, cs, cq, c5);
    const double b11 = g13_bsum((const double *)N, (const double *)S1 + 2, (const double *)S2, sl, ql, cs, cq, c5);
    const double b22 = g13_bsum((const double *)N, (const double *)S1, (const double *)S2 + 2, sl, ql, cs, cq, c5);
    out[0] = K * b0;
    out[1 + A] = K * (bn + ul[0] * b0);
    out[1 + T1] = K * (b1 + ul[1] * b0);
    out[1 + T2] = K * (b2 + ul[2] * b0);
    const double uu = ul[0] * ul[0] + ul[1] * ul[1] + ul[2] * ul[2];
    const double e0 = bnn + b11 + b22 + 2.0 * (ul[0] * bn + ul[1] * b1 + ul[2] * b2) + uu * b0;
    const double sr = rl[0] * N[1] * S1[0] * S2[0] + rl[1] * N[0] * S1[1] * S2[0] + rl[2] * N[0] * S1[0] * S2[1];
    const double f1 = dia ? K * (h1 * b0 + cr * sr) : 0.0;
    out[4] = K * e0 + f1;
    out[5] = f1;
}

// The flux of boundary face dir when the cell holds the Grad-13 distributions
// of Eq. (G13_VDF) of its state P and sq = (sigma, q, qr) (Eq. GSIS-DVM-flux),
// with the face's boundary rule (a wall's density from zero net mass flux):
//   f0 = M [1 + sigma:cc / (rho Tt^2) + 2 (q.c) / (rho Tt^2) (2 |c|^2 / (5 Tt) - 1)],
//   f1 = (dr/2) Tr f0 + 2 M (qr.c) / (rho Tt),
// velocities in sqrt(2 R T0) (these forms give back rho, u, Tt, sigma, q, Tr
// and qr as the moments of Eq. getmoment).  A group of GW lanes per face, as
// group_equilibrium_flux.
template <int GW, bool LIST, class PV>
__device__ __forceinline__ void group_g13_flux(const Geo &g, const BcInfo &bc, const Dev &d, const PV &P, const double sq[12], int dir,
                               int b, int sub, double F[6])
{
    const int a = dir / 2;
    const double sg = (dir & 1) ? 1.0 : -1.0;
    const double T = P[4], iT = 1.0 / T;
    const double piT = PI * T;
    const double K = P[0] / (piT * sqrt(piT)) * sg;
    const double u[3] = {P[1], P[2], P[3]};
    const double irT2 = 1.0 / (P[0] * T * T);
    const double cs = irT2, cq = 2.0 * irT2, c5 = 2.0 / (5.0 * T);
    const double cr = 2.0 / (P[0] * T);
    const bool dia = g.species == 1;
    const double h1 = dia ? 0.5 * g.dr * P[5] : 0.0;
    const gptr<const double> in = G((const double *)d.inpsi) + (b * 6 + dir) * 6;
    double out[6];
    if constexpr (LIST) {
        double s0 = 0.0, s1[3] = {0.0, 0.0, 0.0}, s4 = 0.0, sr = 0.0;
        const gptr<const double> nt = G((const double *)d.nt64);
        for (int k = sub; k < g.nv; k += GW) {
            const double x = nt[4 * (size_t)k + a];
            if (!(sg * x > 0.0)) continue;
            const double v0 = nt[4 * (size_t)k], v1 = nt[4 * (size_t)k + 1], v2 = nt[4 * (size_t)k + 2];
            const double cx = v0 - u[0], cy = v1 - u[1], cz = v2 - u[2];
            const double cc = cx * cx + cy * cy + cz * cz;
            const double e = nt[4 * (size_t)k + 3] * exp_core(fmax(-cc * iT, -745.0)) * x;
            const double scc = sq[0] * cx * cx + sq[1] * cy * cy + sq[2] * cz * cz
                             + 2.0 * (sq[3] * cx * cy + sq[4] * cx * cz + sq[5] * cy * cz);
            const double qc = sq[6] * cx + sq[7] * cy + sq[8] * cz;
            const double eb = e * (1.0 + cs * scc + cq * qc * (c5 * cc - 1.0));
            s0 += eb;
            s1[0] += eb * v0;
            s1[1] += eb * v1;
            s1[2] += eb * v2;
            s4 += eb * (v0 * v0 + v1 * v1 + v2 * v2);
            if (dia) sr += e * (sq[9] * cx + sq[10] * cy + sq[11] * cz);
        }
        s0 = group_sum<GW>(s0);
#pragma unroll
        for (int q = 0; q < 3; ++q) s1[q] = group_sum<GW>(s1[q]);
        s4 = group_sum<GW>(s4);
        sr = group_sum<GW>(sr);
        out[0] = K * s0;
#pragma unroll
        for (int q = 0; q < 3; ++q) out[1 + q] = K * s1[q];
        const double f1 = dia ? K * (h1 * s0 + cr * sr) : 0.0;
        out[4] = K * s4 + f1;
        out[5] = f1;
    } else {
        if (a == 0) g13_tensor_flux<GW, 0>(g, d, u, sq, sg, iT, K, cs, cq, c5, cr, h1, dia, sub, out);
        else if (a == 1) g13_tensor_flux<GW, 1>(g, d, u, sq, sg, iT, K, cs, cq, c5, cr, h1, dia, sub, out);
        else g13_tensor_flux<GW, 2>(g, d, u, sq, sg, iT, K, cs, cq, c5, cr, h1, dia, sub, out);
    }
    const double sc = bc.kind[b] == 1 ? bc.rho[b] : out[0] / (-in[0]);
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] = out[k] + sc * in[k];
}

// The box's solve keeps a cell's W (5, diatomic 6) and its residual R side by
// side, and for the diatomic gas the rotational relaxation rate of that state
// and a pad: a row of a tile's cells is then one stretch of memory, whose
// lines are used whole (as [field][cell] every line gave 48 of its 128 bytes,
// and filling them bound the loads).
constexpr int WS_MONO = 10, WS_DIA = 14, WSRC = 12;
typedef double f64x2 __attribute__((ext_vector_type(2)));

// W^{n+1/2} and the old half of the correction record.
__global__ __launch_bounds__(128) void k_mac_init(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    const gptr<const double> m = G((const double *)d.cm) + (size_t)cell * NMOM;
    double rho = m[0], Tt = m[4];
    double uu = m[1] * m[1] + m[2] * m[2] + m[3] * m[3];
    double Er = g.species == 1 ? 0.5 * g.dr * rho * m[14] : 0.0;
    const size_t n = g.ncell;
    double W[6];
    W[0] = rho;
    W[1] = rho * m[1]; W[2] = rho * m[2]; W[3] = rho * m[3];
    W[4] = rho * uu + 1.5 * rho * Tt + Er;
    W[5] = Er;
    if (g.umesh) {
        const Soa<double> Wd = soa(d.W, n, cell);
        for (int k = 0; k < 6; ++k) Wd[k] = W[k];
    } else {
        const bool dia = g.species == 1;
        const gptr<double> Wd = G(d.W) + (size_t)cell * (dia ? WS_DIA : WS_MONO);
        for (int k = 0; k < (dia ? 6 : 5); ++k) Wd[k] = W[k];
    }
    const gptr<double> c = G(d.corr) + (size_t)cell * NCORR;
    c[6] = rho; c[7] = m[1]; c[8] = m[2]; c[9] = m[3]; c[10] = Tt;
    c[11] = g.species == 1 ? m[14] : Tt;
    prim_from_W(g, W, soa(d.P, n, cell));
}

// Central gradients of u at W^{n+1/2}, one (cell, axis) per thread: one-sided
// next to a non-fluid neighbour, zero with none.
__global__ __launch_bounds__(256) void k_mac_grad(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int npa = grad_axis_blocks(g), a = blk / npa;
    const int cell = (blk - a * npa) * (int)blockDim.x + (int)threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    const int nm = G(d.nbr)[(size_t)(2 * a) * g.ncell + cell], np = G(d.nbr)[(size_t)(2 * a + 1) * g.ncell + cell];
    const size_t n = g.ncell;
    const Soa<double> Pm = soa(d.P, n, nm >= 0 ? nm : cell);
    const Soa<double> Pp = soa(d.P, n, np >= 0 ? np : cell);
    const double iden = (nm >= 0 && np >= 0) ? 0.5 * g.invh[a] : g.invh[a];
    const Soa<double> Gd = soa(d.grad, n, cell);
#pragma unroll
    for (int b = 0; b < 3; ++b) Gd[b * 3 + a] = (nm < 0 && np < 0) ? 0.0 : (Pp[1 + b] - Pm[1 + b]) * iden;
}

// High-order terms at the faces (cell, cell + e_a), frozen at the kinetic
// state: the kinetic scheme's face flux of the moments of f^{n+1/2} (first-order
// upwind: the xi_a > 0 octant sums of the cell plus the xi_a < 0 octant sums of
// the neighbour) minus the macroscopic face flux at W^{n+1/2}, six values per
// face; the face flux of an iterate is its macroscopic flux plus these.  Zero
// for the Euler relations.
__global__ __launch_bounds__(128) void k_mac_hot(GSIS_SPAN_ARGS, int euler)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    const size_t n = g.ncell;
    const int m2row[3][3] = {{4, 7, 8}, {7, 5, 9}, {8, 9, 6}};
    for (int a = 0; a < 3; ++a) {
        const gptr<double> fx = G(d.hot) + ((size_t)a * n + cell) * 6;
        const int nb = G(d.nbr)[(size_t)(2 * a + 1) * g.ncell + cell];
        if (euler || nb < 0) {
            for (int k = 0; k < 6; ++k) fx[k] = 0.0;
            continue;
        }
        double Fk[6] = {0, 0, 0, 0, 0, 0};
        for (int o = 0; o < 8; ++o) {
            const int up = ((o >> a) & 1) ? nb : cell;   // xi_a < 0: the neighbour's value enters the face
            const gptr<const double> m = G((const double *)d.mom8) + ((size_t)up * 8 + o) * NRS;
            Fk[0] += m[1 + a];
            for (int b = 0; b < 3; ++b) Fk[1 + b] += m[m2row[a][b]];
            Fk[4] += m[10 + a] + m[14 + a];
            Fk[5] += m[14 + a];
        }
        const Soa<double> PL = soa(d.P, n, cell), PR = soa(d.P, n, nb);
        double F[6], Gam;
        face_flux(g, PL, PR, soa(d.grad, n, cell), soa(d.grad, n, nb), a, g.invh[a], false, F, &Gam);
        for (int k = 0; k < 6; ++k) fx[k] = Fk[k] - F[k];
        if (g.species != 1) fx[5] = 0.0;
    }
}

// Fixed part of each boundary face flux, F_kin(f^{n+1/2}) - F_eq(W^{n+1/2}).
// One group of FG lanes per face.
// G13: compiled with the Grad-13 wall flux for the cases that take it (the
// plain instantiation keeps its registers for the common path).
template <bool G13>
__global__ __launch_bounds__(256) void k_mac_fbfix(GSIS_SPAN_ARGS, int euler)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const BcInfo &bc = C.bc;
    const int f = (int)(blk * blockDim.x + threadIdx.x) / FG;
    const int sub = threadIdx.x & (FG - 1);
    if (f >= g.nface) return;
    const int cell = G(d.face_cell)[f], dir = G(d.face_dir)[f], b = G(d.face_bc)[f];
    const int a = dir / 2;
    const int neg = (dir & 1) ? 0 : 1;
    const double sg = neg ? -1.0 : 1.0;
    double out[6] = {0, 0, 0, 0, 0, 0};
    const int m2row[3][3] = {{4, 7, 8}, {7, 5, 9}, {8, 9, 6}};
    for (int o = 0; o < 8; ++o) {
        if (((o >> a) & 1) != neg) continue;
        const gptr<const double> m = G((const double *)d.mom8) + ((size_t)cell * 8 + o) * NRS;
        out[0] += m[1 + a];
        for (int c = 0; c < 3; ++c) out[1 + c] += m[m2row[a][c]];
        out[4] += m[10 + a] + m[14 + a];
        out[5] += m[14 + a];
    }
    for (int k = 0; k < 6; ++k) out[k] *= sg;
    const gptr<const double> in = G((const double *)d.inpsi) + (b * 6 + dir) * 6;
    const double sc = bc.kind[b] == 1 ? bc.rho[b] : out[0] / (-in[0]);
    const Soa<double> P = soa(d.P, g.ncell, cell);
    double Fe[6];
    if (G13 && g.wall_flux == 1 && !euler) {
        // Grad-13 wall flux: the cell's high-order terms, HoT_c = kinetic stress
        // and heat fluxes of f^{n+1/2} - NSF_c(W^{n+1/2}), kept per face, and the
        // flux of the distributions of NSF_c + HoT_c
        int who = cell;
        bool has = false;
        if (sub < 6) {
            const int nb = G(d.nbr)[(size_t)sub * g.ncell + cell];
            if (nb >= 0) { who = nb; has = true; }
        }
        const Soa<double> Pw = soa(d.P, g.ncell, who);
        const double v[5] = {Pw[1], Pw[2], Pw[3], Pw[4], Pw[5]};
        double sq[12];
        group_cell_nsf<FG>(g, v, has, P[9], sq);
        const gptr<const double> m = G((const double *)d.cm) + (size_t)cell * NMOM;
        const bool dia = g.species == 1;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            // cm: sigma at 5..10, q at 11..13, qr at 15..17
            const double kin = k < 9 ? m[5 + k] : (dia ? m[6 + k] : 0.0);
            const double hot = kin - sq[k];
            if ((k & (FG - 1)) == sub) G(d.ghot)[(size_t)k * g.nface + f] = hot;
            sq[k] += hot;
        }
        if (g.vlist) group_g13_flux<FG, true>(g, bc, d, P, sq, dir, b, sub, Fe);
        else group_g13_flux<FG, false>(g, bc, d, P, sq, dir, b, sub, Fe);
    } else if (g.vlist) {
        group_equilibrium_flux<FG, true>(g, bc, d, P, dir, b, sub, Fe);
    } else {
        group_equilibrium_flux<FG, false>(g, bc, d, P, dir, b, sub, Fe);
    }
    if (sub < 6) {
        // Euler: the boundary flux is the iterate's own F_eq, no fixed kinetic part
        G(d.fbfix)[(size_t)sub * g.nface + f] = euler ? 0.0 : out[sub] + sc * in[sub] - Fe[sub];
    }
}

// What the residual of a cell keeps through the whole solve: minus the sum
// over its faces, outward, of the high-order terms of the interior ones and
// the fixed parts of the boundary ones, over h.  Six values per cell instead
// of six per face in every iteration.
__global__ __launch_bounds__(128) void k_mac_const(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    const size_t n = g.ncell;
    double s[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int dir = 0; dir < 6; ++dir) {
        const int a = dir >> 1, nb = G(d.nbr)[(size_t)dir * n + cell];
        const double ih = g.invh[a];
        if (nb < 0) {
            for (int k = 0; k < 6; ++k) s[k] -= G(d.fbfix)[(size_t)k * g.nface - nb - 1] * ih;
        } else {
            const gptr<const double> h = G((const double *)d.hot) + ((size_t)a * n + ((dir & 1) ? cell : nb)) * 6;
            for (int k = 0; k < 6; ++k) s[k] -= ((dir & 1) ? h[k] : -h[k]) * ih;
        }
    }
    for (int k = 0; k < 6; ++k) G(d.Rc)[(size_t)cell * 6 + k] = s[k];
}

// ------------------------------------------------------- one inner iteration
// One launch per inner iteration.  A block owns a 4 x 4 x 4 tile of cells:
//   1. its threads step the tile's cells and their halo to the new state,
//      W' = W + R / D* (D* the largest diagonal of the launch before), and
//      stage the prims in LDS (the tile writes its own W');
//   2. one thread per face of the tile (240) forms the face flux with the
//      gradients taken from the staged velocities; boundary faces go into a
//      list, whose 1-D half-range sums are shared out over the block (four
//      lanes per face and axis) and finished by one thread (four with the
//      Grad-13 wall flux) per face;
//   3. a thread per cell and pair of components adds the six face terms into
//      the residual R of the new state, and D goes into the partial maxima.
// The halo is one cell wide without its corners: a face needs its two cells
// and, for the tangential gradients, their neighbours across the other axes.
// It is stepped again by every tile that sees it (208 cells for 64), which
// costs less than the launch and the round trip through memory that writing
// the prims first would take; every face is formed once per tile (3.75 per
// cell) instead of once from each side, and what the high-order terms and the
// fixed boundary parts add to a cell is summed once per solve (k_mac_const).
// Measured, us per inner iteration, against a residual launch (every face from
// both sides) and an advance launch per iteration: cavity of 48^3 cells 18.9
// (32.6), nitrogen block of 64 x 48 x 48 cells 29.2 (45.7), cavity of 12 x 11
// x 13 cells with the Grad-13 wall flux 11.8 (20.7).  What bounds it now: an
// iteration fetches 16.6 MB and writes 9.0 MB between the XCDs' caches and the
// memory side on 48^3 cells (FETCH_SIZE, WRITE_SIZE; about 5 us of the 18.9 at
// the rate of a large copy), then the latency of the three dependent phases,
// twice over for the tiles that do not fit the chip at once (five blocks of
// 30 KB LDS per CU); the boundary faces' 1-D sums add 3.6 us.
constexpr int MT = 4, MH = MT + 2, MHN = MH * MH * MH;
constexpr int MFN = 3 * (MT + 1) * MT * MT;   // faces of a tile
constexpr int MBC = 48;                       // boundary faces finished together

// Half of an axis in tiles, rounded up.  Blocks go to the 8 XCDs in turn, so
// block b takes a tile of octant b mod 8 of the box: an XCD reads its own
// octant and one layer of cells around it, which fit its L2, where tiles dealt
// out in turn had every XCD fetch nearly every line of every field from the
// memory side (48^3 cells: 35 against 20 us per iteration).  An octant that an
// odd number of tiles leaves smaller has blocks without a tile.
__host__ __device__ inline int mtile_half(int n) { return ((n + MT - 1) / MT + 1) / 2; }
__host__ __device__ inline int mtile_blocks(const Geo &g)
{
    return 8 * mtile_half(g.nx) * mtile_half(g.ny) * mtile_half(g.nz);
}

// D* of the launch that filled partial set `set`: 16 lanes share out the
// partial slots, and every row of 16 lanes does the same
constexpr int BSLOT = 16;
__device__ __forceinline__ double partial_diagonal(const Dev &d, int set)
{
    return __longlong_as_double((long long)G(d.dmax)[(size_t)(set * DSLOT + (threadIdx.x & (BSLOT - 1))) * DSTRIDE]);
}
__device__ __forceinline__ double row_max(double v)
{
    v = fmax(v, row_perm<0xB1>(v));
    v = fmax(v, row_perm<0x4E>(v));
    v = fmax(v, row_perm<0x141>(v));
    return fmax(v, row_perm<0x140>(v));
}
__device__ __forceinline__ double largest_diagonal(const Dev &d, int set) { return row_max(partial_diagonal(d, set)); }

// W of a cell after the pseudo-time step of launch it (none before the first)
// from its record: W + R / D* (as R times 1/D*), the rotational-energy row with
// its relaxation source on the diagonal.
template <bool DIA, class PV>
__device__ __forceinline__ void stepped_W(PV rec, int it, double Dm, double iDm, double Wn[6])
{
    constexpr int NW = DIA ? 6 : 5;
#pragma unroll
    for (int k = 0; k < 6; ++k) Wn[k] = k < NW ? rec[k] : 0.0;
    if (it > 0) {
#pragma unroll
        for (int k = 0; k < 5; ++k) Wn[k] += rec[NW + k] * iDm;
        if (DIA) Wn[5] += quot(rec[NW + 5], Dm + rec[DIA ? WSRC : 0]);
    }
}

// rho, u, Tt, Tr, E, Er, c_s of a state
template <bool DIA>
__device__ __forceinline__ void short_prims(const Geo &g, const double W[6], double P[9])
{
    const double rho = W[0], irho = recip(rho);
    const double u0 = W[1] * irho, u1 = W[2] * irho, u2 = W[3] * irho;
    const double Er = DIA ? W[5] : 0.0;
    const double Tt = (2.0 / 3.0) * (W[4] - Er - rho * (u0 * u0 + u1 * u1 + u2 * u2)) * irho;
    P[0] = rho; P[1] = u0; P[2] = u1; P[3] = u2; P[4] = Tt;
    P[5] = DIA ? 2.0 * Er / (g.dr * rho) : Tt;
    P[6] = W[4];
    P[7] = Er;
    P[8] = sqrt(0.5 * g.gam * Tt);
}

// Node list: the boundary-face fluxes of the state that launch it steps to,
// one wave per face (the sums run over every node, too long for a tile's
// share of lanes); k_mac_iter takes them from Fb and Gb.
template <bool DIA, bool EULER, bool G13>
__global__ __launch_bounds__(256) void k_mac_bface(GSIS_SPAN_ARGS, int it)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const BcInfo &bc = C.bc;
    const int f = __builtin_amdgcn_readfirstlane(blk * 4 + (int)(threadIdx.x >> 6));
    if (f >= g.nface) return;
    const int sub = threadIdx.x & 63;
    const gptr<const double> src = G((const double *)((it & 1) ? d.W2 : d.W));
    double Dm = 1.0;
    if (it > 0) Dm = largest_diagonal(d, (it - 1) % DSETS);
    const double iDm = 1.0 / Dm;
    const int cell = G(d.face_cell)[f], dir = G(d.face_dir)[f], b = G(d.face_bc)[f];
    double Wn[6], P[9], Fe[6];
    constexpr int WS = DIA ? WS_DIA : WS_MONO;
    stepped_W<DIA>(src + (size_t)cell * WS, it, Dm, iDm, Wn);
    short_prims<DIA>(g, Wn, P);
    const double mu = quot(pow_line(P[4], g.omega), g.delta, g.idelta);
    if (G13 && !EULER && g.wall_flux == 1) {
        // NSF_c from the new states of the cell and its neighbours (one per lane) plus the cell's HoT_c
        int who = cell;
        bool has = false;
        if (sub < 6) {
            const int nb = G(d.nbr)[(size_t)sub * g.ncell + cell];
            if (nb >= 0) { who = nb; has = true; }
        }
        double Ww[6], Pw[9], sq[12];
        stepped_W<DIA>(src + (size_t)who * WS, it, Dm, iDm, Ww);
        short_prims<DIA>(g, Ww, Pw);
        const double v[5] = {Pw[1], Pw[2], Pw[3], Pw[4], Pw[5]};
        group_cell_nsf<64>(g, v, has, mu, sq);
#pragma unroll
        for (int k = 0; k < 12; ++k) sq[k] += G(d.ghot)[(size_t)k * g.nface + f];
        group_g13_flux<64, true>(g, bc, d, P, sq, dir, b, sub, Fe);
    } else {
        group_equilibrium_flux<64, true>(g, bc, d, P, dir, b, sub, Fe);
    }
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if (sub == k) G(d.Fb)[(size_t)k * g.nface + f] = Fe[k];
    if (sub == 0)
        G(d.Gb)[f] = fabs(P[1 + dir / 2]) + P[8] + (EULER ? 0.0 : g.Cd * mu / (P[0] * g.h[dir / 2]));
}

// sum over the four lanes of a quad, the same bits in each
__device__ __forceinline__ double quad_sum(double v)
{
    v += row_perm<0xB1>(v);
    return v + row_perm<0x4E>(v);
}

template <bool DIA, bool EULER, bool G13>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_mac_iter(GSIS_SPAN_ARGS, int it)
{
    constexpr int NW = DIA ? 6 : 5;
    constexpr int WS = DIA ? WS_DIA : WS_MONO;
    constexpr int NS = G13 ? 6 : 3;      // 1-D sums of a boundary face per axis
    // staged prims: rho, u, Tt, E, c_s, then Tr, Er
    enum { QR = 0, QU = 1, QT = 4, QE = 5, QC = 6, QTR = DIA ? 7 : 4, QER = DIA ? 8 : 5, NQ = DIA ? 9 : 7 };
    // Records as read (WS words per halo cell), then, in the same space, the
    // prims, the face terms along +axis and Gamma, and the boundary faces' sums
    constexpr int NB = MBC * (3 * NS + (G13 ? 8 : 0));
    constexpr int NLDS = NQ * MHN + (NW + 1) * MFN + NB > WS * MHN ? NQ * MHN + (NW + 1) * MFN + NB : WS * MHN;
    __shared__ __attribute__((aligned(16))) double lds[NLDS];
    double(&sp)[NQ][MHN] = *(double(*)[NQ][MHN])lds;
    double(&sf)[NW + 1][MFN] = *(double(*)[NW + 1][MFN])(lds + NQ * MHN);
    double *const ssum = lds + NQ * MHN + (NW + 1) * MFN, *const sb = ssum + MBC * 3 * NS;
    __shared__ int sflag[MHN];
    __shared__ int2 slist[MFN];          // boundary faces: (face | the cell's halo position << 8 | direction << 16 | slot << 20, index)
    __shared__ int scount;

    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const BcInfo &bc = C.bc;
    const int t = threadIdx.x;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const gptr<const double> src = G((const double *)((it & 1) ? d.W2 : d.W));
    const gptr<double> dst = G((it & 1) ? d.W : d.W2);
    const size_t nc = (size_t)g.ncell;
    // The tile in its octant, counted from the octant's outer corner: the layers
    // on the box's boundary (z, then y, then x) first, as their tiles take longest
    const int mx = mtile_half(nx), my = mtile_half(ny), mz = mtile_half(nz);
    int q = blk >> 3, ox, oy, oz;
    if (q < mx * my) {
        oz = 0; oy = q / mx; ox = q - oy * mx;
    } else if ((q -= mx * my) < mx * (mz - 1)) {
        oy = 0; oz = q / mx; ox = q - oz * mx; ++oz;
    } else if ((q -= mx * (mz - 1)) < (my - 1) * (mz - 1)) {
        ox = 0; oz = q / (my - 1); oy = q - oz * (my - 1) + 1; ++oz;
    } else {
        q -= (my - 1) * (mz - 1);
        const int r = q / (mx - 1);
        ox = q - r * (mx - 1) + 1; oz = r / (my - 1); oy = r - oz * (my - 1) + 1; ++oz;
    }
    // the upper half of an axis counts down from its last tile
    const int ntx = (nx + MT - 1) / MT, nty = (ny + MT - 1) / MT, ntz = (nz + MT - 1) / MT;
    const int tx = blk & 1 ? ntx - 1 - ox : ox, ty = blk & 2 ? nty - 1 - oy : oy, tz = blk & 4 ? ntz - 1 - oz : oz;
    const bool none = (blk & 1 && tx < mx) || (blk & 2 && ty < my) || (blk & 4 && tz < mz);
    const int x0 = tx * MT - 1, y0 = ty * MT - 1, z0 = tz * MT - 1;
    if (blk == 0 && t < BSLOT) G(d.dmax)[(size_t)((it + 1) % DSETS * DSLOT + t) * DSTRIDE] = 0ull;
    if (none) return;   // an octant with fewer tiles; uniform over the block
    if (t == 0) scount = 0;

    // the reads of D* (a partial slot per lane) and of this thread's cell of the halo
    double Dp = 1.0;
    if (it > 0) Dp = partial_diagonal(d, (it - 1) % DSETS);
    const int hx = t % MH, hy = t / MH % MH, hz = t / (MH * MH);
    const bool ex = hx == 0 || hx == MH - 1, ey = hy == 0 || hy == MH - 1, ez = hz == 0 || hz == MH - 1;
    const int hi = x0 + hx, hj = y0 + hy, hk = z0 + hz;
    const int hcell = hi + nx * (hj + ny * hk);
    const bool staged = t < MHN && hi >= 0 && hi < nx && hj >= 0 && hj < ny && hk >= 0 && hk < nz && !(ex && ey && ez);
    const bool solids = g.nfluid != g.ncell;
    const int hfl = staged ? (solids ? G(d.cflag)[hcell] : 1) : 0;
    // the records of the halo box, row after row, 16 bytes a thread and step
    constexpr int VC = WS / 2, VR = MH * VC, VN = MH * MH * VR, NV = (VN + 255) / 256;
    f64x2 rec[NV];
#pragma unroll
    for (int r = 0; r < NV; ++r) {
        const int v = t + 256 * r, row = v / VR, c = v - row * VR;
        const int i = x0 + c / VC, j = y0 + row % MH, k = z0 + row / MH;
        rec[r] = f64x2{0.0, 0.0};
        if (v < VN && i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz)
            rec[r] = ((gptr<const f64x2>)src)[(ptrdiff_t)(x0 + nx * (j + ny * k)) * VC + c];
    }

    // This thread's face: axis a, position fq along it and (fv, fw) along the
    // other axes b1, b2.  Waves 0 to 2 take the faces 0..3 of axes 0 to 2, the
    // last wave face 4 of each axis (48 lanes).
    const bool isface = t < MFN;
    const int fl6 = t & 63;
    const bool wave3 = t >= 192;
    const int a = wave3 ? fl6 >> 4 : t >> 6;
    const int fq = wave3 ? MT : fl6 & 3, fv = wave3 ? fl6 & 3 : (fl6 >> 2) & 3, fw = wave3 ? (fl6 >> 2) & 3 : fl6 >> 4;
    const int Sa = a == 0 ? 1 : (a == 1 ? MH : MH * MH);
    const int S1 = a == 0 ? MH : (a == 1 ? MH * MH : 1), S2 = a == 0 ? MH * MH : (a == 1 ? 1 : MH);
    const int b1 = a == 2 ? 0 : a + 1, b2 = a == 0 ? 2 : a - 1;
    const int hL = fq * Sa + (fv + 1) * S1 + (fw + 1) * S2, hR = hL + Sa;
    int nL = 0, nR = 0, fbc = 0;
    if (isface && (solids || x0 < 0 || y0 < 0 || z0 < 0 || x0 + MT + 2 > nx || y0 + MT + 2 > ny || z0 + MT + 2 > nz)) {
        // the neighbour table of a face that may be a boundary face, read before the prims are there
        const int step = a == 0 ? 1 : (a == 1 ? nx : nx * ny);
        const int s1 = a == 0 ? nx : (a == 1 ? nx * ny : 1), s2 = a == 0 ? nx * ny : (a == 1 ? 1 : nx);
        const int at = (a == 0 ? x0 : (a == 1 ? y0 : z0)) + fq, na = a == 0 ? nx : (a == 1 ? ny : nz);
        const int p1 = (b1 == 0 ? x0 : (b1 == 1 ? y0 : z0)) + 1 + fv, n1 = b1 == 0 ? nx : (b1 == 1 ? ny : nz);
        const int p2 = (b2 == 0 ? x0 : (b2 == 1 ? y0 : z0)) + 1 + fw, n2 = b2 == 0 ? nx : (b2 == 1 ? ny : nz);
        const int cL = at * step + p1 * s1 + p2 * s2;
        if (at < na && p1 < n1 && p2 < n2) {
            if (at >= 0) {
                if (solids || at + 1 == na) nL = G(d.nbr)[(size_t)(2 * a + 1) * nc + cL];
            }
            if ((solids || at < 0) && at + 1 < na) nR = G(d.nbr)[(size_t)(2 * a) * nc + cL + step];
        }
    }
    // the cell and the pair of components this thread adds up at the end, and their constant part
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), c = t & 63;
    const int cx = c & 3, cy = (c >> 2) & 3, cz = c >> 4;
    const int ci = x0 + 1 + cx, cj = y0 + 1 + cy, ck = z0 + 1 + cz, cell = ci + nx * (cj + ny * ck);
    f64x2 rc = {0.0, 0.0};
    if (w < 3 && ci < nx && cj < ny && ck < nz) rc = ((gptr<const f64x2>)d.Rc)[(size_t)cell * 3 + w];

    // 1. the new state of the tile and its halo
#pragma unroll
    for (int r = 0; r < NV; ++r)
        if (t + 256 * r < VN) ((f64x2 *)lds)[t + 256 * r] = rec[r];
    const double Dm = row_max(Dp), iDm = recip(Dm);
    if (t < MHN) sflag[t] = hfl;
    __syncthreads();
    double Wn[6];
    if (staged) stepped_W<DIA>(lds + t * WS, it, Dm, iDm, Wn);
    __syncthreads();
    if (staged) {
        double P[9];
        short_prims<DIA>(g, Wn, P);   // a solid cell's is not used
#pragma unroll
        for (int q = 0; q < 5; ++q) sp[q][t] = P[q];
        sp[QE][t] = P[6];
        sp[QC][t] = P[8];
        if (DIA) {
            sp[QTR][t] = P[5];
            sp[QER][t] = P[7];
        }
        if (hfl && !ex && !ey && !ez) {
            const gptr<double> w = dst + (size_t)hcell * WS;
#pragma unroll
            for (int q = 0; q < NW; ++q) w[q] = Wn[q];
        }
    }
    // A boundary face's slot, read while the prims are staged.  The table holds
    // -1 for a solid cell, so the smaller entry is the fluid cell's.
    if (isface && g.nface > 0 && min(nL, nR) < 0) fbc = G(d.face_bc)[-min(nL, nR) - 1];
    __syncthreads();

    // 2. faces
    if (isface) {
        const bool fL = sflag[hL] != 0, fR = sflag[hR] != 0;
        const double ih = a == 0 ? g.invh[0] : (a == 1 ? g.invh[1] : g.invh[2]);
        if (fL && fR) {
            const double rl = sp[QR][hL], rr = sp[QR][hR];
            const double ul = sp[QU + a][hL], ur = sp[QU + a][hR];
            const double vl = sp[QU + b1][hL], vr = sp[QU + b1][hR];
            const double wl = sp[QU + b2][hL], wr = sp[QU + b2][hR];
            const double tl = sp[QT][hL], tr = sp[QT][hR];
            const double el = sp[QE][hL], er = sp[QE][hR];
            double sA = 0.0, s1 = 0.0, s2 = 0.0, qn = 0.0, qr = 0.0, mu = 0.0;
            if (!EULER) {
                mu = quot(pow_line(0.5 * (tl + tr), g.omega), g.delta, g.idelta);
                // twice the mean over the face's two cells of the derivatives along the axis of stride S
                // of the velocity components qa (normal) and qb (that axis)
                auto tangential = [&](int S, int qa, int qb, double invh, double &da, double &db) {
                    da = db = 0.0;
#pragma unroll
                    for (int side = 0; side < 2; ++side) {
                        const int h = side ? hR : hL;
                        const bool m = sflag[h - S] != 0, p = sflag[h + S] != 0;
                        const int hm = m ? h - S : h, hp = p ? h + S : h;
                        const double id = (m && p) ? 0.5 * invh : invh;
                        da += (sp[qa][hp] - sp[qa][hm]) * id;
                        db += (sp[qb][hp] - sp[qb][hm]) * id;
                    }
                };
                double da1, d11, da2, d22;
                tangential(S1, QU + a, QU + b1, b1 == 0 ? g.invh[0] : (b1 == 1 ? g.invh[1] : g.invh[2]), da1, d11);
                tangential(S2, QU + a, QU + b2, b2 == 0 ? g.invh[0] : (b2 == 1 ? g.invh[1] : g.invh[2]), da2, d22);
                const double dn = (ur - ul) * ih;
                const double div = dn + 0.5 * (d11 + d22);
                sA = -mu * (2.0 * dn - (2.0 / 3.0) * div);
                s1 = -mu * ((vr - vl) * ih + 0.5 * da1);
                s2 = -mu * ((wr - wl) * ih + 0.5 * da2);
                qn = -g.kt * mu * (tr - tl) * ih;
                if (DIA) qr = -g.kr * mu * (sp[QTR][hR] - sp[QTR][hL]) * ih;
            }
            const double sL = fabs(ul) + sp[QC][hL], sR = fabs(ur) + sp[QC][hR];
            const double smax = sL > sR ? sL : sR, hs = 0.5 * smax;
            const double pl = rl * tl, pr = rr * tr, ml = rl * ul, mr = rr * ur;
            const double Fa = 0.5 * (ml * ul + 0.5 * pl + (mr * ur + 0.5 * pr)) - hs * (mr - ml) + 0.5 * sA;
            const double F1 = 0.5 * (ml * vl + mr * vr) - hs * (rr * vr - rl * vl) + 0.5 * s1;
            const double F2 = 0.5 * (ml * wl + mr * wr) - hs * (rr * wr - rl * wl) + 0.5 * s2;
            const double Fe = 0.5 * ((el + pl) * ul + (er + pr) * ur) - hs * (er - el)
                              + (sA * (0.5 * (ul + ur)) + s1 * (0.5 * (vl + vr)) + s2 * (0.5 * (wl + wr)) + qn + qr);
            sf[0][t] = (0.5 * (ml + mr) - hs * (rr - rl)) * ih;
            sf[1 + a][t] = Fa * ih;
            sf[1 + b1][t] = F1 * ih;
            sf[1 + b2][t] = F2 * ih;
            sf[4][t] = Fe * ih;
            if (DIA) {
                const double gl = sp[QER][hL], gr = sp[QER][hR];
                sf[NW - 1][t] = (0.5 * (gl * ul + gr * ur) - hs * (gr - gl) + qr) * ih;
            }
            sf[NW][t] = (EULER ? smax : smax + quot(g.Cd * mu * ih, 0.5 * (rl + rr))) * ih;
        } else if ((fL && fq > 0) || (fR && fq < MT)) {
            // the boundary face of a cell of this tile (at most one of the two is fluid)
            const int e = atomicAdd(&scount, 1);
            slist[e] = make_int2(t | (fR ? hR : hL) << 8 | (2 * a + (fR ? 0 : 1)) << 16 | fbc << 20, -(fR ? nR : nL) - 1);
        }
    }
    __syncthreads();
    const int nbf = scount;
    for (int base = 0; base < nbf; base += MBC) {   // uniform over the block
        const int nf = min(MBC, nbf - base);
        constexpr int QF = G13 ? 4 : 1;   // lanes that finish a face
        double in[6];                     // the finishing lane's incoming moments, read ahead
        if (!g.vlist && t < nf * QF) {
            const int2 fe = slist[base + t / QF];
            const gptr<const double> inp = G((const double *)d.inpsi) + ((fe.x >> 20) * 6 + ((fe.x >> 16) & 7)) * 6;
#pragma unroll
            for (int k = 0; k < 6; ++k) in[k] = inp[k];
        }
        if (!g.vlist) {
            // 1-D sums of w e^{-(xi - u)^2 / T} z^p (times xi on the outgoing half
            // along the normal), z = xi, with the Grad-13 wall flux xi - u: a quad
            // of lanes per face and axis
            for (int task = t; task < nf * 12; task += 256) {
                const int fa = task >> 2, e = fa / 3, j = fa - 3 * e;
                const int2 fe = slist[base + e];
                const int h = (fe.x >> 8) & 255, dir = (fe.x >> 16) & 7;
                int ax = (dir >> 1) + j;
                ax = ax > 2 ? ax - 3 : ax;
                const gptr<const double> xs = G((const double *)(ax == 0 ? d.xi64[0] : (ax == 1 ? d.xi64[1] : d.xi64[2])));
                const gptr<const double> ws = G((const double *)(ax == 0 ? d.w64[0] : (ax == 1 ? d.w64[1] : d.w64[2])));
                const int n = ax == 0 ? g.n1[0] : (ax == 1 ? g.n1[1] : g.n1[2]);
                const int kz = ax == 0 ? g.k0[0] : (ax == 1 ? g.k0[1] : g.k0[2]);
                const int lo = j == 0 && (dir & 1) ? kz : 0, hi = j == 0 && !(dir & 1) ? kz : n;
                const double u = sp[QU + ax][h], niT = -recip(sp[QT][h]);
                const bool g13 = G13 && !EULER && g.wall_flux == 1;
                double S[NS];
#pragma unroll
                for (int p = 0; p < NS; ++p) S[p] = 0.0;
                // two nodes a step: two exponentials under way (past the end, the last node with weight 0)
                for (int k = lo + (task & 3); k < hi; k += 8) {
                    const int kb = min(k + 4, hi - 1);
                    const double x[2] = {xs[k], xs[kb]}, wt[2] = {ws[k], k + 4 < hi ? ws[kb] : 0.0};
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const double c = x[q] - u, z = g13 ? c : x[q];
                        double v = wt[q] * exp_core(fmax(c * c * niT, -745.0));
                        if (j == 0) v *= x[q];
#pragma unroll
                        for (int p = 0; p < NS; ++p) {
                            S[p] += v;
                            v *= z;
                        }
                    }
                }
#pragma unroll
                for (int p = 0; p < NS; ++p) S[p] = quad_sum(S[p]);
                if ((task & 3) == 0) {
#pragma unroll
                    for (int p = 0; p < NS; ++p) ssum[fa * NS + p] = S[p];
                }
            }
            __syncthreads();
        }
        if (t < nf * QF) {
            const int e = t / QF;
            const int2 fe = slist[base + e];
            const int tf = fe.x & 255, h = (fe.x >> 8) & 255, dir = (fe.x >> 16) & 7, f = fe.y, ba = dir >> 1;
            const double ih = ba == 0 ? g.invh[0] : (ba == 1 ? g.invh[1] : g.invh[2]);
            const double sg = (dir & 1) ? ih : -ih;
            double Fe[6], gam;
            if (g.vlist) {
#pragma unroll
                for (int k = 0; k < NW; ++k) Fe[k] = G(d.Fb)[(size_t)k * g.nface + f];
                gam = G(d.Gb)[f];
            } else {
                const int b = fe.x >> 20;
                const double rho = sp[QR][h], T = sp[QT][h];
                const double mu = EULER ? 0.0 : quot(pow_line(T, g.omega), g.delta, g.idelta);
                const double piT = PI * T;
                const double K = quot(rho, piT * sqrt(piT)) * ((dir & 1) ? 1.0 : -1.0);
                const double e1 = DIA ? 0.5 * g.dr * sp[QTR][h] : 0.0;
                const double *S0 = ssum + e * 3 * NS, *S1 = S0 + NS, *S2 = S1 + NS;
                const int bb1 = ba == 2 ? 0 : ba + 1;
                double oA, o1, o2;   // momentum along the normal, b1 and b2
                if (G13 && !EULER && g.wall_flux == 1) {
                    double dv[3][5], sq[12];
                    bool hm[3], hp[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const int S = c == 0 ? 1 : (c == 1 ? MH : MH * MH);
                        hm[c] = sflag[h - S] != 0;
                        hp[c] = sflag[h + S] != 0;
                        const int m = hm[c] ? h - S : h, p = hp[c] ? h + S : h;
#pragma unroll
                        for (int k = 0; k < 4; ++k) dv[c][k] = sp[QU + k][p] - sp[QU + k][m];
                        dv[c][4] = sp[QTR][p] - sp[QTR][m];
                    }
                    cell_nsf(g, dv, hm, hp, mu, sq);
#pragma unroll
                    for (int k = 0; k < 12; ++k) sq[k] += G(d.ghot)[(size_t)k * g.nface + f];
                    // sigma, q, qr in the face's axes (ba, b1, b2): the diagonal 0..2, then (ba b1), (ba b2), (b1 b2)
                    auto rot = [&](int i, int ax) { return ax == 0 ? sq[i] : (ax == 1 ? sq[i + 1] : sq[i + 2]); };
                    const int bb2 = ba == 0 ? 2 : ba - 1;
                    const double sl[6] = {rot(0, ba), rot(0, bb1), rot(0, bb2),
                                          ba == 0 ? sq[3] : (ba == 1 ? sq[5] : sq[4]),
                                          ba == 0 ? sq[4] : (ba == 1 ? sq[3] : sq[5]),
                                          ba == 0 ? sq[5] : (ba == 1 ? sq[4] : sq[3])};
                    const double ql[3] = {rot(6, ba), rot(6, bb1), rot(6, bb2)};
                    const double rl[3] = {rot(9, ba), rot(9, bb1), rot(9, bb2)};
                    const double cs = recip(rho * T * T), c5 = quot(2.0, 5.0 * T);
                    // the seven bracketed sums (1, c_n, c_1, c_2, c_n^2, c_1^2, c_2^2), shared out over the quad
                    double *B = sb + e * 8;
                    for (int k = t & 3; k < 7; k += 4) {
                        const int en = k == 1 ? 1 : (k == 4 ? 2 : 0), f1 = k == 2 ? 1 : (k == 5 ? 2 : 0),
                                  f2 = k == 3 ? 1 : (k == 6 ? 2 : 0);
                        B[k] = g13_bsum(S0 + en, S1 + f1, S2 + f2, sl, ql, cs, 2.0 * cs, c5);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    const double ul0 = sp[QU + ba][h], ul1 = sp[QU + bb1][h], ul2 = sp[QU + bb2][h];
                    Fe[0] = K * B[0];
                    oA = K * (B[1] + ul0 * B[0]);
                    o1 = K * (B[2] + ul1 * B[0]);
                    o2 = K * (B[3] + ul2 * B[0]);
                    const double uu = ul0 * ul0 + ul1 * ul1 + ul2 * ul2;
                    const double e0 = B[4] + B[5] + B[6] + 2.0 * (ul0 * B[1] + ul1 * B[2] + ul2 * B[3]) + uu * B[0];
                    const double sr = rl[0] * S0[1] * S1[0] * S2[0] + rl[1] * S0[0] * S1[1] * S2[0] + rl[2] * S0[0] * S1[0] * S2[1];
                    Fe[5] = DIA ? K * (e1 * B[0] + quot(2.0, rho * T) * sr) : 0.0;
                    Fe[4] = K * e0 + Fe[5];
                } else {
                    const double s12 = S1[0] * S2[0];
                    Fe[0] = K * S0[0] * s12;
                    oA = K * S0[1] * s12;
                    o1 = K * S0[0] * S1[1] * S2[0];
                    o2 = K * S0[0] * S1[0] * S2[1];
                    Fe[5] = e1 * Fe[0];
                    Fe[4] = K * (S0[2] * s12 + S0[0] * (S1[2] * S2[0] + S1[0] * S2[2])) + Fe[5];
                }
                Fe[1] = ba == 0 ? oA : (ba == 1 ? o2 : o1);
                Fe[2] = ba == 1 ? oA : (ba == 2 ? o2 : o1);
                Fe[3] = ba == 2 ? oA : (ba == 0 ? o2 : o1);
                const double sc = bc.kind[b] == 1 ? bc.rho[b] : quot(Fe[0], -in[0]);
#pragma unroll
                for (int k = 0; k < NW; ++k) Fe[k] += sc * in[k];
                gam = fabs(sp[QU + ba][h]) + sp[QC][h] + (EULER ? 0.0 : quot(g.Cd * mu * ih, rho));
            }
            if (QF == 1 || (t & 3) == 0) {
#pragma unroll
                for (int k = 0; k < NW; ++k) sf[k][tf] = Fe[k] * sg;
                sf[NW][tf] = gam * ih;
            }
        }
        __syncthreads();
    }

    // 3. residual and diagonal: wave w adds components 2 w and 2 w + 1, the last wave D
    const int h = (cx + 1) + MH * ((cy + 1) + MH * (cz + 1));
    const bool live = sflag[h] != 0;
    // the faces below and above the cell along each axis
    const int xl = cx + 4 * cy + 16 * cz, xh = cx < 3 ? xl + 1 : 192 + cy + 4 * cz;
    const int yl = 64 + cy + 4 * cz + 16 * cx, yh = cy < 3 ? yl + 1 : 208 + cz + 4 * cx;
    const int zl = 128 + cz + 4 * cx + 16 * cy, zh = cz < 3 ? zl + 1 : 224 + cx + 4 * cy;
    if (w < 3) {
        if (!live) return;
        const gptr<double> R = dst + (size_t)cell * WS;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int k = 2 * w + q;
            if (k >= NW) break;
            double res = rc[q] + (sf[k][xl] - sf[k][xh]) + (sf[k][yl] - sf[k][yh]) + (sf[k][zl] - sf[k][zh]);
            if (DIA && k == 5) {
                const double T = sp[QT][h], Tr = sp[QTR][h], rho = sp[QR][h];
                const double rate = g.delta * rho * T / (pow_line(T, g.omega) * g.Zr);   // 1 / (Z tau)
                const double Tm = (3.0 * T + g.dr * Tr) / (3.0 + g.dr);
                res += 0.5 * g.dr * rho * (Tm - Tr) * rate;
                R[WSRC] = rate;
            }
            R[NW + k] = res;
        }
        return;
    }
    double D = 0.0;
    if (live) {
        const double u0 = sp[QU][h], u1 = sp[QU + 1][h], u2 = sp[QU + 2][h], T = sp[QT][h];
        const double sumG = ((sf[NW][xl] + sf[NW][xh]) + (sf[NW][yl] + sf[NW][yh])) + (sf[NW][zl] + sf[NW][zh]);
        const double vis = EULER ? 0.0 : quot(g.Cd * quot(pow_line(T, g.omega), g.delta, g.idelta), sp[QR][h] * g.hmin);
        const double idt = (sqrt(u0 * u0 + u1 * u1 + u2 * u2) + sp[QC][h] + vis) / (g.macro_cfl * g.hmin);
        D = idt + 0.5 * sumG;
        if (!(D > 0.0 && isfinite(D))) {
            atomicOr(d.errflag, 2);
            D = 0.0;
        }
    }
    D = row_max(D);
    D = fmax(D, __shfl_xor(D, 16, 64));
    D = fmax(D, __shfl_xor(D, 32, 64));
    if (c == 0 && D > 0.0)
        atomicMax(&d.dmax[(size_t)(it % DSETS * DSLOT + (blk & (BSLOT - 1))) * DSTRIDE],
                  (unsigned long long)__double_as_longlong(D));
}

// one block per case
__global__ void k_mac_reset(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    for (int j = threadIdx.x; j < DSETS * DSLOT; j += blockDim.x) G(C.d.dmax)[(size_t)j * DSTRIDE] = 0ull;
}

// New half of the correction record; flags non-physical states.
__global__ __launch_bounds__(128) void k_mac_final(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    const Soa<double> P = soa(d.P, g.ncell, cell);
    const gptr<double> c = G(d.corr) + (size_t)cell * NCORR;
    c[0] = P[0]; c[1] = P[1]; c[2] = P[2]; c[3] = P[3]; c[4] = P[4];
    c[5] = g.species == 1 ? P[5] : P[4];
    if (!(P[0] > 0.0) || !(P[4] > 0.0) || !isfinite(P[6]) || (g.species == 1 && !(P[5] > 0.0))) atomicOr(d.errflag, 4);
}

// The last step of the solve on the box (none for iters = 0) and the new half
// of the correction record; flags non-physical states.
template <bool DIA>
__global__ __launch_bounds__(128) void k_mac_close(GSIS_SPAN_ARGS, int iters)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    double Dm = 1.0;
    if (iters > 0) Dm = largest_diagonal(d, (iters - 1) % DSETS);
    const int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !G(d.cflag)[cell]) return;
    double W[6], P[9];
    stepped_W<DIA>(G((const double *)((iters & 1) ? d.W2 : d.W)) + (size_t)cell * (DIA ? WS_DIA : WS_MONO), iters, Dm,
                   1.0 / Dm, W);
    short_prims<DIA>(g, W, P);
    const gptr<double> c = G(d.corr) + (size_t)cell * NCORR;
#pragma unroll
    for (int k = 0; k < 6; ++k) c[k] = P[k];
    if (!(P[0] > 0.0) || !(P[4] > 0.0) || !isfinite(P[6]) || (DIA && !(P[5] > 0.0))) atomicOr(d.errflag, 4);
}

// Launch it of an inner loop of iters forms the residual of iterate it (from
// iterate it - 1, its residual and D*); k_mac_close takes the last step.
template <bool DIA, bool EULER, bool G13>
static void mac_loop(const Target &t, int iters, hipStream_t s)
{
    for (int it = 0; it < iters; ++it) {
        if (t.vlist && t.host[0].g.nface > 0)
            hipLaunchKernelGGL((k_mac_bface<DIA, EULER, G13>), dim3((t.host[0].g.nface + 3) / 4), dim3(256), 0, s,
                               GSIS_SPAN(t.span(K_CELL1)), it);
        hipLaunchKernelGGL((k_mac_iter<DIA, EULER, G13>), dim3(t.nblk[K_MTILE]), dim3(256), 0, s,
                           GSIS_SPAN(t.span(K_MTILE)), it);
    }
    hipLaunchKernelGGL(k_mac_close<DIA>, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(t.span(K_CELL128)), iters);
}

hipError_t launch_gsis_macro(const Target &t, int iters, hipStream_t s, int euler)
{
    hipLaunchKernelGGL(k_mac_reset, dim3(t.nblk[K_CASE]), dim3(64), 0, s, GSIS_SPAN(t.span(K_CASE)));
    hipLaunchKernelGGL(k_mac_init, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(t.span(K_CELL128)));
    hipLaunchKernelGGL(k_mac_grad, dim3(t.nblk[K_GRAD]), dim3(256), 0, s, GSIS_SPAN(t.span(K_GRAD)));
    hipLaunchKernelGGL(k_mac_hot, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(t.span(K_CELL128)), euler);
    if (t.nblk[K_FACE8] > 0) {
        if (t.g13) hipLaunchKernelGGL(k_mac_fbfix<true>, dim3(t.nblk[K_FACE8]), dim3(256), 0, s, GSIS_SPAN(t.span(K_FACE8)), euler);
        else hipLaunchKernelGGL(k_mac_fbfix<false>, dim3(t.nblk[K_FACE8]), dim3(256), 0, s, GSIS_SPAN(t.span(K_FACE8)), euler);
    }
    hipLaunchKernelGGL(k_mac_const, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(t.span(K_CELL128)));
    // the Euler form and the Grad-13 wall flux are their own instantiations: as
    // run-time flags they would cost the common path registers
    if (t.dia) {
        if (euler) mac_loop<true, true, false>(t, iters, s);
        else if (t.g13) mac_loop<true, false, true>(t, iters, s);
        else mac_loop<true, false, false>(t, iters, s);
    } else {
        if (euler) mac_loop<false, true, false>(t, iters, s);
        else if (t.g13) mac_loop<false, false, true>(t, iters, s);
        else mac_loop<false, false, false>(t, iters, s);
    }
    return hipGetLastError();
}

// ------------------------------------------------ unstructured mesh solve
// The same solve on an unstructured mesh (one case): faces of any normal n
// (out of the owner), area S, cells of volume V.  Velocity gradient of a cell
// by least squares over its face neighbours (weights from the host: the
// inverse of sum_j d_j d_j^T on its range applied to d_j), face gradient the
// mean of the two cells' corrected along d = x_R - x_L to the two-cell
// difference, normal heat fluxes -k mu (T_R - T_L) / h with h = d . n (twice
// the centroid-to-face distance along n on a boundary), Rusanov; fluxes per
// unit area times S / V in the residual and the diagonal; the high-order
// terms at every face the kinetic flux of f^{n+1/2} minus the macroscopic
// flux of W^{n+1/2}; on a boundary face F_kin + F_eq(W^m) - F_eq(W^{n+1/2}).

// Rusanov + NSF flux across face f from L to R (no high-order terms).
template <class PV, class GV>
__device__ __forceinline__ void uface_flux(const Geo &g, const PV &L, const PV &R, const GV &gL, const GV &gR,
                                           const double fg[9], bool euler, double F[6], double *Gam)
{
    const double n[3] = {fg[1], fg[2], fg[3]}, h = fg[4], dl = fg[5], e[3] = {fg[6], fg[7], fg[8]};
    const double TF = 0.5 * (L[4] + R[4]), rF = 0.5 * (L[0] + R[0]);
    // Euler constitutive relations: no stress or heat flux, no diffusive part in Gamma
    const double mu = euler ? 0.0 : pow_pos(TF, g.omega) / g.delta;
    double G[9];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double gm[3], gd = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            gm[c] = 0.5 * (gL[b * 3 + c] + gR[b * 3 + c]);
            gd += gm[c] * e[c];
        }
        const double corr = (R[1 + b] - L[1 + b]) / dl - gd;
#pragma unroll
        for (int c = 0; c < 3; ++c) G[b * 3 + c] = gm[c] + corr * e[c];
    }
    const double div = G[0] + G[4] + G[8];
    double sN[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double acc = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) acc += (G[b * 3 + c] + G[c * 3 + b]) * n[c];
        sN[b] = -mu * (acc - (2.0 / 3.0) * div * n[b]);
    }
    const double qN = -g.kt * mu * (R[4] - L[4]) / h;
    const double qrN = g.species == 1 ? -g.kr * mu * (R[5] - L[5]) / h : 0.0;
    double Phi[2][6], Wv[2][6], un[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const PV &P = k ? R : L;
        const double rho = P[0], p = P[0] * P[4];
        un[k] = P[1] * n[0] + P[2] * n[1] + P[3] * n[2];
        Phi[k][0] = rho * un[k];
#pragma unroll
        for (int b = 0; b < 3; ++b) Phi[k][1 + b] = rho * P[1 + b] * un[k] + 0.5 * p * n[b];
        Phi[k][4] = (P[6] + p) * un[k];
        Phi[k][5] = P[7] * un[k];
        Wv[k][0] = rho;
#pragma unroll
        for (int b = 0; b < 3; ++b) Wv[k][1 + b] = rho * P[1 + b];
        Wv[k][4] = P[6];
        Wv[k][5] = P[7];
    }
    const double sL = fabs(un[0]) + L[8], sR = fabs(un[1]) + R[8];
    const double smax = sL > sR ? sL : sR;
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] = 0.5 * (Phi[0][k] + Phi[1][k]) - 0.5 * smax * (Wv[1][k] - Wv[0][k]);
#pragma unroll
    for (int b = 0; b < 3; ++b) F[1 + b] += 0.5 * sN[b];
    F[4] += sN[0] * 0.5 * (L[1] + R[1]) + sN[1] * 0.5 * (L[2] + R[2]) + sN[2] * 0.5 * (L[3] + R[3]) + qN + qrN;
    F[5] += qrN;
    *Gam = euler ? smax : smax + g.Cd * mu / (rF * h);
}

// Velocity gradient of every cell: G[b][c] = sum over its interior face
// entries of (u_j - u_i)_b w_c.
__device__ __forceinline__ void ucell_grad(const Geo &g, const Dev &d, int cell)
{
    if (cell >= g.ncell) return;
    const size_t n = g.ncell;
    const Soa<double> P = soa(d.P, n, cell);
    const double ui[3] = {P[1], P[2], P[3]};
    double Gc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int first = G(d.ucf_first)[cell], cnt = G(d.ucf_first)[cell + 1] - first;
    for (int k = 0; k < cnt; ++k) {
        const int e = first + k;
        const int j = G(d.ucf_nb)[e];
        if (j < 0) continue;
        const Soa<double> Pj = soa(d.P, n, j);
        const double w0 = G(d.ucf_lsq)[3 * (size_t)e], w1 = G(d.ucf_lsq)[3 * (size_t)e + 1], w2 = G(d.ucf_lsq)[3 * (size_t)e + 2];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double du = Pj[1 + b] - ui[b];
            Gc[b * 3] += du * w0;
            Gc[b * 3 + 1] += du * w1;
            Gc[b * 3 + 2] += du * w2;
        }
    }
    const Soa<double> Gd = soa(d.grad, n, cell);
#pragma unroll
    for (int k = 0; k < 9; ++k) Gd[k] = Gc[k];
}

__global__ __launch_bounds__(256) void k_umac_grad(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    ucell_grad(C.g, C.d, blk * (int)blockDim.x + (int)threadIdx.x);
}

// Kinetic flux of every face out of its owner, one wave per face: sum over
// the nodes of w (xi.n) psi f_face, psi = (1, xi, |xi|^2 f0 + f1, f1), f_face
// the upwind cell's value inside; on a boundary face the owner's value going
// out and the boundary value coming in, the wall density from this f (zero
// mass flux).  A boundary face also keeps the incoming half-range
// psi-moments of its boundary Maxwellian, w (xi.n) psi M_b over xi.n < 0.
template <typename T, bool DIA>
__global__ __launch_bounds__(256) void k_umac_kin(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int f = __builtin_amdgcn_readfirstlane(blk * 4 + (int)(threadIdx.x >> 6));
    if (f >= g.unface) return;
    const int lane = threadIdx.x & 63;
    const int L = G(d.uf_cell)[2 * (size_t)f], R = G(d.uf_cell)[2 * (size_t)f + 1];
    const Soa<double> fg = soa(d.uf_geo, (size_t)g.unface, f);
    const double n0 = fg[1], n1 = fg[2], n2 = fg[3];
    const size_t nv = (size_t)g.nv;
    const gptr<const T> f0L = (gptr<const T>)d.f0 + (size_t)L * nv;
    const gptr<const T> f1L = DIA ? (gptr<const T>)d.f1 + (size_t)L * nv : f0L;
    const int Rr = R >= 0 ? R : L;
    const gptr<const T> f0R = (gptr<const T>)d.f0 + (size_t)Rr * nv;
    const gptr<const T> f1R = DIA ? (gptr<const T>)d.f1 + (size_t)Rr * nv : f0R;
    const gptr<const double> nt = G((const double *)d.nt64);
    const int bf = R >= 0 ? 0 : -1 - R;
    const int slot = R >= 0 ? 0 : G(d.ubf_slot)[bf];
    const gptr<const double> mb = G((const double *)d.mb64) + (size_t)slot * nv;
    const gptr<const double> mb1 = G((const double *)d.mb1_64) + (size_t)slot * nv;
    double acc[6] = {0, 0, 0, 0, 0, 0}, bin[6] = {0, 0, 0, 0, 0, 0}, out = 0.0, in = 0.0;
    for (int pos = lane; pos < g.nv; pos += 64) {
        const double x0 = nt[4 * (size_t)pos], x1 = nt[4 * (size_t)pos + 1], x2 = nt[4 * (size_t)pos + 2];
        const double w = nt[4 * (size_t)pos + 3];
        const double xn = x0 * n0 + x1 * n1 + x2 * n2;
        if (xn == 0.0) continue;
        double a0, a1;
        bool add = true;
        if (xn > 0.0) {
            a0 = (double)f0L[pos];
            a1 = DIA ? (double)f1L[pos] : 0.0;
            if (R < 0) out += w * xn * a0;
        } else if (R >= 0) {
            a0 = (double)f0R[pos];
            a1 = DIA ? (double)f1R[pos] : 0.0;
        } else {
            a0 = mb[pos];
            a1 = DIA ? mb1[pos] : 0.0;
            in += w * (-xn) * a0;
            add = false;   // into bin: scaled by the wall density once it is known
        }
        const double ww = w * xn, xx = x0 * x0 + x1 * x1 + x2 * x2;
        const double c[6] = {ww * a0, ww * x0 * a0, ww * x1 * a0, ww * x2 * a0, ww * (xx * a0 + a1), ww * a1};
        if (add) {
#pragma unroll
            for (int k = 0; k < 6; ++k) acc[k] += c[k];
        } else {
#pragma unroll
            for (int k = 0; k < 6; ++k) bin[k] += c[k];
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) acc[k] = wave_sum(acc[k]);
    if (R < 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) bin[k] = wave_sum(bin[k]);
        out = wave_sum(out);
        in = wave_sum(in);
        const double sc = C.bc.kind[slot] == 1 ? C.bc.rho[slot] : out / in;
#pragma unroll
        for (int k = 0; k < 6; ++k) acc[k] += sc * bin[k];
        if (lane < 6) G(d.ubin)[6 * (size_t)bf + lane] = bin[lane];
    }
    if (lane < 6) G(d.uFk)[6 * (size_t)f + lane] = acc[lane];
}

// A face's fixed part plus F, its Gamma and area, one 64-byte record for the
// cells that gather it.
__device__ __forceinline__ void store_face(const Dev &d, size_t f, const double F[6], double Gam, double S)
{
    const gptr<const f64x2> fix = (gptr<const f64x2>)d.ufix + 3 * f;
    const gptr<f64x2> o = (gptr<f64x2>)d.uFf + 4 * f;
#pragma unroll
    for (int k = 0; k < 3; ++k) o[k] = f64x2{F[2 * k] + fix[k].x, F[2 * k + 1] + fix[k].y};
    o[3] = f64x2{Gam, S};
}

// Interior faces, one thread each: the macroscopic flux of the current W;
// mode 0 keeps F_kin - F as the face's high-order terms, mode 1 stores
// F + HoT and Gamma for the residual.
__global__ __launch_bounds__(256) void k_umac_iflux(GSIS_SPAN_ARGS, int mode, int euler)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int f = blk * blockDim.x + threadIdx.x;
    if (f >= g.unface) return;
    const int L = G(d.uf_cell)[2 * (size_t)f], R = G(d.uf_cell)[2 * (size_t)f + 1];
    if (R < 0) return;
    const size_t n = g.ncell;
    double fg[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) fg[k] = G(d.uf_geo)[(size_t)k * g.unface + f];
    double F[6], Gam;
    uface_flux(g, soa(d.P, n, L), soa(d.P, n, R), soa(d.grad, n, L), soa(d.grad, n, R), fg, euler != 0, F, &Gam);
    if (mode == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) G(d.ufix)[6 * (size_t)f + k] = G(d.uFk)[6 * (size_t)f + k] - F[k];
        if (g.species != 1) G(d.ufix)[6 * (size_t)f + 5] = 0.0;
    } else {
        store_face(d, f, F, Gam, fg[0]);
    }
}

// Stress and heat fluxes of the Grad-13 wall flux at every boundary face's
// cell, one thread per boundary face: the NSF values of the current iterate
// (its least-squares velocity gradient and the gradients of Tt and Tr with the
// same weights) plus the cell's high-order terms.  Mode 0 (at W^{n+1/2})
// forms and keeps those terms, the kinetic stress and heat fluxes of
// f^{n+1/2} minus the NSF values; mode 1 adds the kept terms.  ubsq[12][unbf]
// = (sigma xx yy zz xy xz yz, q, qr).
__global__ __launch_bounds__(256) void k_umac_g13s(GSIS_SPAN_ARGS, int mode)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int bf = blk * blockDim.x + threadIdx.x;
    if (bf >= g.unbf) return;
    const size_t n = g.ncell, nb = g.unbf;
    const int cell = G(d.ubf_cell)[bf];
    const Soa<double> P = soa(d.P, n, cell);
    const Soa<double> Gu = soa(d.grad, n, cell);
    double gt[3] = {0, 0, 0}, gr[3] = {0, 0, 0};
    const int first = G(d.ucf_first)[cell], cnt = G(d.ucf_first)[cell + 1] - first;
    for (int k = 0; k < cnt; ++k) {
        const int e = first + k;
        const int j = G(d.ucf_nb)[e];
        if (j < 0) continue;
        const Soa<double> Pj = soa(d.P, n, j);
        const double dt = Pj[4] - P[4], dr = Pj[5] - P[5];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double w = G(d.ucf_lsq)[3 * (size_t)e + c];
            gt[c] += dt * w;
            gr[c] += dr * w;
        }
    }
    const double mu = P[9];
    double G9[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) G9[k] = Gu[k];
    const double div = G9[0] + G9[4] + G9[8];
    double sq[12];
    sq[0] = -mu * (2.0 * G9[0] - (2.0 / 3.0) * div);
    sq[1] = -mu * (2.0 * G9[4] - (2.0 / 3.0) * div);
    sq[2] = -mu * (2.0 * G9[8] - (2.0 / 3.0) * div);
    sq[3] = -mu * (G9[1] + G9[3]);
    sq[4] = -mu * (G9[2] + G9[6]);
    sq[5] = -mu * (G9[5] + G9[7]);
    const bool dia = g.species == 1;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        sq[6 + c] = -g.kt * mu * gt[c];
        sq[9 + c] = dia ? -g.kr * mu * gr[c] : 0.0;
    }
    const gptr<double> hot = G(d.ubhot);
    if (mode == 0) {
        // cm: sigma at 5..10, q at 11..13, qr at 15..17
        const gptr<const double> m = G((const double *)d.cm) + (size_t)cell * NMOM;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const double kin = k < 9 ? m[5 + k] : (dia ? m[6 + k] : 0.0);
            const double h = kin - sq[k];
            hot[(size_t)k * nb + bf] = h;
            sq[k] += h;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) sq[k] += hot[(size_t)k * nb + bf];
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) G(d.ubsq)[(size_t)k * nb + bf] = sq[k];
}

// Boundary faces, two of one outward direction to a wave: F_eq of the owner's
// Maxwellian (outgoing half-range sums over the nodes, incoming part the
// boundary Maxwellian at the face's density rule).  The wave walks the runs of
// nodes whose classes leave through that direction and reads every node once
// for both faces.  Mode 0 keeps F_kin - F_eq(W^{n+1/2}), mode 1 stores fixed
// part + F_eq(W^m) and Gamma.  G13: the same with the outgoing half of the
// owner's Grad-13 distributions of Eq. (G13_VDF) (stress and heat fluxes
// from k_umac_g13s), f0 = M B(c), f1 = (dr/2) Tr f0 + 2 M (qr.c) / (rho Tt).
// A lane takes the nodes at its place in every aligned stretch of 64, in
// order, and nodes outside a run count zero, so that every sum is formed as in
// a walk over all nodes: the first corrections of a hypersonic start pass
// through cells near vacuum that blow a change of rounding up from 1e-16 to
// 1e-8 in the fields.  Splitting the sums over waves, or factoring the
// exponential by axis, is therefore left out, although it takes 39 us.
// Measured on 124k tetrahedra with 9648 boundary faces and 7788 nodes: 65 us a
// call (95 with every node walked; the gradients' blocks, 9 us on their own,
// run beside it), of which the FP64 instructions, 49 per face and node, are 51.
constexpr int UBF = 2;

template <bool G13>
__global__ __launch_bounds__(256) void k_umac_bflux(GSIS_SPAN_ARGS, int mode, int euler)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int nbb = (g.ubgn + 3) / 4;
    if (blk >= nbb) {   // the velocity gradients of the same state, beside the boundary faces
        ucell_grad(g, d, (blk - nbb) * (int)blockDim.x + (int)threadIdx.x);
        return;
    }
    const int pair = __builtin_amdgcn_readfirstlane(blk * 4 + (int)(threadIdx.x >> 6));
    if (pair >= g.ubgn) return;
    const cptr<int> bfp = (cptr<int>)(d.ubg + pair);
    const int lane = threadIdx.x & 63;
    const bool dia = g.species == 1;
    const size_t nc = (size_t)g.ncell, nfc = (size_t)g.unface;
    double n[UBF][3], u[UBF][3], iT[UBF], s0[UBF], s1[UBF][3], s4[UBF];
    // Grad-13: the bracket's coefficients per face, sigma / (rho Tt^2),
    // 2 q / (rho Tt^2), 2 / (5 Tt), 2 qr / (rho Tt), and the q_r sum
    double sg[G13 ? UBF : 1][6], qv[G13 ? UBF : 1][3], c5[G13 ? UBF : 1], qr[G13 ? UBF : 1][3], sr[G13 ? UBF : 1];
    // the faces' state and normals are the same for every lane: scalar loads
#pragma unroll
    for (int q = 0; q < UBF; ++q) {
        const int bf = bfp[q] >= 0 ? bfp[q] : bfp[0];   // a missing face repeats the first
        const cptr<double> fg = (cptr<double>)d.uf_geo + ((cptr<int>)d.ubf_face)[bf];
        const cptr<double> P = (cptr<double>)d.P + ((cptr<int>)d.ubf_cell)[bf];
        n[q][0] = fg[nfc];
        n[q][1] = fg[2 * nfc];
        n[q][2] = fg[3 * nfc];
        u[q][0] = P[nc];
        u[q][1] = P[2 * nc];
        u[q][2] = P[3 * nc];
        iT[q] = 1.0 / P[4 * nc];
        s0[q] = s4[q] = 0.0;
        s1[q][0] = s1[q][1] = s1[q][2] = 0.0;
        if constexpr (G13) {
            const size_t nb = g.unbf;
            const cptr<double> b = (cptr<double>)d.ubsq + bf;
            const double irT2 = 1.0 / (P[0] * P[4 * nc] * P[4 * nc]);
            const double cr = 2.0 / (P[0] * P[4 * nc]);
#pragma unroll
            for (int k = 0; k < 6; ++k) sg[q][k] = b[(size_t)k * nb] * irT2;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                qv[q][k] = 2.0 * irT2 * b[(size_t)(6 + k) * nb];
                qr[q][k] = dia ? cr * b[(size_t)(9 + k) * nb] : 0.0;
            }
            c5[q] = 2.0 / (5.0 * P[4 * nc]);
            sr[q] = 0.0;
        }
    }
    const gptr<const double> nt = G((const double *)d.nt64);
    const int dq = ((cptr<int>)d.ubgd)[pair];
    int rr = ((cptr<int>)d.ubro)[dq] - 1, p0 = 0, p1 = 0, at = 0;
    const int rb = ((cptr<int>)d.ubro)[dq + 1];
    // the wave's next stretch of 64 nodes, from the multiple of 64 below a run's first
    auto next = [&]() -> bool {
        at += 64;
        while (at >= p1) {
            if (++rr >= rb) return false;
            p0 = ((cptr<int>)d.ubr)[2 * rr];
            p1 = ((cptr<int>)d.ubr)[2 * rr + 1];
            at = p0 & ~63;
        }
        return true;
    };
    struct Node { double x[3], w; };
    auto read = [&](Node &v) {   // a lane outside the run reads an end of it with weight 0
        const int pos = at + lane;
        const gptr<const double> t = nt + 4 * (size_t)min(max(pos, p0), p1 - 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) v.x[k] = t[k];
        v.w = pos >= p0 && pos < p1 ? t[3] : 0.0;
    };
    // the next stretch is read while the sums of this one are formed
    Node cur, nxt;
    bool more = next();
    if (more) read(cur);
    while (more) {
        more = next();
        if (more) read(nxt);
        const double x0 = cur.x[0], x1 = cur.x[1], x2 = cur.x[2], w = cur.w, xx = x0 * x0 + x1 * x1 + x2 * x2;
#pragma unroll
        for (int q = 0; q < UBF; ++q) {
            const double xn = fmax(x0 * n[q][0] + x1 * n[q][1] + x2 * n[q][2], 0.0);
            const double cx = x0 - u[q][0], cy = x1 - u[q][1], cz = x2 - u[q][2];
            const double cc = cx * cx + cy * cy + cz * cz;
            const double e = w * exp_core(fmax(-cc * iT[q], -745.0)) * xn;
            double ex = e;
            if constexpr (G13) {
                const double scc = sg[q][0] * cx * cx + sg[q][1] * cy * cy + sg[q][2] * cz * cz
                                 + 2.0 * (sg[q][3] * cx * cy + sg[q][4] * cx * cz + sg[q][5] * cy * cz);
                const double qc = qv[q][0] * cx + qv[q][1] * cy + qv[q][2] * cz;
                ex = e * (1.0 + scc + qc * (c5[q] * cc - 1.0));
                sr[q] += e * (qr[q][0] * cx + qr[q][1] * cy + qr[q][2] * cz);
            }
            s0[q] += ex;
            s1[q][0] += ex * x0;
            s1[q][1] += ex * x1;
            s1[q][2] += ex * x2;
            s4[q] += ex * xx;
        }
        cur = nxt;
    }
    // lane q finishes face q
    const int bf = bfp[lane < UBF ? lane : 0] >= 0 ? bfp[lane < UBF ? lane : 0] : bfp[0];
    const size_t ff = (size_t)G(d.ubf_face)[bf];
    const int slot = G(d.ubf_slot)[bf];
    const Soa<double> P = soa(d.P, nc, G(d.ubf_cell)[bf]), fg = soa(d.uf_geo, nfc, (int)ff);
    const gptr<const double> bin = G((const double *)d.ubin) + 6 * (size_t)bf;
#pragma unroll
    for (int q = 0; q < UBF; ++q) {
        s0[q] = wave_sum(s0[q]);
#pragma unroll
        for (int k = 0; k < 3; ++k) s1[q][k] = wave_sum(s1[q][k]);
        s4[q] = wave_sum(s4[q]);
        if constexpr (G13) sr[q] = wave_sum(sr[q]);
    }
    if (lane >= UBF || bfp[lane] < 0) return;
    auto mine = [&](double a0, double a1) { return lane == 0 ? a0 : a1; };
    static_assert(UBF == 2, "a pair of faces");
    const double t0 = mine(s0[0], s0[1]), t4 = mine(s4[0], s4[1]);
    const double rho = P[0], T = P[4];
    const double piT = PI * T, K = rho / (piT * sqrt(piT));
    const double h1 = g.species == 1 ? 0.5 * g.dr * P[5] : 0.0;
    double out[6];
    out[0] = K * t0;
#pragma unroll
    for (int k = 0; k < 3; ++k) out[1 + k] = K * mine(s1[0][k], s1[1][k]);
    if constexpr (G13) {
        const double f1 = dia ? K * (h1 * t0 + mine(sr[0], sr[1])) : 0.0;
        out[4] = K * t4 + f1;
        out[5] = f1;
    } else {
        out[4] = K * t4 + h1 * out[0];
        out[5] = h1 * out[0];
    }
    const double sc = C.bc.kind[slot] == 1 ? C.bc.rho[slot] : out[0] / (-bin[0]);
    double Fe[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) Fe[k] = out[k] + sc * bin[k];
    if (mode == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) G(d.ufix)[6 * ff + k] = G(d.uFk)[6 * ff + k] - Fe[k];
    } else {
        const double un = P[1] * fg[1] + P[2] * fg[2] + P[3] * fg[3];
        store_face(d, ff, Fe, fabs(un) + P[8] + (euler ? 0.0 : g.Cd * P[9] / (rho * fg[4])), fg[0]);
    }
}

// Residual and diagonal of every cell from the face fluxes (S / V per face,
// the sign of the owner's side), the rotational relaxation on the Er row; one
// atomic max of D per wave into the slot's partials.
__global__ __launch_bounds__(256) void k_umac_res(GSIS_SPAN_ARGS, int slot, int euler)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    const int cell = blk * blockDim.x + threadIdx.x;
    double D = 0.0;
    if (cell < g.ncell) {
        const size_t n = g.ncell;
        const Soa<double> P = soa(d.P, n, cell);
        double res[6] = {0, 0, 0, 0, 0, 0}, sumG = 0.0;
        const double iV = 1.0 / G(d.uvol)[cell];
        const int first = G(d.ucf_first)[cell], cnt = G(d.ucf_first)[cell + 1] - first;
        for (int k = 0; k < cnt; ++k) {
            const int fs = G(d.ucf_face)[first + k], f = fs >> 1;
            const gptr<const f64x2> r = (gptr<const f64x2>)d.uFf + 4 * (size_t)f;
            const f64x2 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
            const double o[6] = {r0.x, r0.y, r1.x, r1.y, r2.x, r2.y};
            const double sv = r3.y * iV, sg = (fs & 1) ? -1.0 : 1.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) res[q] -= sg * o[q] * sv;
            sumG += r3.x * sv;
        }
        if (g.species != 1) res[5] = 0.0;
        const double invtau = P[10];
        if (g.species == 1) {
            const double T = (3.0 * P[4] + g.dr * P[5]) / (3.0 + g.dr);
            res[5] += 0.5 * g.dr * P[0] * (T - P[5]) * invtau / g.Zr;
        }
        const double umag = sqrt(P[1] * P[1] + P[2] * P[2] + P[3] * P[3]);
        const double vis = euler ? 0.0 : g.Cd * P[9] / (P[0] * g.uhmin);
        const double idt = (umag + P[8] + vis) / (g.macro_cfl * g.uhmin);
        D = idt + 0.5 * sumG;
        const Soa<double> r = soa(d.R, n, cell);
#pragma unroll
        for (int q = 0; q < 6; ++q) r[q] = res[q];
        G(d.Src)[cell] = g.species == 1 ? invtau / g.Zr : 0.0;
        if (!(D > 0.0 && isfinite(D))) {
            atomicOr(d.errflag, 2);
            D = 0.0;
        }
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) D = fmax(D, __shfl_xor(D, m, 64));
    if ((threadIdx.x & 63) == 0 && D > 0.0)
        atomicMax(&d.dmax[(size_t)(slot * DSLOT + ((blk * 4 + (int)(threadIdx.x >> 6)) & (DSLOT - 1))) * DSTRIDE],
                  (unsigned long long)__double_as_longlong(D));
}

// W += R / D* (the Er row with its relaxation on the diagonal) and the new
// prims; block 0 clears the partials of the other slot (the previous
// iteration's).
__global__ __launch_bounds__(256) void k_umac_advance(GSIS_SPAN_ARGS, int slot)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    double Dm = __longlong_as_double((long long)G(d.dmax)[(size_t)(slot * DSLOT + (threadIdx.x & (DSLOT - 1))) * DSTRIDE]);
#pragma unroll
    for (int m = 1; m < DSLOT; m <<= 1) Dm = fmax(Dm, __shfl_xor(Dm, m, 64));
    if (blk == 0 && (int)threadIdx.x < DSLOT) G(d.dmax)[(size_t)((slot ^ 1) * DSLOT + threadIdx.x) * DSTRIDE] = 0ull;
    const int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell) return;
    const size_t n = g.ncell;
    const double iDm = 1.0 / Dm;
    const Soa<double> W = soa(d.W, n, cell);
    const Soa<double> r = soa(d.R, n, cell);
    double Wn[6];
#pragma unroll
    for (int k = 0; k < 5; ++k) Wn[k] = W[k] + r[k] * iDm;
    Wn[5] = g.species == 1 ? W[5] + r[5] / (Dm + G(d.Src)[cell]) : W[5];
#pragma unroll
    for (int k = 0; k < 6; ++k) W[k] = Wn[k];
    prim_from_W(g, Wn, soa(d.P, n, cell));
}

// Euler steps: no high-order terms, the boundary flux of the iterate's own
// Maxwellian -- every fixed part zero.
__global__ __launch_bounds__(256) void k_umac_nofix(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const int i = blk * blockDim.x + threadIdx.x;
    if (i < 6 * C.g.unface) G(C.d.ufix)[i] = 0.0;
}

hipError_t launch_umacro(const Target &t, int iters, hipStream_t s, int euler)
{
    const Geo &g = t.host->g;
    const Span sp{t.cases, nullptr};
    const dim3 cells((g.ncell + 255) / 256), faces((g.unface + 255) / 256);
    const dim3 fwaves((g.unface + 3) / 4), bwaves((g.ubgn + 3) / 4), bthreads((std::max(g.unbf, 1) + 255) / 256);
    // the Grad-13 wall flux: its stress and heat fluxes first, then its flux
    const bool g13 = t.g13 && !euler;
    // the boundary faces' fluxes, with grad the velocity gradients in the same
    // launch (those of the Grad-13 stress are needed before it)
    auto bflux = [&](int mode, bool grad) {
        const dim3 gr(bwaves.x + (grad && !g13 ? cells.x : 0));
        if (g13) {
            if (grad) hipLaunchKernelGGL(k_umac_grad, cells, dim3(256), 0, s, GSIS_SPAN(sp));
            if (gr.x == 0) return;
            hipLaunchKernelGGL(k_umac_g13s, bthreads, dim3(256), 0, s, GSIS_SPAN(sp), mode);
            hipLaunchKernelGGL(k_umac_bflux<true>, gr, dim3(256), 0, s, GSIS_SPAN(sp), mode, euler);
        } else if (gr.x > 0) {
            hipLaunchKernelGGL(k_umac_bflux<false>, gr, dim3(256), 0, s, GSIS_SPAN(sp), mode, euler);
        }
    };
    hipLaunchKernelGGL(k_mac_reset, dim3(1), dim3(64), 0, s, GSIS_SPAN(sp));
    hipLaunchKernelGGL(k_mac_init, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(sp));
    hipLaunchKernelGGL(k_umac_grad, cells, dim3(256), 0, s, GSIS_SPAN(sp));
    // the kinetic face fluxes, and the boundary Maxwellians' incoming moments the boundary fluxes need
    if (t.fp32) {
        if (t.dia) hipLaunchKernelGGL((k_umac_kin<float, true>), fwaves, dim3(256), 0, s, GSIS_SPAN(sp));
        else hipLaunchKernelGGL((k_umac_kin<float, false>), fwaves, dim3(256), 0, s, GSIS_SPAN(sp));
    } else {
        if (t.dia) hipLaunchKernelGGL((k_umac_kin<double, true>), fwaves, dim3(256), 0, s, GSIS_SPAN(sp));
        else hipLaunchKernelGGL((k_umac_kin<double, false>), fwaves, dim3(256), 0, s, GSIS_SPAN(sp));
    }
    if (euler) {
        hipLaunchKernelGGL(k_umac_nofix, dim3((6 * g.unface + 255) / 256), dim3(256), 0, s, GSIS_SPAN(sp));
    } else {
        hipLaunchKernelGGL(k_umac_iflux, faces, dim3(256), 0, s, GSIS_SPAN(sp), 0, 0);
        if (g.unbf > 0) bflux(0, false);
    }
    for (int it = 0; it < iters; ++it) {
        const int slot = it & 1;
        bflux(1, it > 0);
        hipLaunchKernelGGL(k_umac_iflux, faces, dim3(256), 0, s, GSIS_SPAN(sp), 1, euler);
        hipLaunchKernelGGL(k_umac_res, cells, dim3(256), 0, s, GSIS_SPAN(sp), slot, euler);
        hipLaunchKernelGGL(k_umac_advance, cells, dim3(256), 0, s, GSIS_SPAN(sp), slot);
    }
    hipLaunchKernelGGL(k_mac_final, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(sp));
    return hipGetLastError();
}

// blocks one case needs for each launch shape
int kind_blocks(const Geo &g, Kind k)
{
    switch (k) {
    case K_CELL64: return (g.ncell + 63) / 64;
    case K_CELL128: return (g.ncell + 127) / 128;
    case K_CELL256: return (g.ncell + 255) / 256;
    case K_CELL1: return g.ncell;
    case K_FACE256: return (g.nface + 255) / 256;
    case K_FACE8: return face_blocks(g);
    case K_GRAD: return grad_blocks(g);
    case K_MTILE: return mtile_blocks(g);
    case K_MOM: return (g.ncell + 16 * MOM_WAVES - 1) / (16 * MOM_WAVES) * (g.species == 1 ? 16 : 8);
    case K_MSUM: return (g.ncell + 15) / 16 * 8;
    case K_CASE: return 1;
    default: return 0;
    }
}

}  // namespace gsis
