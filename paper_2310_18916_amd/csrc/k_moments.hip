// Moment reduction of Eq. (getmoment).
//
// k_moments: raw moments of every (cell, velocity octant) about the origin,
// accumulated in FP64 whatever the VDF precision: per-octant sums, from which
// every half-range wall flux follows.  k_moment_totals: the same from the
// segments that the sweep forms of a large state.
//
// k_derive: central moments (rho, u, Tt, sigma, q, Tr, qr) of every cell from
// the octant sums.
//
// k_commit_correction: adds to the octant sums the discrete raw moments of
// M(W') - M(W) of Eq. (updatef), which factor into 1-D sums on the tensor grid,
// so the corrected state's moments are exact without touching the VDF.
//
// On a node list (a refined or unstructured velocity mesh, Sec. 3.1) the
// correction doesn't factor: k_commit_correction_list sums over the nodes, one
// wave per (cell, octant).  k_moments_mesh is the moment kernel of an
// unstructured spatial mesh.
#include "gsis_common.h"
#include "gsis_launch.h"

namespace gsis {

// Octant sums of a box case, tensor grid or node list, as a matrix product:
// [cells x nodes] times [nodes x 13 monomials] on the FP64 matrix cores.
//
// The order of a cell's sum depends on the octant's size alone, whoever forms
// it: MCHUNK = 64 consecutive nodes are one chunk, multiplied in 16 products
// of v_mfma_f64_16x16x4 (product t takes nodes 16 q + t, q = 0..3) in chains of
// four, ((p0 + p1) + p2) + p3; four chunks are a segment, (c0 + c1) + (c2 + c3), a
// missing one zero; segments are added in order, with the rounding of each
// addition carried along, and so are the octants (k_derive).  Root-mean-square
// error of the cells' moments from an emulation in extended precision (sums along
// rows with a lane tree, before; this order), in units of 2^-52, 16^3 nodes:
// density 0.49 and 0.44, velocity 0.12 and 0.13, temperature 0.66 and 0.58, stress
// 0.34 and 0.31, heat flux 0.34 and 0.35; 32^3: 0.43 and 0.29, 0.12 and 0.08, 0.66
// and 0.45, 0.31 and 0.28, 0.30 and 0.23.  The sweep forms the segments of its tiles while the
// values are in registers (k_sweep), and k_moment_totals adds them up;
// k_moments does all of it from the stored VDF, for a state that was set and
// for tiles that don't form segments, with the same result to the bit.
//
// k_moments: lane l of a product supplies f(cell l & 15, node 16 (l >> 4) + t)
// and monomial l & 15 of that node.  A block is one wave for 16 G cells of one
// octant; its loads take whole stretches of 1 / G KB of a row and pass through
// LDS, the next chunk's in flight while one is multiplied.  One VDF is held to two
// waves per SIMD (286 registers otherwise: 15.1 against 11.4 ms in FP32); two VDFs
// spill 400 bytes there (9.8 against 6.0 ms).  Bound by reading the VDF in FP64:
// 11.7 ms for 75.5 GB (64 x 48 x 48 cells, 40^3 nodes), 6.4 TB/s; in FP32 by the
// products' LDS reads, 11.4 ms for 51.5 GB.  (Sums along the rows of the tensor
// grid with a reduction over lanes read 6.8 and 5.8 TB/s, but in an order that the
// sweep can't form; with the segments in the sweep this kernel runs for small
// states, where both take 0.03 to 0.05 ms, and once when a state is set.)
template <typename T, bool DIA>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(DIA ? 1 : 2))) void k_moments(GSIS_SPAN_ARGS)
{
    typedef double d4 __attribute__((ext_vector_type(4)));
    typedef double d2 __attribute__((ext_vector_type(2)));
    constexpr int G = MOM_GROUPS;
    constexpr int V = 16 / (int)sizeof(T);   // values of one 16-byte load
    constexpr int LR = 64 / G;               // lanes along a row
    constexpr int NCH = LR * V / MCHUNK;     // chunks of a stretch
    constexpr int PITCH = 1024 + 16;         // 16 rows at one offset take all LDS banks
    constexpr int ND = DIA ? 2 : 1;
    // a row starts at any element
    typedef T vec __attribute__((ext_vector_type(V)));
    typedef T uvec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    __shared__ __attribute__((aligned(16))) char sv[16 * PITCH];
    __shared__ d2 sn[NCH * MCHUNK * 2];
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const int o = blk & 7, c0 = (blk >> 3) * 16 * G;
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int n = g.osize[o], ob = g.obase[o], ncell = g.ncell;
    const size_t nv = (size_t)g.nv;
    const gptr<const d2> nt = (gptr<const d2>)C.d.nt64 + 2 * (size_t)ob;
    // load k reads G cells' rows
    const int lr = lane / LR, lv = (lane % LR) * V;
    auto rowp = [&](int d, int k) {
        const int c = min(c0 + G * k + lr, ncell - 1);
        return (d ? (gptr<const T>)C.d.f1 : (gptr<const T>)C.d.f0) + (size_t)c * nv + ob;
    };
    const Monomial mono(i);
    d4 tot[ND][G], err[ND][G], seg[ND][G], pair[ND][G];
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int k = 0; k < G; ++k) tot[d][k] = err[d][k] = seg[d][k] = pair[d][k] = d4{0.0, 0.0, 0.0, 0.0};
    vec pv[16];
    d2 pn[NCH * 2];
    auto load = [&](int d, int n0) {
        if (n0 + NCH * MCHUNK <= n) {
#pragma unroll
            for (int k = 0; k < 16; ++k) pv[k] = __builtin_nontemporal_load((gptr<const uvec>)(rowp(d, k) + n0 + lv));
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int l = n0 + lv + e;
                    const T f = rowp(d, k)[min(l, n - 1)];
                    pv[k][e] = l < n ? f : T(0);
                }
        }
        if (d == 0) {
#pragma unroll
            for (int k = 0; k < NCH * 2; ++k) pn[k] = nt[min(2 * n0 + 64 * k + lane, 2 * n - 1)];
        }
    };
    if (n > 0) load(0, 0);
    for (int n0 = 0; n0 < n; n0 += NCH * MCHUNK)
#pragma unroll
        for (int d = 0; d < ND; ++d) {
#pragma unroll
            for (int k = 0; k < 16; ++k) *(vec *)(sv + k * PITCH + lane * 16) = pv[k];
            if (d == 0) {
#pragma unroll
                for (int k = 0; k < NCH * 2; ++k) sn[64 * k + lane] = pn[k];
            }
            __syncthreads();
            if (d + 1 < ND) load(d + 1, n0);
            else if (n0 + NCH * MCHUNK < n) load(0, n0 + NCH * MCHUNK);
#pragma unroll
            for (int h = 0; h < NCH; ++h) {
                d4 acc[G];
#pragma unroll 2
                for (int s4 = 0; s4 < 16; s4 += 4) {
                    d4 p[G];
#pragma unroll
                    for (int k = 0; k < G; ++k) p[k] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int s = s4; s < s4 + 4; s += V) {
                        vec a[G];
#pragma unroll
                        for (int k = 0; k < G; ++k)
                            a[k] = *(const vec *)(sv + i * PITCH + k * (1024 / G) + (h * MCHUNK + 16 * q + s) * sizeof(T));
#pragma unroll
                        for (int e = 0; e < V; ++e) {
                            const int l = h * MCHUNK + 16 * q + s + e;
                            const d2 t0 = sn[2 * l], t1 = sn[2 * l + 1];
                            const double m = mono(t0.x, t0.y, t1.x, t1.y);
#pragma unroll
                            for (int k = 0; k < G; ++k) p[k] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[k][e], m, p[k], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < G; ++k) acc[k] = s4 == 0 ? p[k] : acc[k] + p[k];
                }
                const int c = (n0 / MCHUNK + h) & 3;   // uniform
                const bool last = n0 + (h + 1) * MCHUNK >= n;
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    const d4 p = acc[k];
                    if (c == 0) seg[d][k] = p;
                    else if (c == 1) seg[d][k] += p;
                    else if (c == 2) pair[d][k] = p;
                    else pair[d][k] += p;
                    if (c == 3 || last) {
                        add_compensated(tot[d][k], err[d][k], seg[d][k] + (c < 2 ? d4{0.0, 0.0, 0.0, 0.0} : pair[d][k]));
                    }
                }
                if (last) break;
            }
            __syncthreads();
        }
    // lane l holds sum (l & 15) of rows 4 r + (l >> 4), r = 0..3
    const gptr<double> mom8 = (gptr<double>)C.d.mom8;
    const gptr<const int> cflag = (gptr<const int>)C.d.cflag;
#pragma unroll
    for (int k = 0; k < G; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int cell = c0 + G * (4 * r + q) + k;
            if (cell >= ncell) continue;
            const bool live = cflag[cell] != 0;
            const gptr<double> out = mom8 + ((size_t)cell * 8 + o) * NRS;
            if (i < 13) out[i] = live ? tot[0][k][r] + err[0][k][r] : 0.0;
            if (i < 4) out[13 + i] = DIA && live ? tot[ND - 1][k][r] + err[ND - 1][k][r] : 0.0;
        }
}

// The octant sums from the segments that the sweep stored: 16 cells of one
// octant per block, a thread per (cell, sum).
__global__ __launch_bounds__(256) void k_moment_totals(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const int o = blk & 7, cell = (blk >> 3) * 16 + (threadIdx.x >> 4), j = threadIdx.x & 15;
    if (cell >= g.ncell) return;
    const int s0 = g.oseg[o], s1 = g.oseg[o + 1];
    const bool live = ((gptr<const int>)C.d.cflag)[cell] != 0;
    const gptr<double> out = (gptr<double>)C.d.mom8 + ((size_t)cell * 8 + o) * NRS;
    const size_t step = (size_t)g.ncell * 16;
    gptr<const double> p = (gptr<const double>)C.d.mseg + s0 * step + (size_t)cell * 16 + j;
    double t = 0.0, e = 0.0;
#pragma unroll 8
    for (int s = s0; s < s1; ++s, p += step) add_compensated(t, e, *p);
    if (j < 13) out[j] = live ? t + e : 0.0;
    if (j < 4) {
        double t1 = 0.0, e1 = 0.0;
        if (g.species == 1) {
            gptr<const double> p1 = (gptr<const double>)C.d.mseg1 + s0 * (step / 4) + (size_t)cell * 4 + j;
#pragma unroll 8
            for (int s = s0; s < s1; ++s, p1 += step / 4) add_compensated(t1, e1, *p1);
        }
        out[13 + j] = live ? t1 + e1 : 0.0;
    }
}

// The 13 raw monomials of one node times its weight: 1, x, y, z, xx, yy, zz,
// xy, xz, yz, x|xi|^2, y|xi|^2, z|xi|^2.
__device__ __forceinline__ void node_monomials(const double *t, double m[13])
{
    const double x = t[0], y = t[1], z = t[2], w = t[3];
    m[0] = w;
    m[1] = w * x;
    m[2] = w * y;
    m[3] = w * z;
    m[4] = m[1] * x;
    m[5] = m[2] * y;
    m[6] = m[3] * z;
    m[7] = m[1] * y;
    m[8] = m[1] * z;
    m[9] = m[2] * z;
    const double s2 = x * x + y * y + z * z;
    m[10] = m[1] * s2;
    m[11] = m[2] * s2;
    m[12] = m[3] * s2;
}

// Writes the NRS sums of one (cell, octant) from the lanes' partial sums
// acc[0..12] (f0) and acc1[0..3] (f1), reduced over the wave in a fixed order.
template <bool DIA>
__device__ __forceinline__ void store_octant_sums(const double *acc, const double *acc1, int lane, gptr<double> out,
                                                  bool add)
{
    constexpr int NR = DIA ? 32 : 16;
    double v[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) v[k] = k < 13 ? acc[k < 13 ? k : 0] : (DIA && k < NRS ? acc1[k < NRS ? k - 13 : 0] : 0.0);
    int idx;
    const double r = wave_reduce_scatter<NR>(v, lane, &idx);
    if ((lane & (64 / NR - 1)) == 0 && idx < NRS) {
        if (add) out[idx] += r;
        else out[idx] = r;
    }
    if (!DIA && !add && lane == 0) out[NRS - 1] = 0.0;
}

// Unstructured spatial mesh: one wave (block) per octant of a group of CG consecutive cells.
// A lane takes the octant's nodes 64 apart, reads each node's (xi, w) once
// and applies its monomials to the node's value in every cell of the group,
// so the node table is read once per CG cells while each VDF load covers 64
// consecutive nodes of one cell.  Two nodes per lane and step, and the loads
// of all cells issued unconditionally (rows clamped to the last cell, a dead
// or missing cell's sums discarded at the end), keep 2 CG loads in flight.
template <typename T, bool DIA, int CG>
__global__ __launch_bounds__(64) void k_moments_mesh(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const gptr<const int> cflag = (gptr<const int>)C.d.cflag;
    const gptr<const double> nt = (gptr<const double>)C.d.nt64;
    const gptr<double> mom8 = (gptr<double>)C.d.mom8;
    const int o = blk & 7;
    const int cell0 = (blk >> 3) * CG;
    const int lane = threadIdx.x;
    const int n = g.osize[o], ob = g.obase[o];
    const size_t nv = (size_t)g.nv;
    gptr<const T> r0[CG], r1[CG];
    bool live[CG];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        const int cc = min(cell0 + c, g.ncell - 1);
        live[c] = cell0 + c < g.ncell && cflag[cc];   // uniform over the wave
        r0[c] = (gptr<const T>)C.d.f0 + (size_t)cc * nv + ob;
        r1[c] = DIA ? (gptr<const T>)C.d.f1 + (size_t)cc * nv + ob : r0[c];
    }
    double acc[CG][13], acc1[CG][4];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
#pragma unroll
        for (int k = 0; k < 13; ++k) acc[c][k] = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc1[c][k] = 0.0;
    }
    for (int l0 = 0; l0 < n; l0 += 128) {
        int li[2];
        double sc[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int l = l0 + h * 64 + lane;
            li[h] = min(l, n - 1);
            sc[h] = l < n ? 1.0 : 0.0;   // a repeated last node counts zero
        }
        T v[2][CG], v1[2][CG];
        double t[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                v[h][c] = r0[c][li[h]];
                if (DIA) v1[h][c] = r1[c][li[h]];
            }
            const gptr<const double> tp = nt + 4 * ((size_t)ob + li[h]);
#pragma unroll
            for (int q = 0; q < 4; ++q) t[h][q] = tp[q];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            t[h][3] *= sc[h];
            double m[13];
            node_monomials(t[h], m);
#pragma unroll
            for (int c = 0; c < CG; ++c) {
                const double x = (double)v[h][c];
#pragma unroll
                for (int k = 0; k < 13; ++k) acc[c][k] += m[k] * x;
                if (DIA) {
                    const double x1 = (double)v1[h][c];
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc1[c][k] += m[k] * x1;
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CG; ++c) {
        if (cell0 + c >= g.ncell) break;
        if (!live[c]) {
#pragma unroll
            for (int k = 0; k < 13; ++k) acc[c][k] = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) acc1[c][k] = 0.0;
        }
        store_octant_sums<DIA>(acc[c], acc1[c], lane, mom8 + ((size_t)(cell0 + c) * 8 + o) * NRS, false);
    }
}

// Central moments from the octant sums (octants added in a fixed order).
__global__ __launch_bounds__(256) void k_derive(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    // the octants' sums of 64 cells, read along the rows, the roundings carried (on
    // a mesh the plain sum, which is the first part of this one: its corrections
    // pass through cells near vacuum that blow up any change of rounding)
    constexpr int DC = 64;
    __shared__ double sm[DC * NRS];
    for (int idx = threadIdx.x; idx < DC * NRS; idx += blockDim.x) {
        const int c = blk * DC + idx / NRS, k = idx % NRS;
        if (c >= g.ncell) break;
        const gptr<const double> mo = (gptr<const double>)d.mom8 + (size_t)c * 8 * NRS + k;
        double t = 0.0, e = 0.0;
#pragma unroll
        for (int o = 0; o < 8; ++o) add_compensated(t, e, mo[o * NRS]);
        sm[idx] = g.umesh ? t : t + e;
    }
    __syncthreads();
    const int cell = blk * DC + (int)threadIdx.x;
    if (threadIdx.x >= DC || cell >= g.ncell) return;
    double *out = d.cm + (size_t)cell * NMOM;
    if (!d.cflag[cell]) {
        for (int k = 0; k < NMOM; ++k) out[k] = __builtin_nan("");
        return;
    }
    double m[NRS];
    for (int k = 0; k < NRS; ++k) m[k] = sm[threadIdx.x * NRS + k];
    double rho = m[0];
    double u[3] = {m[1] / rho, m[2] / rho, m[3] / rho};
    // second raw moments as a matrix
    double M2[3][3] = {{m[4], m[7], m[8]}, {m[7], m[5], m[9]}, {m[8], m[9], m[6]}};
    double S[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) S[a][b] = M2[a][b] - rho * u[a] * u[b];
    double tr = S[0][0] + S[1][1] + S[2][2];
    double Tt = (2.0 / 3.0) * tr / rho;
    double tr2 = M2[0][0] + M2[1][1] + M2[2][2];
    double u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    out[0] = rho;
    out[1] = u[0];
    out[2] = u[1];
    out[3] = u[2];
    out[4] = Tt;
    out[5] = 2.0 * (S[0][0] - tr / 3.0);
    out[6] = 2.0 * (S[1][1] - tr / 3.0);
    out[7] = 2.0 * (S[2][2] - tr / 3.0);
    out[8] = 2.0 * S[0][1];
    out[9] = 2.0 * S[0][2];
    out[10] = 2.0 * S[1][2];
    // q_a = sum c_a |c|^2 f = m3_a - 2 (M2 u)_a - u_a tr(M2) + 2 rho u_a |u|^2
    for (int a = 0; a < 3; ++a) {
        double m2u = M2[a][0] * u[0] + M2[a][1] * u[1] + M2[a][2] * u[2];
        out[11 + a] = m[10 + a] - 2.0 * m2u - u[a] * tr2 + 2.0 * rho * u[a] * u2;
    }
    if (g.species == 1) {
        double e1 = m[13];
        out[14] = 2.0 * e1 / (g.dr * rho);
        for (int a = 0; a < 3; ++a) out[15 + a] = m[14 + a] - u[a] * e1;
    } else {
        out[14] = out[15] = out[16] = out[17] = 0.0;
    }
    if (!(rho > 0.0) || !(Tt > 0.0)) atomicOr(d.errflag, 1);
}

// 1-D sums over the negative (h = 0) and positive (h = 1) halves of one axis:
// R[h][p] = sum_k w_k xi_k^p exp(-(xi_k - u)^2 / T), p = 0..3.
__device__ void half_sums(const double *xi, const double *w, int n, int k0, double u, double T, double R[2][4])
{
    for (int h = 0; h < 2; ++h)
        for (int p = 0; p < 4; ++p) R[h][p] = 0.0;
    for (int k = 0; k < n; ++k) {
        double x = xi[k], c = x - u;
        double e = w[k] * exp(-c * c / T);
        int h = k >= k0;
        R[h][0] += e;
        R[h][1] += e * x;
        R[h][2] += e * x * x;
        R[h][3] += e * x * x * x;
    }
}

// Raw octant moments (13 on f0, 4 on f1) of K * prod_a exp(-(xi_a-u_a)^2/T) given the
// half sums of each axis; f1 gets the factor h1.
__device__ void octant_monomials(const double X[4], const double Y[4], const double Z[4], double K, double h1,
                                 double *m)
{
    m[0] = K * X[0] * Y[0] * Z[0];
    m[1] = K * X[1] * Y[0] * Z[0];
    m[2] = K * X[0] * Y[1] * Z[0];
    m[3] = K * X[0] * Y[0] * Z[1];
    m[4] = K * X[2] * Y[0] * Z[0];
    m[5] = K * X[0] * Y[2] * Z[0];
    m[6] = K * X[0] * Y[0] * Z[2];
    m[7] = K * X[1] * Y[1] * Z[0];
    m[8] = K * X[1] * Y[0] * Z[1];
    m[9] = K * X[0] * Y[1] * Z[1];
    m[10] = K * (X[3] * Y[0] * Z[0] + X[1] * Y[2] * Z[0] + X[1] * Y[0] * Z[2]);
    m[11] = K * (X[2] * Y[1] * Z[0] + X[0] * Y[3] * Z[0] + X[0] * Y[1] * Z[2]);
    m[12] = K * (X[2] * Y[0] * Z[1] + X[0] * Y[2] * Z[1] + X[0] * Y[0] * Z[3]);
    m[13] = h1 * m[0];
    m[14] = h1 * m[1];
    m[15] = h1 * m[2];
    m[16] = h1 * m[3];
}

// Octant sums += moments of M(W') - M(W) (and (dr/2)[Tr' M(W') - Tr M(W)] on f1).
__global__ __launch_bounds__(128) void k_commit_correction(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const Dev &d = C.d;
    int cell = blk * blockDim.x + threadIdx.x;
    if (cell >= g.ncell || !d.cflag[cell]) return;
    const double *c = d.corr + (size_t)cell * NCORR;
    double Rn[3][2][4], Ro[3][2][4];
    for (int a = 0; a < 3; ++a) {
        half_sums(d.xi64[a], d.w64[a], g.n1[a], g.k0[a], c[1 + a], c[4], Rn[a]);
        half_sums(d.xi64[a], d.w64[a], g.n1[a], g.k0[a], c[7 + a], c[10], Ro[a]);
    }
    double Kn = c[0] * pow(PI * c[4], -1.5), Ko = c[6] * pow(PI * c[10], -1.5);
    double hn = g.species == 1 ? 0.5 * g.dr * c[5] : 0.0;
    double ho = g.species == 1 ? 0.5 * g.dr * c[11] : 0.0;
    for (int o = 0; o < 8; ++o) {
        int hx = (o & 1) ? 0 : 1, hy = (o & 2) ? 0 : 1, hz = (o & 4) ? 0 : 1;
        double mn[NRS], mo[NRS];
        octant_monomials(Rn[0][hx], Rn[1][hy], Rn[2][hz], Kn, hn, mn);
        octant_monomials(Ro[0][hx], Ro[1][hy], Ro[2][hz], Ko, ho, mo);
        double *dst = d.mom8 + ((size_t)cell * 8 + o) * NRS;
        for (int k = 0; k < NRS; ++k) dst[k] += mn[k] - mo[k];
    }
}

// Node list: octant sums += moments of M(W') - M(W) (and (dr/2)[Tr' M(W') -
// Tr M(W)] on f1), one wave per octant of one cell, summed over the nodes.
__global__ __launch_bounds__(512) void k_commit_correction_list(GSIS_SPAN_ARGS)
{
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const int cell = blk;
    const gptr<const int> cflag = (gptr<const int>)C.d.cflag;
    if (!cflag[cell]) return;   // uniform over the block
    const int o = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const gptr<const double> nt = (gptr<const double>)C.d.nt64;
    const gptr<const double> c = (gptr<const double>)C.d.corr + (size_t)cell * NCORR;
    const double pn = PI * c[4], po = PI * c[10];
    const double Kn = c[0] / (pn * sqrt(pn)), Ko = c[6] / (po * sqrt(po));
    const double itn = 1.0 / c[4], ito = 1.0 / c[10];
    const bool dia = g.species == 1;
    const double hn = dia ? 0.5 * g.dr * c[5] : 0.0, ho = dia ? 0.5 * g.dr * c[11] : 0.0;
    double acc[13], acc1[4];
#pragma unroll
    for (int k = 0; k < 13; ++k) acc[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) acc1[k] = 0.0;
    const int n = g.osize[o], ob = g.obase[o];
    for (int l = lane; l < n; l += 64) {
        const size_t node = (size_t)ob + l;
        const double t[4] = {nt[4 * node], nt[4 * node + 1], nt[4 * node + 2], nt[4 * node + 3]};
        const double nx = t[0] - c[1], ny = t[1] - c[2], nz = t[2] - c[3];
        const double ox = t[0] - c[7], oy = t[1] - c[8], oz = t[2] - c[9];
        const double en = Kn * exp_core(fmax(-(nx * nx + ny * ny + nz * nz) * itn, -745.0));
        const double eo = Ko * exp_core(fmax(-(ox * ox + oy * oy + oz * oz) * ito, -745.0));
        const double d0 = en - eo, d1 = hn * en - ho * eo;
        double m[13];
        node_monomials(t, m);
#pragma unroll
        for (int k = 0; k < 13; ++k) acc[k] += m[k] * d0;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc1[k] += m[k] * d1;
    }
    const gptr<double> out = (gptr<double>)C.d.mom8 + ((size_t)cell * 8 + o) * NRS;
    if (dia) store_octant_sums<true>(acc, acc1, lane, out, true);
    else store_octant_sums<false>(acc, acc1, lane, out, true);
}

// ------------------------------------------------------------------ launches
template <typename T, bool DIA>
static void moments(const Target &t, hipStream_t s)
{
    if (t.host[0].g.umesh) {
        constexpr int CG = DIA ? 2 : 4;   // cells per block
        const int ncell = t.host[0].g.ncell;
        hipLaunchKernelGGL((k_moments_mesh<T, DIA, CG>), dim3(8 * ((ncell + CG - 1) / CG)), dim3(64), 0, s,
                           GSIS_SPAN(t.span(K_CELL1)));
        return;
    }
    hipLaunchKernelGGL((k_moments<T, DIA>), dim3(t.nblk[K_MOM]), dim3(64), 0, s, GSIS_SPAN(t.span(K_MOM)));
}

hipError_t launch_moments(const Target &t, hipStream_t s, bool swept)
{
    if (swept && sweep_forms_sums(t)) {
        hipLaunchKernelGGL(k_moment_totals, dim3(t.nblk[K_MSUM]), dim3(256), 0, s, GSIS_SPAN(t.span(K_MSUM)));
        return hipGetLastError();
    }
    if (t.fp32) { if (t.dia) moments<float, true>(t, s); else moments<float, false>(t, s); }
    else { if (t.dia) moments<double, true>(t, s); else moments<double, false>(t, s); }
    return hipGetLastError();
}

hipError_t launch_derive(const Target &t, hipStream_t s)
{
    hipLaunchKernelGGL(k_derive, dim3(t.nblk[K_CELL64]), dim3(256), 0, s, GSIS_SPAN(t.span(K_CELL64)));
    return hipGetLastError();
}

hipError_t launch_commit_correction(const Target &t, hipStream_t s)
{
    if (t.vlist) {
        hipLaunchKernelGGL(k_commit_correction_list, dim3(t.host[0].g.ncell), dim3(512), 0, s,
                           GSIS_SPAN(t.span(K_CELL1)));
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_commit_correction, dim3(t.nblk[K_CELL128]), dim3(128), 0, s, GSIS_SPAN(t.span(K_CELL128)));
    return hipGetLastError();
}

}  // namespace gsis
