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
// of v_mfma_f64_16x16x4 (product t takes nodes mom_node(q, t), q = 0..3) in chains of
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
// k_moments: a wave takes 16 cells of one octant and one VDF; lane l of product t
// supplies f(cell l & 15, node mom_node(l >> 4, t)).  Loads take 512 bytes of a row at
// a time, the next stretch's in flight while this one, brought to the lanes through
// the wave's own LDS tile, is multiplied.  The monomials come from a table
// (k_monomials, 128 bytes a node, in the XCD's L2 as blocks of one octant go to one
// XCD), a chunk at a time through LDS for the four waves of a block: formed in the
// kernel they took a third of its instructions.
// Bound in FP64 by reading the VDF, 11.4 ms for 75.5 GB (64 x 48 x 48 cells, 40^3 nodes,
// 6.6 TB/s); in FP32 by instructions, the products' 1024 cycles a chunk and the
// conversions, 9.3 ms for 51.5 GB (96 x 64 x 64, 32^3) and 18.3 for 100.7 (40^3); two
// VDFs 5.3 for 32.6 GB and 3.4 for 16.3.  The kernel that formed its monomials, a wave
// per block, took 12.0, 11.3, 22.0, 6.1 and 5.7; sums along the rows of the tensor grid
// with a reduction over lanes, in an order that the sweep can't form, 11.3, 8.7, 15.9,
// 5.8 and 3.5.  It runs for states under 256 MB and with few nodes an octant, for a
// caller's tile that forms no sums (tile_forms_sums), for a lean workspace, and once
// when a state is set.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_moments(GSIS_SPAN_ARGS)
{
    typedef double d4 __attribute__((ext_vector_type(4)));
    typedef double d2 __attribute__((ext_vector_type(2)));
    constexpr int V = 16 / (int)sizeof(T);   // values of a load
    constexpr int ROW = 512, NROW = ROW / (int)sizeof(T), NCH = NROW / MCHUNK;   // bytes, nodes, chunks of a stretch
    constexpr int PITCH = ROW + 16;          // 16 rows at one offset take all LDS banks
    // a row starts at any element
    typedef T vec __attribute__((ext_vector_type(V)));
    typedef T uvec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
    __shared__ __attribute__((aligned(16))) char stile[MOM_WAVES][16 * PITCH];
    __shared__ d2 smono2[2][16 * 32];
    int blk;
    const Case &C = case_of(span_cases, span_map, blk);
    const Geo &g = C.g;
    const bool dia = g.species == 1;
    const int o = blk & 7, d = dia ? (blk >> 3) & 1 : 0, r = blk >> (dia ? 4 : 3);
    const int t = threadIdx.x, lane = t & 63, i = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int c0 = (r * MOM_WAVES + w) * 16;   // the wave's cells
    const int n = g.osize[o], ob = g.obase[o], ncell = g.ncell;
    const int nch = (n + MCHUNK - 1) / MCHUNK;
    const bool live = c0 < ncell;   // uniform over the wave
    const gptr<const d2> tab = (gptr<const d2>)C.d.mono + (size_t)mom_chunk(g, o) * (16 * 32) + 2 * t;
    // load k reads two cells' rows
    const int lr = lane >> 5, lv = (lane & 31) * V;
    const gptr<const T> f = d ? (gptr<const T>)C.d.f1 : (gptr<const T>)C.d.f0;
    auto row = [&](int k) { return f + (size_t)min(c0 + 2 * k + lr, ncell - 1) * (size_t)g.nv + ob; };
    vec pv[8];
    auto load = [&](int n0) {
        if (n0 + NROW <= n) {
#pragma unroll
            for (int k = 0; k < 8; ++k) pv[k] = __builtin_nontemporal_load((gptr<const uvec>)(row(k) + n0 + lv));
        } else {   // nodes past the end read the last one (and weigh 0)
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) pv[k][e] = row(k)[min(n0 + lv + e, n - 1)];
        }
    };
    // monomials of a chunk, a part per thread, read before the values that are in flight longer
    struct Mono { d2 a, b; };
    auto read = [&](int h) {
        const gptr<const d2> p = tab + (size_t)min(h, nch - 1) * (16 * 32);
        return Mono{p[0], p[1]};
    };
    auto place = [&](int h, const Mono &m) {
        smono2[h & 1][2 * t] = m.a;
        smono2[h & 1][2 * t + 1] = m.b;
    };
    d4 tot, err, seg, pair;
    const d4 zero = {0.0, 0.0, 0.0, 0.0};
    tot = err = seg = pair = zero;
    Mono m1;
    if (n > 0) {
        place(0, read(0));
        m1 = read(1);
        if (live) load(0);
        __syncthreads();
    }
    for (int h0 = 0; h0 < nch; h0 += NCH) {
        if (live) {
#pragma unroll
            for (int k = 0; k < 8; ++k) *(vec *)(stile[w] + (2 * k + lr) * PITCH + (lane & 31) * 16) = pv[k];
            // LDS accesses of one wave complete in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int h = h0 + c;
            if (h >= nch) break;
            place(h + 1, m1);
            m1 = read(h + 2);
            const double *const smono = (const double *)smono2[h & 1];
            if (c == 0 && live && h0 + NCH < nch) load((h0 + NCH) * MCHUNK);
            if (live) {
                d4 sum, p;
#pragma unroll
                for (int s = 0; s < 16; s += V) {
                    const vec a = *(const vec *)(stile[w] + i * PITCH + (c * MCHUNK + mom_node<T>(q, s)) * sizeof(T));
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        p = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[e], smono[(s + e) * 64 + lane],
                                                                 (s + e) % 4 == 0 ? zero : p, 0, 0, 0);
                        if (s + e == 3) sum = p;
                        else if ((s + e) % 4 == 3) sum += p;
                    }
                }
                const int m = h & 3;   // uniform
                if (m == 0) seg = sum;
                else if (m == 1) seg += sum;
                else if (m == 2) pair = sum;
                else pair += sum;
                if (m == 3 || h + 1 == nch) add_compensated(tot, err, seg + (m < 2 ? zero : pair));
            }
            __syncthreads();
        }
    }
    if (!live) return;
    // lane l holds sum (l & 15) of rows 4 j + (l >> 4), j = 0..3
    const gptr<double> mom8 = (gptr<double>)C.d.mom8;
    const gptr<const int> cflag = (gptr<const int>)C.d.cflag;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int cell = c0 + 4 * j + q;
        if (cell >= ncell) continue;
        const double v = cflag[cell] != 0 ? tot[j] + err[j] : 0.0;
        const gptr<double> out = mom8 + ((size_t)cell * 8 + o) * NRS;
        if (d == 0 && i < 13) out[i] = v;
        if (d == 1 && i < 4) out[13 + i] = v;
        if (!dia && i < 4) out[13 + i] = 0.0;
    }
}

// The monomials of every chunk of an octant as k_moments multiplies them: for product
// p and lane l monomial l & 15 of node mom_node(l >> 4, p), zero past the octant's end
// (a block per chunk).
template <typename T>
__global__ __launch_bounds__(256) void k_monomials(Geo g, Dev d)
{
    const int chunk = (int)blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int o = 0;
    while (o < 7 && chunk >= mom_chunk(g, o + 1)) ++o;
    const Monomial mono(lane & 15);
    for (int p = w; p < 16; p += 4) {
        const int l = (chunk - mom_chunk(g, o)) * MCHUNK + mom_node<T>(lane >> 4, p);
        const double *t = d.nt64 + 4 * ((size_t)g.obase[o] + min(l, g.osize[o] - 1));
        d.mono[((size_t)chunk * 16 + p) * 64 + lane] = mono(t[0], t[1], t[2], l < g.osize[o] ? t[3] : 0.0);
    }
}

hipError_t launch_monomials(const Geo &g, const Dev &d, bool fp32, hipStream_t s)
{
    const dim3 grid(mom_chunk(g, 8));
    if (fp32) hipLaunchKernelGGL(k_monomials<float>, grid, dim3(256), 0, s, g, d);
    else hipLaunchKernelGGL(k_monomials<double>, grid, dim3(256), 0, s, g, d);
    return hipGetLastError();
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
    hipLaunchKernelGGL(k_moments<T>, dim3(t.nblk[K_MOM]), dim3(64 * MOM_WAVES), 0, s, GSIS_SPAN(t.span(K_MOM)));
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
