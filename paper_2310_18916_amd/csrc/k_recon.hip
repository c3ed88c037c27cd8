// Second-order right-hand side of the kinetic update (Sec. 3.2).
//
// The interface values of the explicit flux divergence r^n of Eq.
// (delta_equations) are reconstructed from the upwind cell,
// f_up + phi_up grad f_up . (x_face - x_up), with a least-squares gradient
// over the fluid face neighbours and the Venkatakrishnan limiter phi; the
// increments on the left-hand side stay first-order upwind.  On the Cartesian
// grid the least-squares normal matrix is diagonal, so each gradient
// component is a central difference, one-sided next to a box face or a solid
// cell, and zero along an axis with no fluid neighbour.  Faces on the box or
// a solid surface keep first-order values (the cell's own value leaving, the
// boundary value entering), so the wall density balance is unchanged.
//
// The sweep keeps its first-order implicit operator in direct form; the
// difference of the two divergences, D2 - D1, moves to its right-hand side:
// it reads inv_dt f^n - (D2 - D1) per point from the buffer written here.
//
// With G_a = phi grad_a f of a cell the term is the sum over the axes of
//   (xi_a / 2) (G_a of the cell [downwind face interior]
//               - G_a of the upwind cell [upwind face interior]),
// so one pass over the VDF does it: a block of four waves takes PX x PY columns
// of cells for 64 nodes of one octant and walks them downwind in z.  A wave
// holds one row of PX columns, the x-upwind column beside it and 2 of the PX
// y-upwind columns, with the values at k - 1, k, k + 1 (and the ones ahead) in
// registers; a plane's values meet in LDS for the y neighbours, G_y goes
// through LDS to the next row, G_x and G_z stay in registers.  Limiters are
// formed for (PX PY + PX + PY) / (PX PY) = 1.375 of the points and VDF values
// read 2.2 times, mostly from L2.  Bound by two waves per SIMD between the
// memory floor (33.6 GB, 7.8 ms) and the limiter's arithmetic: 13.4 ms on 40^3
// cells x 32^3 nodes in FP64, 6.9 without the limiter on 48^3 x 24^3 (24.5 GB,
// 5.7).  Two passes (every point's limiter stored and read back, neighbours from
// L2, 15 reads per point, six divisions) took 35.6; this pass with the six
// divisions replaced by cross products 20.7.
#include "gsis_common.h"
#include "gsis_launch.h"

#include <algorithm>

namespace gsis {

constexpr int PX = 8, PY = 4;          // columns of a block
constexpr int NCOL = PX + 3;           // columns of a wave

// Venkatakrishnan's psi of a face whose neighbourhood leaves D >= 0 on the side of
// the reconstruction's change x >= 0; D2 = D^2 + eps^2, y = 2 x.  (0 / 0, of values
// whose squares underflow, limits nothing: fmin passes over it.)
template <typename T>
__device__ __forceinline__ T psi(T D, T D2, T x)
{
    const T y = T(2) * x;
    return fma(D, y, D2) / fma(D, x, fma(y, x, D2));
}

// Venkatakrishnan phi of one point, the least psi over its interior faces (at most
// 1), and its gradient G = phi grad f along the octant's axes: f[2 a] the upwind
// and f[2 a + 1] the downwind neighbour along axis a; e2 = (K h)^3, multiplied
// here by the square of the stencil's largest |f|.
//
// Below 1 (x > D / 2) psi falls with x and grows with D.  Where all six neighbours
// are fluid cells both faces of an axis have the same x, one with D = max - f and
// one with f - min, so the least is psi(least D, largest x): one division
// instead of six.
template <typename T>
__device__ __forceinline__ void limited_gradient(const T *invh, bool limited, T fc, const T *f, T e2, T *G)
{
    T mx = fc, mn = fc, x = T(0), df[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        mx = fmax(mx, fmax(f[2 * a], f[2 * a + 1]));
        mn = fmin(mn, fmin(f[2 * a], f[2 * a + 1]));
        df[a] = f[2 * a + 1] - f[2 * a];
        x = fmax(x, fabs(df[a]));
    }
    T phi = T(0.5);
    if (limited) {
        const T S = fmax(fabs(mx), fabs(mn)), D = fmin(mx - fc, fc - mn);
        phi *= fmin(T(1), psi<T>(D, fma(D, D, e2 * (S * S)), T(0.25) * x));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) G[a] = phi * (df[a] * invh[a]);
}

// The same with neighbours missing (has: the neighbour is a fluid cell): a
// gradient component is one-sided where one is, zero where both are, and only the
// faces that are there limit it.
template <typename T>
__device__ __forceinline__ void limited_gradient(const T *invh, const T *half, bool limited, T fc, const T *f,
                                                 const bool *has, T e2, T *G)
{
    T mx = fc, mn = fc, xu = T(0), xd = T(0), ga[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T fm = has[2 * a] ? f[2 * a] : fc, fp = has[2 * a + 1] ? f[2 * a + 1] : fc;
        mx = fmax(mx, fmax(fm, fp));
        mn = fmin(mn, fmin(fm, fp));
        ga[a] = (fp - fm) * (has[2 * a] && has[2 * a + 1] ? T(0.5) * invh[a] : invh[a]);
        const T x = fabs(ga[a]) * half[a];
        const bool rise = ga[a] > T(0);   // towards the downwind face
        if (has[2 * a + 1]) { xu = fmax(xu, rise ? x : T(0)); xd = fmax(xd, rise ? T(0) : x); }
        if (has[2 * a]) { xd = fmax(xd, rise ? x : T(0)); xu = fmax(xu, rise ? T(0) : x); }
    }
    T phi = T(1);
    if (limited) {
        const T S = fmax(fabs(mx), fabs(mn)), up = mx - fc, dn = fc - mn, eps = e2 * (S * S);
        phi = fmin(fmin(phi, psi<T>(up, fma(up, up, eps), xu)), psi<T>(dn, fma(dn, dn, eps), xd));
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) G[a] = phi * ga[a];
}

// Logical block = (octant, 64 nodes) * patches + patch; blocks are dealt to the 8
// XCDs round robin, so logical block (b mod 8) (nblk / 8) + b / 8 gives every XCD
// one contiguous range, whose patches share their edges in its L2.
template <typename T, bool MASK>
__global__ __launch_bounds__(256) void k_recon(Geo g, Dev d, int nvb, int npx, int npy)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int LX = PX + 3, LY = PY + 3;   // a plane from two upwind to one downwind column
    __shared__ T sf[LY][LX][64], sg[PY][PX][64];
    const int nblk = (int)gridDim.x;
    int b = (int)blockIdx.x;
    if ((nblk & 7) == 0) b = (b & 7) * (nblk >> 3) + (b >> 3);
    const int patch = b % (npx * npy), run = b / (npx * npy);
    const int o = run / nvb, l0 = (run - o * nvb) * 64;
    if (l0 >= g.osize[o]) return;             // uniform over the block
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool act = l0 + lane < g.osize[o];
    const size_t node = (size_t)g.obase[o] + min(l0 + lane, g.osize[o] - 1);
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int sx = o & 1, sy = (o >> 1) & 1, sz = (o >> 2) & 1;
    const int i0 = (patch % npx) * PX, j0 = (patch / npx) * PY;   // in the octant's frame: upwind is one step back
    const gptr<const T> f = (gptr<const T>)(blockIdx.y ? d.f1 : d.f0);
    const gptr<T> out = (gptr<T>)(blockIdx.y ? d.ho1 : d.ho0);
    const gptr<const int> cflag = (gptr<const int>)d.cflag;
    T ax[3], invh[3], half[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ax[a] = T(0.5) * fabs(F32 ? (T)((gptr<const float>)d.nt32)[4 * node + a] : (T)((gptr<const double>)d.nt64)[4 * node + a]);
        invh[a] = (T)g.invh[a];
        half[a] = T(0.5) * (T)g.h[a];
    }
    const T idt = (T)g.inv_dt, e2 = (T)g.venk_e2;
    const bool limited = g.limited != 0;
    const size_t rowb = (size_t)g.nv * sizeof(T);
    const unsigned loff = (unsigned)node * (unsigned)sizeof(T);
    // cell of frame column (a, b) of the block at frame height k, clamped into the box
    auto cell_at = [&](int a, int bb, int k) -> int {
        const int ii = min(max(i0 + a, 0), nx - 1), jj = min(max(j0 + bb, 0), ny - 1), kk = min(max(k, 0), nz - 1);
        return (sx ? nx - 1 - ii : ii) + nx * ((sy ? ny - 1 - jj : jj) + ny * (sz ? nz - 1 - kk : kk));
    };
    auto value = [&](int a, int bb, int k) -> T {
        return *(gptr<const T>)((gptr<const char>)f + (size_t)cell_at(a, bb, k) * rowb + loff);
    };
    // columns of this wave: its row, the x-upwind one, two y-upwind ones
    auto col_a = [&](int c) { return c < PX ? c : (c == PX ? -1 : 2 * w + (c - PX - 1)); };
    auto col_b = [&](int c) { return c <= PX ? w : -1; };
    // the outer columns this wave brings to the plane
    constexpr int NOUT = 7;
    auto out_a = [&](int m) { return m == 0 ? -2 : (m == 1 ? PX : (m < 6 ? 2 * w + (m & 1) : (w == 2 ? PX : -1))); };
    auto out_b = [&](int m) { return m < 2 ? w : (m < 4 ? -2 : (m < 6 ? PY : (w == 1 ? PY : -1))); };

    // Fluid cells of a plane as one word: bit 5 c + q of column c, q = 0 the cell
    // itself, 1 and 2 its upwind and downwind neighbour along x, 3 and 4 along y.
    const int fe = min(lane, 5 * NCOL - 1), fcol = fe / 5, fq = fe - 5 * fcol;
    const int fa = (fcol < PX ? fcol : (fcol == PX ? -1 : 2 * w + (fcol - PX - 1))) + (fq == 2) - (fq == 1);
    const int fb = (fcol <= PX ? w : -1) + (fq == 4) - (fq == 3);
    const bool fin = lane < 5 * NCOL && i0 + fa >= 0 && i0 + fa < nx && j0 + fb >= 0 && j0 + fb < ny;
    const unsigned long long inxy = __ballot(fin);
    auto flag_of = [&](int k) -> int { return MASK ? cflag[cell_at(fa, fb, k)] : 1; };
    auto word_of = [&](int flag, int k) -> unsigned long long {
        if (k >= nz) return 0ull;
        return MASK ? __ballot(fin && flag != 0) : inxy;
    };
    unsigned long long prv = 0ull, cur = word_of(flag_of(0), 0), nxt = word_of(flag_of(1), 1);

    T fm[NCOL], fc[NCOL], fp[NCOL], fx[NCOL], ov[NOUT], gz[PX];
#pragma unroll
    for (int c = 0; c < NCOL; ++c) {
        fc[c] = value(col_a(c), col_b(c), 0);
        fp[c] = value(col_a(c), col_b(c), 1);
        fm[c] = fc[c];
    }
#pragma unroll
    for (int m = 0; m < NOUT; ++m) ov[m] = value(out_a(m), out_b(m), 0);
#pragma unroll
    for (int c = 0; c < PX; ++c) gz[c] = T(0);
    for (int k = 0; k < nz; ++k) {
#pragma unroll
        for (int c = 0; c < NCOL; ++c) sf[col_b(c) + 2][col_a(c) + 2][lane] = fc[c];
#pragma unroll
        for (int m = 0; m < NOUT; ++m) sf[out_b(m) + 2][out_a(m) + 2][lane] = ov[m];
        __syncthreads();
        // ahead
#pragma unroll
        for (int c = 0; c < NCOL; ++c) fx[c] = value(col_a(c), col_b(c), k + 2);
#pragma unroll
        for (int m = 0; m < NOUT; ++m) ov[m] = value(out_a(m), out_b(m), k + 1);
        const int flag2 = flag_of(k + 2);
        T xz[PX], gy[PX], gup = T(0);
        auto gradient = [&](int c, T *G) {
            const int a = col_a(c), bb = col_b(c);
            const T v[6] = {sf[bb + 2][a + 1][lane], sf[bb + 2][a + 3][lane], sf[bb + 1][a + 2][lane],
                            sf[bb + 3][a + 2][lane], fm[c], fp[c]};
            const unsigned m = (unsigned)(cur >> (5 * c)), zu = (unsigned)(prv >> (5 * c)) & 1u, zd = (unsigned)(nxt >> (5 * c)) & 1u;
            if ((m & 31u) == 31u && zu && zd) {   // uniform
                limited_gradient<T>(invh, limited, fc[c], v, e2, G);
            } else {
                const bool has[6] = {(m & 2u) != 0, (m & 4u) != 0, (m & 8u) != 0, (m & 16u) != 0, zu != 0, zd != 0};
                limited_gradient<T>(invh, half, limited, fc[c], v, has, e2, G);
            }
        };
        T G[3];
#pragma unroll
        for (int c = PX + 1; c < NCOL; ++c) {
            gradient(c, G);
            sg[0][col_a(c)][lane] = G[1];
        }
        gradient(PX, G);
        gup = G[0];
#pragma unroll
        for (int c = 0; c < PX; ++c) {
            gradient(c, G);
            const unsigned m = (unsigned)(cur >> (5 * c));
            const T tx = (m & 4u ? G[0] : T(0)) - (m & 2u ? gup : T(0));
            const T tz = ((nxt >> (5 * c)) & 1u ? G[2] : T(0)) - ((prv >> (5 * c)) & 1u ? gz[c] : T(0));
            xz[c] = fma(ax[0], tx, ax[2] * tz);
            gy[c] = m & 16u ? G[1] : T(0);
            gup = G[0];
            gz[c] = G[2];
            if (w + 1 < PY) sg[w + 1][c][lane] = G[1];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < PX; ++c) {
            const unsigned m = (unsigned)(cur >> (5 * c));
            const T ty = gy[c] - (m & 8u ? sg[w][c][lane] : T(0));
            const T v = idt * fc[c] - fma(ax[1], ty, xz[c]);
            if (act && (m & 1u))
                __builtin_nontemporal_store(v, (gptr<T>)((gptr<char>)out + (size_t)cell_at(c, w, k) * rowb + loff));
        }
#pragma unroll
        for (int c = 0; c < NCOL; ++c) { fm[c] = fc[c]; fc[c] = fp[c]; fp[c] = fx[c]; }
        prv = cur;
        cur = nxt;
        nxt = word_of(flag2, k + 2);
    }
}

hipError_t launch_recon(const Geo &g, const Dev &d, bool fp32, hipStream_t s)
{
    int omax = 0;
    for (int o = 0; o < 8; ++o) omax = std::max(omax, g.osize[o]);
    const int nvb = (omax + 63) / 64, npx = (g.nx + PX - 1) / PX, npy = (g.ny + PY - 1) / PY;
    const long long nblk = (long long)npx * npy * 8 * nvb;
    if (nblk <= 0 || nblk > 0x7fffffffll) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)nblk, g.species == 1 ? 2 : 1), block(256);
    const bool mask = g.nfluid != g.ncell;
    if (fp32) {
        if (mask) hipLaunchKernelGGL((k_recon<float, true>), grid, block, 0, s, g, d, nvb, npx, npy);
        else hipLaunchKernelGGL((k_recon<float, false>), grid, block, 0, s, g, d, nvb, npx, npy);
    } else {
        if (mask) hipLaunchKernelGGL((k_recon<double, true>), grid, block, 0, s, g, d, nvb, npx, npy);
        else hipLaunchKernelGGL((k_recon<double, false>), grid, block, 0, s, g, d, nvb, npx, npy);
    }
    return hipGetLastError();
}

}  // namespace gsis
