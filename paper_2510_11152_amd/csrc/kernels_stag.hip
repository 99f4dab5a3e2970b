// Kernels of the staggered-grid FAS solver (Section 4.1, Appendices C-D) and of the
// first-order projection step (Section 4.2, Scheme 1).
//
// Point formulas (one fixed evaluation tree each; the library is built with
// -ffp-contract=off so every kernel rounds them identically):
//   s = (W + E) + (S + N)             neighbours, 0.0 for ghosts and wall points
//   k = 4 + (#odd ghosts) - (#even ghosts),   D = a h^2 + c k
//   sweep update   w = (c s + h^2 f) / D
//   operator       L w = (D w - c s) * (1 / h^2),    residual r = f - L w
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "fas_device.h"
#include "fas_internal.h"
#include "march_util.h"
#include "stag_internal.h"

namespace fas {
namespace stag {

namespace {

__device__ __forceinline__ double kshift(int kind) { return kind == K_CN ? -1.0 : (kind == K_CD ? 1.0 : 0.0); }

// k of the point (x, y) of level L.
__device__ __forceinline__ double kcount(const Lev& L, int x, int y)
{
    double k = 4.0;
    if (x == 0) k += kshift(L.kx);
    if (x == L.nx - 1) k += kshift(L.kx);
    if (y == 0) k += kshift(L.ky);
    if (y == L.ny - 1) k += kshift(L.ky);
    return k;
}

__device__ __forceinline__ double diag(const Lev& L, int x, int y) { return L.a * L.h2 + L.c * kcount(L, x, y); }

__device__ __forceinline__ double nbsum(const Lev& L, const double* u, int x, int y)
{
    const size_t i = (size_t)y * L.nx + x;
    const double W = x > 0 ? u[i - 1] : 0.0;
    const double E = x < L.nx - 1 ? u[i + 1] : 0.0;
    const double S = y > 0 ? u[i - L.nx] : 0.0;
    const double N = y < L.ny - 1 ? u[i + L.nx] : 0.0;
    return (W + E) + (S + N);
}

__device__ __forceinline__ double resid_at(const Lev& L, const double* f, const double* u, int x, int y)
{
    const size_t i = (size_t)y * L.nx + x;
    return f[i] - (diag(L, x, y) * u[i] - L.c * nbsum(L, u, x, y)) * L.ih2;
}

// ---- transfers ------------------------------------------------------------------------------
// Restriction (Appendix C for cells; Appendix D's six-point form for edges) of the iterate
// and of the residual (computed at the fine taps on the fly) at coarse point (K, J).
template <int LOC>
__device__ __forceinline__ void restrict_point(const Lev& Lf, const double* f, const double* u, int K, int J,
                                               double& ru, double& rr)
{
    if (LOC == LOC_CELL) {
        const int x = 2 * K, y = 2 * J;
        const size_t i = (size_t)y * Lf.nx + x;
        ru = ((u[i] + u[i + 1]) + (u[i + Lf.nx] + u[i + Lf.nx + 1])) * 0.25;
        rr = ((resid_at(Lf, f, u, x, y) + resid_at(Lf, f, u, x + 1, y)) +
              (resid_at(Lf, f, u, x, y + 1) + resid_at(Lf, f, u, x + 1, y + 1))) * 0.25;
    } else if (LOC == LOC_EDGE_X) {
        double gu[2], gr[2];
        for (int q = 0; q < 2; ++q) {
            const int y = 2 * J + q, x = 2 * K;
            const size_t i = (size_t)y * Lf.nx + x;
            gu[q] = (u[i] + 2.0 * u[i + 1]) + u[i + 2];
            gr[q] = (resid_at(Lf, f, u, x, y) + 2.0 * resid_at(Lf, f, u, x + 1, y)) + resid_at(Lf, f, u, x + 2, y);
        }
        ru = (gu[0] + gu[1]) * 0.125;
        rr = (gr[0] + gr[1]) * 0.125;
    } else {
        double gu[2], gr[2];
        for (int q = 0; q < 2; ++q) {
            const int x = 2 * K + q, y = 2 * J;
            const size_t i = (size_t)y * Lf.nx + x;
            gu[q] = (u[i] + 2.0 * u[i + Lf.nx]) + u[i + 2 * (size_t)Lf.nx];
            gr[q] = (resid_at(Lf, f, u, x, y) + 2.0 * resid_at(Lf, f, u, x, y + 1)) + resid_at(Lf, f, u, x, y + 2);
        }
        ru = (gu[0] + gu[1]) * 0.125;
        rr = (gr[0] + gr[1]) * 0.125;
    }
}

// Prolongation of the correction e = uc - uc0 (Appendix C: injection; Appendix D: linear
// along the cell-centred axis with odd ghosts first, then midpoint means along the edge axis
// with 0 at the wall points).  Coarse (stag_internal.h) gives e(K, J).
// Linear interpolation along a cell-centred axis from the coarse value of the cell and that
// of its neighbour on the side of the fine point (odd ghost beyond the last cell).
__device__ __forceinline__ double lin_cell(double e0, double enb) { return (3.0 * e0 + enb) * 0.25; }

// P e at fine point (x, y).
template <int LOC>
__device__ __forceinline__ double prolong_point(const Coarse& C, int x, int y)
{
    if (LOC == LOC_CELL) return C.e(x >> 1, y >> 1);
    if (LOC == LOC_EDGE_X) {
        const int J = y >> 1;
        auto col = [&](int K) {
            const double e0 = C.e(K, J);
            const double nb = (y & 1) ? (J < C.ncy - 1 ? C.e(K, J + 1) : -e0) : (J > 0 ? C.e(K, J - 1) : -e0);
            return lin_cell(e0, nb);
        };
        const int K = x >> 1;
        if (x & 1) return col(K);
        const double left = K >= 1 ? col(K - 1) : 0.0;
        const double right = K <= C.ncx - 1 ? col(K) : 0.0;
        return (left + right) * 0.5;
    }
    const int K = x >> 1;
    auto row = [&](int J) {
        const double e0 = C.e(K, J);
        const double nb = (x & 1) ? (K < C.ncx - 1 ? C.e(K + 1, J) : -e0) : (K > 0 ? C.e(K - 1, J) : -e0);
        return lin_cell(e0, nb);
    };
    const int J = y >> 1;
    if (y & 1) return row(J);
    const double below = J >= 1 ? row(J - 1) : 0.0;
    const double above = J <= C.ncy - 1 ? row(J) : 0.0;
    return (below + above) * 0.5;
}

template <int LOC>
__global__ __launch_bounds__(256) void k_restrict(Lev Lf, const double* __restrict__ f, const double* __restrict__ u,
                                                  int ncx, int ncy, double* __restrict__ uc,
                                                  double* __restrict__ uc0, double* __restrict__ rc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)ncx * ncy) return;
    double ru, rr;
    restrict_point<LOC>(Lf, f, u, (int)(t % ncx), (int)(t / ncx), ru, rr);
    uc[t] = ru;
    uc0[t] = ru;
    rc[t] = rr;
}

__global__ __launch_bounds__(256) void k_form_rhs(Lev L, const double* __restrict__ r, const double* __restrict__ u,
                                                  double* __restrict__ f)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)L.nx * L.ny) return;
    const int x = (int)(t % L.nx), y = (int)(t / L.nx);
    f[t] = r[t] + (diag(L, x, y) * u[t] - L.c * nbsum(L, u, x, y)) * L.ih2;
}

__global__ __launch_bounds__(256) void k_coarse_rhs(Lev L, double* __restrict__ f, const double* __restrict__ u)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)L.nx * L.ny) return;
    const int x = (int)(t % L.nx), y = (int)(t / L.nx);
    f[t] = f[t] + (diag(L, x, y) * u[t] - L.c * nbsum(L, u, x, y)) * L.ih2;
}

template <int LOC>
__global__ __launch_bounds__(256) void k_correct(Lev Lf, Coarse C, const double* usrc, double* udst)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)Lf.nx * Lf.ny) return;
    udst[t] = usrc[t] + prolong_point<LOC>(C, (int)(t % Lf.nx), (int)(t / Lf.nx));
}

// The FAS corrections of a lane's window columns (x0, x0 + 1) and rows yw .. yw + RPW - 1.  A
// lane loads e(K, J) for its own coarse column K = x0 / 2 and the RPW/2 + 3 coarse rows
// around its rows, and takes what the neighbouring columns give from the neighbouring lanes
// (the window's first even and last odd column come out wrong: one column of margin).
// add<PAR, I>() corrects row yw + I (yw of parity PAR) with the operations of prolong_point,
// so the result is the same bit for bit; entries outside the coarse grid are never used.
template <int LOC, int RPW>
struct CorrTable {
    static constexpr int NJ = RPW / 2 + 3;
    double E[NJ];
    int K, Jb;
    __device__ __forceinline__ void load(const Coarse& C, int x0, int yw)
    {
        K = x0 >> 1;
        Jb = (yw >> 1) - 1;
        double c0[NJ];
        const int Kl = min(max(K, 0), C.ncx - 1);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            const size_t i = (size_t)min(max(Jb + jj, 0), C.ncy - 1) * C.ncx + Kl;
            E[jj] = C.uc[i];
            c0[jj] = C.uc0[i];
        }
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) E[jj] = E[jj] - c0[jj];
    }
    template <int PAR, int I>
    __device__ __forceinline__ void add(const Coarse& C, bool in0, bool in1, double& u0, double& u1) const
    {
        constexpr int jj = ((PAR + I) >> 1) + 1;  // J - Jb
        constexpr bool yodd = ((PAR + I) & 1) != 0;
        const int J = Jb + jj;
        double p0, p1;
        if constexpr (LOC == LOC_CELL) {
            p0 = p1 = E[jj];
        } else if constexpr (LOC == LOC_EDGE_X) {
            // linear along y in column K; the even point takes the mean with column K - 1
            const double e0 = E[jj];
            const double nb = yodd ? (J < C.ncy - 1 ? E[jj + 1] : -e0) : (J > 0 ? E[jj - 1] : -e0);
            p1 = lin_cell(e0, nb);
            const double l = dpp_move<kShr1>(p1);
            const double left = K >= 1 ? l : 0.0, right = K <= C.ncx - 1 ? p1 : 0.0;
            p0 = (left + right) * 0.5;
        } else {
            // linear along x in coarse row j; an even row takes the mean of rows J - 1 and J
            auto row = [&](int j, double& r0, double& r1) {
                const double e0 = E[j], l = dpp_move<kShr1>(E[j]), r = dpp_move<kShl1>(E[j]);
                r0 = lin_cell(e0, K > 0 ? l : -e0);
                r1 = lin_cell(e0, K < C.ncx - 1 ? r : -e0);
            };
            if constexpr (yodd) {
                row(jj, p0, p1);
            } else {
                double b0, b1, a0, a1;
                row(jj - 1, b0, b1);
                row(jj, a0, a1);
                const bool below = J >= 1, above = J <= C.ncy - 1;
                p0 = ((below ? b0 : 0.0) + (above ? a0 : 0.0)) * 0.5;
                p1 = ((below ? b1 : 0.0) + (above ? a1 : 0.0)) * 0.5;
            }
        }
        u0 = in0 ? u0 + p0 : u0;
        u1 = in1 ? u1 + p1 : u1;
    }
};

template <int LOC, int RPW, int PAR, int... I>
__device__ __forceinline__ void corr_rows(const CorrTable<LOC, RPW>& T, const Coarse& C, int yw, int ny, bool in0,
                                          bool in1, double (&u0)[RPW], double (&u1)[RPW],
                                          std::integer_sequence<int, I...>)
{
    ((yw + I >= 0 && yw + I < ny ? T.template add<PAR, I>(C, in0, in1, u0[I], u1[I]) : (void)0), ...);
}

// ---- red-black sweeps on a window held in registers -----------------------------------------
// A 512-thread block (8 waves) loads a 128-column window of the iterate and right-hand side:
// lane l of a wave owns the column pair (2l, 2l + 1) of the window and each wave WY/8 rows, all
// in registers.  x-neighbours come from the adjacent lane by DPP; before each half-sweep the
// waves trade the first and last row of their bands through LDS (double-buffered: one barrier
// per half-sweep).  Half-sweep k updates values at distance >= k from the window's edge
// correctly, so after 2 nu half-sweeps the values at distance >= 2 nu are exactly what nu
// sweeps over the whole grid give.  Values outside the grid stay 0 (the 0.0 neighbours of the
// point formula).  Window geometry (rows, margins of the written region): sweep_geom(); the
// window origin is an even column and a row of fixed parity, so the column of a pair that a
// half-sweep updates is known at compile time, row by row.
//
// What bounds it: memory on the large levels (an edge row is odd, so rows start at any 8-byte
// boundary; a pair is one 16-byte access all the same), the chain of half-sweeps on the small
// ones.  The form that kept the window in LDS (two planes, every neighbour an LDS read) was
// bound by its LDS accesses: at 4096^2, two sweeps with the restriction took 124-132 us, with
// correction and norm 126 (cells), 142 (EW) and 177 us (NS edges); now 96-107 and 116-123 us
// (4.4-5 TB/s), and 7-8 instead of 9 us on small levels.  Eight waves, two blocks per compute
// unit: blocks of 5 and 10 waves took 134-175 us (they fill the SIMDs unevenly), and 80 VGPRs
// for a third block spill.  Divisions by a precomputed reciprocal and two corrections (the
// same bits) gained 1.5% and were not worth their range checks.
//
// XE: the window reaches past a domain x-edge; the other windows need no column masks and
// have one diagonal.
//
// Variants (each a fixed set of point formulas of the per-level kernels, so the results are
// the same bit for bit):
//   CORR  the FAS correction is applied as the window is loaded (u = uin + P e, as k_correct);
//   NORM  one more ring of margin; each block writes the sum of the squared residuals of the
//         values it wrote to io.partials (one value per block), replacing a residual pass;
//   RHS   f holds the restricted residual r of the finer level: the FAS right-hand side
//         f = r + L u is formed from the loaded window before the sweeps (as k_coarse_rhs)
//         and written to io.fout;
//   RES   after the sweeps, the residual is formed and the block restricts its written region
//         into the coarse level (as k_restrict): io.uc0 = R u, io.rc = R r.  Along an edge axis
//         the third tap of a coarse point lies one column (the next lane) or one row (the next
//         wave's first, traded through LDS) past the region.
typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));  // a pair at any 8-byte boundary

struct SweepShared {
    double2 xch[2][kSweepWaves][2][kTile];  // two buffers of each wave's first and last row
    double red[kSweepWaves];      // wave sums of the norm
};

// The entry of a PointCoef table for a point at an x wall (bx) and / or a y wall (by).
__device__ __forceinline__ double by_wall(bool bx, bool by, double v0, double v1, double v2, double v3)
{
    const double a = by ? v2 : v0, b = by ? v3 : v1;
    return bx ? b : a;
}

template <int NU, int LOC, bool CORR, bool NORM, bool RHS, bool RES, bool XE>
__device__ __forceinline__ void sweep_pass(const Lev& L, const PointCoef& P, const double* __restrict__ f,
                                           const double* __restrict__ uin, double* __restrict__ uout, int tx, int ty,
                                           const SweepIO& io, SweepShared& sh)
{
    constexpr SweepGeom G = sweep_geom(NU, CORR, NORM, RES);
    constexpr int WV = kSweepWaves, RPW = G.wy / WV, HX = G.hx, HY = G.hy, OX = G.ox, OY = G.oy;
    static_assert(HX % 2 == 0 && OX % 2 == 0 && OY % 2 == 0 && RPW % 2 == 0, "window geometry");
    static_assert(!RES || HY % 2 == 0, "2 x 2 blocks of the restriction");
    auto& xch = sh.xch;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int x0 = tx * OX - HX + 2 * lane;  // grid column of the lane's even column
    const int yw = ty * OY - HY + w * RPW;   // grid row of the wave's first row (parity of HY)
    const bool in0 = !XE || (x0 >= 0 && x0 < L.nx), in1 = !XE || (x0 + 1 >= 0 && x0 + 1 < L.nx);
    double u0[RPW], u1[RPW], f0[RPW], f1[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        const int gy = yw + i;
        const bool row = gy >= 0 && gy < L.ny;
        const size_t idx = (size_t)min(max(gy, 0), L.ny - 1) * L.nx;
        if constexpr (!XE) {
            const pair_t vu = *reinterpret_cast<const pair_t*>(uin + idx + x0);
            const pair_t vf = *reinterpret_cast<const pair_t*>(f + idx + x0);
            u0[i] = row ? vu.x : 0.0;
            u1[i] = row ? vu.y : 0.0;
            f0[i] = row ? vf.x : 0.0;
            f1[i] = row ? vf.y : 0.0;
        } else {
            const size_t a = idx + (in0 ? x0 : 0), b = idx + (in1 ? x0 + 1 : 0);
            const double v0 = uin[a], v1 = uin[b], g0 = f[a], g1 = f[b];
            u0[i] = row && in0 ? v0 : 0.0;
            u1[i] = row && in1 ? v1 : 0.0;
            f0[i] = row && in0 ? g0 : 0.0;
            f1[i] = row && in1 ? g1 : 0.0;
        }
    }
    if constexpr (CORR) {
        // the coarse values are loaded with the window, then P e is added row by row
        CorrTable<LOC, RPW> T;
        T.load(io.C, x0, yw);
        corr_rows<LOC, RPW, HY & 1>(T, io.C, yw, L.ny, in0, in1, u0, u1, std::make_integer_sequence<int, RPW>{});
    }
    // walls: of the two columns along x, of a row along y
    const bool bx0 = XE && (x0 == 0 || x0 == L.nx - 1), bx1 = XE && (x0 + 1 == 0 || x0 + 1 == L.nx - 1);
    const double D0 = P.D[0], D1 = P.D[1], D2 = P.D[2], D3 = P.D[3];
    const int ny = L.ny;
    auto D_at = [=](bool bx, int i) { return by_wall(XE && bx, yw + i == 0 || yw + i == ny - 1, D0, D1, D2, D3); };
    // The row above the wave's band (the next wave's first) and below it (the previous wave's
    // last), as they stand after the last half-sweep.  Exchange e writes buffer e & 1: a wave
    // can only overwrite a buffer after the next barrier, which every wave passes only once
    // it has read that buffer.
    double2 dn, up;
    auto exchange = [&](int e) {
        xch[e & 1][w][0][lane] = double2{u0[0], u1[0]};
        xch[e & 1][w][1][lane] = double2{u0[RPW - 1], u1[RPW - 1]};
        __syncthreads();
        dn = double2{0.0, 0.0};
        up = dn;
        if (w > 0) dn = xch[e & 1][w - 1][1][lane];
        if (w < WV - 1) up = xch[e & 1][w + 1][0][lane];
    };
    // neighbour sums of the even / odd point of row i
    auto sum_even = [&](int i) {
        const double S = i > 0 ? u0[i - 1] : dn.x, N = i < RPW - 1 ? u0[i + 1] : up.x;
        return (dpp_move<kShr1>(u1[i]) + u1[i]) + (S + N);
    };
    auto sum_odd = [&](int i) {
        const double S = i > 0 ? u1[i - 1] : dn.y, N = i < RPW - 1 ? u1[i + 1] : up.y;
        return (u0[i] + dpp_move<kShl1>(u0[i])) + (S + N);
    };
    auto Lu_even = [&](int i) { return (D_at(bx0, i) * u0[i] - L.c * sum_even(i)) * L.ih2; };
    auto Lu_odd = [&](int i) { return (D_at(bx1, i) * u1[i] - L.c * sum_odd(i)) * L.ih2; };
    exchange(0);
    if constexpr (RHS) {
        // f = r + L u from the values as loaded
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            f0[i] = f0[i] + Lu_even(i);
            f1[i] = f1[i] + Lu_odd(i);
        }
    }
#pragma unroll
    for (int hs = 0; hs < 2 * NU; ++hs) {
        if (hs > 0) exchange(hs);
        const int colour = (hs & 1) ^ 1;  // sets 1-2 (odd index sum) first
        double q[RPW];
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const bool odd = (colour + HY + i) & 1;  // the pair's column with this colour
            q[i] = (L.c * (odd ? sum_odd(i) : sum_even(i)) + L.h2 * (odd ? f1[i] : f0[i])) / D_at(odd ? bx1 : bx0, i);
        }
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const bool odd = (colour + HY + i) & 1;
            const bool row = yw + i >= 0 && yw + i < L.ny;
            if (odd)
                u1[i] = row && in1 ? q[i] : u1[i];
            else
                u0[i] = row && in0 ? q[i] : u0[i];
        }
    }
    if constexpr (NORM || RES) exchange(2 * NU);
    const bool colw = 2 * lane >= HX && 2 * lane < HX + OX;  // the lane's pair is written
    double acc = 0.0;
    if (colw) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int r = w * RPW + i, gy = yw + i;
            if (r < HY || r >= HY + OY || gy < 0 || gy >= L.ny) continue;
            const size_t o = (size_t)gy * L.nx + x0;
            if constexpr (!XE) {
                *reinterpret_cast<pair_t*>(uout + o) = pair_t{u0[i], u1[i]};
                if constexpr (RHS) *reinterpret_cast<pair_t*>(io.fout + o) = pair_t{f0[i], f1[i]};
            } else {
                if (in0) uout[o] = u0[i];
                if (in1) uout[o + 1] = u1[i];
                if constexpr (RHS) {
                    if (in0) io.fout[o] = f0[i];
                    if (in1) io.fout[o + 1] = f1[i];
                }
            }
        }
    }
    if constexpr (NORM || RES) {
        // residuals f - L u in place of f (right wherever every neighbour is final: the written
        // region and, with RES, one ring around it)
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            f0[i] = f0[i] - Lu_even(i);
            f1[i] = f1[i] - Lu_odd(i);
        }
    }
    if constexpr (NORM) {
        if (colw) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                const int r = w * RPW + i, gy = yw + i;
                if (r < HY || r >= HY + OY || gy < 0 || gy >= L.ny) continue;
                if (in0) acc = acc + f0[i] * f0[i];
                if (in1) acc = acc + f1[i] * f1[i];
            }
        }
        // fixed-order reduction: butterfly within each wave, then the wave sums in order
        for (int o = 32; o > 0; o >>= 1) acc = acc + __shfl_xor(acc, o, 64);
        if (lane == 0) sh.red[w] = acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = sh.red[0];
            for (int k = 1; k < WV; ++k) t = t + sh.red[k];
            io.partials[blockIdx.x] = t;
        }
    }
    if constexpr (RES) {
        // the third tap of an edge axis: the next lane's even column (EDGE_X), the next
        // wave's first row (EDGE_Y; its values of u are the row above the band)
        double nx0[RPW], nu0[RPW];
        double2 rup = double2{0.0, 0.0};
        if constexpr (LOC == LOC_EDGE_X) {
#pragma unroll
            for (int i = 0; i < RPW; ++i) {
                nx0[i] = dpp_move<kShl1>(f0[i]);
                nu0[i] = dpp_move<kShl1>(u0[i]);
            }
        }
        if constexpr (LOC == LOC_EDGE_Y) {
            constexpr int b = (2 * NU + 1) & 1;  // the buffer of the exchange before the last
            xch[b][w][0][lane] = double2{f0[0], f1[0]};
            __syncthreads();
            if (w < WV - 1) rup = xch[b][w + 1][0][lane];
        }
        if (colw) {
            const int K = x0 >> 1;  // x0 >= 0 here
#pragma unroll
            for (int p = 0; p < RPW / 2; ++p) {
                const int r = w * RPW + 2 * p, gy = yw + 2 * p;  // gy even
                if (r < HY || r >= HY + OY || gy < 0) continue;
                const int J = gy >> 1;
                if (J >= io.ncy || K >= io.ncx) continue;
                double ru, rr;
                if (LOC == LOC_CELL) {
                    ru = ((u0[2 * p] + u1[2 * p]) + (u0[2 * p + 1] + u1[2 * p + 1])) * 0.25;
                    rr = ((f0[2 * p] + f1[2 * p]) + (f0[2 * p + 1] + f1[2 * p + 1])) * 0.25;
                } else if (LOC == LOC_EDGE_X) {
                    const double gu0 = (u0[2 * p] + 2.0 * u1[2 * p]) + nu0[2 * p];
                    const double gu1 = (u0[2 * p + 1] + 2.0 * u1[2 * p + 1]) + nu0[2 * p + 1];
                    const double gr0 = (f0[2 * p] + 2.0 * f1[2 * p]) + nx0[2 * p];
                    const double gr1 = (f0[2 * p + 1] + 2.0 * f1[2 * p + 1]) + nx0[2 * p + 1];
                    ru = (gu0 + gu1) * 0.125;
                    rr = (gr0 + gr1) * 0.125;
                } else {
                    const bool last = 2 * p + 2 >= RPW;
                    const double v0 = last ? up.x : u0[(2 * p + 2) % RPW], v1 = last ? up.y : u1[(2 * p + 2) % RPW];
                    const double e2 = last ? rup.x : f0[(2 * p + 2) % RPW], o2 = last ? rup.y : f1[(2 * p + 2) % RPW];
                    const double gu0 = (u0[2 * p] + 2.0 * u0[2 * p + 1]) + v0;
                    const double gu1 = (u1[2 * p] + 2.0 * u1[2 * p + 1]) + v1;
                    const double gr0 = (f0[2 * p] + 2.0 * f0[2 * p + 1]) + e2;
                    const double gr1 = (f1[2 * p] + 2.0 * f1[2 * p + 1]) + o2;
                    ru = (gu0 + gu1) * 0.125;
                    rr = (gr0 + gr1) * 0.125;
                }
                const size_t c = (size_t)J * io.ncx + K;
                io.uc0[c] = ru;
                io.rc[c] = rr;
            }
        }
    }
}

template <int NU, int LOC, bool CORR, bool NORM, bool RHS, bool RES>
__global__ __launch_bounds__(64 * kSweepWaves) void k_sweep(Lev L, PointCoef P, const double* __restrict__ f,
                                               const double* __restrict__ uin, double* __restrict__ uout, int tiles_x,
                                               SweepIO io)
{
    constexpr SweepGeom G = sweep_geom(NU, CORR, NORM, RES);
    if (io.act && !io.act[0]) return;
    const unsigned b = xcd_block(blockIdx.x, gridDim.x);
    const int tx = (int)(b % (unsigned)tiles_x), ty = (int)(b / (unsigned)tiles_x);
    const int x0 = tx * G.ox - G.hx;
    __shared__ SweepShared sh;
    if (x0 <= 0 || x0 + 2 * kTile >= L.nx)
        sweep_pass<NU, LOC, CORR, NORM, RHS, RES, true>(L, P, f, uin, uout, tx, ty, io, sh);
    else
        sweep_pass<NU, LOC, CORR, NORM, RHS, RES, false>(L, P, f, uin, uout, tx, ty, io, sh);
}

// ---- persistent coarse tail ------------------------------------------------------------------
// One 512-thread workgroup runs the V-cycle of the coarsest levels (top .. coarsest) with
// every array in LDS: the top level's iterate and right-hand side are loaded once and the
// iterate is written back at the end, instead of five launches per level.  Each step uses
// the point formulas of the per-level kernels, so the result is the same bit for bit.
//
// One compute unit issues everything, so a half-sweep costs its instructions on the large
// levels and its latency chain on the small ones (the coarsest alone takes 32 half-sweeps).
// As in the cell-centred tail, a thread owns blocks of 2 x 2 points (the last of an odd axis
// is half a block whose missing points hold 0): half of a point's neighbours are the thread's
// registers, the others come from LDS planes (one per point of a block, indexed by block,
// index 0 a zero) at indices worked out once per visit of a level, and levels of at most 64
// blocks run in one wave without block barriers.  With a point per thread and step, all
// neighbours and diagonals worked out at each, 64^2 to 4^2 took 54.6 us (cells) and 59.5 us
// (edges); now 29.1 and 32.1 us.
constexpr int kTailThreads = 512;

__device__ __forceinline__ int div_by(int t, unsigned g) { return g ? (int)__umulhi((unsigned)t, g) : t; }

// A thread's block on one level; point c is (c & 1, c >> 1).
struct StagBlock {
    bool on;
    int o, I, J;
    int nb[4];       // LDS indices of the blocks at x-, x+, y-, y+ (0: outside)
    unsigned valid;  // points inside the level
    bool bx[2], by[2];  // the points at 0 / 1 along x and y lie at a wall
    double u[4], f[4], D[4];
};

template <int LOC, bool BIG>
struct StagTail {
    static constexpr int CAP = stag_tail_cap(BIG), CAP0 = stag_tail_cap0(BIG), KB = stag_tail_kb(BIG);
    static_assert((size_t)(8 * CAP + 4 * CAP0) * sizeof(double) <= 160 * 1024, "LDS of one workgroup");
    const TailArgs& a;
    double* const lds;

    __device__ __forceinline__ double* U(int c) const { return lds + c * CAP; }
    __device__ __forceinline__ double* F(int c) const { return lds + (4 + c) * CAP; }

    // Between steps that read what other threads wrote: a barrier, or inside one wave (whose
    // LDS accesses are in order) only the compiler's order.
    template <bool ONE>
    static __device__ __forceinline__ void sync()
    {
        if constexpr (ONE) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    }

    __device__ __forceinline__ void setup(const TailLev& L, int t, StagBlock& B) const
    {
        B.on = t < L.nb;
        if (!B.on) t = 0;
        B.J = div_by(t, L.g0);
        B.I = t - B.J * L.m0;
        B.o = L.off + t;
        B.nb[0] = B.I > 0 ? B.o - 1 : 0;
        B.nb[1] = B.I < L.m0 - 1 ? B.o + 1 : 0;
        B.nb[2] = B.J > 0 ? B.o - L.m0 : 0;
        B.nb[3] = B.J < L.m1 - 1 ? B.o + L.m0 : 0;
        const bool x1 = 2 * B.I + 1 < L.nx, y1 = 2 * B.J + 1 < L.ny;
        B.valid = 1u | (x1 ? 2u : 0u) | (y1 ? 4u : 0u) | (x1 && y1 ? 8u : 0u);
        B.bx[0] = B.I == 0 || 2 * B.I == L.nx - 1;
        B.bx[1] = 2 * B.I + 1 == L.nx - 1;
        B.by[0] = B.J == 0 || 2 * B.J == L.ny - 1;
        B.by[1] = 2 * B.J + 1 == L.ny - 1;
#pragma unroll
        for (int c = 0; c < 4; ++c) B.D[c] = by_wall(B.bx[c & 1], B.by[c >> 1], L.D[0], L.D[1], L.D[2], L.D[3]);
    }

    // Neighbour sum of point c: inside the block from registers, else from LDS.
    __device__ __forceinline__ double sum_of(const StagBlock& B, int c) const
    {
        const bool x = c & 1, y = c >> 1;
        const int ox = c ^ 1, oy = c ^ 2;
        const double W = x ? B.u[ox] : U(ox)[B.nb[0]], E = x ? U(ox)[B.nb[1]] : B.u[ox];
        const double S = y ? B.u[oy] : U(oy)[B.nb[2]], N = y ? U(oy)[B.nb[3]] : B.u[oy];
        return (W + E) + (S + N);
    }
    __device__ __forceinline__ double Lu(const TailLev& L, const StagBlock& B, int c) const
    {
        return (B.D[c] * B.u[c] - L.c * sum_of(B, c)) * L.ih2;
    }

    // One half-sweep: the points of index-sum parity P.
    template <int P>
    __device__ __forceinline__ void phase(const TailLev& L, StagBlock& B) const
    {
        constexpr int c0 = P, c1 = 3 - P;  // (P, 0) and (1 - P, 1)
        const double v0 = (L.c * sum_of(B, c0) + L.h2 * B.f[c0]) / B.D[c0];
        const double v1 = (L.c * sum_of(B, c1) + L.h2 * B.f[c1]) / B.D[c1];
        B.u[c0] = B.valid >> c0 & 1 ? v0 : 0.0;
        B.u[c1] = B.valid >> c1 & 1 ? v1 : 0.0;
        U(c0)[B.o] = B.u[c0];
        U(c1)[B.o] = B.u[c1];
    }

    template <int NB, bool ONE>
    __device__ __forceinline__ void smooth(const TailLev& L, StagBlock (&B)[NB], int nu) const
    {
        for (int s = 0; s < nu; ++s) {
            // sets 1-2 (odd index sum) first
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (B[k].on) phase<1>(L, B[k]);
            sync<ONE>();
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (B[k].on) phase<0>(L, B[k]);
            sync<ONE>();
        }
    }

    // LDS plane offset and index of coarse point (K, J).
    static __device__ __forceinline__ int cell_of(int K, int J) { return (K & 1) + 2 * (J & 1); }
    static __device__ __forceinline__ int index_of(const TailLev& Lc, int K, int J)
    {
        return (K >> 1) + Lc.m0 * (J >> 1);
    }

    // Own points of every block: from LDS, or on the top level (gu != nullptr) from memory into
    // registers and LDS.  Points that are not there become 0 in both.
    template <int NB, bool ONE>
    __device__ __forceinline__ void load(const TailLev& L, StagBlock (&B)[NB], const double* gu, const double* gf) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) setup(L, (int)threadIdx.x + k * kTailThreads, B[k]);
        if (gu) {
            // every load of the thread is issued before the first use (missing points and
            // blocks read a point that is there)
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int x = 2 * B[k].I + (B[k].valid & 2 ? c & 1 : 0), y = 2 * B[k].J + (B[k].valid & 4 ? c >> 1 : 0);
                    B[k].u[c] = gu[y * L.nx + x];
                    B[k].f[c] = gf[y * L.nx + x];
                }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (!gu) {
                    B[k].u[c] = U(c)[B[k].o];
                    B[k].f[c] = F(c)[B[k].o];
                }
                const bool in = B[k].valid >> c & 1;
                B[k].u[c] = in ? B[k].u[c] : 0.0;
                B[k].f[c] = in ? B[k].f[c] : 0.0;
                if (gu || !in) {
                    U(c)[B[k].o] = B[k].u[c];
                    F(c)[B[k].o] = B[k].f[c];
                }
            }
        }
        if (gu) sync<ONE>();
    }

    // f = r + L u in place (the level's f holds r).
    template <int NB, bool ONE>
    __device__ __forceinline__ void form(const TailLev& L, StagBlock (&B)[NB]) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                B[k].f[c] = B[k].f[c] + Lu(L, B[k], c);
                F(c)[B[k].o] = B[k].f[c];
            }
        }
        sync<ONE>();
    }

    // Down: pre-smoothing, then the restricted iterate and residual (as restrict_point).
    template <int NB, bool ONE>
    __device__ __forceinline__ void down(int lv, const double* gu, const double* gf) const
    {
        const TailLev& L = a.lev[lv];
        const TailLev& Lc = a.lev[lv + 1];
        StagBlock B[NB];
        load<NB, ONE>(L, B, gu, gf);
        if (lv > 0 || a.r) form<NB, ONE>(L, B);
        smooth<NB, ONE>(L, B, a.nu1);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on || B[k].I >= Lc.nx || B[k].J >= Lc.ny) continue;
            const StagBlock& b = B[k];
            double r[4], ru, rr;
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = b.f[c] - Lu(L, b, c);
            if constexpr (LOC == LOC_CELL) {
                ru = ((b.u[0] + b.u[1]) + (b.u[2] + b.u[3])) * 0.25;
                rr = ((r[0] + r[1]) + (r[2] + r[3])) * 0.25;
            } else if constexpr (LOC == LOC_EDGE_X) {
                // the third tap: the first column of the block at x+
                const int R = b.nb[1], Rm = b.nb[2] ? R - L.m0 : 0, Rp = b.nb[3] ? R + L.m0 : 0;
                const bool wall = 2 * b.I + 2 == L.nx - 1;
                double u2[2] = {U(0)[R], U(2)[R]}, r2[2];
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    const double D = by_wall(wall, b.by[y], L.D[0], L.D[1], L.D[2], L.D[3]);
                    const double s = (b.u[1 + 2 * y] + U(1 + 2 * y)[R]) +
                                     (y ? u2[0] + U(0)[Rp] : U(2)[Rm] + u2[1]);
                    r2[y] = F(2 * y)[R] - (D * u2[y] - L.c * s) * L.ih2;
                }
                ru = (((b.u[0] + 2.0 * b.u[1]) + u2[0]) + ((b.u[2] + 2.0 * b.u[3]) + u2[1])) * 0.125;
                rr = (((r[0] + 2.0 * r[1]) + r2[0]) + ((r[2] + 2.0 * r[3]) + r2[1])) * 0.125;
            } else {
                // the third tap: the first row of the block at y+
                const int A = b.nb[3], Am = b.nb[0] ? A - 1 : 0, Ap = b.nb[1] ? A + 1 : 0;
                const bool wall = 2 * b.J + 2 == L.ny - 1;
                double u2[2] = {U(0)[A], U(1)[A]}, r2[2];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const double D = by_wall(b.bx[x], wall, L.D[0], L.D[1], L.D[2], L.D[3]);
                    const double s = (x ? u2[0] + U(0)[Ap] : U(1)[Am] + u2[1]) + (b.u[x + 2] + U(x + 2)[A]);
                    r2[x] = F(x)[A] - (D * u2[x] - L.c * s) * L.ih2;
                }
                ru = (((b.u[0] + 2.0 * b.u[2]) + u2[0]) + ((b.u[1] + 2.0 * b.u[3]) + u2[1])) * 0.125;
                rr = (((r[0] + 2.0 * r[2]) + r2[0]) + ((r[1] + 2.0 * r[3]) + r2[1])) * 0.125;
            }
            const int c = cell_of(b.I, b.J), p = index_of(Lc, b.I, b.J);
            U(c)[Lc.off + p] = ru;
            lds[8 * CAP + c * CAP0 + Lc.off0 + p] = ru;
            F(c)[Lc.off + p] = rr;
        }
        sync<ONE>();
    }

    template <int NB, bool ONE>
    __device__ __forceinline__ void coarsest(const double* gu, const double* gf, double* gout) const
    {
        const TailLev& L = a.lev[a.nlev - 1];
        StagBlock B[NB];
        load<NB, ONE>(L, B, gu, gf);
        if (a.nlev > 1 || a.r) form<NB, ONE>(L, B);
        smooth<NB, ONE>(L, B, a.nuc);  // Remark 1
        if (gout) store<NB>(L, B, gout);
    }

    // Up: u += P (u_c - R u) (as prolong_point), post-smoothing.
    template <int NB, bool ONE>
    __device__ __forceinline__ void up(int lv, double* gout) const
    {
        const TailLev& L = a.lev[lv];
        const TailLev& Lc = a.lev[lv + 1];
        StagBlock B[NB];
        load<NB, ONE>(L, B, nullptr, nullptr);
        // e = uc - uc0 (out of range: a value that is not used)
        auto e = [&](int K, int J) {
            K = min(max(K, 0), Lc.nx - 1);
            J = min(max(J, 0), Lc.ny - 1);
            const int c = cell_of(K, J), p = index_of(Lc, K, J);
            return lds[c * CAP + Lc.off + p] - lds[8 * CAP + c * CAP0 + Lc.off0 + p];
        };
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
            const int K = B[k].I, J = B[k].J;
            double p[4];
            if constexpr (LOC == LOC_CELL) {
                p[0] = p[1] = p[2] = p[3] = e(K, J);
            } else if constexpr (LOC == LOC_EDGE_X) {
                const double e0 = e(K, J), m = e(K - 1, J);
                const double em = J > 0 ? e(K, J - 1) : -e0, mm = J > 0 ? e(K - 1, J - 1) : -m;
                const double ep = J < Lc.ny - 1 ? e(K, J + 1) : -e0, mp = J < Lc.ny - 1 ? e(K - 1, J + 1) : -m;
                const bool l = K >= 1, r = K <= Lc.nx - 1;
                p[1] = lin_cell(e0, em);
                p[3] = lin_cell(e0, ep);
                p[0] = ((l ? lin_cell(m, mm) : 0.0) + (r ? p[1] : 0.0)) * 0.5;
                p[2] = ((l ? lin_cell(m, mp) : 0.0) + (r ? p[3] : 0.0)) * 0.5;
            } else {
                const double e0 = e(K, J), m = e(K, J - 1);
                const double em = K > 0 ? e(K - 1, J) : -e0, mm = K > 0 ? e(K - 1, J - 1) : -m;
                const double ep = K < Lc.nx - 1 ? e(K + 1, J) : -e0, mp = K < Lc.nx - 1 ? e(K + 1, J - 1) : -m;
                const bool b = J >= 1, t = J <= Lc.ny - 1;
                p[2] = lin_cell(e0, em);
                p[3] = lin_cell(e0, ep);
                p[0] = ((b ? lin_cell(m, mm) : 0.0) + (t ? p[2] : 0.0)) * 0.5;
                p[1] = ((b ? lin_cell(m, mp) : 0.0) + (t ? p[3] : 0.0)) * 0.5;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                B[k].u[c] = B[k].valid >> c & 1 ? B[k].u[c] + p[c] : 0.0;
                U(c)[B[k].o] = B[k].u[c];
            }
        }
        sync<ONE>();
        smooth<NB, ONE>(L, B, a.nu2);
        if (gout) store<NB>(L, B, gout);
    }

    template <int NB>
    __device__ __forceinline__ void store(const TailLev& L, StagBlock (&B)[NB], double* gout) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (B[k].valid >> c & 1) gout[(2 * B[k].J + (c >> 1)) * L.nx + 2 * B[k].I + (c & 1)] = B[k].u[c];
        }
    }

    __device__ __forceinline__ void run() const
    {
        const int last = a.nlev - 1;
        const double* const gf = a.r ? a.r : a.f;
        if (threadIdx.x < 4) U((int)threadIdx.x)[0] = 0.0;
        __syncthreads();
        // blocks per level fall, so one wave runs the levels from a.one on
        for (int l = 0; l < a.one && l < last; ++l) down<KB, false>(l, l ? nullptr : a.uin, gf);
        if (a.one < a.nlev) {
            if (threadIdx.x < 64) {
                for (int l = a.one; l < last; ++l) down<1, true>(l, l ? nullptr : a.uin, gf);
                coarsest<1, true>(last ? nullptr : a.uin, gf, last ? nullptr : a.u);
                for (int l = last - 1; l >= a.one; --l) up<1, true>(l, l ? nullptr : a.u);
            }
            __syncthreads();
        } else {
            coarsest<KB, false>(last ? nullptr : a.uin, gf, last ? nullptr : a.u);
        }
        for (int l = (a.one < last ? a.one : last) - 1; l >= 0; --l) up<KB, false>(l, l ? nullptr : a.u);
    }
};

template <int LOC, bool BIG>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs args)
{
    // levels are picked at run time: read the arguments where they are, as constants (a copy
    // would go through scratch)
    (void)args;
    const TailArgs& a =
        *(const TailArgs*)(const __attribute__((address_space(4))) TailArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    if (a.act && !a.act[0]) return;
    using Tl = StagTail<LOC, BIG>;
    __shared__ double lds[8 * Tl::CAP + 4 * Tl::CAP0];
    const Tl tail{a, lds};
    tail.run();
}

// ---- residual norm -------------------------------------------------------------------------
__device__ __forceinline__ double block_sum(double v, double* sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + o];
        __syncthreads();
    }
    return sh[0];
}

__global__ __launch_bounds__(256) void k_resnorm(Lev L, const double* __restrict__ f, const double* __restrict__ u,
                                                 double* __restrict__ r, double* __restrict__ partials)
{
    __shared__ double sh[256];
    const int64_t n = (int64_t)L.nx * L.ny;
    double acc = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) {
        const int x = (int)(t % L.nx), y = (int)(t / L.nx);
        const double rv = resid_at(L, f, u, x, y);
        if (r) r[t] = rv;
        acc = acc + rv * rv;
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void k_sum(const double* __restrict__ partials, int n, double* __restrict__ out)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc = acc + partials[i];
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) out[0] = s;
}

// The norm of cycle k and the stopping test (Status).  1024 threads with four loads in flight
// each: the few thousand sums of a 4096^2 launch took 9.7 us with 256 threads.
__global__ __launch_bounds__(1024) void k_status(const double* __restrict__ partials, int n, double s2max, int k,
                                                 int* __restrict__ act, Status* host)
{
    if (k > 0 && !act[0]) return;
    __shared__ double sh[1024];
    double acc = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += 1024) acc = acc + partials[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] = sh[threadIdx.x] + sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double s2 = sh[0];
    const bool active = isfinite(s2) && s2 > s2max;
    act[0] = active ? 1 : 0;
    // (not ordered, as a release to the host would write the L2 back: the host reads s2 once the
    // stream has ended)
    __hip_atomic_store(&host->s2, s2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host->seen, status_word(k, active), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void k_copy(const double* __restrict__ src, double* __restrict__ dst, int64_t n)
{
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) dst[t] = src[t];
}

// ---- projection step ------------------------------------------------------------------------
constexpr double kWenoEps = 1e-6;

// Third-order WENO derivatives (Hamilton-Jacobi form, Jiang-Shu smoothness ratio) at the
// centre of five values along one axis: the left-biased phi^- and the right-biased phi^+.
__device__ __forceinline__ void weno_pair(double pm2, double pm1, double p0, double pp1, double pp2, double ih,
                                          double& minus, double& plus)
{
    const double d0 = pm1 - pm2, d1 = p0 - pm1, d2 = pp1 - p0;
    const double rm = (kWenoEps + (d1 - d0) * (d1 - d0)) / (kWenoEps + (d2 - d1) * (d2 - d1));
    const double wm = 1.0 / (1.0 + 2.0 * (rm * rm));
    minus = ((d1 + d2) - wm * ((d0 - 2.0 * d1) + d2)) * (0.5 * ih);
    const double e0 = pp2 - pp1, e1 = pp1 - p0, e2 = p0 - pm1;
    const double rp = (kWenoEps + (e1 - e0) * (e1 - e0)) / (kWenoEps + (e2 - e1) * (e2 - e1));
    const double wp = 1.0 / (1.0 + 2.0 * (rp * rp));
    plus = ((e1 + e2) - wp * ((e0 - 2.0 * e1) + e2)) * (0.5 * ih);
}

// Branch-free upwinding: max(a, 0) phi^- + min(a, 0) phi^+.
__device__ __forceinline__ double upwind(double a, double minus, double plus)
{
    return (a > 0.0 ? a : 0.0) * minus + (a < 0.0 ? a : 0.0) * plus;
}

__device__ __forceinline__ double forcing(const NsArgs& A, const double* const* F, size_t i)
{
    double s = 0.0;
    for (int k = 0; k < A.nforce; ++k) s = k == 0 ? A.coef[0] * F[0][i] : s + A.coef[k] * F[k][i];
    return s;
}

// u extended by two layers beyond each wall: wall points x = 0, 1 hold 0, their odd
// reflections beyond; along y cell-type ghosts 2 g - mirror (g = 0 below, lid above).
__device__ __forceinline__ double u_ext(const double* u, int m, int ny, int a, int b, double lid)
{
    if (b >= 0 && b < ny) {
        if (a >= 0 && a < m) return u[(size_t)b * m + a];
        if (a == -1 || a == m) return 0.0;
        if (a == -2) return 2.0 * 0.0 - u[(size_t)b * m];
        return 2.0 * 0.0 - u[(size_t)b * m + m - 1];  // a == m + 1
    }
    if (b == -1) return 2.0 * 0.0 - u[a];
    if (b == -2) return 2.0 * 0.0 - u[(size_t)m + a];
    if (b == ny) return 2.0 * lid - u[(size_t)(ny - 1) * m + a];
    return 2.0 * lid - u[(size_t)(ny - 2) * m + a];  // b == ny + 1
}

// v extended likewise: wall points y = 0, 1 hold 0 with odd reflections beyond; along x
// cell-type ghosts 2 * 0 - mirror.
__device__ __forceinline__ double v_ext(const double* v, int nx, int m, int ii, int jj)
{
    if (ii >= 0 && ii < nx) {
        if (jj >= 0 && jj < m) return v[(size_t)jj * nx + ii];
        if (jj == -1 || jj == m) return 0.0;
        if (jj == -2) return 2.0 * 0.0 - v[ii];
        return 2.0 * 0.0 - v[(size_t)(m - 1) * nx + ii];  // jj == m + 1
    }
    if (ii == -1) return 2.0 * 0.0 - v[(size_t)jj * nx];
    if (ii == -2) return 2.0 * 0.0 - v[(size_t)jj * nx + 1];
    if (ii == nx) return 2.0 * 0.0 - v[(size_t)jj * nx + nx - 1];
    return 2.0 * 0.0 - v[(size_t)jj * nx + nx - 2];  // ii == nx + 1
}

__global__ __launch_bounds__(256) void k_rhs_u(NsArgs A, const double* __restrict__ u, const double* __restrict__ v,
                                               const double* __restrict__ p, double* __restrict__ fu)
{
    const int m = A.nx - 1, ny = A.ny;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)m * ny) return;
    const int a = (int)(t % m), b = (int)(t / m);
    const double u0 = u[t];
    double xm, xp, ym, yp;
    weno_pair(u_ext(u, m, ny, a - 2, b, A.lid), u_ext(u, m, ny, a - 1, b, A.lid), u0,
              u_ext(u, m, ny, a + 1, b, A.lid), u_ext(u, m, ny, a + 2, b, A.lid), A.ih, xm, xp);
    weno_pair(u_ext(u, m, ny, a, b - 2, A.lid), u_ext(u, m, ny, a, b - 1, A.lid), u0,
              u_ext(u, m, ny, a, b + 1, A.lid), u_ext(u, m, ny, a, b + 2, A.lid), A.ih, ym, yp);
    // mean of the four v around the point (wall values 0 below the first, above the last row)
    const int nx = A.nx;
    const double sW = b > 0 ? v[(size_t)(b - 1) * nx + a] : 0.0;
    const double sE = b > 0 ? v[(size_t)(b - 1) * nx + a + 1] : 0.0;
    const double nW = b < ny - 1 ? v[(size_t)b * nx + a] : 0.0;
    const double nE = b < ny - 1 ? v[(size_t)b * nx + a + 1] : 0.0;
    const double vbar = ((sW + sE) + (nW + nE)) * 0.25;
    const double conv = upwind(u0, xm, xp) + upwind(vbar, ym, yp);
    const double gp = (p[(size_t)b * nx + a + 1] - p[(size_t)b * nx + a]) * A.ih;
    const double F = forcing(A, A.fu, (size_t)t);
    double r = u0 + A.dt * ((F - conv) - gp);
    if (b == ny - 1) r = r + A.lift;
    fu[t] = r;
}

__global__ __launch_bounds__(256) void k_rhs_v(NsArgs A, const double* __restrict__ u, const double* __restrict__ v,
                                               const double* __restrict__ p, double* __restrict__ fv)
{
    const int nx = A.nx, m = A.ny - 1;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)m * nx) return;
    const int ii = (int)(t % nx), jj = (int)(t / nx);
    const double v0 = v[t];
    double xm, xp, ym, yp;
    weno_pair(v_ext(v, nx, m, ii - 2, jj), v_ext(v, nx, m, ii - 1, jj), v0, v_ext(v, nx, m, ii + 1, jj),
              v_ext(v, nx, m, ii + 2, jj), A.ih, xm, xp);
    weno_pair(v_ext(v, nx, m, ii, jj - 2), v_ext(v, nx, m, ii, jj - 1), v0, v_ext(v, nx, m, ii, jj + 1),
              v_ext(v, nx, m, ii, jj + 2), A.ih, ym, yp);
    // mean of the four u around the point (wall values 0 left of the first, right of the
    // last column)
    const int mu = nx - 1;
    const double sW = ii > 0 ? u[(size_t)jj * mu + ii - 1] : 0.0;
    const double sE = ii < nx - 1 ? u[(size_t)jj * mu + ii] : 0.0;
    const double nW = ii > 0 ? u[(size_t)(jj + 1) * mu + ii - 1] : 0.0;
    const double nE = ii < nx - 1 ? u[(size_t)(jj + 1) * mu + ii] : 0.0;
    const double ubar = ((sW + sE) + (nW + nE)) * 0.25;
    const double conv = upwind(ubar, xm, xp) + upwind(v0, ym, yp);
    const double gp = (p[(size_t)(jj + 1) * nx + ii] - p[(size_t)jj * nx + ii]) * A.ih;
    const double F = forcing(A, A.fv, (size_t)t);
    fv[t] = v0 + A.dt * ((F - conv) - gp);
}

__global__ __launch_bounds__(256) void k_neg_div(NsArgs A, const double* __restrict__ ut, const double* __restrict__ vt,
                                                 double* __restrict__ fp)
{
    const int nx = A.nx, ny = A.ny;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nx * ny) return;
    const int i = (int)(t % nx), j = (int)(t / nx);
    const int mu = nx - 1;
    const double uW = i > 0 ? ut[(size_t)j * mu + i - 1] : 0.0;
    const double uE = i < nx - 1 ? ut[(size_t)j * mu + i] : 0.0;
    const double vS = j > 0 ? vt[(size_t)(j - 1) * nx + i] : 0.0;
    const double vN = j < ny - 1 ? vt[(size_t)j * nx + i] : 0.0;
    fp[t] = -(((uE - uW) + (vN - vS)) * A.ih);
}

__global__ __launch_bounds__(256) void k_project(NsArgs A, const double* __restrict__ ut, const double* __restrict__ vt,
                                                 const double* __restrict__ pt, const double* p_in,
                                                 double* __restrict__ u_out, double* __restrict__ v_out,
                                                 double* p_out)
{
    const int nx = A.nx, ny = A.ny;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)nx * ny) return;
    const int i = (int)(t % nx), j = (int)(t / nx);
    const double pc = pt[t];
    if (i < nx - 1) {
        const size_t k = (size_t)j * (nx - 1) + i;
        u_out[k] = ut[k] - A.dt * ((pt[t + 1] - pc) * A.ih);
    }
    if (j < ny - 1) v_out[t] = vt[t] - A.dt * ((pt[t + nx] - pc) * A.ih);
    p_out[t] = p_in[t] + pc;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

template <int NU, int LOC, bool CORR, bool NORM, bool RHS, bool RES>
void sweep_go(hipStream_t s, dim3 grid, const Lev& L, const double* f, const double* uin, double* uout, int tx,
              const SweepIO& io)
{
    hipLaunchKernelGGL((k_sweep<NU, LOC, CORR, NORM, RHS, RES>), grid, dim3(64 * kSweepWaves), 0, s, L, point_coef(L), f, uin, uout,
                       tx, io);
}

template <int NU, int LOC>
void sweep_flags(hipStream_t s, dim3 grid, const Lev& L, const double* f, const double* uin, double* uout, int tx,
                 const SweepIO& io, unsigned flags)
{
    switch (flags) {
    case 0: sweep_go<NU, LOC_CELL, false, false, false, false>(s, grid, L, f, uin, uout, tx, io); break;
    case SW_CORR: sweep_go<NU, LOC, true, false, false, false>(s, grid, L, f, uin, uout, tx, io); break;
    case SW_CORR | SW_NORM: sweep_go<NU, LOC, true, true, false, false>(s, grid, L, f, uin, uout, tx, io); break;
    case SW_RHS: sweep_go<NU, LOC_CELL, false, false, true, false>(s, grid, L, f, uin, uout, tx, io); break;
    case SW_RES: sweep_go<NU, LOC, false, false, false, true>(s, grid, L, f, uin, uout, tx, io); break;
    case SW_RHS | SW_RES: sweep_go<NU, LOC, false, false, true, true>(s, grid, L, f, uin, uout, tx, io); break;
    default: throw Error(FAS_ERR_ARG, "internal: unsupported sweep variant");
    }
}

PointCoef point_coef(const Lev& L)
{
    auto shift = [](int kind) { return kind == K_CN ? -1.0 : (kind == K_CD ? 1.0 : 0.0); };
    PointCoef P;
    for (int i = 0; i < 4; ++i) {
        const double k = 4.0 + (i & 1 ? shift(L.kx) : 0.0) + (i & 2 ? shift(L.ky) : 0.0);
        P.D[i] = L.a * L.h2 + L.c * k;
    }
    return P;
}

int sweep_blocks(const Lev& L, int nu, unsigned flags, int* tiles_x)
{
    const SweepGeom g = sweep_geom(nu, (flags & SW_CORR) != 0, (flags & SW_NORM) != 0, (flags & SW_RES) != 0);
    const int tx = (L.nx + g.ox - 1) / g.ox, ty = (L.ny + g.oy - 1) / g.oy;
    if (tiles_x) *tiles_x = tx;
    return tx * ty;
}

int launch_sweep(hipStream_t s, int loc, const Lev& L, int nu, const double* f, const double* uin, double* uout,
                 const SweepIO& io, unsigned flags)
{
    int tx;
    const int nb = sweep_blocks(L, nu, flags, &tx);
    const dim3 grid(nb);
    if (loc == LOC_CELL) {
        if (nu == 1) sweep_flags<1, LOC_CELL>(s, grid, L, f, uin, uout, tx, io, flags);
        else sweep_flags<2, LOC_CELL>(s, grid, L, f, uin, uout, tx, io, flags);
    } else if (loc == LOC_EDGE_X) {
        if (nu == 1) sweep_flags<1, LOC_EDGE_X>(s, grid, L, f, uin, uout, tx, io, flags);
        else sweep_flags<2, LOC_EDGE_X>(s, grid, L, f, uin, uout, tx, io, flags);
    } else {
        if (nu == 1) sweep_flags<1, LOC_EDGE_Y>(s, grid, L, f, uin, uout, tx, io, flags);
        else sweep_flags<2, LOC_EDGE_Y>(s, grid, L, f, uin, uout, tx, io, flags);
    }
    return nb;
}

void launch_form_rhs(hipStream_t s, const Lev& L, const double* r, const double* u, double* f)
{
    hipLaunchKernelGGL(k_form_rhs, dim3(blocks_for((int64_t)L.nx * L.ny)), dim3(256), 0, s, L, r, u, f);
}

void launch_status(hipStream_t s, const double* partials, int n, double s2max, int k, int* act, Status* host)
{
    hipLaunchKernelGGL(k_status, dim3(1), dim3(1024), 0, s, partials, n, s2max, k, act, host);
}

TailLev tail_lev(const Lev& L)
{
    TailLev T{};
    T.nx = L.nx;
    T.ny = L.ny;
    T.m0 = (L.nx + 1) / 2;
    T.m1 = (L.ny + 1) / 2;
    T.nb = T.m0 * T.m1;
    T.g0 = T.m0 > 1 ? (unsigned)((((uint64_t)1 << 32) + (uint64_t)T.m0 - 1) / (uint64_t)T.m0) : 0u;
    T.c = L.c;
    T.h2 = L.h2;
    T.ih2 = L.ih2;
    const PointCoef P = point_coef(L);
    for (int i = 0; i < 4; ++i) T.D[i] = P.D[i];
    return T;
}

// LDS layout of the levels in A.lev (their off, off0) and the first level one wave runs;
// returns whether it takes the small (0) or the big (1) planes, or -1 when neither hold it.
namespace {
int tail_class(TailArgs& A)
{
    int off = 1, off0 = 0;  // block 0: the zeros outside the grid
    A.one = A.nlev;
    for (int k = 0; k < A.nlev; ++k) {
        A.lev[k].off = off;
        A.lev[k].off0 = off0;
        off += A.lev[k].nb;
        if (k > 0) off0 += A.lev[k].nb;  // the top level keeps no restricted copy
        if (A.lev[k].nb <= 64 && A.one == A.nlev) A.one = k;
    }
    for (int big = 0; big < 2; ++big)
        if (off <= stag_tail_cap(big) && off0 <= stag_tail_cap0(big) &&
            A.lev[0].nb <= kTailThreads * stag_tail_kb(big))
            return big;
    return -1;
}
}  // namespace

bool tail_fits(const int* nx, const int* ny, int nlev)
{
    TailArgs A{};
    A.nlev = nlev;
    for (int k = 0; k < nlev; ++k) {
        Lev L{};
        L.nx = nx[k];
        L.ny = ny[k];
        A.lev[k] = tail_lev(L);
    }
    return tail_class(A) >= 0;
}

void launch_tail(hipStream_t s, int loc, TailArgs& A)
{
    const int big = tail_class(A);
    if (big < 0) throw Error(FAS_ERR_ARG, "internal: tail levels exceed the tail's LDS");
#define FAS_STAG_TAIL(LOC_)                                                                              \
    do {                                                                                                 \
        if (big)                                                                                         \
            hipLaunchKernelGGL((k_tail<LOC_, true>), dim3(1), dim3(kTailThreads), 0, s, A);              \
        else                                                                                             \
            hipLaunchKernelGGL((k_tail<LOC_, false>), dim3(1), dim3(kTailThreads), 0, s, A);             \
    } while (0)
    if (loc == LOC_CELL)
        FAS_STAG_TAIL(LOC_CELL);
    else if (loc == LOC_EDGE_X)
        FAS_STAG_TAIL(LOC_EDGE_X);
    else
        FAS_STAG_TAIL(LOC_EDGE_Y);
#undef FAS_STAG_TAIL
}

void launch_restrict(hipStream_t s, int loc, const Lev& Lf, const double* f, const double* u, int ncx, int ncy,
                     double* uc, double* uc0, double* rc)
{
    const unsigned nb = blocks_for((int64_t)ncx * ncy);
    if (loc == LOC_CELL)
        hipLaunchKernelGGL(k_restrict<LOC_CELL>, dim3(nb), dim3(256), 0, s, Lf, f, u, ncx, ncy, uc, uc0, rc);
    else if (loc == LOC_EDGE_X)
        hipLaunchKernelGGL(k_restrict<LOC_EDGE_X>, dim3(nb), dim3(256), 0, s, Lf, f, u, ncx, ncy, uc, uc0, rc);
    else
        hipLaunchKernelGGL(k_restrict<LOC_EDGE_Y>, dim3(nb), dim3(256), 0, s, Lf, f, u, ncx, ncy, uc, uc0, rc);
}

void launch_coarse_rhs(hipStream_t s, const Lev& Lc, double* f, const double* u)
{
    hipLaunchKernelGGL(k_coarse_rhs, dim3(blocks_for((int64_t)Lc.nx * Lc.ny)), dim3(256), 0, s, Lc, f, u);
}

void launch_correct(hipStream_t s, int loc, const Lev& Lf, const double* uc, const double* uc0, int ncx, int ncy,
                    const double* usrc, double* udst)
{
    const Coarse C{uc, uc0, ncx, ncy};
    const unsigned nb = blocks_for((int64_t)Lf.nx * Lf.ny);
    if (loc == LOC_CELL)
        hipLaunchKernelGGL(k_correct<LOC_CELL>, dim3(nb), dim3(256), 0, s, Lf, C, usrc, udst);
    else if (loc == LOC_EDGE_X)
        hipLaunchKernelGGL(k_correct<LOC_EDGE_X>, dim3(nb), dim3(256), 0, s, Lf, C, usrc, udst);
    else
        hipLaunchKernelGGL(k_correct<LOC_EDGE_Y>, dim3(nb), dim3(256), 0, s, Lf, C, usrc, udst);
}

int launch_resnorm_partials(hipStream_t s, const Lev& L, const double* f, const double* u, double* r, double* partials)
{
    const int64_t n = (int64_t)L.nx * L.ny;
    const int nb = (int)std::min<int64_t>(kNormBlocks, (n + 255) / 256);
    hipLaunchKernelGGL(k_resnorm, dim3(nb), dim3(256), 0, s, L, f, u, r, partials);
    return nb;
}

void launch_resnorm(hipStream_t s, const Lev& L, const double* f, const double* u, double* r, double* partials,
                    double* out)
{
    const int nb = launch_resnorm_partials(s, L, f, u, r, partials);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, partials, nb, out);
}

void launch_copy(hipStream_t s, const double* src, double* dst, int64_t n)
{
    const unsigned nb = (unsigned)std::min<int64_t>(4096, (n + 255) / 256);
    hipLaunchKernelGGL(k_copy, dim3(nb), dim3(256), 0, s, src, dst, n);
}

void launch_rhs_u(hipStream_t s, const NsArgs& a, const double* u, const double* v, const double* p, double* fu)
{
    hipLaunchKernelGGL(k_rhs_u, dim3(blocks_for((int64_t)(a.nx - 1) * a.ny)), dim3(256), 0, s, a, u, v, p, fu);
}

void launch_rhs_v(hipStream_t s, const NsArgs& a, const double* u, const double* v, const double* p, double* fv)
{
    hipLaunchKernelGGL(k_rhs_v, dim3(blocks_for((int64_t)a.nx * (a.ny - 1))), dim3(256), 0, s, a, u, v, p, fv);
}

void launch_neg_div(hipStream_t s, const NsArgs& a, const double* ut, const double* vt, double* fp)
{
    hipLaunchKernelGGL(k_neg_div, dim3(blocks_for((int64_t)a.nx * a.ny)), dim3(256), 0, s, a, ut, vt, fp);
}

void launch_project(hipStream_t s, const NsArgs& a, const double* ut, const double* vt, const double* pt,
                    const double* p_in, double* u_out, double* v_out, double* p_out)
{
    hipLaunchKernelGGL(k_project, dim3(blocks_for((int64_t)a.nx * a.ny)), dim3(256), 0, s, a, ut, vt, pt, p_in, u_out,
                       v_out, p_out);
}

}  // namespace stag
}  // namespace fas
