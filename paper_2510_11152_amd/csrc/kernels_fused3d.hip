// Fused 3D plane-march kernels for large levels (constant kappa): one or two X-MCGS
// sweeps (each both colour phases, Appendix B sets 1-4 then 5-8) per pass, fused with the
// residual and restriction, or with the prolongation correction, or with the residual norm.
//
// Geometry.  A block owns an x-y tile of 64 columns and 2 TR rows (thread (px, py) holds the
// cell pair 2px, 2px+1 of rows 2py and 2py+1) and marches along z through a segment of planes,
// keeping a ring of planes in registers.  x-neighbours come from the adjacent lane by a
// DPP shift (a wavefront holds two row pairs; the lanes where the shift crosses rows are
// halo columns), y-neighbours from the thread's other row or through a double-buffered LDS
// exchange (one barrier per plane), z-neighbours from the ring.  Phase s = 1 .. S (S = 2 per
// sweep) updates plane t - s - LAG when plane t arrives; the residual follows on plane
// t - S - 1 - LAG.  A halo of H cells on each side of the tile and H planes below the segment
// are recomputed (neighbouring tiles overlap): each phase reaches one cell further, so H = S
// covers the phases, and a pass that also takes the residual needs S + 1, rounded up to even
// to keep 2 x 2 x 2 blocks aligned (one sweep: H = 2 or 4; two sweeps: 4 or 6).  Point formulas
// are those of fas_device.h.
//
// Why row pairs: which cell of a pair a phase updates depends on the row's parity, so with one
// row per thread a wave of two neighbouring rows runs both cases for every phase; a pair of
// rows has one of each, known at compile time, half of its y-neighbours in registers, and the
// 2 x 2 x 2 blocks of the transfers to itself (no second barrier for the restriction).  The
// passes are bound by their issue and by the halo (a two-sweep FP64 tile writes 52 x 20 of its
// 64 x 32 cells), no longer by either alone.  512^3 FP64: pre pass (two sweeps, residual,
// restriction) 1289-1309 -> 1036-1056 us, post pass with the norm 1237 -> 1073 us; FP32 pre
// pass 919 -> 647 us; 48 batched periodic 128^3 FP32 1017 / 995 -> 553 / 565 us; 256^3 FP64
// 239 / 172 -> 147 / 115 us.
//
// Modes: 0 = sweep + residual + restriction (u_c = R u, r_c = R r);
//        1 = correction u += P(u_c - R u) + sweep;  2 = sweep only;
//        3 = no sweep (FP64): the residual r = f - A u cast to FP32 for the inner solve of
//            the mixed form, with the partial sums of r^2 (and of f^2 if asked).
// RHS (the first pass of a coarse level, mode 2): f holds r = R(f - A u) of the finer
// level, and the pass first forms the FAS right-hand side f = r + A u, one plane ahead of
// the sweep while every neighbour still holds its initial value, then uses it and writes
// it for the level's later passes.
// Any mode with NORM leaves one partial sum of the squared residual per block.
// Inner solves of the mixed form (FP32 only): zero_in makes a pass start from u = 0 without
// reading u; acc64 makes a pass add its result into an FP64 iterate (acc64 += fp64(u))
// instead of storing u.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fas_device.h"
#include "fas_fused.h"
#include "fas_internal.h"

namespace fas {

namespace {

constexpr int kTPX = 32;                   // pairs per row
constexpr int kWX = 2 * kTPX;              // tile width in cells (64)
constexpr int kMinSegPlanes = 4;

// Row pairs of a tile.  FP64: 16 (512 threads of 256 VGPRs: the ring of two rows and eight to
// ten planes takes 128 to 160).  FP32: 24 (768 threads of 168 VGPRs), whose 48-row tile writes
// 36 rows with two sweeps and the residual, a 32-row tile 20: 512^3 646 against 729 us per
// pre pass (32 pairs, 1024 threads of 128 VGPRs, spill: 653 us), 20 batched 64^3 47 against
// 64 us, a single 64^3 level 25 against 22 us.
template <typename T>
constexpr int kRows3 = sizeof(T) == 8 ? 16 : 24;

template <typename T>
struct March3Args {
    int n0, n1, n2;
    int bc;
    T k;
    T q[16];
    int tiles_x, tiles_y, segs, seg_planes;
    int batch;
    int64_t stride, cstride;
    const int* act;
    const T* f;
    const T* u_in;
    T* u_out;
    T* uc;
    T* rc;
    T* fout;  // RHS passes: the formed right-hand side
    double* partials;
    float* r32;          // mode 3: the FP32 residual
    double* fpartials;   // mode 3 (nullable): partial sums of f^2
    int zero_in;         // FP32: 1: u_in is taken as 0 and not read (modes 0 and 2)
    double* acc64;       // FP32 (nullable): acc64 += fp64(u) in place of storing u_out
};

constexpr int kShr1 = 0x138;  // wave_shr:1 (lane i gets lane i - 1)
constexpr int kShl1 = 0x130;  // wave_shl:1 (lane i gets lane i + 1)

template <int CTRL>
__device__ __forceinline__ float dpp3(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

template <int CTRL>
__device__ __forceinline__ double dpp3(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

template <typename T>
struct Pair3;
template <>
struct Pair3<double> {
    using V = double2;
};
template <>
struct Pair3<float> {
    using V = float2;
};

__device__ __forceinline__ int wrap3(int g, int n)
{
    int w = g < 0 ? g + n : g - n;
    if (w < 0 || w >= n) w = ((g % n) + n) % n;
    return w;
}

template <typename T>
__device__ __forceinline__ T pick_q3(const March3Args<T>& a, int W)
{
    T v = a.q[6];
    v = W == 3 ? a.q[3] : v;
    v = W == 4 ? a.q[4] : v;
    v = W == 5 ? a.q[5] : v;
    v = W == 7 ? a.q[7] : v;
    v = W == 8 ? a.q[8] : v;
    v = W == 9 ? a.q[9] : v;
    return v;
}

// halo of a pass: even, >= the phases' reach (one cell per phase), +1 when the residual
// is taken
constexpr int halo3(int ns, int mode, bool norm)
{
    return (2 * ns + ((mode == 0 || mode == 3 || norm) ? 1 : 0) + 1) & ~1;
}

template <typename T, int NS, int MODE, bool NORM, bool RHS>
struct Geom3 {
    static constexpr int TR = kRows3<T>;        // row pairs of the tile
    static constexpr int S = 2 * NS;            // colour phases in the pass
    static constexpr int H = halo3(NS, MODE, NORM);
    static constexpr bool RES = MODE == 0 || MODE == 3 || NORM;  // residual of the final plane
    // the correction (mode 1) and the right-hand side (RHS) need the plane below untouched
    static constexpr int LAG = (MODE == 1 || RHS) ? 1 : 0;
    static constexpr int PF = 2;                // planes loaded ahead
    static constexpr int RING = (S + 3 + LAG + PF + 1) & ~1;  // planes held: >= S + 3 + LAG + PF, even
    static constexpr int THREADS = kTPX * TR;
    // LDS exchange slots per buffer: per phase the cells that the row pairs above and below
    // read, both cells of both rows for the residual, and for the right-hand side
    static constexpr int SLOTS = 2 * S + (RES ? 4 : 0) + (RHS ? 4 : 0);
    static constexpr int UX = kWX - 2 * H;      // cells written per tile in x
    static constexpr int UY = 2 * TR - 2 * H;   // rows written per tile
};

// LDS exchange area: two buffers; the norm reduction reuses it after the march.
template <typename T, int SLOTS, int THREADS>
struct Xchg {
    T buf[2][SLOTS][THREADS];
};

// Per-problem arrays of a batched launch (the kernel arguments stay in place).
template <typename T>
struct Arrays3 {
    const T* f;
    const T* u_in;
    T* u_out;
    T* uc;
    T* rc;
    T* fout;
    float* r32;
    double* acc64;
};

// Where a block stands: inside (no index leaves the domain), over a periodic edge (indices
// wrap, nothing else differs) or over a wall (cells outside are 0 and stay so, cells at the
// wall have their own diagonals).
enum { IN_DOMAIN = 0, AT_WALL = 1, AT_WRAP = 2 };

template <typename T, int NS, int MODE, bool NORM, bool RHS, int PLACE, int FIRST>
__device__ __forceinline__ void march3(const March3Args<T>& a, const Arrays3<T> A,
                                       Xchg<T, Geom3<T, NS, MODE, NORM, RHS>::SLOTS, kTPX * kRows3<T>>& X, int tx,
                                       int ty, int seg, double* red)
{
    using G = Geom3<T, NS, MODE, NORM, RHS>;
    using V = typename Pair3<T>::V;
    static_assert(!RHS || MODE == 2, "the right-hand side is formed by a level's first, sweep-only pass");
    constexpr int S = G::S, H = G::H, RING = G::RING, PF = G::PF, LAG = G::LAG, TR = G::TR, NT = G::THREADS;
    const int tid = threadIdx.x;
    const int px = tid % kTPX, py = tid / kTPX;
    constexpr bool WALL = PLACE == AT_WALL;
    const int x0 = tx * G::UX, y0 = ty * G::UY;
    const int gxe = x0 - H + 2 * px;
    const int gy0 = y0 - H + 2 * py;  // the thread's even row
    const int z0 = seg * a.seg_planes;
    const int rA = z0 - H;
    const int zend = min(z0 + a.seg_planes, a.n2);
    const int nsteps = zend - rA + S + 1 + LAG;
    // x / y position of the 2 x 2 cells: wrapped (periodic) or in / out of the domain (sizes and
    // origins are even: all four are on one side)
    bool xyin = true;
    int gxl = gxe, gyl = gy0;
    if constexpr (PLACE == AT_WRAP) {
        gxl = wrap3(gxe, a.n0);
        gyl = wrap3(gy0, a.n1);
    } else if constexpr (WALL) {
        xyin = gxe >= 0 && gxe < a.n0 && gy0 >= 0 && gy0 < a.n1;
        gxl = min(max(gxe, 0), a.n0 - 2);
        gyl = min(max(gy0, 0), a.n1 - 2);
    }
    const bool own = px >= H / 2 && px < kTPX - H / 2 && py >= H / 2 && py < TR - H / 2 && gxe < a.n0 && gy0 < a.n1;
    // boundary faces across x of the even / odd cell, across y of the even / odd row
    const int dsgn = a.bc == BC_DIRICHLET ? 1 : -1;
    const int bx[2] = {WALL && gxe == 0, WALL && gxe + 2 == a.n0};
    const int by[2] = {WALL && gy0 == 0, WALL && gy0 + 2 == a.n1};
    const T k = a.k;
    // 1 / (1 + k W) of cell (row r, column c) inside and on a z boundary
    T qin[2][2], qzb[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            qin[r][c] = a.q[6];
            qzb[r][c] = a.q[6];
            if constexpr (WALL) {
                const int W = 6 + dsgn * (bx[c] + by[r]);
                qin[r][c] = pick_q3(a, W);
                qzb[r][c] = pick_q3(a, W + dsgn);
            }
        }
    const int64_t plane = (int64_t)a.n0 * a.n1;
    const int mc0 = a.n0 >> 1, mc1 = a.n1 >> 1;
    const int64_t cplane = (int64_t)mc0 * mc1;
    const int ym = py > 0 ? tid - kTPX : tid;          // row pairs below and above (those at the
    const int yp = py < TR - 1 ? tid + kTPX : tid;     // tile's edge read themselves: halo rows)

    T u[RING][2][2], f[RING][2][2], cr[RING];  // [plane][row][column]
    T su_prev[2] = {0, 0}, sr_prev[2] = {0, 0};  // restriction: pair sums of the previous plane
    double acc = 0.0, facc = 0.0;

    auto plane_of = [&](int rho, int& gz) -> bool {
        gz = rA + rho;
        if constexpr (PLACE == IN_DOMAIN) return true;
        if (gz >= 0 && gz < a.n2) return true;
        if constexpr (PLACE == AT_WRAP) {
            gz = wrap3(gz, a.n2);
            return true;
        }
        gz = min(max(gz, 0), a.n2 - 1);
        return false;
    };
    auto load_plane = [&](int rho, int p, bool odd) {
        int gz;
        const bool zin = plane_of(rho, gz);
        const int64_t off = (int64_t)gz * plane + (int64_t)gyl * a.n0 + gxl;
        const bool in = !WALL || (zin && xyin);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            V zu;
            if (sizeof(T) == 4 && a.zero_in) {
                zu.x = (T)0;
                zu.y = (T)0;
            } else {
                zu = *reinterpret_cast<const V*>(A.u_in + off + r * a.n0);
            }
            const V zf = *reinterpret_cast<const V*>(A.f + off + r * a.n0);
            u[p][r][0] = in ? zu.x : (T)0;
            u[p][r][1] = in ? zu.y : (T)0;
            f[p][r][0] = in ? zf.x : (T)0;
            f[p][r][1] = in ? zf.y : (T)0;
        }
        if constexpr (MODE == 1) {
            cr[p] = (T)0;
            if (odd) cr[p] = A.uc[(int64_t)(gz >> 1) * cplane + (int64_t)(gyl >> 1) * mc0 + (gxl >> 1)];
        }
    };
    auto zbound = [&](int gz) -> bool { return WALL && (gz == 0 || gz == a.n2 - 1); };

    // Neighbour sum of cell (r, c) of ring plane a0 (planes am below, ap above); yb: the value
    // across the row pair's edge (below row 0 or above row 1).
    auto nb_sum = [&](int r, int c, int a0, int am, int ap, T yb) -> T {
        const T xs = c == 0 ? dpp3<kShr1>(u[a0][r][1]) + u[a0][r][1] : u[a0][r][0] + dpp3<kShl1>(u[a0][r][0]);
        const T ys = r == 0 ? yb + u[a0][1][c] : u[a0][0][c] + yb;
        return (xs + ys) + (u[am][r][c] + u[ap][r][c]);
    };
    // (A u) of that cell, given its neighbour sum.
    auto apply = [&](int r, int c, int a0, T Ssum, bool zb) -> T {
        const T W = (T)(WALL ? 6 + dsgn * (bx[c] + by[r] + (zb ? 1 : 0)) : 6);
        return u[a0][r][c] + k * (W * u[a0][r][c] - Ssum);
    };
    // Both cells of both rows, for the row pairs below (slots 0, 1) and above (slots 2, 3).
    auto publish4 = [&](T (*B)[NT], int a0) {
        B[0][tid] = u[a0][0][0];
        B[1][tid] = u[a0][0][1];
        B[2][tid] = u[a0][1][0];
        B[3][tid] = u[a0][1][1];
    };

#pragma unroll
    for (int p = 0; p < PF; ++p) load_plane(p, p, p & 1);

    // whole ring turns; loads past the last visited plane repeat that plane (no new
    // memory traffic), and the steps past it only touch planes that are never written
    const int nturns = (nsteps + RING - 1) / RING;
    for (int turn = 0; turn < nturns; ++turn) {
        const int rb = turn * RING;
#pragma unroll
        for (int j = 0; j < RING; ++j) {
            const int rho = rb + j;
            load_plane(min(rho + PF, nsteps - 1), (j + PF) % RING, ((j + PF) & 1) != 0);
            constexpr int sh = 4 * RING;
            T(*const B)[NT] = X.buf[j & 1];
            T(*const BR)[NT] = B + 2 * S;                   // residual
            T(*const BF)[NT] = B + 2 * S + (G::RES ? 4 : 0);  // right-hand side
            // publish the values the neighbouring row pairs read in this step (colour of a
            // cell: (x + y + z) parity with x, y, z local; all origins even): phase s updates
            // column c of row 0 and column 1 - c of row 1, in every row pair
#pragma unroll
            for (int s = 1; s <= S; ++s) {
                const int a0 = (j - s - LAG + sh) % RING;
                const int c = ((j - s - LAG + sh) & 1) ^ ((s - 1) & 1) ^ FIRST;
                B[2 * s - 2][tid] = u[a0][1][c];      // below row 0 of the pair above
                B[2 * s - 1][tid] = u[a0][0][1 - c];  // above row 1 of the pair below
            }
            if constexpr (G::RES) publish4(BR, (j - S - 1 - LAG + sh) % RING);
            if constexpr (RHS) publish4(BF, (j - LAG + sh) % RING);  // plane rho - 1, initial values
            __syncthreads();
            if constexpr (RHS) {
                // FAS right-hand side of plane rho - LAG (f held r)
                const int r3 = rho - LAG;
                int gz;
                const bool zin = plane_of(r3, gz);
                if (r3 >= 1 && (!WALL || zin)) {
                    const int a0 = (j - LAG + sh) % RING;
                    const int am = (j - LAG - 1 + sh) % RING;
                    const int ap = (j - LAG + 1 + sh) % RING;
                    const bool zb = zbound(gz);
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const T yb = r == 0 ? BF[2 + c][ym] : BF[c][yp];
                            f[a0][r][c] = f[a0][r][c] + apply(r, c, a0, nb_sum(r, c, a0, am, ap, yb), zb);
                        }
                    const int graw = rA + r3;
                    if (graw >= z0 && graw < zend && own) {
                        T* const o = A.fout + (int64_t)graw * plane + (int64_t)gy0 * a.n0 + gxe;
                        store_pair_nt(o, f[a0][0][0], f[a0][0][1]);
                        store_pair_nt(o + a.n0, f[a0][1][0], f[a0][1][1]);
                    }
                }
            }
            if constexpr (MODE == 1) {
                // fine grid correction on planes (rho - 1, rho) when rho is odd: the thread's
                // cells of the two planes are the children of one coarse cell
                if (j & 1) {
                    int gz;
                    const bool zin = plane_of(rho, gz);
                    const int jp = (j + RING - 1) % RING;
                    const T s00 = u[jp][0][0] + u[jp][0][1], s10 = u[jp][1][0] + u[jp][1][1];
                    const T s01 = u[j][0][0] + u[j][0][1], s11 = u[j][1][0] + u[j][1][1];
                    const T old = ((s00 + s10) + (s01 + s11)) * (T)0.125;
                    const T c = cr[j] - old;
                    const bool ok = !WALL || (zin && xyin);
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            u[jp][r][x] = ok ? u[jp][r][x] + c : u[jp][r][x];
                            u[j][r][x] = ok ? u[j][r][x] + c : u[j][r][x];
                        }
                }
            }
            // colour phases
#pragma unroll
            for (int s = 1; s <= S; ++s) {
                const int r3 = rho - s - LAG;
                if (r3 < 1) continue;
                int gz;
                const bool zin = plane_of(r3, gz);
                if (WALL && !zin) continue;
                const int a0 = (j - s - LAG + sh) % RING;
                const int am = (j - s - LAG - 1 + sh) % RING;
                const int ap = (j - s - LAG + 1 + sh) % RING;
                const int c = ((j - s - LAG + sh) & 1) ^ ((s - 1) & 1) ^ FIRST;
                const bool zb = zbound(gz);
                const T S0 = nb_sum(0, c, a0, am, ap, B[2 * s - 2][ym]);
                const T S1 = nb_sum(1, 1 - c, a0, am, ap, B[2 * s - 1][yp]);
                const T v0 = (f[a0][0][c] + k * S0) * (zb ? qzb[0][c] : qin[0][c]);
                const T v1 = (f[a0][1][1 - c] + k * S1) * (zb ? qzb[1][1 - c] : qin[1][1 - c]);
                u[a0][0][c] = (!WALL || xyin) ? v0 : u[a0][0][c];
                u[a0][1][1 - c] = (!WALL || xyin) ? v1 : u[a0][1][1 - c];
            }
            // plane rho - S - 1 - LAG is final: write, residual, restriction / norm
            {
                const int r3 = rho - S - 1 - LAG;
                if (r3 >= 1) {
                    int gz;
                    plane_of(r3, gz);
                    const int graw = rA + r3;
                    const bool inseg = graw >= z0 && graw < zend;
                    const int a0 = (j - S - 1 - LAG + sh) % RING;
                    const int am = (j - S - 2 - LAG + sh) % RING;
                    const int ap = (j - S - LAG + sh) % RING;
                    T res[2][2] = {};
                    if constexpr (G::RES) {
                        const bool zb = zbound(gz);
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                const T yb = r == 0 ? BR[2 + c][ym] : BR[c][yp];
                                res[r][c] = f[a0][r][c] - apply(r, c, a0, nb_sum(r, c, a0, am, ap, yb), zb);
                            }
                    }
                    if (inseg && own) {
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const int64_t o = (int64_t)graw * plane + (int64_t)(gy0 + r) * a.n0 + gxe;
                            if constexpr (MODE == 3) {
                                float2 rv;
                                rv.x = (float)res[r][0];
                                rv.y = (float)res[r][1];
                                *reinterpret_cast<float2*>(A.r32 + o) = rv;
                                if (a.fpartials) {
                                    facc += (double)f[a0][r][0] * (double)f[a0][r][0];
                                    facc += (double)f[a0][r][1] * (double)f[a0][r][1];
                                }
                            } else if (sizeof(T) == 4 && A.acc64) {
                                double2* const d = reinterpret_cast<double2*>(A.acc64 + o);
                                double2 v = *d;
                                v.x = v.x + (double)u[a0][r][0];
                                v.y = v.y + (double)u[a0][r][1];
                                *d = v;
                            } else {
                                store_pair_nt(A.u_out + o, u[a0][r][0], u[a0][r][1]);
                            }
                            if constexpr (NORM) {
                                acc += (double)res[r][0] * (double)res[r][0];
                                acc += (double)res[r][1] * (double)res[r][1];
                            }
                        }
                    }
                    if constexpr (MODE == 0) {
                        const T su[2] = {u[a0][0][0] + u[a0][0][1], u[a0][1][0] + u[a0][1][1]};
                        const T sr[2] = {res[0][0] + res[0][1], res[1][0] + res[1][1]};
                        // planes (r - 1, r) form coarse plane graw / 2 when r is odd
                        if (((j - S - 1 - LAG + sh) & 1) && graw - 1 >= z0 && inseg && own) {
                            // children summed along x (pair), then y (rows), then z
                            const T ucv = ((su_prev[0] + su_prev[1]) + (su[0] + su[1])) * (T)0.125;
                            const T rcv = ((sr_prev[0] + sr_prev[1]) + (sr[0] + sr[1])) * (T)0.125;
                            const int64_t P = (int64_t)(graw >> 1) * cplane + (int64_t)(gy0 >> 1) * mc0 + (gxe >> 1);
                            __builtin_nontemporal_store(ucv, A.uc + P);
                            __builtin_nontemporal_store(rcv, A.rc + P);
                        }
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            su_prev[r] = su[r];
                            sr_prev[r] = sr[r];
                        }
                    }
                }
            }
        }
    }
    if constexpr (NORM) {
        // red aliases the exchange area; mode 3 sums f^2 beside r^2 in red[NT ..)
        __syncthreads();
        red[tid] = acc;
        if constexpr (MODE == 3) red[NT + tid] = facc;
        __syncthreads();
        for (int s = 512; s > 0; s >>= 1) {  // NT <= 1024, not always a power of two
            if (tid < s && tid + s < NT) {
                red[tid] = red[tid] + red[tid + s];
                if constexpr (MODE == 3) red[NT + tid] = red[NT + tid] + red[NT + tid + s];
            }
            __syncthreads();
        }
    }
}

template <typename T, int NS, int MODE, bool NORM, bool RHS>
__global__ __launch_bounds__(kTPX * kRows3<T>) void k_march3(March3Args<T> a, int first)
{
    using G = Geom3<T, NS, MODE, NORM, RHS>;
    static_assert(!NORM || sizeof(Xchg<T, G::SLOTS, G::THREADS>) >= (MODE == 3 ? 2 : 1) * G::THREADS * sizeof(double),
                  "norm reductions fit the exchange area");
    static_assert(MODE != 3 || (NS == 0 && NORM && !RHS && sizeof(T) == 8), "mode 3: FP64 residual pass");
    __shared__ Xchg<T, G::SLOTS, G::THREADS> X;
    double* red = reinterpret_cast<double*>(&X.buf[0][0][0]);
    // (dispatch order, tile x fastest: the blocks resident at one time cover one z-segment
    // of neighbouring tiles across all XCDs; renumbering so that each XCD takes a contiguous
    // range of a segment's tiles changed the passes by -4 to +3%, of all tiles by +8 to +14%)
    const int per = a.tiles_x * a.tiles_y * a.segs;
    const int b = blockIdx.x / per, w = blockIdx.x % per;
    if (a.act && !a.act[b]) return;
    Arrays3<T> A;
    A.f = a.f + b * a.stride;
    A.u_in = a.u_in + b * a.stride;
    A.u_out = a.u_out + b * a.stride;
    A.uc = a.uc ? a.uc + b * a.cstride : nullptr;
    A.rc = a.rc ? a.rc + b * a.cstride : nullptr;
    A.fout = a.fout ? a.fout + b * a.stride : nullptr;
    A.r32 = a.r32 ? a.r32 + b * a.stride : nullptr;
    A.acc64 = a.acc64 ? a.acc64 + b * a.stride : nullptr;
    const int tx = w % a.tiles_x, ty = (w / a.tiles_x) % a.tiles_y, seg = w / (a.tiles_x * a.tiles_y);
    const int x0 = tx * G::UX, y0 = ty * G::UY, z0 = seg * a.seg_planes;
    const int planes_read = a.seg_planes + G::H + G::S + 1 + G::LAG;  // the steps of a full segment
    const bool edge = x0 - G::H < 0 || x0 - G::H + kWX > a.n0 || y0 - G::H < 0 || y0 - G::H + 2 * G::TR > a.n1 ||
                      z0 - G::H < 0 || z0 - G::H + planes_read > a.n2;
#define FAS_MARCH3(PLACE_)                                                           \
    do {                                                                             \
        if (first)                                                                   \
            march3<T, NS, MODE, NORM, RHS, PLACE_, 1>(a, A, X, tx, ty, seg, red);    \
        else                                                                         \
            march3<T, NS, MODE, NORM, RHS, PLACE_, 0>(a, A, X, tx, ty, seg, red);    \
    } while (0)
    if (!edge)
        FAS_MARCH3(IN_DOMAIN);
    else if (a.bc == BC_PERIODIC)
        FAS_MARCH3(AT_WRAP);
    else
        FAS_MARCH3(AT_WALL);
#undef FAS_MARCH3
    if constexpr (NORM) {
        if (threadIdx.x == 0) {
            a.partials[(int64_t)b * per + w] = red[0];
            if constexpr (MODE == 3) {
                if (a.fpartials) a.fpartials[(int64_t)b * per + w] = red[G::THREADS];
            }
        }
    }
}

// Planes per segment: a launch takes about (rounds of blocks over the compute units) x (planes
// of a segment + `extra` planes of halo and lag) steps; the number of segments that makes this
// least.  With 64-plane segments,
// halved until there were 512 blocks, 64^3 to 256^3 levels ran up to twice the steps (a launch
// of 260 blocks on 256 compute units takes two rounds): 256^3 FP64 pre pass 201 -> 147 us,
// 128^3 60 -> 44 us.
int segment_planes(int64_t tiles, int n2, int extra)
{
    const unsigned cus = (unsigned)device_cus();
    unsigned best = (unsigned)n2;
    uint64_t least = ~(uint64_t)0;
    for (unsigned segs = 1; segs <= (unsigned)n2 / kMinSegPlanes; ++segs) {
        const unsigned planes = 2 * (((unsigned)n2 + 2 * segs - 1) / (2 * segs));  // even: 2 x 2 x 2 blocks
        const unsigned n = (unsigned)tiles * (((unsigned)n2 + planes - 1) / planes);
        const uint64_t steps = (uint64_t)((n + cus - 1) / cus) * (planes + (unsigned)extra);
        if (steps < least) {
            least = steps;
            best = planes;
        }
    }
    return (int)best;
}

template <typename T>
March3Args<T> make_args3(const fas_grid* g, int l, const Coef& c, int ns, int mode, bool norm)
{
    March3Args<T> a{};
    a.n0 = g->lev[l].n[0];
    a.n1 = g->lev[l].n[1];
    a.n2 = g->lev[l].n[2];
    a.bc = g->bc;
    a.k = (T)c.kd;
    for (int W = 0; W < 16; ++W) a.q[W] = (T)c.q[W];
    const int H = halo3(ns, mode, norm);
    a.tiles_x = (a.n0 + (kWX - 2 * H) - 1) / (kWX - 2 * H);
    a.tiles_y = (a.n1 + (2 * kRows3<T> - 2 * H) - 1) / (2 * kRows3<T> - 2 * H);
    a.seg_planes = segment_planes((int64_t)g->batch * a.tiles_x * a.tiles_y, a.n2, H + 2 * ns + 2);
    if (g->seg_rows[l]) a.seg_planes = g->seg_rows[l];
    if (g->seg_force) a.seg_planes = g->seg_force < a.n2 ? g->seg_force : a.n2;
    a.segs = (a.n2 + a.seg_planes - 1) / a.seg_planes;
    a.batch = g->batch;
    a.stride = g->lev[l].N;
    a.cstride = l < g->L ? g->lev[l + 1].N : 0;
    a.act = active_flags(g);
    return a;
}

inline void check_launch3()
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw Error(FAS_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

template <typename T, int NS, int MODE, bool NORM, bool RHS = false>
void go3(const fas_grid* g, const March3Args<T>& a, int first)
{
    const unsigned blocks = (unsigned)((int64_t)a.batch * a.tiles_x * a.tiles_y * a.segs);
    k_march3<T, NS, MODE, NORM, RHS><<<blocks, kTPX * kRows3<T>, 0, g->stream>>>(a, first);
}

template <typename T>
void dispatch3(const fas_grid* g, int l, const Coef& c, int first, int mode, int ns, bool norm, const void* f,
               const void* u_in, void* u_out, void* uc, void* rc, double* partials, void* fout, bool zero_in,
               double* acc64)
{
    if ((zero_in && (sizeof(T) != 4 || mode == 1 || fout)) || (acc64 && (sizeof(T) != 4 || mode == 0)))
        throw Error(FAS_ERR_ARG, "internal: zero start / FP64 accumulation on a pass that cannot take it");
    March3Args<T> a = make_args3<T>(g, l, c, ns, mode, norm && mode != 0);
    a.zero_in = zero_in ? 1 : 0;
    a.acc64 = acc64;
    a.f = (const T*)f;
    a.u_in = (const T*)u_in;
    a.u_out = (T*)u_out;
    a.uc = (T*)uc;
    a.rc = (T*)rc;
    a.partials = partials;
    a.fout = (T*)fout;
    if (ns != 1 && ns != 2) throw Error(FAS_ERR_ARG, "internal: 3D march kernels run one or two sweeps per pass");
    if (fout && (mode != 2 || norm || ns != 1))
        throw Error(FAS_ERR_ARG, "internal: right-hand side formed by a one-sweep, sweep-only pass");
    if (fout) {
        go3<T, 1, 2, false, true>(g, a, first);
    } else if (ns == 1) {
        if (mode == 0) go3<T, 1, 0, false>(g, a, first);
        else if (mode == 1) norm ? go3<T, 1, 1, true>(g, a, first) : go3<T, 1, 1, false>(g, a, first);
        else norm ? go3<T, 1, 2, true>(g, a, first) : go3<T, 1, 2, false>(g, a, first);
    } else {
        if (mode == 0) go3<T, 2, 0, false>(g, a, first);
        else if (mode == 1) norm ? go3<T, 2, 1, true>(g, a, first) : go3<T, 2, 1, false>(g, a, first);
        else norm ? go3<T, 2, 2, true>(g, a, first) : go3<T, 2, 2, false>(g, a, first);
    }
    check_launch3();
}

}  // namespace

bool fused3_ok(const fas_grid* g, int l, bool variable)
{
    if (!g->fused || g->dim != 3 || variable || l >= g->L) return false;
    return g->lev[l].n[0] >= 64 && g->lev[l].n[1] >= 32 && g->lev[l].n[2] >= 16;
}

int fused3_seg_candidates(const fas_grid* g, int l, int ns, int out[kMaxSegCandidates])
{
    const int n2 = g->lev[l].n[2];
    const int rule = g->dtype == FAS_F64 ? make_args3<double>(g, l, g->coef[l], ns, 0, false).seg_planes
                                         : make_args3<float>(g, l, g->coef[l], ns, 0, false).seg_planes;
    const int segs = (n2 + rule - 1) / rule;
    auto planes = [&](int s) { return s < 1 ? n2 : 2 * ((n2 + 2 * s - 1) / (2 * s)); };
    int n = 0;
    for (int p : {rule, planes(segs - 1), planes(segs + 1), 8, 16, 32, 64, 128})
        if (p >= kMinSegPlanes && p <= n2 && std::find(out, out + n, p) == out + n) out[n++] = p;
    return n;
}

int fused3_partials(const fas_grid* g, int l, int ns)
{
    auto blocks = [](const auto& a) { return a.tiles_x * a.tiles_y * a.segs; };
    return g->dtype == FAS_F64 ? blocks(make_args3<double>(g, l, g->coef[l], ns, 2, true))
                               : blocks(make_args3<float>(g, l, g->coef[l], ns, 2, true));
}

int launch_march3_resid(const fas_grid* g, const Coef& c, const void* f, const void* u, void* r32, double* partials,
                        double* fpartials)
{
    if (g->dtype != FAS_F64 || !fused3_ok(g, 0, g->lev[0].kap != nullptr)) return 0;
    March3Args<double> a = make_args3<double>(g, 0, c, 0, 3, true);
    const int per = a.tiles_x * a.tiles_y * a.segs;
    if (per > g->npartials / g->batch) return 0;
    a.f = (const double*)f;
    a.u_in = (const double*)u;
    a.r32 = (float*)r32;
    a.partials = partials;
    a.fpartials = fpartials;
    go3<double, 0, 3, true>(g, a, 0);
    check_launch3();
    return per;
}

void launch_march3(const fas_grid* g, int l, const Coef& c, int first, int mode, int ns, bool norm, const void* f,
                   const void* u_in, void* u_out, void* uc, void* rc, double* partials, void* fout, bool zero_in,
                   double* acc64)
{
    if (g->dtype == FAS_F64)
        dispatch3<double>(g, l, c, first, mode, ns, norm, f, u_in, u_out, uc, rc, partials, fout, zero_in, acc64);
    else
        dispatch3<float>(g, l, c, first, mode, ns, norm, f, u_in, u_out, uc, rc, partials, fout, zero_in, acc64);
}

}  // namespace fas
