// Fused 3D passes of small levels (constant kappa) as bricks: a workgroup holds a brick of
// 8^3 or 16^3 cells with its halo at once (u in LDS, u and f in registers) and runs the pass
// colour phase by colour phase, one barrier each.  The plane marches (kernels_fused3d.hip)
// visit a segment's planes one after another, at least (planes + halo) dependent steps, which
// on a level too small to fill the device is their time: a 64^3 level took two launches of
// 30 and 26 us a cycle, and a level below the marches' sizes some eleven launches of 5-7 us.
// A brick pass waits on memory once, then on its phases: V(2,2)-cycles of 64^3 cells
// 106 -> 49 us (FP64), 95 -> 40 us (FP32), of 32^3 54 -> 29 us, of 48^3 96 -> 37 us; with
// bricks of 16^3 (more to do: brick_side) of 96^3 153 -> 68 us, of 128^3 184 -> 111 us.
//
// Geometry.  A thread owns a block of 2 x 2 x 2 cells (of large bricks two blocks), the
// children of one coarse cell: half of a cell's neighbours are its registers, the cells that
// a phase updates are the same for every thread, and the transfers need no neighbour; LDS
// keeps one plane per cell of the block, indexed by block (as kernels_tail.hip).  A value
// reaches one cell further along one axis per phase, so a pass reads u within R cells of its
// brick in the sum of the distances along the axes, not in a cube around it: with two sweeps
// and the residual (R = 5) 528 blocks of the cube's 1000 (8^3) or 1984 of 2744 (16^3, whose
// cube would not fit LDS), and f and the phases need fewer still.  The threads are numbered
// over those blocks only, by a list made at compile time: first the brick's own, so that few
// waves have all of the output work, then the rest in the order of memory (by distance
// instead: 128^3 FP64 in bricks of 8^3 98 -> 80 us for the pre pass; the whole cube: 102 us).
// Waves without a boundary face take phases without the selection of their coefficients, and
// neighbours lie at constant LDS offsets (80 -> 76 us); neighbouring bricks run under one L2
// (76 -> 71 us, the post pass 41 -> 37).  Large bricks take 34 and 28 us there (march: 46 and
// 28), at 256^3 258 us (march: 148): the price of the short chain, hence only small levels.
// (64 VGPRs, for two large FP32 bricks per compute unit, spill: 22.6 -> 24.9 us.)
//
// Passes (Alg. 1): pre = nu sweeps, then u_c = R u and r_c = R (f - A u), on a coarse level
// forming the FAS right-hand side f = r + A u first; post = u += P (u_c - R u), nu sweeps,
// optionally one sum of r^2 per brick.  For the inner solves of the mixed form (FP32) a pre
// pass can start from zero and a post pass add into an FP64 iterate.  Point formulas are those
// of fas_device.h.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fas_device.h"
#include "fas_fused.h"
#include "fas_internal.h"
#include "march_util.h"

namespace fas {

namespace {

// Rules of brick_side and brick_ok, in bricks of 8^3 cells over all problems.
constexpr int64_t kBrickLarge = 768;                        // from here on bricks of 16^3
constexpr int64_t kBrickMarch = 6144, kBrickMarchNarrow = 24576, kBrickMarch32 = 4096;  // most where marches could run

// Distance (sum over the axes) from a brick up to which a pass reads u: one cell per colour
// phase, one more for a residual.  f is read one cell less far.
constexpr int brick_reach(int nu, bool residual) { return 2 * nu + (residual ? 1 : 0); }

// Blocks of 2 x 2 x 2 cells within reach R of a brick of BS^3 cells: M along each axis of
// their bounding cube, N of them in all, KB to each thread.
template <int R, int BS>
struct BrickShape {
    static constexpr int D = (R + 1) / 2, M = BS / 2 + 2 * D;
    static constexpr int out(int i)  // cells between block i of an axis and the brick, plus one (0: inside)
    {
        const int d = i < D ? D - i : (i >= D + BS / 2 ? i - (D + BS / 2) + 1 : 0);
        return d > 0 ? 2 * d - 1 : 0;
    }
    static constexpr int dist(int i, int j, int k) { return out(i) + out(j) + out(k); }
    static constexpr int count()
    {
        int n = 0;
        for (int k = 0; k < M; ++k)
            for (int j = 0; j < M; ++j)
                for (int i = 0; i < M; ++i) n += dist(i, j, k) <= R ? 1 : 0;
        return n;
    }
    static constexpr int N = count();
    // threads, in whole waves: one for each block; of large bricks for every second one
    static constexpr int KB = BS > 8 ? 2 : 1, NT = ((N + KB - 1) / KB + 63) & ~63;
    // LDS indices of one cell of the blocks: rows of M, and of a large brick only the rows that
    // have blocks (the whole cube would not fit).  Neighbours that no result needs may lie in
    // other rows, or in the padding.
    static constexpr bool TRIM = BS > 8;
    static constexpr int PAD = TRIM ? M + 1 : (R % 2 ? 0 : M * M);
    static constexpr bool has_row(int j, int k) { return !TRIM || out(j) + out(k) <= R; }
    static constexpr int index(int i, int j, int k)
    {
        int o = PAD + i;
        for (int z = 0; z < M; ++z)
            for (int y = 0; y < M; ++y) {
                if (z > k || (z == k && y >= j)) return o;
                o += has_row(y, z) ? M : 0;
            }
        return o;
    }
    static constexpr int CAP = index(0, M, M - 1) + PAD;
};

// The blocks, the brick's own first, the others in the order of memory: v = i | j << 4 | k << 8
// | distance << 12; of large bricks also the LDS indices of the block and of those below and
// above it.
template <int R, int BS>
struct BrickList {
    using B = BrickShape<R, BS>;
    unsigned short v[B::N];
    unsigned short o[B::TRIM ? B::N : 1], below[B::TRIM ? B::N : 1], above[B::TRIM ? B::N : 1];
    constexpr BrickList() : v(), o(), below(), above()
    {
        int row[B::M][B::M] = {};  // LDS index of each row
        for (int k = 0, at = B::PAD; k < B::M; ++k)
            for (int j = 0; j < B::M; ++j) {
                row[k][j] = at;
                at += B::has_row(j, k) ? B::M : 0;
            }
        int n = 0;
        for (int halo = 0; halo <= 1; ++halo)
            for (int k = 0; k < B::M; ++k)
                for (int j = 0; j < B::M; ++j)
                    for (int i = 0; i < B::M; ++i) {
                        const int d = B::dist(i, j, k);
                        if (d > R || (d > 0) != (halo == 1)) continue;
                        v[n] = (unsigned short)(i | j << 4 | k << 8 | d << 12);
                        if (B::TRIM) {
                            // (a row that is not there holds nothing a result needs)
                            o[n] = (unsigned short)(row[k][j] + i);
                            below[n] = k > 0 && B::has_row(j, k - 1) ? (unsigned short)(row[k - 1][j] + i) : o[n];
                            above[n] = k < B::M - 1 && B::has_row(j, k + 1) ? (unsigned short)(row[k + 1][j] + i) : o[n];
                        }
                        ++n;
                    }
    }
};

template <typename T>
struct BrickArgs {
    int n0, n1, n2;
    int bc;
    T k;
    T q[4];            // 1 / (1 + k W) with 0 .. 3 boundary faces
    int b0, b1, b2;    // bricks along each axis
    int64_t stride, cstride;
    const int* act;
    const T* f;
    const T* u_in;
    T* u_out;
    T* uc;             // pre: R u out; post: new coarse values in
    T* rc;             // pre: R r out
    T* fout;           // pre forming the right-hand side (f then holds r)
    double* partials;  // post: sum of r^2 per brick
    int zero_in;       // FP32 pre: u_in is taken as 0 and not read
    double* acc64;     // FP32 post (nullable): acc64 += fp64(result) in place of storing u_out
};

// A thread's block of the window; cell c is (c & 1, c >> 1 & 1, c >> 2).
template <typename T>
struct BrickBlock {
    bool on;              // the window has this block
    bool in;              // it lies in the domain (always, on periodic grids)
    bool own;             // the brick writes it
    int dist;             // of its nearest cell from the brick
    int o, zm, zp;        // LDS index of the block, and (large bricks) of those below and above
    bool lo[3], hi[3];    // the cells at 0 / at 1 along an axis have a boundary face
    unsigned row[4];      // byte offsets of its cell pairs in the domain (wrapped or clamped)
    unsigned coarse;      // and of its coarse cell
    T u[8], f[8];
};

// The pass of one brick; returns the thread's share of the sum of r^2.
template <typename T, int NU, bool POST, bool RHS, bool NORM, int BS>
__device__ __forceinline__ double brick_pass(const BrickArgs<T>& a, int first, int prob, int bx, int by, int bz, T* lds)
{
    constexpr bool RES = !POST || NORM;
    constexpr int R = brick_reach(NU, RES);
    using Shape = BrickShape<R, BS>;
    constexpr int D = Shape::D, M = Shape::M, CAP = Shape::CAP, KB = Shape::KB;
    static constexpr BrickList<R, BS> list{};
    static_assert(!(POST && RHS), "a pre pass forms the right-hand side");
    // a row's cell pair (base pointers need not be aligned to pairs)
    typedef T V __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    typedef double V64 __attribute__((ext_vector_type(2), aligned(8)));
    const bool periodic = a.bc == BC_PERIODIC;
    const int n[3] = {a.n0, a.n1, a.n2};
    auto U = [&](int c) { return lds + c * CAP; };
    // cell pairs and coarse values of this problem's arrays by byte offset
    auto pair_at = [&](const T* v, unsigned byte) {
        return reinterpret_cast<V*>(reinterpret_cast<char*>(const_cast<T*>(v + prob * a.stride)) + byte);
    };
    auto coarse_at = [&](T* v, unsigned byte) {
        return reinterpret_cast<T*>(reinterpret_cast<char*>(v + prob * a.cstride) + byte);
    };
    // 0 .. 3 boundary faces of cell c -> one of four values
    auto by_faces = [](auto walls, const BrickBlock<T>& B, int c, T v0, T v1, T v2, T v3) {
        if (!decltype(walls)::value) return v0;
        const bool x = c & 1 ? B.hi[0] : B.lo[0], y = c & 2 ? B.hi[1] : B.lo[1], z = c & 4 ? B.hi[2] : B.lo[2];
        const bool all = x && y && z, two = (x && y) || (x && z) || (y && z), any = x || y || z;
        return all ? v3 : (two ? v2 : (any ? v1 : v0));
    };
    auto nb_sum = [&](const BrickBlock<T>& B, int c) {
        const int below[3] = {B.o - 1, B.o - M, Shape::TRIM ? B.zm : B.o - M * M};
        const int above[3] = {B.o + 1, B.o + M, Shape::TRIM ? B.zp : B.o + M * M};
        T v[6];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const int o = c ^ (1 << x);
            const bool hi = (c >> x) & 1;
            v[2 * x] = hi ? B.u[o] : U(o)[below[x]];
            v[2 * x + 1] = hi ? U(o)[above[x]] : B.u[o];
        }
        return nbsum<T, 3>(v);
    };
    const T d = a.bc == BC_DIRICHLET ? (T)1 : (T)-1;
    auto apply = [&](auto walls, const BrickBlock<T>& B, int c) {
        const T W = by_faces(walls, B, c, (T)6, (T)6 + d, (T)6 + (d + d), (T)6 + (d + d + d));
        return B.u[c] + a.k * (W * B.u[c] - nb_sum(B, c));
    };

    // every load is issued before the first use
    BrickBlock<T> blk[KB];
    T cnew[KB];
    bool faces = false;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        BrickBlock<T>& b = blk[kb];
        const int t = (int)threadIdx.x + kb * Shape::NT;
        b.on = t < Shape::N;
        const int at = b.on ? t : 0, code = list.v[at];
        b.dist = code >> 12;
        const int pos[3] = {code & 15, code >> 4 & 15, code >> 8 & 15};
        const int org[3] = {bx * BS - 2 * D, by * BS - 2 * D, bz * BS - 2 * D};
        int g[3];
        if constexpr (Shape::TRIM)
            b.o = list.o[at], b.zm = list.below[at], b.zp = list.above[at];
        else
            b.o = Shape::PAD + pos[0] + M * (pos[1] + M * pos[2]);
        b.in = b.on;
        b.own = b.on && b.dist == 0;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            g[x] = org[x] + 2 * pos[x];
            b.own = b.own && g[x] < n[x];
            b.lo[x] = !periodic && g[x] == 0;
            b.hi[x] = !periodic && g[x] + 2 == n[x];
            if (periodic) {  // sizes and origins are even: a block never straddles the edge
                g[x] = wrap(g[x], n[x]);
            } else {
                b.in = b.in && g[x] >= 0 && g[x] < n[x];
                g[x] = min(max(g[x], 0), n[x] - 2);
            }
            faces = faces || b.lo[x] || b.hi[x];
        }
        const unsigned first_cell = g[0] + (unsigned)a.n0 * (g[1] + (unsigned)a.n1 * g[2]);
        b.coarse = (g[0] / 2 + (unsigned)(a.n0 / 2) * (g[1] / 2 + (unsigned)(a.n1 / 2) * (g[2] / 2))) * sizeof(T);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b.row[i] = (first_cell + (i & 1) * (unsigned)a.n0 + (i >> 1) * (unsigned)(a.n0 * a.n1)) * sizeof(T);
            V vu = {(T)0, (T)0}, vf = {(T)0, (T)0};
            if (b.in && b.dist < R) vf = *pair_at(a.f, b.row[i]);
            if (b.in && !(sizeof(T) == 4 && a.zero_in)) vu = *pair_at(a.u_in, b.row[i]);
            b.u[2 * i] = vu.x;
            b.u[2 * i + 1] = vu.y;
            b.f[2 * i] = vf.x;
            b.f[2 * i + 1] = vf.y;
        }
        if constexpr (POST) cnew[kb] = *coarse_at(a.uc, b.coarse);
    }
    // whether any block of the wave has a boundary face
    const bool walls = __any(faces) != 0;
    auto with_walls = [&](auto&& body) {
        if (walls)
            body(std::true_type{});
        else
            body(std::false_type{});
    };
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        BrickBlock<T>& b = blk[kb];
        if constexpr (POST) {
            // the fine grid correction: the block's cells are the children of one coarse cell
            const T c = cnew[kb] - restrict8(b.u[0], b.u[1], b.u[2], b.u[3], b.u[4], b.u[5], b.u[6], b.u[7]);
#pragma unroll
            for (int i = 0; i < 8; ++i) b.u[i] = b.in ? b.u[i] + c : b.u[i];
        }
        if (b.on) {
#pragma unroll
            for (int c = 0; c < 8; ++c) U(c)[b.o] = b.u[c];
        }
    }
    __syncthreads();
    if constexpr (RHS) {
        // FAS right-hand side from the initial values: f = r + A u
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            BrickBlock<T>& b = blk[kb];
            with_walls([&](auto wl) {
                if (b.dist >= R) return;
#pragma unroll
                for (int c = 0; c < 8; ++c) b.f[c] = b.f[c] + apply(wl, b, c);
            });
            if (b.own) {
#pragma unroll
                for (int i = 0; i < 4; ++i) *pair_at(a.fout, b.row[i]) = V{b.f[2 * i], b.f[2 * i + 1]};
            }
        }
        __syncthreads();
    }
    // colour phases
    auto phase = [&](auto step, auto par, auto wl, BrickBlock<T>& b) {
        constexpr int s = decltype(step)::value, P = decltype(par)::value;
        // blocks outside the domain stay 0; from this far off no value reaches a result any more
        if (!b.in || b.dist > R - 1 - s) return;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if ((((c & 1) + ((c >> 1) & 1) + (c >> 2)) & 1) != P) continue;
            b.u[c] = (b.f[c] + a.k * nb_sum(b, c)) * by_faces(wl, b, c, a.q[0], a.q[1], a.q[2], a.q[3]);
            U(c)[b.o] = b.u[c];
        }
    };
    auto colour = [&](auto step) {
        with_walls([&](auto wl) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (((decltype(step)::value & 1) ^ first) != 0)
                    phase(step, std::integral_constant<int, 1>{}, wl, blk[kb]);
                else
                    phase(step, std::integral_constant<int, 0>{}, wl, blk[kb]);
            }
        });
        __syncthreads();
    };
    colour(std::integral_constant<int, 0>{});
    colour(std::integral_constant<int, 1>{});
    if constexpr (NU == 2) {
        colour(std::integral_constant<int, 2>{});
        colour(std::integral_constant<int, 3>{});
    }
    // (a thread's own block is its first)
    static_assert(BS * BS * BS / 8 <= Shape::NT, "own blocks");
    const BrickBlock<T>& b = blk[0];
    double acc = 0.0;
    if (b.own) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (POST && sizeof(T) == 4 && a.acc64) {
                V64* const q = reinterpret_cast<V64*>(reinterpret_cast<char*>(a.acc64 + prob * a.stride) + 2 * (size_t)b.row[i]);
                const V64 v = *q;
                *q = V64{v.x + (double)b.u[2 * i], v.y + (double)b.u[2 * i + 1]};
            } else {
                *pair_at(a.u_out, b.row[i]) = V{b.u[2 * i], b.u[2 * i + 1]};
            }
        }
        if constexpr (RES) {
            T r[8];
            with_walls([&](auto wl) {
#pragma unroll
                for (int c = 0; c < 8; ++c) r[c] = b.f[c] - apply(wl, b, c);
            });
            if constexpr (POST) {
#pragma unroll
                for (int c = 0; c < 8; ++c) acc += (double)r[c] * (double)r[c];
            } else {
                *coarse_at(a.uc, b.coarse) = restrict8(b.u[0], b.u[1], b.u[2], b.u[3], b.u[4], b.u[5], b.u[6], b.u[7]);
                *coarse_at(a.rc, b.coarse) = restrict8(r[0], r[1], r[2], r[3], r[4], r[5], r[6], r[7]);
            }
        }
    }
    return acc;
}

// threads of a pass's workgroup
template <int NU, bool RES, int BS>
constexpr int kBrickThreads = BrickShape<brick_reach(NU, RES), BS>::NT;

template <typename T, int NU, bool POST, bool RHS, bool NORM, int BS>
__global__ __launch_bounds__((kBrickThreads<NU, !POST || NORM, BS>)) void k_brick(BrickArgs<T> a, int first)
{
    using B = BrickShape<brick_reach(NU, !POST || NORM), BS>;
    __shared__ T lds[8 * B::CAP];
    const int per = a.b0 * a.b1 * a.b2;
    // neighbouring bricks share most of what they read: each of the 8 L2 caches (blocks go to
    // them in turn) gets a contiguous eighth of the bricks
    const int share = gridDim.x / 8, more = gridDim.x % 8, xcd = blockIdx.x % 8;
    const int brick = xcd * share + min(xcd, more) + blockIdx.x / 8;
    const int prob = brick / per, w = brick % per;
    if (a.act && !a.act[prob]) return;
    const int bx = w % a.b0, by = (w / a.b0) % a.b1, bz = w / (a.b0 * a.b1);
    const double acc = brick_pass<T, NU, POST, RHS, NORM, BS>(a, first, prob, bx, by, bz, lds);
    if constexpr (NORM) {
        // the brick's own blocks are the first waves': a fixed butterfly over the lanes of each,
        // then the waves in order
        constexpr int OWN = BS * BS * BS / 8 / 64;
        __shared__ double red[OWN];
        double v = acc;
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if constexpr (OWN == 1) {
            if (threadIdx.x == 0) a.partials[(int64_t)prob * per + w] = v;
        } else {
            if ((int)threadIdx.x < 64 * OWN && (threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
            __syncthreads();
            if (threadIdx.x == 0) {
                double s = 0.0;
                for (int i = 0; i < OWN; ++i) s += red[i];
                a.partials[(int64_t)prob * per + w] = s;
            }
        }
    }
}

inline void check_launch()
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw Error(FAS_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

// Bricks of level l of bs^3 cells, for one problem.
int64_t brick_blocks(const fas_grid* g, int l, int bs)
{
    int64_t n = 1;
    for (int a = 0; a < 3; ++a) n *= (g->lev[l].n[a] + bs - 1) / bs;
    return n;
}

// Cells along the axes of level l's bricks: large ones compute 3.9 times what they write, small
// ones 8.25 times, but a large one takes 13 us on a compute unit to itself, two small ones 8.
// Pre + post pass, small against large: 512 small bricks (64^3) 25 and 29 us (FP64), 19 and 24
// (FP32), 768 (96 x 64 x 64) 31 and 31, 25 and 24, 1024 (two 64^3 with norms) 47 and 35, 36
// and 28.  Bricks that a level's axes leave mostly empty are not worth it (one axis of 8: 108
// and 91 us; two: 189 and 261).
int brick_side(const fas_grid* g, int l)
{
    const int64_t small = brick_blocks(g, l, 8);
    return g->batch * small >= kBrickLarge && small >= 3 * brick_blocks(g, l, 16) ? 16 : 8;
}

template <typename T>
BrickArgs<T> make_brick_args(const fas_grid* g, int l, const Coef& c)
{
    const int bs = brick_side(g, l);
    BrickArgs<T> a{};
    a.n0 = g->lev[l].n[0];
    a.n1 = g->lev[l].n[1];
    a.n2 = g->lev[l].n[2];
    a.bc = g->bc;
    a.k = (T)c.kd;
    for (int no = 0; no < 4; ++no) a.q[no] = (T)c.q[diag_count(g->bc, 3, no)];
    a.b0 = (a.n0 + bs - 1) / bs;
    a.b1 = (a.n1 + bs - 1) / bs;
    a.b2 = (a.n2 + bs - 1) / bs;
    a.stride = g->lev[l].N;
    a.cstride = g->lev[l + 1].N;
    a.act = active_flags(g);
    return a;
}

template <typename T, bool POST, bool RHS, bool NORM, int BS>
void launch_brick_side(const fas_grid* g, const BrickArgs<T>& a, int nu, int first)
{
    const unsigned blocks = (unsigned)((int64_t)g->batch * a.b0 * a.b1 * a.b2);
    constexpr bool RES = !POST || NORM;
    if (nu == 1)
        k_brick<T, 1, POST, RHS, NORM, BS><<<blocks, kBrickThreads<1, RES, BS>, 0, g->stream>>>(a, first);
    else if (nu == 2)
        k_brick<T, 2, POST, RHS, NORM, BS><<<blocks, kBrickThreads<2, RES, BS>, 0, g->stream>>>(a, first);
    else
        throw Error(FAS_ERR_ARG, "internal: brick passes take one or two sweeps");
    check_launch();
}

template <typename T, bool POST, bool RHS, bool NORM>
void launch_brick(const fas_grid* g, int l, const BrickArgs<T>& a, int nu, int first)
{
    if (brick_side(g, l) == 8)
        launch_brick_side<T, POST, RHS, NORM, 8>(g, a, nu, first);
    else
        launch_brick_side<T, POST, RHS, NORM, 16>(g, a, nu, first);
}

template <typename T>
void brick_pre(const fas_grid* g, int l, const Coef& c, int first, int nu, const void* f, const void* u_in, void* u_out,
               void* uc, void* rc, void* fout, bool zero)
{
    BrickArgs<T> a = make_brick_args<T>(g, l, c);
    a.f = (const T*)f, a.u_in = (const T*)u_in, a.u_out = (T*)u_out;
    a.uc = (T*)uc, a.rc = (T*)rc, a.fout = (T*)fout, a.zero_in = zero ? 1 : 0;
    if (fout)
        launch_brick<T, false, true, false>(g, l, a, nu, first);
    else
        launch_brick<T, false, false, false>(g, l, a, nu, first);
}

template <typename T>
void brick_post(const fas_grid* g, int l, const Coef& c, int first, int nu, const void* f, const void* u_in,
                const void* uc, void* u_out, double* partials, double* acc64)
{
    BrickArgs<T> a = make_brick_args<T>(g, l, c);
    a.f = (const T*)f, a.u_in = (const T*)u_in, a.u_out = (T*)u_out;
    a.uc = (T*)const_cast<void*>(uc), a.partials = partials, a.acc64 = acc64;
    if (partials)
        launch_brick<T, true, false, true>(g, l, a, nu, first);
    else
        launch_brick<T, true, false, false>(g, l, a, nu, first);
}

}  // namespace

bool brick_ok(const fas_grid* g, int l, int nu_pre, int nu_post, bool variable)
{
    if (!g->fused || g->dim != 3 || variable || l >= g->L) return false;
    if (nu_pre < 1 || nu_pre > 2 || nu_post < 1 || nu_post > 2) return false;
    if (g->lev[l].N * (int64_t)g->elem() > 0xffffffffll) return false;  // 32-bit byte offsets
    const int64_t blocks = g->batch * brick_blocks(g, l, 8);
    // Where marches could run, pre + post pass (us, march against bricks): FP64 512 bricks
    // (64^3) 56 -> 25, 1728 (96^3) 62 -> 33, 4096 (128^3) 74 -> 63, 6144 (192 x 128 x 128) 87
    // and 87, 8000 (160^3) 104 and 113, 32768 (256^3) 262 and 469; marches leave two tiles half
    // empty on 64 columns: 8192 (16 problems of 64^3, norms) 152 -> 123, 24576 (48) 415 -> 358,
    // 49152 683 and 704.  FP32 512 49 -> 19, 4096 54 -> 43, 6144 59 and 60, 8192 (16 of 64^3)
    // 78 and 82; but below the finest level marches need a pass more for the right-hand side:
    // cycles of 384 x 256 x 256 with 6144 bricks there 393 -> 379, of 48 problems of 128^3 with
    // 24576 of 64 columns 1600 -> 1516, of 384^3 with 13824 732 and 746.
    if (fused3_ok(g, l, variable)) {
        // options of the marches hold for every level that can take one
        if (g->seg_force || g->march3_ns == 1) return false;
        if (g->dtype == FAS_F32 && l == 0) return blocks <= kBrickMarch32;
        return blocks <= (g->lev[l].n[0] <= 64 ? kBrickMarchNarrow : kBrickMarch);
    }
    // Elsewhere the per-level kernels are the alternative: their launches cost as much as some
    // `launches` cells, then their time grows with the cells, that of bricks with the bricks
    // however empty they are.  Whole cycles, per-level against bricks (us): full bricks, 1024
    // problems of 32^3 2388 -> 848 (FP64) and 1367 -> 681 (FP32), 48 x 48 x 8192 1430 -> 587,
    // 8 x 8 x 65536 (8192 small ones) 213 and 206, 152 -> 148; partly filled ones, FP64 / FP32:
    //   large, a quarter: 4 x 512 x 512 (1024) 136 -> 125 / 114 -> 103, 4 x 32 x 16384 (2048)
    //     162 and 202 / 143 and 159, 4 x 1024 x 1024 (4096) 278 and 379 / 201 and 288
    //   large, three eighths: 8 x 12 x 65536 (4096) 373 -> 358 / 270 and 285
    //   large, a half: 8 x 1024 x 1024 (4096) 462 -> 415 / 332 -> 319, 8 x 2048 x 2048 (16384)
    //     1845 -> 1614 / 1060 and 1207
    //   small, a quarter: 4 x 4 x 8192 (1024) 78 -> 71 / 74 -> 63, 4 x 4 x 32768 (4096) 90 and
    //     134 / 85 and 105
    //   small, a half: 4 x 8 x 16384 (2048) 91 and 104 / 85 -> 80, 4 x 8 x 65536 153 and 236 /
    //     140 and 177
    const bool large = brick_side(g, l) == 16, f32 = g->dtype == FAS_F32;
    const int64_t cells = large ? (f32 ? 2150 : 1680) : 600;  // that the per-level kernels do in a brick's time
    const int64_t launches = f32 ? (large ? 1300000 : 800000) : 700000;
    const int64_t bricks = large ? g->batch * brick_blocks(g, l, 16) : blocks;
    return bricks * cells <= g->batch * (int64_t)g->lev[l].N + launches;
}

int brick_partials(const fas_grid* g, int l) { return (int)brick_blocks(g, l, brick_side(g, l)); }

void launch_brick_pre(const fas_grid* g, int l, const Coef& c, int first, int nu, const void* f, const void* u_in,
                      void* u_out, void* uc, void* rc, void* fout, bool zero)
{
    if (zero && (fout || g->dtype != FAS_F32))
        throw Error(FAS_ERR_ARG, "internal: a zero-start pre pass is an FP32 pass that forms nothing else");
    if (g->dtype == FAS_F64)
        brick_pre<double>(g, l, c, first, nu, f, u_in, u_out, uc, rc, fout, zero);
    else
        brick_pre<float>(g, l, c, first, nu, f, u_in, u_out, uc, rc, fout, zero);
}

void launch_brick_post(const fas_grid* g, int l, const Coef& c, int first, int nu, const void* f, const void* u_in,
                       const void* uc, void* u_out, double* partials, double* acc64)
{
    if (acc64 && (partials || g->dtype != FAS_F32))
        throw Error(FAS_ERR_ARG, "internal: the accumulating post pass is an FP32 pass without a norm");
    if (g->dtype == FAS_F64)
        brick_post<double>(g, l, c, first, nu, f, u_in, uc, u_out, partials, acc64);
    else
        brick_post<float>(g, l, c, first, nu, f, u_in, uc, u_out, partials, acc64);
}

}  // namespace fas
