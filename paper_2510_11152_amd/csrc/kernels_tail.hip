// Persistent coarse tail: every level from `top` down to the coarsest, in one workgroup
// whose LDS holds u and f of all those levels (Remark 2's recursion below `top`, and
// Remark 1's smoothing on the coarsest level).  One launch replaces a dozen tiny
// launches per level; the per-point formulas are those of fas_device.h, so the values
// are bit-identical to running the per-level kernels.
//
// What bounds it: one compute unit issues every instruction, so a phase costs its
// instruction count on the large levels and its latency chain (LDS reads, the sums, the
// write, a barrier) on the small ones.  Hence
//   - a thread owns a block of 2^d cells, the children of one coarse cell: in each colour
//     phase it updates half of them, half of their neighbours are its own registers, the
//     cells updated are the same for every thread, and restriction and correction need
//     no neighbour at all;
//   - LDS keeps one plane per cell of the block (u and f), indexed by block, so every
//     access of a wave is 64 consecutive values and a neighbour is an index worked out
//     once per visit of a level (index 0 is a zero: the neighbours across a boundary);
//   - levels of at most 64 blocks (16^2, 8^3 and below) run in one wave without block
//     barriers while the other waves wait once.
// With 64^2 to 4^2 (FP64, constant kappa) a launch took 37.2 us with one cell per thread and
// step, all neighbours gathered, and takes 19.5 us now; 16^3 to 4^3 58.8 us and 13.1 us;
// 64^2 with a cell kappa 56.1 us and 38.4 us; 1189 FP32 tails in one launch 168 us and 47 us.
// (A 3D cell kappa needs 36 face weights per block, more registers than 1024 threads have:
// it keeps the gather form, below.)
#include <hip/hip_runtime.h>
#include <string.h>

#include <algorithm>

#include "fas_batch.h"
#include "fas_device.h"
#include "fas_internal.h"
#include "fas_tail.h"

namespace fas {

namespace {

// 512 threads: 256 VGPRs each, so that a thread can own several blocks (u, f, the diagonal
// or face weights of up to 5 blocks stay in registers; with 1024 threads 3D blocks spill).
constexpr int kTailThreads = 512;
constexpr int kTailThreadsK3 = 1024;
constexpr int kTailLds = 96 * 1024;     // budget of tail_top(): bytes of u and f of the tail levels
constexpr int kTailLdsKV = 156 * 1024;  // cell kappa: u and f, and in 2D the face weights of one
                                        // level (3D: kappa per level)

// One level as blocks of 2^d cells (an odd axis of the coarsest level ends in half a block).
template <typename T>
struct TailLevel {
    int n0, n1, n2;      // cells per axis
    int m0, m1, m2;      // blocks per axis
    int nb;              // blocks
    int off;             // index of the level's first block in the LDS planes
    unsigned g0, g01;    // ceil(2^32 / m0), ceil(2^32 / (m0 m1)) (0: divide by one)
    T k;
    T q[4];              // 1 / (1 + k W) with 0 .. 3 boundary faces
    const T* kap;        // cell kappa, or nullptr
};

template <typename T>
struct TailArgs {
    int nl;                   // levels in the tail (top .. coarsest)
    int one;                  // first level run by a single wave (nl: none)
    int pre, post, nuc;       // sweeps
    int first;                // parity of the first phase of a sweep
    int form_rhs;             // 1: f_top = r_top + A u_top (FAS coarse right-hand side)
    int bc;
    TailLevel<T> lev[kMaxTail];
    T* u_top;                 // in: initial guess of the top level; out: its new values
    const T* r_top;           // in: restricted residual (form_rhs) or the right-hand side
    int64_t stride;           // batched grids: problem b = blockIdx.x at b * stride
    const int* act;           // per-problem active flags (nullable)
};

// Blocks one LDS plane holds, and blocks a thread owns on the largest level of a tail of
// several levels (tail_kb) and of a coarsest level alone (tail_kb_one).  Small: tails from at
// most 64^2 or 16^3 cells; big: all that the byte budget admits (tail_class).  A coarsest level
// alone may take the whole budget, and an odd axis of it ends in half blocks: up to 1554 blocks
// in FP64 and 3087 in FP32 (2D, constant kappa), where the top of several levels has at most
// 1228 and 2457.  Cycles with such a tail against the cell-per-thread form: 220^2 FP32
// (coarsest 110) 50 -> 46 us, 148 x 166 FP64 (coarsest 74) 46 -> 39 us, 36 x 1200 FP32
// (coarsest 18) 81 -> 44 us.
constexpr int tail_cap(int dim, bool big, size_t s)
{
    return dim == 2 ? (!big ? 1368 : (s == 8 ? 1568 : 3120)) : (!big ? 600 : (s == 8 ? 1112 : 2224));
}
constexpr int tail_kb(int dim, bool big, size_t s) { return !big ? (dim == 2 ? 2 : 1) : (s == 8 ? 3 : 5); }
constexpr int tail_kb_one(int dim, bool big, size_t s, bool kv)
{
    return big && dim == 2 && !kv ? (s == 8 ? 4 : 7) : tail_kb(dim, big, s);
}

__device__ __forceinline__ int div_by(int t, unsigned g) { return g ? (int)__umulhi((unsigned)t, g) : t; }

// A thread's block on one level.  Cell c of the block is (c & 1, c >> 1 & 1, c >> 2).
// LEAN (big tails): f stays in LDS and the diagonal is picked at each use, for registers.
template <typename T, int DIM, bool KV, bool LEAN>
struct TailBlock {
    static constexpr int C = 1 << DIM;
    bool on;            // the level has this block
    int o;              // LDS index of the block
    int nb[2 * DIM];    // LDS indices of the neighbouring blocks (x-, x+, y-, y+, z-, z+), 0 outside
    int I, J, K;
    bool lo[DIM], hi[DIM];  // the cells at 0 / at 1 along an axis have a boundary face
    unsigned valid;         // cells inside the level (half blocks)
    T u[C], f[LEAN ? 1 : C];
    T q[KV || LEAN ? 1 : C];
    // 2D cell kappa: face weights (rows y of x faces, columns x of y faces: before, inside and
    // after the block) and 1 + k Wt of each cell
    T wx[KV ? 3 : 1][2], wy[KV ? 3 : 1][2], d[KV ? C : 1];
};

template <typename T, int DIM, bool KV, bool BIG>
struct Tail {
    static constexpr int C = 1 << DIM;
    static constexpr int CAP = tail_cap(DIM, BIG, sizeof(T)), KB = tail_kb(DIM, BIG, sizeof(T));
    static constexpr int KB1 = tail_kb_one(DIM, BIG, sizeof(T), KV);
    static constexpr int PLANES = (KV ? 3 : 2) * C;
    using Block = TailBlock<T, DIM, KV, BIG>;
    using Level = TailLevel<T>;
    static_assert(!KV || DIM == 2, "2D cell kappa");
    static_assert((size_t)PLANES * CAP * sizeof(T) <= 160 * 1024, "LDS of one workgroup");

    const TailArgs<T>& a;
    T* const lds;

    __device__ __forceinline__ T* U(int c) const { return lds + c * CAP; }
    __device__ __forceinline__ T* F(int c) const { return lds + (C + c) * CAP; }
    __device__ __forceinline__ T* KP(int c) const { return lds + (2 * C + c) * CAP; }

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

    // v[W] of a cell with W = 0 .. DIM boundary faces, from the flags of cell c.
    static __device__ __forceinline__ T by_faces(const Block& B, int c, T v0, T v1, T v2, T v3)
    {
        const bool x = c & 1 ? B.hi[0] : B.lo[0], y = c & 2 ? B.hi[1] : B.lo[1];
        if constexpr (DIM == 2) {
            return x && y ? v2 : (x || y ? v1 : v0);
        } else {
            const bool z = c & 4 ? B.hi[2] : B.lo[2];
            const bool all = x && y && z, two = (x && y) || (x && z) || (y && z), any = x || y || z;
            return all ? v3 : (two ? v2 : (any ? v1 : v0));
        }
    }
    // The diagonal count W of cell c.
    __device__ __forceinline__ T diag_of(const Block& B, int c) const
    {
        const T d = a.bc == BC_DIRICHLET ? (T)1 : (T)-1;
        return by_faces(B, c, (T)(2 * DIM), (T)(2 * DIM) + d, (T)(2 * DIM) + (d + d), (T)(2 * DIM) + (d + d + d));
    }

    // 1 / (1 + k W) of cell c.
    static __device__ __forceinline__ T pick_q(const Level& L, const Block& B, int c)
    {
        return by_faces(B, c, L.q[0], L.q[1], L.q[2], L.q[3]);
    }
    __device__ __forceinline__ T f_of(const Block& B, int c) const
    {
        if constexpr (BIG)
            return F(c)[B.o];
        else
            return B.f[c];
    }

    // ODD: the level may end in half blocks (the coarsest only).
    template <bool ODD>
    __device__ __forceinline__ void setup(const Level& L, int t, Block& B) const
    {
        B.on = t < L.nb;
        if (!B.on) t = 0;
        const bool per = a.bc == BC_PERIODIC;
        const int K = DIM == 3 ? div_by(t, L.g01) : 0;
        const int r = DIM == 3 ? t - K * (L.m0 * L.m1) : t;
        const int J = div_by(r, L.g0), I = r - J * L.m0;
        B.I = I, B.J = J, B.K = K;
        B.o = L.off + t;
        const int pos[3] = {I, J, K}, m[3] = {L.m0, L.m1, L.m2}, n[3] = {L.n0, L.n1, L.n2};
        const int step[3] = {1, L.m0, L.m0 * L.m1};
#pragma unroll
        for (int x = 0; x < DIM; ++x) {
            const bool lo = pos[x] == 0, hi = pos[x] == m[x] - 1, half = ODD && 2 * pos[x] + 1 == n[x];
            B.nb[2 * x] = !lo ? B.o - step[x] : (per ? B.o + (m[x] - 1) * step[x] : 0);
            B.nb[2 * x + 1] = !hi ? B.o + step[x] : (per ? B.o - (m[x] - 1) * step[x] : 0);
            // (an axis that ends in half a block has more than one block: lo and half differ)
            B.lo[x] = !per && (lo || half);
            B.hi[x] = !per && hi;
        }
        B.valid = (1u << C) - 1;
        if constexpr (ODD) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                bool in = 2 * I + (c & 1) < L.n0 && 2 * J + ((c >> 1) & 1) < L.n1;
                if constexpr (DIM == 3) in = in && 2 * K + (c >> 2) < L.n2;
                if (!in) B.valid &= ~(1u << c);
            }
        }
        if constexpr (!KV && !BIG) {
#pragma unroll
            for (int c = 0; c < C; ++c) B.q[c] = pick_q(L, B, c);
        } else if constexpr (KV) {
            // harmonic means in the argument order of fas_device.h's gather; a boundary face
            // weighs 2 kappa of its cell (Dirichlet) or 0
            const bool dir = a.bc == BC_DIRICHLET;
            T kp[C];
#pragma unroll
            for (int c = 0; c < C; ++c) kp[c] = KP(c)[B.o];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int xa = 2 * s, xb = 2 * s + 1;  // row s: cells at x = 0, 1
                const int ya = s, yb = s + 2;          // column s: cells at y = 0, 1
                const T wb0 = dir ? (T)2 * kp[xa] : (T)0, wb1 = dir ? (T)2 * kp[xb] : (T)0;
                const T vb0 = dir ? (T)2 * kp[ya] : (T)0, vb1 = dir ? (T)2 * kp[yb] : (T)0;
                B.wx[0][s] = B.nb[0] ? face_w(KP(xb)[B.nb[0]], kp[xa]) : wb0;
                B.wx[1][s] = B.valid >> xb & 1 ? face_w(kp[xa], kp[xb]) : wb0;
                B.wx[2][s] = B.nb[1] ? face_w(kp[xb], KP(xa)[B.nb[1]]) : wb1;
                B.wy[0][s] = B.nb[2] ? face_w(KP(yb)[B.nb[2]], kp[ya]) : vb0;
                B.wy[1][s] = B.valid >> yb & 1 ? face_w(kp[ya], kp[yb]) : vb0;
                B.wy[2][s] = B.nb[3] ? face_w(kp[yb], KP(ya)[B.nb[3]]) : vb1;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int x = c & 1, y = c >> 1;
                const T Wt = (B.wx[x][y] + B.wx[x + 1][y]) + (B.wy[y][x] + B.wy[y + 1][x]);
                B.d[c] = (T)1 + L.k * Wt;
            }
        }
    }

    // Neighbour values of cell c (slot order x-, x+, y-, y+, z-, z+): inside the block from
    // registers, else from the neighbouring block's plane.
    __device__ __forceinline__ void neighbours(const Block& B, int c, T (&v)[2 * DIM]) const
    {
#pragma unroll
        for (int x = 0; x < DIM; ++x) {
            const int o = c ^ (1 << x);
            const bool hi = (c >> x) & 1;
            v[2 * x] = hi ? B.u[o] : U(o)[B.nb[2 * x]];
            v[2 * x + 1] = hi ? U(o)[B.nb[2 * x + 1]] : B.u[o];
        }
    }

    __device__ __forceinline__ T wsum_of(const Block& B, int c, const T (&v)[2 * DIM]) const
    {
        const int x = c & 1, y = (c >> 1) & 1;
        return (B.wx[x][y] * v[0] + B.wx[x + 1][y] * v[1]) + (B.wy[y][x] * v[2] + B.wy[y + 1][x] * v[3]);
    }

    // (A u) of cell c (fas_device.h's apply_value).
    __device__ __forceinline__ T apply(const Level& L, const Block& B, int c) const
    {
        T v[2 * DIM];
        neighbours(B, c, v);
        if constexpr (!KV) {
            const T S = nbsum<T, DIM>(v);
            const T W = diag_of(B, c);
            return B.u[c] + L.k * (W * B.u[c] - S);
        } else {
            const int x = c & 1, y = (c >> 1) & 1;
            const T Sw = wsum_of(B, c, v);
            const T Wt = (B.wx[x][y] + B.wx[x + 1][y]) + (B.wy[y][x] + B.wy[y + 1][x]);
            return B.u[c] + L.k * (Wt * B.u[c] - Sw);
        }
    }

    // One colour phase: the cells of parity P of the block (fas_device.h's gs_value).
    template <int P, bool ODD>
    __device__ __forceinline__ void phase(const Level& L, Block& B) const
    {
        T nv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if ((((c & 1) + ((c >> 1) & 1) + (c >> 2)) & 1) != P) continue;
            T v[2 * DIM];
            neighbours(B, c, v);
            const T f = f_of(B, c);
            if constexpr (KV)
                nv[c] = (f + L.k * wsum_of(B, c, v)) / B.d[c];
            else if constexpr (BIG)
                nv[c] = (f + L.k * nbsum<T, DIM>(v)) * pick_q(L, B, c);
            else
                nv[c] = (f + L.k * nbsum<T, DIM>(v)) * B.q[c];
            if constexpr (ODD) nv[c] = B.valid >> c & 1 ? nv[c] : (T)0;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if ((((c & 1) + ((c >> 1) & 1) + (c >> 2)) & 1) != P) continue;
            B.u[c] = nv[c];
            U(c)[B.o] = nv[c];
        }
    }

    template <int NB, bool ONE, bool ODD>
    __device__ __forceinline__ void smooth(const Level& L, Block (&B)[NB], int sweeps) const
    {
        for (int s = 0; s < 2 * sweeps; ++s) {
            if (((s & 1) ^ a.first) != 0) {
#pragma unroll
                for (int k = 0; k < NB; ++k)
                    if (B[k].on) phase<1, ODD>(L, B[k]);
            } else {
#pragma unroll
                for (int k = 0; k < NB; ++k)
                    if (B[k].on) phase<0, ODD>(L, B[k]);
            }
            sync<ONE>();
        }
    }

    // LDS index, and cell, of the coarse cell that block B's cells form.
    __device__ __forceinline__ int coarse_at(const Level& Lc, const Block& B) const
    {
        int p = Lc.off + (B.I >> 1) + Lc.m0 * (B.J >> 1);
        int c = (B.I & 1) + 2 * (B.J & 1);
        if constexpr (DIM == 3) {
            p += Lc.m0 * Lc.m1 * (B.K >> 1);
            c += 4 * (B.K & 1);
        }
        return c * CAP + p;
    }

    static __device__ __forceinline__ T restricted(const T (&x)[C])
    {
        if constexpr (DIM == 2)
            return restrict4(x[0], x[1], x[2], x[3]);
        else
            return restrict8(x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]);
    }

    __device__ __forceinline__ int64_t cell_of(const Level& L, const Block& B, int c) const
    {
        return cell_index(L.n0, L.n1, 2 * B.I + (c & 1), 2 * B.J + ((c >> 1) & 1), DIM == 3 ? 2 * B.K + (c >> 2) : 0);
    }

    // Own cells of every block from LDS, or on the top level (gu != nullptr) from memory into
    // registers and LDS.
    template <int NB, bool ONE, bool ODD>
    __device__ __forceinline__ void load(const Level& L, Block (&B)[NB], const T* gu, const T* gr) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) setup<ODD>(L, (int)threadIdx.x + k * kTailThreads, B[k]);
        if (!gu) {
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                if (!B[k].on) continue;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    B[k].u[c] = U(c)[B[k].o];
                    if constexpr (ODD) B[k].u[c] = B[k].valid >> c & 1 ? B[k].u[c] : (T)0;
                    if constexpr (!BIG) B[k].f[c] = F(c)[B[k].o];
                }
            }
            return;
        }
        // every load of the thread is issued before the first use (blocks that are not there
        // read block 0)
        T fv[NB][C];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
#pragma unroll
            for (int c = 0; c < C; c += 2) {
                const int64_t p = cell_of(L, B[k], c);
                if constexpr (!ODD) {
                    // the row's cell pair (base pointers need not be aligned to pairs)
                    typedef T V __attribute__((ext_vector_type(2), aligned(sizeof(T))));
                    const V vu = *reinterpret_cast<const V*>(gu + p), vf = *reinterpret_cast<const V*>(gr + p);
                    B[k].u[c] = vu.x, B[k].u[c + 1] = vu.y;
                    fv[k][c] = vf.x, fv[k][c + 1] = vf.y;
                } else {
                    const bool in0 = B[k].valid >> c & 1, in1 = B[k].valid >> (c + 1) & 1;
                    B[k].u[c] = in0 ? gu[p] : (T)0, B[k].u[c + 1] = in1 ? gu[p + 1] : (T)0;
                    fv[k][c] = in0 ? gr[p] : (T)0, fv[k][c + 1] = in1 ? gr[p + 1] : (T)0;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                U(c)[B[k].o] = B[k].u[c];
                F(c)[B[k].o] = fv[k][c];
                if constexpr (!BIG) B[k].f[c] = fv[k][c];
            }
        }
        sync<ONE>();
    }

    // f = r + A u in place (the level's f holds r).
    template <int NB, bool ONE>
    __device__ __forceinline__ void form(const Level& L, Block (&B)[NB]) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T f = f_of(B[k], c) + apply(L, B[k], c);
                if constexpr (!BIG) B[k].f[c] = f;
                F(c)[B[k].o] = f;
            }
        }
        sync<ONE>();
    }

    // Down: pre-smoothing, then u_c = R u and r_c = R (f - A u).
    template <int NB, bool ONE>
    __device__ __forceinline__ void down(int lv, const T* gu, const T* gr) const
    {
        const Level& L = a.lev[lv];
        const Level& Lc = a.lev[lv + 1];
        Block B[NB];
        load<NB, ONE, false>(L, B, gu, gr);
        if (lv > 0 || a.form_rhs) form<NB, ONE>(L, B);
        smooth<NB, ONE, false>(L, B, a.pre);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
            T r[C];
#pragma unroll
            for (int c = 0; c < C; ++c) r[c] = f_of(B[k], c) - apply(L, B[k], c);
            const int p = coarse_at(Lc, B[k]);
            U(0)[p] = restricted(B[k].u);
            F(0)[p] = restricted(r);
        }
        sync<ONE>();
    }

    // Coarsest level: smoothing only (Remark 1).
    template <int NB, bool ONE>
    __device__ __forceinline__ void coarsest(const T* gu, const T* gr, T* gout) const
    {
        const Level& L = a.lev[a.nl - 1];
        Block B[NB];
        load<NB, ONE, true>(L, B, gu, gr);
        if (a.nl > 1 || a.form_rhs) form<NB, ONE>(L, B);
        smooth<NB, ONE, true>(L, B, a.nuc);
        if (gout) store<NB>(L, B, gout);
    }

    // Up: u += P (u_c - R u), post-smoothing.
    template <int NB, bool ONE>
    __device__ __forceinline__ void up(int lv, T* gout) const
    {
        const Level& L = a.lev[lv];
        const Level& Lc = a.lev[lv + 1];
        Block B[NB];
        load<NB, ONE, false>(L, B, nullptr, nullptr);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
            const T c = U(0)[coarse_at(Lc, B[k])] - restricted(B[k].u);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                B[k].u[i] = B[k].u[i] + c;
                U(i)[B[k].o] = B[k].u[i];
            }
        }
        sync<ONE>();
        smooth<NB, ONE, false>(L, B, a.post);
        if (gout) store<NB>(L, B, gout);
    }

    template <int NB>
    __device__ __forceinline__ void store(const Level& L, Block (&B)[NB], T* gout) const
    {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (!B[k].on) continue;
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (B[k].valid >> c & 1) gout[cell_of(L, B[k], c)] = B[k].u[c];
        }
    }

    // The tail of one problem: its top level's u (in and out) and r (or f).
    __device__ __forceinline__ void run(T* const u_top, const T* const r_top) const
    {
        const int last = a.nl - 1;
        if (threadIdx.x < (unsigned)C) U((int)threadIdx.x)[0] = (T)0;
        if constexpr (KV) {
            for (int l = 0; l < a.nl; ++l) {
                const Level& L = a.lev[l];
                const int N = L.n0 * L.n1;
                for (int p = threadIdx.x; p < N; p += kTailThreads) {
                    const int j = p / L.n0, i = p - j * L.n0;
                    KP((i & 1) + 2 * (j & 1))[L.off + (i >> 1) + L.m0 * (j >> 1)] = L.kap[p];
                }
            }
        }
        __syncthreads();
        // blocks per level fall by 2^d, so one wave runs the levels from a.one on
        // (each step has one call in each of the two forms: the code is large, and a launch
        // fetches it anew)
        for (int l = 0; l < a.one && l < last; ++l) down<KB, false>(l, l ? nullptr : u_top, l ? nullptr : r_top);
        if (a.one < a.nl) {
            if (threadIdx.x < 64) {
                for (int l = a.one; l < last; ++l) down<1, true>(l, l ? nullptr : u_top, l ? nullptr : r_top);
                coarsest<1, true>(last ? nullptr : u_top, last ? nullptr : r_top, last ? nullptr : u_top);
                for (int l = last - 1; l >= a.one; --l) up<1, true>(l, l ? nullptr : u_top);
            }
            __syncthreads();
        } else {
            coarsest<KB1, false>(last ? nullptr : u_top, last ? nullptr : r_top, last ? nullptr : u_top);
        }
        for (int l = (a.one < last ? a.one : last) - 1; l >= 0; --l) up<KB, false>(l, l ? nullptr : u_top);
    }
};

// Problem b = blockIdx.x of a stacked batch (arrays b * stride apart).
template <typename T, int DIM, bool KV, bool BIG>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs<T> args)
{
    // levels are picked at run time: read the arguments where they are, as constants (a copy
    // would go through scratch)
    (void)args;
    const TailArgs<T>& a = *(const TailArgs<T>*)(const __attribute__((address_space(4))) TailArgs<T>*)
                               __builtin_amdgcn_kernarg_segment_ptr();
    if (a.act && !a.act[blockIdx.x]) return;
    using Tl = Tail<T, DIM, KV, BIG>;
    __shared__ T lds[Tl::PLANES * Tl::CAP];
    const Tl tail{a, lds};
    tail.run(a.u_top + blockIdx.x * a.stride, a.r_top + blockIdx.x * a.stride);
}

// Table launch (array-form batches, 2D): problem blockIdx.x's descriptor.
template <typename T, bool KV, bool BIG>
__global__ __launch_bounds__(kTailThreads) void k_tail_table(TableLaunch tl)
{
    // descriptors do not change during a launch: read them as constants (scalar loads)
    const TailArgs<T>& a = *(const TailArgs<T>*)(const __attribute__((address_space(4))) TailArgs<T>*)(
        reinterpret_cast<uintptr_t>(tl.desc[blockIdx.x]));
    if (a.act && !a.act[0]) return;
    using Tl = Tail<T, 2, KV, BIG>;
    __shared__ T lds[Tl::PLANES * Tl::CAP];
    const Tl tail{a, lds};
    tail.run(a.u_top, a.r_top);
}

// ---- 3D cell kappa: u, f and kappa of every level in LDS, neighbours gathered per cell ------
template <typename T>
struct TailArgsK3 {
    int nl, pre, post, nuc, first, form_rhs;  // as TailArgs
    int lds_off[kMaxTail];    // element offset of u of each level; f follows u
    int kap_off[kMaxTail];    // element offset of each level's kappa copy
    Op<T> op[kMaxTail];
    T* u_top;
    const T* r_top;
    const int* act;
};

// Cells are visited row by row: the 1024 threads form TX columns by kTailThreadsK3 / TX
// rows (x fastest), TX the smallest power of two >= the row's work items (at most 32), so
// narrow levels keep every lane busy and no thread divides by a level size.
constexpr int kTX = 32;
struct TMap {
    int tx, ty, TX, TY;
};
__device__ __forceinline__ TMap tmap(int width)
{
    int lg = 0;
    while ((1 << lg) < width && (1 << lg) < kTX) ++lg;
    return TMap{(int)threadIdx.x & ((1 << lg) - 1), (int)threadIdx.x >> lg, 1 << lg, kTailThreadsK3 >> lg};
}

template <typename T>
__device__ void tail_smooth_k3(const Op<T>& op, T* U, const T* F, int sweeps, int first)
{
    const int half = (op.n0 + 1) >> 1;
    const int rows = op.n1 * op.n2;
    const TMap m = tmap(half);
    for (int s = 0; s < 2 * sweeps; ++s) {
        const int parity = (s & 1) ^ first;
        for (int row = m.ty; row < rows; row += m.TY) {
            const int l = row / op.n1, j = row - l * op.n1;
            const int odd = (parity + j + l) & 1;
            for (int tt = m.tx; tt < half; tt += m.TX) {
                const int i = 2 * tt + odd;
                if (i >= op.n0) continue;
                Nbhd<T, 3> nb;
                gather<T, 3, true>(op, U, i, j, l, nb);
                const int p = (int)cell_index(op.n0, op.n1, i, j, l);
                U[p] = gs_value<T, 3, true>(op, nb, F[p]);
            }
        }
        __syncthreads();
    }
}

template <typename T>
__global__ __launch_bounds__(kTailThreadsK3) void k_tail_k3(TailArgsK3<T> a)
{
    if (a.act && !a.act[0]) return;
    T* const u_top = a.u_top;
    const T* const r_top = a.r_top;
    __shared__ __attribute__((aligned(16))) char lds[kTailLdsKV];
    T* base = reinterpret_cast<T*>(lds);
    auto U = [&](int l) { return base + a.lds_off[l]; };
    auto F = [&](int l) { return base + a.lds_off[l] + (a.op[l].n0 * a.op[l].n1 * a.op[l].n2); };
    // the operator of level l, its cell kappa read from the LDS copy
    auto OP = [&](int l) {
        Op<T> o = a.op[l];
        o.kap = base + a.kap_off[l];
        return o;
    };
    const int N0 = a.op[0].n0 * a.op[0].n1 * a.op[0].n2;
    for (int p = threadIdx.x; p < N0; p += kTailThreadsK3) {
        U(0)[p] = u_top[p];
        F(0)[p] = r_top[p];
    }
    for (int l = 0; l < a.nl; ++l) {
        const int Nl = a.op[l].n0 * a.op[l].n1 * a.op[l].n2;
        T* const kl = base + a.kap_off[l];
        const T* const kg = a.op[l].kap;
        for (int p = threadIdx.x; p < Nl; p += kTailThreadsK3) kl[p] = kg[p];
    }
    __syncthreads();
    // f = r + A u of a level whose f holds r
    auto form = [&](int lv) {
        const Op<T> op = OP(lv);
        const TMap m = tmap(op.n0);
        for (int row = m.ty; row < op.n1 * op.n2; row += m.TY) {
            const int l = row / op.n1, j = row - l * op.n1;
            for (int i = m.tx; i < op.n0; i += m.TX) {
                const int p = (int)cell_index(op.n0, op.n1, i, j, l);
                Nbhd<T, 3> nb;
                gather<T, 3, true>(op, U(lv), i, j, l, nb);
                F(lv)[p] = F(lv)[p] + apply_value<T, 3, true>(op, nb, U(lv)[p]);
            }
        }
        __syncthreads();
    };
    if (a.form_rhs) form(0);
    // descend: pre-smoothing, then u_c = R u, f_c = R (f - A u) + A_c u_c
    for (int lv = 0; lv + 1 < a.nl; ++lv) {
        const Op<T> op = OP(lv);
        const Op<T> oc = OP(lv + 1);
        T* u = U(lv);
        const T* f = F(lv);
        tail_smooth_k3<T>(op, u, f, a.pre, a.first);
        const TMap m = tmap(oc.n0);
        for (int crow = m.ty; crow < oc.n1 * oc.n2; crow += m.TY)
        for (int I = m.tx; I < oc.n0; I += m.TX) {
            const int K = crow / oc.n1, J = crow - K * oc.n1;
            const int P = (int)cell_index(oc.n0, oc.n1, I, J, K);
            T uu[8], rr[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int i = 2 * I + (c & 1), j = 2 * J + ((c >> 1) & 1), l = 2 * K + (c >> 2);
                const int p = (int)cell_index(op.n0, op.n1, i, j, l);
                Nbhd<T, 3> nb;
                gather<T, 3, true>(op, u, i, j, l, nb);
                uu[c] = u[p];
                rr[c] = f[p] - apply_value<T, 3, true>(op, nb, uu[c]);
            }
            U(lv + 1)[P] = restrict8(uu[0], uu[1], uu[2], uu[3], uu[4], uu[5], uu[6], uu[7]);
            F(lv + 1)[P] = restrict8(rr[0], rr[1], rr[2], rr[3], rr[4], rr[5], rr[6], rr[7]);
        }
        __syncthreads();
        form(lv + 1);
    }
    // coarsest level: smoothing only (Remark 1)
    tail_smooth_k3<T>(OP(a.nl - 1), U(a.nl - 1), F(a.nl - 1), a.nuc, a.first);
    // ascend: u += P(u_c - R u), post-smoothing
    for (int lv = a.nl - 2; lv >= 0; --lv) {
        const Op<T> op = OP(lv);
        const Op<T> oc = OP(lv + 1);
        T* u = U(lv);
        const TMap m = tmap(oc.n0);
        for (int crow = m.ty; crow < oc.n1 * oc.n2; crow += m.TY)
        for (int I = m.tx; I < oc.n0; I += m.TX) {
            const int K = crow / oc.n1, J = crow - K * oc.n1;
            const int P = (int)cell_index(oc.n0, oc.n1, I, J, K);
            const int i = 2 * I, j = 2 * J, l = 2 * K;
            const T old = restrict8(
                u[cell_index(op.n0, op.n1, i, j, l)], u[cell_index(op.n0, op.n1, i + 1, j, l)],
                u[cell_index(op.n0, op.n1, i, j + 1, l)], u[cell_index(op.n0, op.n1, i + 1, j + 1, l)],
                u[cell_index(op.n0, op.n1, i, j, l + 1)], u[cell_index(op.n0, op.n1, i + 1, j, l + 1)],
                u[cell_index(op.n0, op.n1, i, j + 1, l + 1)], u[cell_index(op.n0, op.n1, i + 1, j + 1, l + 1)]);
            const T c = U(lv + 1)[P] - old;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const int p = (int)cell_index(op.n0, op.n1, i + (ch & 1), j + ((ch >> 1) & 1), l + (ch >> 2));
                u[p] = u[p] + c;
            }
        }
        __syncthreads();
        tail_smooth_k3<T>(op, u, F(lv), a.post, a.first);
    }
    for (int p = threadIdx.x; p < N0; p += kTailThreadsK3) u_top[p] = U(0)[p];
}

unsigned div_magic(int64_t d) { return d > 1 ? (unsigned)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; }

template <typename T>
TailArgs<T> make_tail_args(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first)
{
    TailArgs<T> a{};
    a.nl = g->L - top + 1;
    a.one = a.nl;
    a.pre = pre;
    a.post = post;
    a.nuc = g->nuc;
    a.first = first;
    a.bc = g->bc;
    int off = 1;  // block 0: the zeros across a boundary
    for (int i = 0; i < a.nl; ++i) {
        const int l = top + i;
        TailLevel<T>& L = a.lev[i];
        L.n0 = g->lev[l].n[0];
        L.n1 = g->lev[l].n[1];
        L.n2 = g->lev[l].n[2];
        L.m0 = (L.n0 + 1) / 2;
        L.m1 = (L.n1 + 1) / 2;
        L.m2 = g->dim == 3 ? (L.n2 + 1) / 2 : 1;
        L.nb = L.m0 * L.m1 * L.m2;
        L.off = off;
        off += L.nb;
        L.g0 = div_magic(L.m0);
        L.g01 = div_magic((int64_t)L.m0 * L.m1);
        L.k = (T)coef[l].kd;
        for (int no = 0; no <= g->dim; ++no) L.q[no] = (T)coef[l].q[diag_count(g->bc, g->dim, no)];
        L.kap = (const T*)g->lev[l].kap;
        if (L.nb <= 64 && a.one == a.nl) a.one = i;
    }
    if (tail_class(g, top) < 0) throw Error(FAS_ERR_ARG, "internal: tail levels exceed the tail's LDS");
    return a;
}

template <typename T>
TailArgsK3<T> make_tail_args_k3(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first)
{
    TailArgsK3<T> a{};
    a.nl = g->L - top + 1;
    a.pre = pre;
    a.post = post;
    a.nuc = g->nuc;
    a.first = first;
    int off = 0;
    for (int i = 0; i < a.nl; ++i) {
        const int l = top + i;
        Op<T>& op = a.op[i];
        op.n0 = g->lev[l].n[0];
        op.n1 = g->lev[l].n[1];
        op.n2 = g->lev[l].n[2];
        op.bc = g->bc;
        op.k = (T)coef[l].kd;
        for (int W = 0; W < 16; ++W) op.q[W] = (T)coef[l].q[W];
        op.kap = (const T*)g->lev[l].kap;
        a.lds_off[i] = off;
        off += 2 * (int)g->lev[l].N;
    }
    for (int i = 0; i < a.nl; ++i) {  // copies after every level's u and f
        a.kap_off[i] = off;
        off += (int)g->lev[top + i].N;
    }
    if ((size_t)off * sizeof(T) > (size_t)kTailLdsKV)
        throw Error(FAS_ERR_ARG, "internal: tail levels exceed the tail's LDS");
    return a;
}

inline void check_launch()
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw Error(FAS_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

template <typename T>
void launch_t(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first, void* u, const void* r,
              int form_rhs)
{
    const unsigned nb = (unsigned)g->batch;
    const bool kv = g->lev[top].kap != nullptr;
    if (kv && g->dim == 3) {  // single-problem grids
        TailArgsK3<T> a = make_tail_args_k3<T>(g, top, coef, pre, post, first);
        a.u_top = (T*)u;
        a.r_top = (const T*)r;
        a.form_rhs = form_rhs;
        a.act = active_flags(g);
        k_tail_k3<T><<<1, kTailThreadsK3, 0, g->stream>>>(a);
        check_launch();
        return;
    }
    TailArgs<T> a = make_tail_args<T>(g, top, coef, pre, post, first);
    a.u_top = (T*)u;
    a.r_top = (const T*)r;
    a.form_rhs = form_rhs;
    a.stride = g->lev[top].N;
    a.act = active_flags(g);
    const bool big = tail_class(g, top) == 1;
#define FAS_TAIL(DIM_, KV_)                                                             \
    do {                                                                                \
        if (big)                                                                        \
            k_tail<T, DIM_, KV_, true><<<nb, kTailThreads, 0, g->stream>>>(a);          \
        else                                                                            \
            k_tail<T, DIM_, KV_, false><<<nb, kTailThreads, 0, g->stream>>>(a);         \
    } while (0)
    if (g->dim == 3)
        FAS_TAIL(3, false);
    else if (kv)
        FAS_TAIL(2, true);
    else
        FAS_TAIL(2, false);
#undef FAS_TAIL
    check_launch();
}

}  // namespace

int tail_class(const fas_grid* g, int top)
{
    const bool kv = (g->flags & FAS_FLAG_VARIABLE_KAPPA) != 0;
    const size_t s = g->elem();
    int64_t blocks = 1, most = 0;  // block 0: the zeros across a boundary
    for (int l = top; l <= g->L; ++l) {
        int64_t nb = 1;
        for (int a = 0; a < g->dim; ++a) nb *= (g->lev[l].n[a] + 1) / 2;
        blocks += nb;
        most = std::max(most, nb);
    }
    for (int big = 0; big < 2; ++big) {
        const int kb = top == g->L ? tail_kb_one(g->dim, big, s, kv) : tail_kb(g->dim, big, s);
        if (blocks <= tail_cap(g->dim, big, s) && most <= (int64_t)kTailThreads * kb) return big;
    }
    return -1;
}

int tail_top(const fas_grid* g)
{
    // the largest level from which every coarser level's u and f (and, on a grid that may
    // take a cell kappa, the top level's face tables in 2D or every level's kappa in 3D) fit
    // the budget in bytes, and whose blocks the planes and the threads hold
    const size_t s = g->elem();
    const bool kv = (g->flags & FAS_FLAG_VARIABLE_KAPPA) != 0;
    const size_t cap = kv ? (size_t)kTailLdsKV : (size_t)kTailLds;
    size_t bytes = 0;
    int top = g->L + 1;
    for (int l = g->L; l >= 0; --l) {
        bytes += (kv && g->dim == 3 ? 3 : 2) * (size_t)g->lev[l].N * s;
        const int64_t n0 = g->lev[l].n[0], n1 = g->lev[l].n[1];
        const size_t faces = kv && g->dim == 2 ? (size_t)((n0 + 1) * n1 + n0 * (n1 + 1)) * s : 0;
        if (bytes + faces > cap || g->L - l + 1 > kMaxTail || tail_class(g, l) < 0) break;
        top = l;
    }
    return top;  // L + 1: not even the coarsest level fits
}

size_t tail_desc_bytes(int dtype)
{
    return dtype == FAS_F64 ? sizeof(TailArgs<double>) : sizeof(TailArgs<float>);
}

template <typename T>
bool fill_tail_desc_t(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first, void* u,
                      const void* r, bool form_rhs, const int* act, void* out)
{
    TailArgs<T> a = make_tail_args<T>(g, top, coef, pre, post, first);
    a.u_top = (T*)u;
    a.r_top = (const T*)r;
    a.form_rhs = form_rhs ? 1 : 0;
    a.stride = 0;
    a.act = act;
    memcpy(out, &a, sizeof(a));
    return tail_class(g, top) == 1;
}

bool fill_tail_desc(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first, void* u, const void* r,
                    bool form_rhs, const int* act, void* out)
{
    if (g->dim != 2 || !u || !r || !act || top < 0 || top > g->L || g->L - top + 1 > kMaxTail)
        throw Error(FAS_ERR_ARG, "internal: tail descriptor with a missing array or level");
    if (g->dtype == FAS_F64)
        return fill_tail_desc_t<double>(g, top, coef, pre, post, first, u, r, form_rhs, act, out);
    return fill_tail_desc_t<float>(g, top, coef, pre, post, first, u, r, form_rhs, act, out);
}

void launch_tail_table(hipStream_t stream, int dtype, bool kv, bool big, const TableLaunch& t)
{
    if (t.np < 1 || t.np > kBatchChunk) throw Error(FAS_ERR_ARG, "internal: table launch size");
    const unsigned nb = (unsigned)t.np;
#define FAS_TAIL_T(T_)                                                                         \
    do {                                                                                       \
        if (kv) {                                                                              \
            if (big) k_tail_table<T_, true, true><<<nb, kTailThreads, 0, stream>>>(t);         \
            else k_tail_table<T_, true, false><<<nb, kTailThreads, 0, stream>>>(t);            \
        } else {                                                                               \
            if (big) k_tail_table<T_, false, true><<<nb, kTailThreads, 0, stream>>>(t);        \
            else k_tail_table<T_, false, false><<<nb, kTailThreads, 0, stream>>>(t);           \
        }                                                                                      \
    } while (0)
    if (dtype == FAS_F64)
        FAS_TAIL_T(double);
    else
        FAS_TAIL_T(float);
#undef FAS_TAIL_T
    check_launch();
}

void launch_tail(const fas_grid* g, int top, const Coef* coef, int pre, int post, int first, void* u, const void* r,
                 bool form_rhs)
{
    if (g->dtype == FAS_F64)
        launch_t<double>(g, top, coef, pre, post, first, u, r, form_rhs ? 1 : 0);
    else
        launch_t<float>(g, top, coef, pre, post, first, u, r, form_rhs ? 1 : 0);
}

}  // namespace fas
