// Nystrom approximation around the sketch (Sec. 5, Alg. 2): with B = A Omega and
// the core C = Omega^T B (both from the product kernels), the approximation is
// A~ = B C^+ B^T.  This file holds the rest of it on the device, in FP64:
//
//   * the pseudo-inverse of the symmetric r x r core: its inverse where no eigenvalue
//     is cut, else by a parallel block Jacobi
//     eigensolver (two-sided, cyclic round-robin over 16-row blocks), with the
//     eigenvalue cut of Sec. 6.2: eigenvalues of modulus at most tol times the
//     largest are treated as zero;
//   * W = B C^+, then rows of A~ = W B^T or the squared Frobenius norms
//     ||A - A~||^2 and ||A||^2 (relative error of Table 2).
//
// Jacobi: S = (C + C^T)/2 is padded with zero rows and columns to Rp, a
// multiple of 32, and split into nb = Rp/16 blocks.  A step pairs the blocks by
// the circle method (nb/2 disjoint pairs; nb-1 steps meet every pair once).
// For each pair, one workgroup runs one cyclic sweep of 2x2 Jacobi rotations on
// the pair's 32 x 32 diagonal tile and keeps their product Q_P.  A second
// launch forms S <- Q^T S Q tile by tile (pair-tile (a, b) becomes
// Q_a^T S_ab Q_b; tiles a <= b are computed and mirrored, so S stays exactly
// symmetric) and V <- V Q.  After each sweep the off-diagonal norm decides
// convergence; the kernels of later sweeps return at once.  Padding rows and
// columns are zero and are never rotated (a rotation needs a non-zero
// off-diagonal entry), so they stay zero and carry the eigenvalue 0.
//
// Every sum runs in a fixed order, so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "sk_internal.hpp"

namespace sk {
namespace {

constexpr int kJB = 16;            // rows of a Jacobi block
constexpr int kJT = 2 * kJB;       // rows of a pair tile
constexpr int kJP = kJT + 1;       // LDS row pitch of a tile (doubles)
constexpr int kJThreads = 256;

// Circle-method pairing of nb (even) players at round s in [0, nb - 1): player 0
// meets 1 + s; for i >= 1 the players 1 + (s + i) mod (nb - 1) and
// 1 + (s - i) mod (nb - 1) meet.
__device__ __forceinline__ void circle_pair(int nb, int s, int i, int& a, int& b) {
    const int m = nb - 1;
    if (i == 0) {
        a = 0;
        b = 1 + s % m;
    } else {
        a = 1 + (s + i) % m;
        b = 1 + (s - i + m) % m;
    }
}

// Global row of tile index t (0..31) of the pair of blocks (I, J).
__device__ __forceinline__ int64_t tile_row(int I, int J, int t) {
    return t < kJB ? (int64_t)I * kJB + t : (int64_t)J * kJB + (t - kJB);
}

struct JacState {
    int converged;      // set once the off-diagonal norm is small enough
    int sweeps;         // sweeps run before convergence
    int inverse;        // 1: C^+ is the inverse of S (no eigenvalue is cut), left in S;
                        // -1: the elimination met a pivot that rules it out
    // of k_jac_sweep, zero between sweeps
    unsigned ticket;    // workgroups started
    alignas(128) unsigned solved;    // pair solves done, over all steps so far
};
static_assert(sizeof(JacState) <= 256, "the state's area of the workspace");

// S = (C + C^T)/2 padded to Rp x Rp, V = I, state cleared.
template <typename TC>
__global__ __launch_bounds__(256) void k_jac_init(const TC* __restrict__ C, int64_t r, int64_t ldc,
                                                  double* __restrict__ S, double* __restrict__ V,
                                                  int64_t Rp, JacState* st) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e == 0) {
        st->converged = 0;
        st->sweeps = 0;
        st->inverse = 0;
        st->ticket = 0;
        st->solved = 0;
    }
    if (e >= Rp * Rp) return;
    const int64_t i = e / Rp, j = e % Rp;
    double s = 0.0;
    if (i < r && j < r) s = 0.5 * ((double)C[i * ldc + j] + (double)C[j * ldc + i]);
    S[e] = s;
    V[e] = (i == j) ? 1.0 : 0.0;
}

// 1/sqrt(x) and 1/x for normal positive x: the hardware estimates refined by
// two Newton steps (each squares the relative error).
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    for (int i = 0; i < 2; ++i) {
        const double e = fma(-(x * y), y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    return y;
}

__device__ __forceinline__ double rcp_nr(double x) {
    double y = __builtin_amdgcn_rcp(x);
    for (int i = 0; i < 2; ++i) y = fma(fma(-x, y, 1.0), y, y);
    return y;
}

// Rotation for the symmetric 2x2 [[app, apq], [apq, aqq]]: J = [[c, s], [-s, c]]
// with t = tan theta = sign(d) e / (|d| + sqrt(d^2 + e^2)), d = aqq - app,
// e = 2 apq, the smaller root of the equation that zeroes the off-diagonal
// entry.  t is evaluated in FP32 (d and e brought into [2^-64, 2^64] by a
// power of two when they lie outside; an angle within a few 2^-24 of the
// exact one leaves that fraction of apq), then c = (1 + t^2)^-1/2 and s = t c
// in FP64, so that J is orthogonal to FP64 rounding.  Identity when apq = 0.
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double& c,
                                                double& s) {
    double d = aqq - app, e = 2.0 * apq;
    const double m = fmax(fabs(d), fabs(e));
    if (m > 0x1p64 || m < 0x1p-64) {
        int ex;
        (void)frexp(m, &ex);
        d = ldexp(d, -ex);
        e = ldexp(e, -ex);
    }
    const float df = (float)d, ef = (float)e;
    const float hf = __builtin_amdgcn_sqrtf(fmaf(df, df, ef * ef));
    const float tf = (df >= 0.f ? ef : -ef) * __builtin_amdgcn_rcpf(fabsf(df) + hf);
    const double t = (double)tf;
    const double cc = rsqrt_nr(fma(t, t, 1.0));
    c = apq == 0.0 ? 1.0 : cc;
    s = apq == 0.0 ? 0.0 : t * cc;
}

// Pairing of the blocks in a launch: kFull pairs blocks (2i, 2i + 1) and runs
// a full inner sweep (every pair of the tile's 32 indices); kCross pairs the
// blocks by the circle method at the given step and rotates only the 256
// pairs (one index of each block).  A sweep of the whole matrix is one kFull
// launch and nb - 1 kCross launches: every pair of indices is rotated at least
// once, in 31 + 16 (nb - 1) rounds.
enum { kFull = 0, kCross = 1 };

template <int MODE>
__device__ __forceinline__ void pair_blocks(int nb, int step, int i, int& I, int& J) {
    if (MODE == kFull) {
        I = 2 * i;
        J = 2 * i + 1;
    } else {
        circle_pair(nb, step, i, I, J);
    }
}

// Inner schedule on the 32 positions of a pair tile: the pairs of a round are
// always the positions (2i, 2i + 1); after each round the entry at position p
// moves to sigma(p).
//  kFull (31 rounds): position p starts with tile index p; sigma is the circle
//   method seen from the positions: position 0 stays, the others carry an
//   offset c in [0, 31) (position 1: c = 0, 2i: c = i, 2i + 1: c = 31 - i) that
//   drops by one each round, so every pair of indices meets once.
//  kCross (16 rounds): position 2k starts with index k of the first block and
//   2k + 1 with index k of the second; even positions stay and the second
//   block's indices step down one odd position per round, so each first-block
//   index meets every second-block index once.
// Both schedules return every index to its starting position.
template <int MODE>
__device__ __forceinline__ int tile_index(int p) {
    return MODE == kFull ? p : (p & 1) ? kJB + p / 2 : p / 2;
}
__device__ __forceinline__ int pos_offset(int p) { return p == 1 ? 0 : (p & 1) ? kJT - 1 - p / 2 : p / 2; }
__device__ __forceinline__ int offset_pos(int c) {
    return c == 0 ? 1 : c < kJT / 2 ? 2 * c : 2 * (kJT - 1 - c) + 1;
}
template <int MODE>
__device__ __forceinline__ int sigma(int p) {
    if (MODE == kCross) return (p & 1) ? 2 * ((p / 2 + kJB - 1) % kJB) + 1 : p;
    return p == 0 ? 0 : offset_pos((pos_offset(p) + kJT - 2) % (kJT - 1));
}
template <int MODE>
constexpr int rounds() { return MODE == kFull ? kJT - 1 : kJB; }

// One inner sweep on each pair's 32 x 32 diagonal tile; Q_P (32 x 32,
// row-major) = the product of its rotations.  512 threads: thread (X, Y) of the
// first 256 keeps the 2x2 block of rows 2X, 2X+1 and columns 2Y, 2Y+1 of the
// tile in registers, the same thread of the second 256 that block of Q.  A
// round computes the 16 rotations (on the diagonal blocks), applies them to
// every block, and moves the entries to their next positions through LDS.
constexpr int kSolveThreads = 2 * kJThreads;

// Accesses to S, V, Q and the norms.  SH: they pass between workgroups inside a launch
// (k_jac_sweep) and go to the device's point of coherence, so that neither side has to
// write back or invalidate a whole L2 around them (with plain accesses under device-scope
// fences r = 256 took 7.7 ms instead of 4.7).
template <bool SH>
__device__ __forceinline__ double mem_load(const double* p) {
    if constexpr (SH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
template <bool SH>
__device__ __forceinline__ void mem_store(double* p, double v) {
    if constexpr (SH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

struct SolveLds {
    // rc and rs far apart: combined into one two-address access, their latency sits in the
    // chain of every round (14.2 us a solve against 13.7)
    double rc[kJT / 2];
    double al[kJT][kJP];
    double ql[kJT][kJP];
    double rs[kJT / 2];
};

// before_store(): until it returns, Q may still be read.
template <int MODE, bool SH, typename Wait>
__device__ __forceinline__ void jac_solve(const double* S, int64_t Rp, double* Q, int nb, int step,
                                          int pair, SolveLds& L, Wait before_store) {
    double (*al)[kJP] = L.al;
    double (*ql)[kJP] = L.ql;
    double* rc = L.rc;
    double* rs = L.rs;
    const bool qrole = threadIdx.x >= kJThreads;
    const int tid = threadIdx.x & (kJThreads - 1), X = tid / 16, Y = tid % 16;
    int I, J;
    pair_blocks<MODE>(nb, step, pair, I, J);
    double a[2][2];
    for (int u = 0; u < 2; ++u)
        for (int v = 0; v < 2; ++v)
            a[u][v] = qrole ? ((2 * X + u == 2 * Y + v) ? 1.0 : 0.0)
                            : mem_load<SH>(S + tile_row(I, J, tile_index<MODE>(2 * X + u)) * Rp +
                                          tile_row(I, J, tile_index<MODE>(2 * Y + v)));
    int sx[2], sy[2];
    for (int u = 0; u < 2; ++u) {
        sx[u] = qrole ? 2 * X + u : sigma<MODE>(2 * X + u);    // Q's rows do not move
        sy[u] = sigma<MODE>(2 * Y + u);
    }
    double (*buf)[kJP] = qrole ? ql : al;
    for (int t = 0; t < rounds<MODE>(); ++t) {
        if (!qrole && X == Y) {
            double c, sn;
            jacobi_rotation(a[0][0], a[1][1], a[0][1], c, sn);
            rc[X] = c;
            rs[X] = sn;
        }
        __syncthreads();
        // J of a pair: [[c, s], [-s, c]] on its two positions
        const double cy = rc[Y], syn = rs[Y];
        const double jy[2][2] = {{cy, syn}, {-syn, cy}};
        double na[2][2];
        if (qrole) {
            for (int u = 0; u < 2; ++u)
                for (int v = 0; v < 2; ++v) na[u][v] = a[u][v] * jy[v][v] + a[u][v ^ 1] * jy[v ^ 1][v];
        } else {
            const double cx = rc[X], sxn = rs[X];
            const double jx[2][2] = {{cx, sxn}, {-sxn, cx}};
            for (int u = 0; u < 2; ++u)
                for (int v = 0; v < 2; ++v) {
                    // (J_X^T A J_Y)(u, v) as (T(u,v) + T(u',v')) + (T(u,v') + T(u',v)),
                    // T(i, j) = (J_X(i, u) J_Y(j, v)) A(i, j): block (Y, X) sums the same
                    // terms, so the tile stays exactly symmetric
                    const int ub = u ^ 1, vb = v ^ 1;
                    const double t1 = (jx[u][u] * jy[v][v]) * a[u][v];
                    const double t4 = (jx[ub][u] * jy[vb][v]) * a[ub][vb];
                    const double t2 = (jx[u][u] * jy[vb][v]) * a[u][vb];
                    const double t3 = (jx[ub][u] * jy[v][v]) * a[ub][v];
                    na[u][v] = (t1 + t4) + (t2 + t3);
                }
        }
        for (int u = 0; u < 2; ++u)
            for (int v = 0; v < 2; ++v) buf[sx[u]][sy[v]] = na[u][v];
        __syncthreads();
        for (int u = 0; u < 2; ++u)
            for (int v = 0; v < 2; ++v) a[u][v] = buf[2 * X + u][2 * Y + v];
    }
    before_store();
    if (qrole) {        // back at the starting positions: Q in tile-index order
        double* Qp = Q + (int64_t)pair * kJT * kJT;
        for (int u = 0; u < 2; ++u)
            for (int v = 0; v < 2; ++v)
                mem_store<SH>(Qp + tile_index<MODE>(2 * X + u) * kJT + tile_index<MODE>(2 * Y + v), a[u][v]);
    }
}

// Fixed-order workgroup sum of two doubles per thread.
template <int TH>
__device__ __forceinline__ void block_sum2(double& x, double& y, double (*red)[TH]) {
    const int tid = threadIdx.x;
    red[0][tid] = x;
    red[1][tid] = y;
    __syncthreads();
    for (int w = TH / 2; w > 0; w >>= 1) {
        if (tid < w) {
            red[0][tid] += red[0][tid + w];
            red[1][tid] += red[1][tid + w];
        }
        __syncthreads();
    }
    x = red[0][0];
    y = red[1][0];
}

// S <- Q^T S Q over the upper pair-tiles (b in [0, nT)) and V <- V Q over
// 32-row blocks of V (b in [nT, nT + nV)).  Each S tile also writes its
// squared off-diagonal and total norms (mirror counted) to part[2 b], part[2 b + 1].
// TH threads: thread (ti, tj) forms rows ti, ti + TH/16, ... and columns tj, tj + 16.
template <int TH>
struct ApplyLds {
    double x[kJT][kJP], qa[kJT][kJP], qb[kJT][kJP], u[kJT][kJP];
    double red[2][TH];
};

// Blocks of rows (Ia, Ja) and columns (Ib, Jb) of piece b: of S, or of V (rows 32 rb ..).
struct Piece {
    bool s;
    int pa, pb, rb;
    int Ia, Ja, Ib, Jb;
};
template <int MODE>
__device__ __forceinline__ Piece jac_piece(int nb, int step, int b) {
    const int np = nb / 2, nT = np * (np + 1) / 2;
    Piece p{};
    p.s = b < nT;
    if (p.s) {
        while (b >= np - p.pa) {
            b -= np - p.pa;
            ++p.pa;
        }
        p.pb = p.pa + b;
        pair_blocks<MODE>(nb, step, p.pa, p.Ia, p.Ja);
        pair_blocks<MODE>(nb, step, p.pb, p.Ib, p.Jb);
    } else {
        p.rb = (b - nT) / np;
        p.pa = (b - nT) % np;
        pair_blocks<MODE>(nb, step, p.pa, p.Ib, p.Jb);
    }
    return p;
}

// Element (i, j) of the piece's tile of S or V.
template <bool SH>
__device__ __forceinline__ double piece_s(const double* S, int64_t Rp, const Piece& p, int i, int j) {
    return mem_load<SH>(S + tile_row(p.Ia, p.Ja, i) * Rp + tile_row(p.Ib, p.Jb, j));
}
template <bool SH>
__device__ __forceinline__ double piece_v(const double* V, int64_t Rp, const Piece& p, int i, int j) {
    return mem_load<SH>(V + ((int64_t)p.rb * kJT + i) * Rp + tile_row(p.Ib, p.Jb, j));
}

// The piece's tile -> L.x, ahead of jac_apply<..., PRE = true>.
template <bool SH, int TH>
__device__ __forceinline__ void jac_apply_load(const double* S, const double* V, int64_t Rp,
                                               const Piece& p, ApplyLds<TH>& L) {
    if (p.s) {
#pragma unroll
        for (int v = 0; v < kJT * kJT / TH; ++v) {
            const int e = threadIdx.x + TH * v, i = e / kJT, j = e % kJT;
            L.x[i][j] = piece_s<SH>(S, Rp, p, i, j);
        }
    } else {
#pragma unroll
        for (int v = 0; v < kJT * kJT / TH; ++v) {
            const int e = threadIdx.x + TH * v, i = e / kJT, j = e % kJT;
            L.x[i][j] = piece_v<SH>(V, Rp, p, i, j);
        }
    }
}

template <bool SH, bool PRE, int TH>
__device__ __forceinline__ void jac_apply(double* S, double* V, int64_t Rp, const double* Q,
                                          const Piece& p, int b, double* part, ApplyLds<TH>& L) {
    constexpr int RS = TH / 16, RN = kJT / RS;            // row step, rows per thread
    const int tid = threadIdx.x;
    const int ti = tid / 16, tj = tid % 16;
    const double* Qa = Q + (int64_t)p.pa * kJT * kJT;
    const double* Qb = Q + (int64_t)p.pb * kJT * kJT;
    if (p.s) {
#pragma unroll
        for (int v = 0; v < kJT * kJT / TH; ++v) {
            const int e = tid + TH * v, i = e / kJT, j = e % kJT;
            if constexpr (!PRE) L.x[i][j] = piece_s<SH>(S, Rp, p, i, j);
            L.qa[i][j] = mem_load<SH>(Qa + e);
            L.qb[i][j] = mem_load<SH>(Qb + e);
        }
    } else {
#pragma unroll
        for (int v = 0; v < kJT * kJT / TH; ++v) {
            const int e = tid + TH * v, i = e / kJT, j = e % kJT;
            if constexpr (!PRE) L.x[i][j] = piece_v<SH>(V, Rp, p, i, j);
            L.qb[i][j] = mem_load<SH>(Qa + e);
        }
    }
    __syncthreads();
    double acc[RN][2];
#pragma unroll
    for (int a = 0; a < RN; ++a) acc[a][0] = acc[a][1] = 0.0;
    for (int z = 0; z < kJT; ++z) {                       // U = X Q_b (V Q)
        const double q0 = L.qb[z][tj], q1 = L.qb[z][tj + 16];
#pragma unroll
        for (int a = 0; a < RN; ++a) {
            const double xv = L.x[ti + RS * a][z];
            acc[a][0] = fma(xv, q0, acc[a][0]);
            acc[a][1] = fma(xv, q1, acc[a][1]);
        }
    }
    if (!p.s) {
#pragma unroll
        for (int a = 0; a < RN; ++a)
            for (int c = 0; c < 2; ++c)
                mem_store<SH>(V + ((int64_t)p.rb * kJT + ti + RS * a) * Rp + tile_row(p.Ib, p.Jb, tj + 16 * c),
                              acc[a][c]);
        return;
    }
#pragma unroll
    for (int a = 0; a < RN; ++a) {
        L.u[ti + RS * a][tj] = acc[a][0];
        L.u[ti + RS * a][tj + 16] = acc[a][1];
        acc[a][0] = acc[a][1] = 0.0;
    }
    __syncthreads();
    for (int z = 0; z < kJT; ++z) {                       // T = Q_a^T U
        const double u0 = L.u[z][tj], u1 = L.u[z][tj + 16];
#pragma unroll
        for (int a = 0; a < RN; ++a) {
            const double q = L.qa[z][ti + RS * a];
            acc[a][0] = fma(q, u0, acc[a][0]);
            acc[a][1] = fma(q, u1, acc[a][1]);
        }
    }
#pragma unroll
    for (int a = 0; a < RN; ++a) {                        // every reader of X is past the barrier
        L.x[ti + RS * a][tj] = acc[a][0];
        L.x[ti + RS * a][tj + 16] = acc[a][1];
    }
    __syncthreads();
    double off = 0.0, tot = 0.0;
#pragma unroll
    for (int v = 0; v < kJT * kJT / TH; ++v) {
        const int e = tid + TH * v, i = e / kJT, j = e % kJT;
        const int64_t gi = tile_row(p.Ia, p.Ja, i), gj = tile_row(p.Ib, p.Jb, j);
        if (p.pa == p.pb) {
            const double t = i <= j ? L.x[i][j] : L.x[j][i];
            mem_store<SH>(S + gi * Rp + gj, t);
            tot += t * t;
            if (i != j) off += t * t;
        } else {
            const double t = L.x[i][j];
            mem_store<SH>(S + gi * Rp + gj, t);
            mem_store<SH>(S + gj * Rp + gi, t);
            tot += 2.0 * t * t;
            off += 2.0 * t * t;
        }
    }
    block_sum2(off, tot, L.red);
    if (tid == 0) {
        mem_store<SH>(part + 2 * b, off);
        mem_store<SH>(part + 2 * b + 1, tot);
    }
}

// One sweep in one launch (r <= kSweepMaxR): the kFull step, then nb - 1 kCross steps (none
// if nb == 2), each np solves and nT + nV applied tiles, and at last the convergence test.
// A workgroup takes the next piece of work in that order when it starts (a ticket), and
// waits only for pieces before its own: a solve for the tiles of the step before, an applied
// tile for these and for the solves of its step.  Whoever holds a smaller ticket has started
// already and itself waits only for still smaller ones, so the first unfinished piece always
// runs and every wait ends, whatever the order or the number of workgroups that the device
// keeps resident.  Solves count up one counter; applied tiles, of which there are many, each
// set their own flag (done[b] = steps finished since the first sweep began), as additions to
// one address come one at a time.
// Hand-over: every access to S, V, Q and the norms is an agent-scope atomic (mem_load,
// mem_store), which goes to the device's point of coherence; the stores of a wave have arrived
// there when its s_waitcnt vmcnt(0) ends, the barrier after it collects the waves, and only
// then does the flag move.  A reader's loads are issued after the flag's value has come back.
// (A release and an acquire of agent scope say the same to the memory model, but write back
// and invalidate whole caches: 7.7 ms at r = 256.)
// After convergence, or when the inverse was taken, a sweep then costs one short launch
// (2.9 us) instead of 2 nb + 1 of 2.7 us each (r = 256, 16 sweeps: 1.4 ms of the inverse's
// 1.6).  A core that needs the sweeps pays for the attempt and, with many tiles, for the
// tickets (separate launches alone, and now): r = 24 307 and 329 us, r = 64 1262 and 1290,
// r = 128 2687 and 2705, r = 200 4615 and 4820, r = 256 5292 and 5577 (5713 while a solve
// waited for every tile of the step before).  The tickets' share grows with r, so larger cores
// keep the launches.
constexpr int64_t kSweepMaxR = 256;

__device__ __forceinline__ void wait_solved(unsigned* solved, unsigned target, unsigned near) {
    if (threadIdx.x == 0) {
        for (;;) {
            const unsigned v = __hip_atomic_load(solved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v >= target) break;
            // a step or more away: look seldom, the counter's own traffic goes first
            if (target - v > near) __builtin_amdgcn_s_sleep(127);
            else __builtin_amdgcn_s_sleep(2);
        }
    }
    __syncthreads();
}

__device__ __forceinline__ void wait_applied(const unsigned* done, unsigned nA, unsigned target) {
    for (;;) {
        bool ok = true;
        unsigned least = target;
        for (unsigned b = threadIdx.x; b < nA; b += kSolveThreads) {
            const unsigned v = __hip_atomic_load(done + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = ok && v >= target;
            least = min(least, v);
        }
        if (__syncthreads_and(ok)) break;
        if (__syncthreads_or(least + 1 < target)) __builtin_amdgcn_s_sleep(127);
        else __builtin_amdgcn_s_sleep(2);
    }
}

// The solve of pair (I, J) at kCross step `step` reads the tile of these two blocks, which the
// step before left in three pieces: wait for those.
__device__ __forceinline__ void wait_tile(const unsigned* done, int nb, int step, int pair,
                                          unsigned target) {
    const int np = nb / 2;
    int I, J;
    circle_pair(nb, step - 1, pair, I, J);
    // the pair a block belonged to in the step before
    auto owner = [&](int block) {
        if (step == 1) return block / 2;
        int p = 0;
        for (int i = 0; i < np; ++i) {
            int a, b;
            circle_pair(nb, step - 2, i, a, b);
            if (a == block || b == block) p = i;
        }
        return p;
    };
    const int pi = owner(I), pj = owner(J);
    const int lo = threadIdx.x == 0 ? pi : threadIdx.x == 1 ? pj : min(pi, pj);
    const int hi = threadIdx.x == 0 ? pi : threadIdx.x == 1 ? pj : max(pi, pj);
    const unsigned* flag = done + (lo * np - lo * (lo - 1) / 2 + hi - lo);   // piece (lo, hi)
    for (;;) {
        const bool ok = threadIdx.x > 2 ||
                        __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target;
        if (__syncthreads_and(ok)) break;
        __builtin_amdgcn_s_sleep(2);
    }
}

__global__ __launch_bounds__(kSolveThreads) void k_jac_sweep(double* S, double* V, int64_t Rp, double* Q,
                                                             int nb, double* part, double tolc,
                                                             unsigned* done, JacState* st) {
    if (st->converged) return;
    __shared__ union {
        SolveLds solve;
        ApplyLds<kSolveThreads> apply;
    } lds;
    __shared__ unsigned word;
    const unsigned np = (unsigned)nb / 2, nT = np * (np + 1) / 2, nA = nT + np * np;
    const unsigned steps = nb > 2 ? (unsigned)nb : 1u;
    const unsigned base = (unsigned)st->sweeps * steps;      // steps before this sweep
    if (threadIdx.x == 0)
        word = __hip_atomic_fetch_add(&st->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned step = word / (np + nA), piece = word % (np + nA);
    if (step == steps) {         // the last ticket: end of the sweep
        wait_applied(done, nA, base + steps);
        double off = 0.0, tot = 0.0;
        for (unsigned i = threadIdx.x; i < nT; i += kSolveThreads) {
            off += mem_load<true>(part + 2 * i);
            tot += mem_load<true>(part + 2 * i + 1);
        }
        block_sum2(off, tot, lds.apply.red);
        if (threadIdx.x == 0) {
            st->sweeps += 1;
            st->ticket = 0;
            st->solved = 0;
            if (off <= tolc * tolc * tot) st->converged = 1;
        }
    } else if (piece < np) {
        // the pieces of the step before also read the Q that this solve replaces: all of them
        // have to be done by then, the tile's own at once
        if (step == 0) {
            wait_applied(done, nA, base);
            jac_solve<kFull, true>(S, Rp, Q, nb, 0, (int)piece, lds.solve, [] {});
        } else {
            wait_tile(done, nb, (int)step, (int)piece, base + step);
            jac_solve<kCross, true>(S, Rp, Q, nb, (int)step - 1, (int)piece, lds.solve,
                                    [&] { wait_applied(done, nA, base + step); });
        }
        // every wave's stores have reached the point of coherence before the count moves
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_fetch_add(&st->solved, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        // the tile is loaded while the step's solves run
        const int b = (int)(piece - np);
        const Piece p = step == 0 ? jac_piece<kFull>(nb, 0, b) : jac_piece<kCross>(nb, (int)step - 1, b);
        wait_applied(done, nA, base + step);
        jac_apply_load<true>(S, V, Rp, p, lds.apply);
        wait_solved(&st->solved, (step + 1) * np, np);
        jac_apply<true, true>(S, V, Rp, Q, p, b, part, lds.apply);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(done + (piece - np), base + step + 1, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The same steps as launches of their own.
template <int MODE>
__global__ __launch_bounds__(kSolveThreads) void k_jac_solve(const double* __restrict__ S,
                                                             int64_t Rp, double* __restrict__ Q,
                                                             int nb, int step, const JacState* st) {
    if (st->converged) return;
    __shared__ SolveLds lds;
    jac_solve<MODE, false>(S, Rp, Q, nb, step, blockIdx.x, lds, [] {});
}

template <int MODE>
__global__ __launch_bounds__(kJThreads) void k_jac_apply(double* __restrict__ S,
                                                         double* __restrict__ V, int64_t Rp,
                                                         const double* __restrict__ Q, int nb,
                                                         int step, double* __restrict__ part,
                                                         const JacState* st) {
    if (st->converged) return;
    __shared__ ApplyLds<kJThreads> lds;
    const Piece p = jac_piece<MODE>(nb, step, blockIdx.x);
    jac_apply<false, false>(S, V, Rp, Q, p, blockIdx.x, part, lds);
}

// End of a sweep: sum the tiles' norms in tile order; converged when
// off <= tolc * total (Frobenius).
__global__ __launch_bounds__(kJThreads) void k_jac_flag(const double* __restrict__ part, int nT,
                                                        double tolc, JacState* st) {
    if (st->converged) return;
    __shared__ double red[2][kJThreads];
    double off = 0.0, tot = 0.0;
    for (int i = threadIdx.x; i < nT; i += kJThreads) {
        off += part[2 * i];
        tot += part[2 * i + 1];
    }
    block_sum2(off, tot, red);
    if (threadIdx.x == 0) {
        st->sweeps += 1;
        if (off <= tolc * tolc * tot) st->converged = 1;
    }
}

// 32 x 32 tile at (i0, j0) of V diag(mu) V^T: sum_l V(i, l) V(j, l) mu_l, l ascending, for
// i, j < r (256 threads, 2 x 2 outputs each, l in chunks of 16 staged in LDS).
constexpr int kGK = 16;

__device__ __forceinline__ void spectral_tile(const double* __restrict__ V, int64_t ldv, int64_t r,
                                              const double* mu, int64_t i0, int64_t j0,
                                              double acc[2][2], double (*xs)[kJT], double (*ys)[kJT]) {
    const int tid = threadIdx.x, ty = tid / 16, tx = tid % 16;
    const int li = tid / 8, lk = (tid % 8) * 2;
    for (int a = 0; a < 2; ++a)
        for (int c = 0; c < 2; ++c) acc[a][c] = 0.0;
    for (int64_t l0 = 0; l0 < r; l0 += kGK) {
        for (int w = 0; w < 2; ++w) {
            const int64_t l = l0 + lk + w;
            const int64_t gi = i0 + li, gj = j0 + li;
            xs[lk + w][li] = (gi < r && l < r) ? V[gi * ldv + l] : 0.0;
            ys[lk + w][li] = (gj < r && l < r) ? V[gj * ldv + l] : 0.0;
        }
        __syncthreads();
        const int kk_end = (int)((r - l0) < kGK ? (r - l0) : kGK);
        for (int kk = 0; kk < kk_end; ++kk) {
            const double m = mu[l0 + kk];
            for (int a = 0; a < 2; ++a)
                for (int c = 0; c < 2; ++c)
                    acc[a][c] = fma(xs[kk][ty * 2 + a] * ys[kk][tx * 2 + c], m, acc[a][c]);
        }
        __syncthreads();
    }
}

// ---- The inverse, where no eigenvalue is cut ----------------------------------------
// If every |lambda| exceeds tol max|lambda|, V diag(mu) V^T is the inverse of S, which
// takes Rp/32 short launches instead of a dozen Jacobi sweeps of 2 Rp/16 each.  A call at
// r = 24 takes 70 us against 252, r = 64 85 against 822, r = 256 220 against 3627 and
// r = 500 (whose idle sweeps stay separate launches, most of its time) 3.1 ms against 8.3; a
// core that needs the sweeps pays for the attempt, 22 us at r = 24 to 0.4 ms at r = 500 (3 to
// 7%), less where an early pivot ends it.
// X = S^-1 by a block Gauss-Jordan elimination without pivoting, R = I - S X as computed,
// and the certificate
//     ||R||_F <= 2^-24,  rho = ||R||_F + (r + 2) u ||S||_F ||X||_F < 1/2  (u = 2^-53)
//     and  1.01 tol ||S||_F ||X||_F < 1 - rho.
// rho bounds the exact residual (the middle term is the rounding of R), so S is not
// singular, min|lambda| >= (1 - rho) / ||X||_F > tol ||S||_F >= tol max|lambda|, and no
// eigenvalue is cut; 1.01 covers the rounding of the norms.  X + X R then has a residual of
// at most ||R||^2 <= 2^-48 besides rounding of order r u ||S|| ||X||, as any inverse.  A
// singular, badly scaled or unluckily indefinite S fails it (NaN included), and the sweeps
// run as they do when the caller asks for the eigenvalues.

// Element (i, j) of a matrix of r x r, continued by the identity.
struct Padded {
    double* p;
    int64_t ld;
    int64_t r;
    __device__ __forceinline__ double get(int64_t i, int64_t j) const {
        return i < r && j < r ? p[i * ld + j] : i == j ? 1.0 : 0.0;
    }
    __device__ __forceinline__ void put(int64_t i, int64_t j, double v) const {
        if (i < r && j < r) p[i * ld + j] = v;
    }
};

// (acc[u]) += sum_k a[ti][k] b[k][4 tj + u] over a 32 x 32 x 32 product.
__device__ __forceinline__ void mul32(const double (*a)[kJP], const double (*b)[kJP], int ti, int tj,
                                      double sign, double (&acc)[4]) {
#pragma unroll 8
    for (int k = 0; k < kJT; ++k) {
        const double x = sign * a[ti][k];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = fma(x, b[k][4 * tj + u], acc[u]);
    }
}

__device__ __forceinline__ void load32(double (*t)[kJP], const Padded& m, int bi, int bj, int ti, int tj) {
#pragma unroll
    for (int u = 0; u < 4; ++u) t[ti][4 * tj + u] = m.get((int64_t)bi * kJT + ti, (int64_t)bj * kJT + 4 * tj + u);
}

// Step k of the elimination, src -> dst: every workgroup forms one 32 x 32 block and
// inverts the pivot block for itself (32 pivots, one barrier each).
// A pivot of at most tol times the diagonal entry of S in its place ends the attempt: a
// semidefinite S then has an eigenvalue to cut (the pivot is at least the smallest one, the
// entry at most the largest), and another S would fail the certificate for the growth of X.
__global__ __launch_bounds__(kJThreads) void k_inv_step(const Padded src, const Padded dst, int k,
                                                        const Padded S, double tol, JacState* st) {
    __shared__ double d[kJT][kJP], a[kJT][kJP], b[kJT][kJP];
    __shared__ double prow[2][kJT], pcol[2][kJT];
    const int ended = st->inverse;         // in flight with the blocks
    const int bi = blockIdx.y, bj = blockIdx.x;
    const int tid = threadIdx.x, ti = tid / 8, tj = tid % 8;
    double e[4], own[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = src.get((int64_t)k * kJT + ti, (int64_t)k * kJT + 4 * tj + u);
    if (bj != k) load32(b, src, k, bj, ti, tj);
    if (bi != k) load32(a, src, bi, k, ti, tj);
    const int64_t pk = (int64_t)k * kJT + (tid & (kJT - 1));
    const double least = tol * fabs(S.get(pk, pk));
    double pivot = 0.0;                    // of column tid % 32
    if (bi != k && bj != k) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            own[u] = src.get((int64_t)bi * kJT + ti, (int64_t)bj * kJT + 4 * tj + u);
    }
    if (ended < 0) return;
#pragma unroll
    for (int p = 0; p < kJT; ++p) {
        double* pr = prow[p & 1];
        double* pc = pcol[p & 1];
        if (ti == p) {
#pragma unroll
            for (int u = 0; u < 4; ++u) pr[4 * tj + u] = e[u];
        }
        if (tj == p / 4) pc[ti] = e[p % 4];
        __syncthreads();
        const double inv = rcp_nr(pr[p]);
        const double f = pc[ti] * inv;
        if ((tid & (kJT - 1)) == p) pivot = pr[p];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = 4 * tj + u;
            const double v = ti == p ? (j == p ? inv : pr[j] * inv)
                                     : (j == p ? -f : fma(-f, pr[j], e[u]));
            e[u] = v;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) d[ti][4 * tj + u] = e[u];
    if (__syncthreads_or(!(fabs(pivot) > least))) {        // NaN too
        if (bi == 0 && bj == 0 && tid == 0) st->inverse = -1;
        return;
    }
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (bi == k && bj == k) {
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = e[u];
    } else if (bj == k) {
        mul32(a, d, ti, tj, -1.0, v);
    } else {
        mul32(d, b, ti, tj, 1.0, v);
        if (bi != k) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                b[ti][4 * tj + u] = v[u];
                v[u] = own[u];
            }
            __syncthreads();
            mul32(a, b, ti, tj, -1.0, v);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) dst.put((int64_t)bi * kJT + ti, (int64_t)bj * kJT + 4 * tj + u, v[u]);
}

// One 32 x 32 block of L M (np blocks of 32 along the contraction): acc of thread (ti, tj);
// the next blocks are loaded while these are multiplied.
__device__ __forceinline__ void block_product(const Padded& L, const Padded& M, int bi, int bj, int np,
                                              int ti, int tj, double (*a)[kJP], double (*b)[kJP],
                                              double sign, double (&acc)[4]) {
    double na[4], nb[4];
    auto fetch = [&](int k) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            na[u] = L.get((int64_t)bi * kJT + ti, (int64_t)k * kJT + 4 * tj + u);
            nb[u] = M.get((int64_t)k * kJT + ti, (int64_t)bj * kJT + 4 * tj + u);
        }
    };
    fetch(0);
    for (int k = 0; k < np; ++k) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[ti][4 * tj + u] = na[u];
            b[ti][4 * tj + u] = nb[u];
        }
        __syncthreads();
        if (k + 1 < np) fetch(k + 1);
        mul32(a, b, ti, tj, sign, acc);
    }
}

// Fixed-order workgroup sum (256 threads).
__device__ __forceinline__ double block_sum1(double x, double* red) {
    red[threadIdx.x] = x;
    __syncthreads();
    for (int w = kJThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

// R = I - S X by blocks; norm[3 t ..] = the block's squares of R, S and X.
__global__ __launch_bounds__(kJThreads) void k_inv_residual(const Padded S, const Padded X,
                                                            const Padded R, double* __restrict__ norm,
                                                            const JacState* st) {
    if (st->inverse < 0) return;
    __shared__ double a[kJT][kJP], b[kJT][kJP];
    __shared__ double red[kJThreads];
    const int bi = blockIdx.y, bj = blockIdx.x, np = gridDim.x;
    const int tid = threadIdx.x, ti = tid / 8, tj = tid % 8;
    const int64_t i = (int64_t)bi * kJT + ti, j0 = (int64_t)bj * kJT + 4 * tj;
    double acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = i == j0 + u ? 1.0 : 0.0;
    block_product(S, X, bi, bj, np, ti, tj, a, b, -1.0, acc);
    double r2 = 0.0, s2 = 0.0, x2 = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (i >= S.r || j0 + u >= S.r) continue;
        const double sv = S.get(i, j0 + u), xv = X.get(i, j0 + u);
        r2 = fma(acc[u], acc[u], r2);
        s2 = fma(sv, sv, s2);
        x2 = fma(xv, xv, x2);
        R.put(i, j0 + u, acc[u]);
    }
    r2 = block_sum1(r2, red);
    s2 = block_sum1(s2, red);
    x2 = block_sum1(x2, red);
    if (tid == 0) {
        double* n = norm + 3 * (bi * np + bj);
        n[0] = r2;
        n[1] = s2;
        n[2] = x2;
    }
}

// With the certificate: S <- X + X R, state "converged".  Without it: V <- I for the
// sweeps, and their flags (in the output, which X or R held) cleared.  (X or R may lie in V:
// every block decides alike.)
__global__ __launch_bounds__(kJThreads) void k_inv_finish(const Padded X, const Padded R,
                                                          const double* __restrict__ norm, double tol,
                                                          double* __restrict__ S, double* __restrict__ V,
                                                          int64_t Rp, unsigned* done, int nA,
                                                          JacState* st) {
    __shared__ double a[kJT][kJP], b[kJT][kJP];
    __shared__ double red[kJThreads];
    const int bi = blockIdx.y, bj = blockIdx.x, np = gridDim.x;
    const int tid = threadIdx.x, ti = tid / 8, tj = tid % 8;
    double q[3] = {0.0, 0.0, 0.0};
    for (int t = tid; t < np * np; t += kJThreads)
#pragma unroll
        for (int c = 0; c < 3; ++c) q[c] += norm[3 * t + c];
#pragma unroll
    for (int c = 0; c < 3; ++c) q[c] = block_sum1(q[c], red);
    const int64_t i = (int64_t)bi * kJT + ti, j0 = (int64_t)bj * kJT + 4 * tj;
    const double kappa = sqrt(q[1]) * sqrt(q[2]);
    const double rho = sqrt(q[0]) + (double)(X.r + 2) * 0x1p-53 * kappa;
    if (st->inverse < 0 || !(q[0] <= 0x1p-48 && rho < 0.5 && 1.01 * tol * kappa < 1.0 - rho)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) V[i * Rp + j0 + u] = i == j0 + u ? 1.0 : 0.0;
        if (bi == 0 && bj == 0)
            for (int t = tid; t < nA; t += kJThreads) done[t] = 0u;
        return;
    }
    double acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = X.get(i, j0 + u);
    block_product(X, R, bi, bj, np, ti, tj, a, b, 1.0, acc);
#pragma unroll
    for (int u = 0; u < 4; ++u) S[i * Rp + j0 + u] = acc[u];
    // every workgroup has found st->inverse at 0 or 1: neither is below 0
    if (bi == 0 && bj == 0 && tid == 0) {
        st->converged = 1;
        st->inverse = 1;
    }
}

// C^+ = V diag(mu) V^T on the first r rows / columns, mu_l = 1 / lambda_l for
// |lambda_l| > tol max|lambda|, else 0 (lambda_l = S(l, l) after convergence).
// (V_il V_jl) mu_l is the same product for (i, j) and (j, i): C^+ is exactly
// symmetric.
__global__ __launch_bounds__(256) void k_pinv_form(const double* __restrict__ S,
                                                   const double* __restrict__ V, int64_t Rp,
                                                   int64_t r, double tol, double* __restrict__ Cp,
                                                   int64_t ldcp, double* __restrict__ eig,
                                                   const JacState* st) {
    constexpr int TM = 32;
    if (st->inverse > 0) {       // the symmetric part of the inverse
        for (int e = threadIdx.x; e < TM * TM; e += 256) {
            const int64_t i = (int64_t)blockIdx.y * TM + e / TM, j = (int64_t)blockIdx.x * TM + e % TM;
            if (i < r && j < r) Cp[i * ldcp + j] = 0.5 * (S[i * Rp + j] + S[j * Rp + i]);
        }
        return;
    }
    __shared__ double xs[kGK][TM], ys[kGK][TM];
    __shared__ double mu[1024];
    __shared__ double red[256];
    const int tid = threadIdx.x;
    double mx = 0.0;
    for (int64_t l = tid; l < r; l += 256) mx = fmax(mx, fabs(S[l * Rp + l]));
    red[tid] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
        __syncthreads();
    }
    const double cut = tol * red[0];
    for (int64_t l = tid; l < r; l += 256) {
        const double lam = S[l * Rp + l];
        mu[l] = fabs(lam) > cut ? 1.0 / lam : 0.0;
        if (eig && blockIdx.x == 0 && blockIdx.y == 0) eig[l] = lam;
    }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.y * TM, j0 = (int64_t)blockIdx.x * TM;
    double acc[2][2];
    spectral_tile(V, Rp, r, mu, i0, j0, acc, xs, ys);
    const int ty = tid / 16, tx = tid % 16;
    for (int a = 0; a < 2; ++a)
        for (int c = 0; c < 2; ++c) {
            const int64_t i = i0 + ty * 2 + a, j = j0 + tx * 2 + c;
            if (i < r && j < r) Cp[i * ldcp + j] = acc[a][c];
        }
}

// FP64 matrix-core tile: out(i, j) = sum_l X(i, l) Y(j, l) for a 128 x 128 tile per workgroup
// (4 waves of 64 x 64, 4 x 4 tiles of v_mfma_f64_16x16x4f64 each), l ascending in steps of
// four.  16 values of l at a time are staged in LDS, [l][row] with a pitch of 16 mod 32
// doubles, so that the four l of an operand read fall on different banks; the next 16 are
// loaded while these are multiplied (64 MFMAs of 64 cycles a wave, which hide them).
// The former tile of 64 x 64 with FP64 FMAs ran at 29 TFLOP/s, two LDS reads for every four
// FMAs; this one at 58, the matrix cores busy 74% of the time (error at n = 16384, r = 256
// with a C^+ that is not bitwise symmetric: 4.78 -> 2.45 ms; n = 5000, r = 100: 229 -> 177 us;
// n = 2048, r = 16: 21 us either way).
typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d_a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kDT = 128;           // rows and columns of a tile
constexpr int kDK = 16;            // contraction values staged at a time
constexpr int kDP = kDT + 16;      // LDS pitch (doubles)
struct TileLds64 {
    double x[2][kDK][kDP], y[2][kDK][kDP];
};

// 8 values p[0 .. 7] -> v, those from `left` on zero.
__device__ __forceinline__ void load8(const double* p, int64_t left, double* v) {
    if (left >= 8) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const v2d_a8 t = *reinterpret_cast<const v2d_a8*>(p + e);
            v[e] = t[0];
            v[e + 1] = t[1];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = e < left ? p[e] : 0.0;
    }
}
__device__ __forceinline__ void load8(const float* p, int64_t left, double* v) {
    if (left >= 8) {
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
            const v4f_a4 t = *reinterpret_cast<const v4f_a4*>(p + e);
#pragma unroll
            for (int u = 0; u < 4; ++u) v[e + u] = (double)t[u];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = e < left ? (double)p[e] : 0.0;
    }
}

// acc[tm][tn]: register r of lane (g, j) is row 64 (wave / 2) + 16 tm + 4 r + g, column
// 64 (wave % 2) + 16 tn + j of the tile.  Rows past mx (my) repeat the last one.
// TAIL: K is no multiple of 16; its last values are multiplied after the loop, without the
// zeros that fill their stage (r = 20 on n = 3001: 42.2 -> 36.4 us).  An instance of its own: with
// the tail's code behind it the loop takes 2% longer at r = 256, with a test in it 5%.
template <bool TAIL, typename TX, typename TY>
__device__ __forceinline__ void tile_mfma64(const TX* __restrict__ X, int64_t ldx, int64_t mx,
                                            const TY* __restrict__ Y, int64_t ldy, int64_t my,
                                            int64_t K, int64_t i0, int64_t j0, v4d (&acc)[4][4],
                                            TileLds64& L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, j = lane & 15;
    const int row = tid >> 1, half = (tid & 1) * 8;      // staging: row, first l
    const TX* xp = X + min(i0 + row, mx - 1) * ldx + half;
    const TY* yp = Y + min(j0 + row, my - 1) * ldy + half;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = v4d{0.0, 0.0, 0.0, 0.0};
    double xv[8], yv[8];
    auto load = [&](int64_t l0) {
        load8(xp + l0, K - l0 - half, xv);
        load8(yp + l0, K - l0 - half, yv);
    };
    auto store = [&](int b) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            L.x[b][half + e][row] = xv[e];
            L.y[b][half + e][row] = yv[e];
        }
    };
    load(0);
    store(0);
    __syncthreads();
    int b = 0;
    auto multiply = [&](const double* xb, const double* yb, int kk) {
        double av[4], bv[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            av[t] = xb[kk * kDP + 16 * t];
            bv[t] = yb[kk * kDP + 16 * t];
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[c], acc[a][c], 0, 0, 0);
    };
    int64_t l0 = 0;
    for (; TAIL ? l0 + kDK <= K : l0 < K; l0 += kDK, b ^= 1) {
        const bool more = l0 + kDK < K;
        if (more) load(l0 + kDK);
        const double* xb = &L.x[b][g][(wave >> 1) * 64 + j];
        const double* yb = &L.y[b][g][(wave & 1) * 64 + j];
#pragma unroll
        for (int kk = 0; kk < kDK; kk += 4) multiply(xb, yb, kk);
        if (more) store(b ^ 1);
        __syncthreads();
    }
    if constexpr (TAIL) {
        const double* xb = &L.x[b][g][(wave >> 1) * 64 + j];
        const double* yb = &L.y[b][g][(wave & 1) * 64 + j];
#pragma unroll
        for (int kk = 0; kk < kDK; kk += 4) {
            if (l0 + kk >= K) break;
            multiply(xb, yb, kk);
        }
    }
}

// W = B C^+ (rows [row0, row0 + mw) of B; C^+ symmetric, so W(i, j) =
// sum_l B(i, l) C^+(j, l)).
template <bool TAIL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_bw(const float* __restrict__ B, int64_t ldb, int64_t mw, int64_t r,
          const double* __restrict__ Cp, int64_t ldcp, double* __restrict__ W, int* sym) {
    __shared__ TileLds64 lds;
    if (sym && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *sym = 1;
    const int64_t i0 = (int64_t)blockIdx.y * kDT, j0 = (int64_t)blockIdx.x * kDT;
    v4d acc[4][4];
    tile_mfma64<TAIL>(B, ldb, mw, Cp, ldcp, r, r, i0, j0, acc, lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = i0 + (wave >> 1) * 64 + 16 * a + 4 * q + (lane >> 4);
                const int64_t j = j0 + (wave & 1) * 64 + 16 * c + (lane & 15);
                if (i < mw && j < r) W[i * r + j] = acc[a][c][q];
            }
}

// *sym (1 on entry, from k_bw) = 0 if C^+ differs from its transpose in any bit: one
// workgroup per 32 x 32 tile, the mirror tile turned round in LDS.
__global__ __launch_bounds__(256) void k_symmetric(const double* __restrict__ Cp, int64_t r,
                                                   int64_t ldcp, int* __restrict__ sym) {
    if (blockIdx.x < blockIdx.y) return;
    __shared__ double m[32][33];
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    const int64_t i0 = (int64_t)blockIdx.y * 32, j0 = (int64_t)blockIdx.x * 32;
    for (int u = y; u < 32; u += 8)
        m[u][x] = (j0 + u < r && i0 + x < r) ? Cp[(j0 + u) * ldcp + i0 + x] : 0.0;
    __syncthreads();
    bool same = true;
    for (int u = y; u < 32; u += 8) {
        const double c = (i0 + u < r && j0 + x < r) ? Cp[(i0 + u) * ldcp + j0 + x] : 0.0;
        same = same && __double_as_longlong(c) == __double_as_longlong(m[x][u]);
    }
    if (!same) *sym = 0;
}

// Rows of A~ = W B^T (out, mr x n) or, with A given, per-tile sums of
// (A - A~)^2 and A^2 over the n x n matrix (part[2 t], part[2 t + 1]).  With a symmetric
// C^+ (*sym), A~ is symmetric: a tile above the diagonal serves its mirror image too, and
// the tiles below the diagonal do nothing.  The tile's elements of A are loaded from clamped
// addresses without a branch, 16 of a lane (32 with the mirror image) in flight.
template <bool ERR, bool TAIL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_nys_tile(const double* __restrict__ W, int64_t mw, const float* __restrict__ B, int64_t ldb,
                int64_t n, int64_t r, const float* __restrict__ A, int64_t lda,
                double* __restrict__ out, int64_t ldo, double* __restrict__ part,
                const int* __restrict__ sym) {
    __shared__ TileLds64 lds;
    __shared__ double red[2][kJThreads];
    const int64_t t = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const bool mirror = ERR && sym && *sym && blockIdx.x != blockIdx.y;
    if (mirror && blockIdx.x < blockIdx.y) {
        if (threadIdx.x == 0) {
            part[2 * t] = 0.0;
            part[2 * t + 1] = 0.0;
        }
        return;
    }
    const int64_t i0 = (int64_t)blockIdx.y * kDT, j0 = (int64_t)blockIdx.x * kDT;
    v4d acc[4][4];
    tile_mfma64<TAIL>(W, r, mw, B, ldb, n, r, i0, j0, acc, lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = (wave >> 1) * 64 + (lane >> 4), lj = (wave & 1) * 64 + (lane & 15);
    if constexpr (!ERR) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t i = i0 + li + 16 * a + 4 * q, j = j0 + lj + 16 * c;
                    if (i < mw && j < n) out[i * ldo + j] = acc[a][c][q];
                }
        return;
    }
    double se = 0.0, sa = 0.0;
    auto add = [&](float a32, bool in, double at) {
        const double av = in ? (double)a32 : 0.0;
        const double d = in ? av - at : 0.0;
        se = fma(d, d, se);
        sa = fma(av, av, sa);
    };
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        float av[4][4], bv[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = min(i0 + li + 16 * a + 4 * q, n - 1), j = min(j0 + lj + 16 * c, n - 1);
                av[c][q] = A[i * lda + j];
                if (mirror) bv[c][q] = A[j * lda + i];
            }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = i0 + li + 16 * a + 4 * q < n && j0 + lj + 16 * c < n;
                add(av[c][q], in, acc[a][c][q]);
                if (mirror) add(bv[c][q], in, acc[a][c][q]);
            }
    }
    block_sum2(se, sa, red);
    if (threadIdx.x == 0) {
        part[2 * t] = se;
        part[2 * t + 1] = sa;
    }
}

// sums = (sum of part[2 t], sum of part[2 t + 1], sqrt(sums[0] / sums[1])): every thread its
// t, t + 256, ... in order, eight loads at a time, then the threads in a fixed tree.
__global__ __launch_bounds__(kJThreads) void k_err_sum(const double* __restrict__ part, int64_t T,
                                                       double* __restrict__ sums) {
    __shared__ double red[2][kJThreads];
    const double2* p = reinterpret_cast<const double2*>(part);
    double se = 0.0, sa = 0.0;
    int64_t t = threadIdx.x;
    for (; t + 7 * kJThreads < T; t += 8 * kJThreads) {
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[t + u * kJThreads];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            se += v[u].x;
            sa += v[u].y;
        }
    }
    for (; t < T; t += kJThreads) {
        se += p[t].x;
        sa += p[t].y;
    }
    block_sum2(se, sa, red);
    if (threadIdx.x == 0) {
        sums[0] = se;
        sums[1] = sa;
        sums[2] = sa > 0.0 ? sqrt(se / sa) : 0.0;
    }
}

__global__ void k_jac_info(const JacState* st, int32_t* info) {
    if (threadIdx.x == 0) {
        info[0] = st->sweeps;
        info[1] = st->converged;
    }
}

inline int64_t jac_rp(int64_t r) { return (r + kJT - 1) / kJT * kJT; }
inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t pinv_workspace_bytes(int64_t r) {
    if (r <= 0) return 0;
    const int64_t Rp = jac_rp(r), np = Rp / kJT;
    const int64_t nT = np * (np + 1) / 2;
    return align256(sizeof(JacState)) + 2 * align256((size_t)(Rp * Rp) * 8) +
           align256((size_t)(np * kJT * kJT) * 8) + align256((size_t)nT * 16);
}

hipError_t launch_core_pinv(const void* C, int c_f64, int64_t r, int64_t ldc, double tol,
                            int max_sweeps, double* Cp, int64_t ldcp, double* eig, int32_t* info,
                            void* ws, hipStream_t s) {
    const int64_t Rp = jac_rp(r), nb = Rp / kJB, np = nb / 2;
    const int64_t nT = np * (np + 1) / 2, nV = (Rp / kJT) * np;
    char* p = static_cast<char*>(ws);
    JacState* st = reinterpret_cast<JacState*>(p);
    p += align256(sizeof(JacState));
    double* S = reinterpret_cast<double*>(p);
    p += align256((size_t)(Rp * Rp) * 8);
    double* V = reinterpret_cast<double*>(p);
    p += align256((size_t)(Rp * Rp) * 8);
    double* Q = reinterpret_cast<double*>(p);
    p += align256((size_t)(np * kJT * kJT) * 8);
    double* part = reinterpret_cast<double*>(p);
    const unsigned gi = (unsigned)((Rp * Rp + 255) / 256);
    if (c_f64)
        k_jac_init<double><<<gi, 256, 0, s>>>(static_cast<const double*>(C), r, ldc, S, V, Rp, st);
    else
        k_jac_init<float><<<gi, 256, 0, s>>>(static_cast<const float*>(C), r, ldc, S, V, Rp, st);
    // flags of k_jac_sweep: nT + nV <= 2 r words, in the output's first row
    unsigned* done = reinterpret_cast<unsigned*>(Cp);
    if (eig == nullptr) {
        // blocks of V and of the output in turn; Q's area (Rp/32 KiB x 8) holds the norms
        const Padded ms{S, Rp, r}, mv{V, Rp, r}, mc{Cp, ldcp, r};
        const dim3 gb((unsigned)np, (unsigned)np);
        for (int k = 0; k < (int)np; ++k)
            k_inv_step<<<gb, kJThreads, 0, s>>>(k == 0 ? ms : k % 2 ? mv : mc, k % 2 ? mc : mv, k, ms,
                                                tol, st);
        const Padded& X = np % 2 ? mv : mc;
        const Padded& R = np % 2 ? mc : mv;
        k_inv_residual<<<gb, kJThreads, 0, s>>>(ms, X, R, Q, st);
        k_inv_finish<<<gb, kJThreads, 0, s>>>(X, R, Q, tol, S, V, Rp, done, (int)(nT + nV), st);
    }
    // off-diagonal Frobenius norm at most 8 Rp units of FP64 rounding of ||S||
    const double tolc = 8.0 * (double)Rp * 0x1p-53;
    const unsigned ga = (unsigned)(nT + nV);
    const unsigned steps = nb > 2 ? (unsigned)nb : 1u;
    // sweeps that may have nothing to do go out as one launch each, the others step by step
    const bool sweep_launch = eig == nullptr && r <= kSweepMaxR;
    for (int sw = 0; sw < max_sweeps; ++sw) {
        if (sweep_launch) {
            k_jac_sweep<<<steps * (unsigned)(np + nT + nV) + 1, kSolveThreads, 0, s>>>(
                S, V, Rp, Q, (int)nb, part, tolc, done, st);
            continue;
        }
        k_jac_solve<kFull><<<(unsigned)np, kSolveThreads, 0, s>>>(S, Rp, Q, (int)nb, 0, st);
        k_jac_apply<kFull><<<ga, kJThreads, 0, s>>>(S, V, Rp, Q, (int)nb, 0, part, st);
        for (int step = 0; nb > 2 && step < nb - 1; ++step) {
            k_jac_solve<kCross><<<(unsigned)np, kSolveThreads, 0, s>>>(S, Rp, Q, (int)nb, step, st);
            k_jac_apply<kCross><<<ga, kJThreads, 0, s>>>(S, V, Rp, Q, (int)nb, step, part, st);
        }
        k_jac_flag<<<1, kJThreads, 0, s>>>(part, (int)nT, tolc, st);
    }
    const unsigned gt = (unsigned)((r + 31) / 32);
    k_pinv_form<<<dim3(gt, gt), 256, 0, s>>>(S, V, Rp, r, tol, Cp, ldcp, eig, st);
    if (info) k_jac_info<<<1, 64, 0, s>>>(st, info);
    return hipGetLastError();
}

// W, then a pair of partial sums for each 64 x 64 tile (more than the kDT-wide tiles fill)
constexpr int kGT = 64;

size_t nystrom_workspace_bytes(int64_t n, int64_t r) {
    if (n <= 0 || r <= 0) return 0;
    const int64_t t = (n + kGT - 1) / kGT;
    return align256((size_t)(n * r) * 8) + align256((size_t)(t * t) * 16);
}

hipError_t launch_nystrom(const float* A, int64_t lda, const float* B, int64_t n, int64_t r,
                          int64_t ldb, const double* Cp, int64_t ldcp, int64_t row0, int64_t mr,
                          double* out, int64_t ldo, double* sums, void* ws, hipStream_t s) {
    double* W = static_cast<double*>(ws);
    char* pp = static_cast<char*>(ws) + align256((size_t)(n * r) * 8);
    double* part = reinterpret_cast<double*>(pp);
    const int64_t t64 = (n + kGT - 1) / kGT;
    // the partial sums of the kDT-wide tiles leave the last 8 bytes of their area free
    // (r < 64: the product is a small part, every tile reads its own A).  Mirrored tiles pay
    // where they save a round of tiles, two to a compute unit (r = 100: n = 3001 94 us without
    // them and 76 with them; n = 2048, one round either way, 57.5 and 60.2; n = 4096, two rounds
    // either way, 108 and 124)
    const int64_t td = (n + kDT - 1) / kDT, slots = 2 * device_cus();
    const bool pays = (td * (td + 1) / 2 + slots - 1) / slots < (td * td + slots - 1) / slots;
    int* sym = A && r >= 64 && pays ? reinterpret_cast<int*>(pp + align256((size_t)(t64 * t64) * 16) - 8)
                            : nullptr;
    const unsigned gr = (unsigned)((r + kDT - 1) / kDT);
    const int64_t mw = A ? n : mr;
    const float* Bw = A ? B : B + row0 * ldb;
    const unsigned gn = (unsigned)((n + kDT - 1) / kDT);
    const unsigned gm = (unsigned)((mw + kDT - 1) / kDT);
    const unsigned g32 = (unsigned)((r + 31) / 32);
    auto run = [&](auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
        k_bw<TAIL><<<dim3(gr, gm), 256, 0, s>>>(Bw, ldb, mw, r, Cp, ldcp, W, sym);
        if (sym) k_symmetric<<<dim3(g32, g32), 256, 0, s>>>(Cp, r, ldcp, sym);
        if (A)
            k_nys_tile<true, TAIL><<<dim3(gn, gm), 256, 0, s>>>(W, mw, B, ldb, n, r, A, lda, nullptr, 0,
                                                                part, sym);
        else
            k_nys_tile<false, TAIL><<<dim3(gn, gm), 256, 0, s>>>(W, mw, B, ldb, n, r, nullptr, 0, out,
                                                                 ldo, nullptr, nullptr);
    };
    if (r % kDK) run(std::true_type{});
    else run(std::false_type{});
    if (A) k_err_sum<<<1, kJThreads, 0, s>>>(part, (int64_t)gn * gm, sums);
    return hipGetLastError();
}

}  // namespace sk
