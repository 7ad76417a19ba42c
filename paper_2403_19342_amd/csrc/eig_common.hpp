// Pieces shared by the local eigensolvers of the set-up phase: the start
// blocks' noise and modes, the small dense eigenproblem, Cholesky factor and
// triangular inverse of one wavefront, the cluster rule and the stopping test.
#pragma once

#include "common.hpp"

namespace specmg {

constexpr int kDeg = 20;          // Chebyshev degree per cycle of a relaxed, warm-started solve
constexpr int kMaxCycles = 300;
constexpr int kWarmCycles = 4;     // cycles a learned start gets to reach the relaxed residual


__device__ __forceinline__ double hash_noise(unsigned a, unsigned b, unsigned c) {
    unsigned h = a * 0x9E3779B1u ^ (b + 0x7F4A7C15u) * 0x85EBCA77u ^ (c + 0x165667B1u) * 0xC2B2AE3Du;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    h *= 0x297A2D39u;
    h ^= h >> 15;
    return (double)(h & 0xFFFFFF) / 8388608.0 - 1.0;   // [-1, 1)
}

// low-frequency cosine modes (p, q, r) by increasing p^2+q^2+r^2
static __constant__ unsigned char kModes[16][3] = {
    {0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {1, 1, 0}, {1, 0, 1}, {0, 1, 1}, {1, 1, 1},
    {2, 0, 0}, {0, 2, 0}, {0, 0, 2}, {2, 1, 0}, {1, 2, 0}, {2, 0, 1}, {0, 2, 1}, {1, 0, 2}};

template <typename T>
__device__ __forceinline__ T harm_e(T a, T b) {
    const T s = a + b;
    return s > T(0) ? (T(2) * a * b) / s : T(0);
}

// ---------------------------------------------------------------------------
// small dense helpers on LDS, run by one thread or one wavefront

// Empty asm statements that take v as an operand: the arithmetic producing v
// runs before them, and no memory access moves across pin().  Used after
// every few columns of an operator apply, so that the compiler cannot hoist
// all of its LDS loads ahead of the arithmetic (a register per loaded value,
// which halves the waves per SIMD).
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)::"memory"); }
__device__ __forceinline__ void pin_value(double& v) { asm volatile("" : "+v"(v)); }

typedef __attribute__((address_space(3))) double lds_double;
typedef __attribute__((address_space(3))) int lds_int;

// 1 / sqrt(x), x > 0: the hardware estimate and one third-order correction
__device__ __forceinline__ double rsqrt_f64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Symmetric eigendecomposition H = Q diag(th) Q^T, eigenvalues ascending,
// by parallel cyclic Jacobi in one wavefront (every lane calls it).  Round
// robin with moving players: the pairs of a round are always the positions
// (2k, 2k + 1), and rows and columns move to the next round's positions as
// they are written back, so every address is the same in every round.  A lane
// owns one 2 x 2 block of H and of Q; the lanes of the diagonal blocks derive
// their rotations from the values they hold.  Stops when the largest
// off-diagonal entry is below rtol times the largest diagonal entry.  H (M*M)
// is destroyed; Q (M*M) receives the eigenvectors as columns; scr holds M
// values.
template <int M>
__device__ __forceinline__ void jacobi_wave(lds_double* H, lds_double* Q, lds_double* th, lds_double* scr,
                                            lds_int* iscr, double rtol = 1e-15) {
    static_assert(M % 2 == 0 && M <= 26, "Jacobi block size");
    typedef double __attribute__((ext_vector_type(2))) dbl2;
    typedef __attribute__((address_space(3))) dbl2 lds_dbl2;
    constexpr int N = M / 2, PER = (N * N + 63) / 64;
    const int lane = threadIdx.x & 63;
    // the position that the row or column at position p moves to
    auto moved = [](int p) {
        const int k = p >> 1;
        const int top = k == 0 ? 0 : (k < N - 1 ? 2 * k + 2 : 2 * N - 1);
        return (p & 1) ? (k == 0 ? (N > 1 ? 2 : 1) : 2 * k - 1) : top;
    };
    int src[PER], r0[PER], r1[PER], c0[PER], c1[PER], bp[PER], bq[PER];
    bool on[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int t = lane + 64 * u;
        on[u] = t < N * N;
        bp[u] = on[u] ? t / N : 0;
        bq[u] = on[u] ? t % N : 0;
        src[u] = 2 * bp[u] * M + 2 * bq[u];
        r0[u] = moved(2 * bp[u]) * M;
        r1[u] = moved(2 * bp[u] + 1) * M;
        c0[u] = moved(2 * bq[u]);
        c1[u] = moved(2 * bq[u] + 1);
        if (on[u]) {
            // symmetrised into registers before anything is written
            const int i = 2 * bp[u], j = 2 * bq[u];
            Q[i * M + j] = i == j ? 1.0 : 0.0;
            Q[i * M + j + 1] = 0.0;
            Q[(i + 1) * M + j] = 0.0;
            Q[(i + 1) * M + j + 1] = i == j ? 1.0 : 0.0;
        }
    }
    double h00[PER], h01[PER], h10[PER], h11[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = 2 * bp[u], j = 2 * bq[u];
        h00[u] = 0.5 * (H[i * M + j] + H[j * M + i]);
        h01[u] = 0.5 * (H[i * M + j + 1] + H[(j + 1) * M + i]);
        h10[u] = 0.5 * (H[(i + 1) * M + j] + H[j * M + i + 1]);
        h11[u] = 0.5 * (H[(i + 1) * M + j + 1] + H[(j + 1) * M + i + 1]);
    }
    wave_sync();
#pragma unroll 1
    for (int sweep = 0;; ++sweep) {
        double off = 0.0, dg = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (on[u]) {
                const double a = fmax(fabs(h00[u]), fabs(h11[u]));
                off = fmax(off, fmax(fabs(h01[u]), fabs(h10[u])));
                if (bp[u] == bq[u]) dg = fmax(dg, a);
                else off = fmax(off, a);
            }
        }
        off = wave_max(off);
        dg = wave_max(dg);
        if (off <= rtol * dg || off == 0.0 || sweep == 30) break;
#pragma unroll 1
        for (int r = 0; r < M - 1; ++r) {
            dbl2 q0[PER], q1[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                q0[u] = *(const lds_dbl2*)(Q + src[u]);
                q1[u] = *(const lds_dbl2*)(Q + src[u] + M);
                // the rotation (by at most pi/4) that annihilates h01 of a
                // diagonal block: rows 0' = c 0 - s 1, 1' = s 0 + c 1
                const double d = h11[u] - h00[u], o = 2.0 * h01[u];
                const double ir = rsqrt_f64(fma(d, d, o * o));
                const double x = fma(0.5 * fabs(d), ir, 0.5);
                const double ic = rsqrt_f64(x);
                const bool rot = o != 0.0;   // nothing to annihilate: the identity (d = 0 would give NaN)
                const double c = rot ? x * ic : 1.0;
                const double s = rot ? 0.5 * (d >= 0.0 ? o : -o) * ir * ic : 0.0;
                if (on[u] && bp[u] == bq[u]) *(lds_dbl2*)(scr + 2 * bp[u]) = dbl2{c, s};
            }
            wave_sync();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const dbl2 p = *(const lds_dbl2*)(scr + 2 * bp[u]), q = *(const lds_dbl2*)(scr + 2 * bq[u]);
                const double a00 = q.x * h00[u] - q.y * h01[u], a01 = q.y * h00[u] + q.x * h01[u];
                const double a10 = q.x * h10[u] - q.y * h11[u], a11 = q.y * h10[u] + q.x * h11[u];
                const bool dia = bp[u] == bq[u];   // the annihilated entries are zero exactly
                if (on[u]) {
                    H[r0[u] + c0[u]] = p.x * a00 - p.y * a10;
                    H[r0[u] + c1[u]] = dia ? 0.0 : p.x * a01 - p.y * a11;
                    H[r1[u] + c0[u]] = dia ? 0.0 : p.y * a00 + p.x * a10;
                    H[r1[u] + c1[u]] = p.y * a01 + p.x * a11;
                    Q[2 * bp[u] * M + c0[u]] = q.x * q0[u].x - q.y * q0[u].y;
                    Q[2 * bp[u] * M + c1[u]] = q.y * q0[u].x + q.x * q0[u].y;
                    Q[(2 * bp[u] + 1) * M + c0[u]] = q.x * q1[u].x - q.y * q1[u].y;
                    Q[(2 * bp[u] + 1) * M + c1[u]] = q.y * q1[u].x + q.x * q1[u].y;
                }
            }
            wave_sync();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const dbl2 a = *(const lds_dbl2*)(H + src[u]), b = *(const lds_dbl2*)(H + src[u] + M);
                h00[u] = a.x;
                h01[u] = a.y;
                h10[u] = b.x;
                h11[u] = b.y;
            }
        }
    }
    // ascending order: lane k < M finds the rank of H[k][k]
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (on[u] && bp[u] == bq[u]) {
            scr[2 * bp[u]] = h00[u];
            scr[2 * bp[u] + 1] = h11[u];
        }
    }
    wave_sync();
    if (lane < M) {
        const double hk = scr[lane];
        int rank = 0;
#pragma unroll
        for (int l = 0; l < M; ++l) {
            const double hl = scr[l];
            rank += (hl < hk || (hl == hk && l < lane)) ? 1 : 0;
        }
        iscr[rank] = lane;
        th[rank] = hk;
    }
    wave_sync();
    constexpr int QPER = (M * M + 63) / 64;
    double nq[QPER];
#pragma unroll
    for (int u = 0; u < QPER; ++u) {
        const int t = lane + 64 * u < M * M ? lane + 64 * u : 0;
        nq[u] = Q[t - t % M + iscr[t % M]];
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < QPER; ++u)
        if (lane + 64 * u < M * M) Q[lane + 64 * u] = nq[u];
    wave_sync();
}

// Generalised Rayleigh-Ritz of a block Y from G = Y^T Y and H = Y^T A Y, by
// one wavefront: C (into Q) with (Y C)^T (Y C) = I and (Y C)^T A (Y C) =
// diag(th).  G is scaled to a unit diagonal and factored G = R^T R with lane l
// holding column l in registers (pivots and rows travel by readlane, so no step
// waits for LDS), then C = D R^-1 Q with Q the eigenvectors of
// (D R^-1)^T H (D R^-1).  Returns the smallest pivot of the scaled G; pivots
// below 1e-12 are raised to that.  When it is below min_ritz the eigenproblem
// is left out and C = D R^-1 (a Cholesky-QR step).  G and H are destroyed (H
// keeps D R^-1 while the eigenproblem runs); scr holds M values.  With nval < M
// the columns nval.. of Y are zero and the others orthonormal: C is the
// eigenvectors' matrix, pad (above the spectrum) the values of the empty
// columns, which sort last.
// A call of its own: inlined, the caller's live registers (the couplings of
// its operator) push this routine's arrays to scratch.
template <int M>
__device__ __attribute__((noinline)) double ritz_wave(lds_double* G, lds_double* H, lds_double* Q, lds_double* scr,
                                                      lds_double* th, lds_int* iscr, double min_ritz, double rtol,
                                                      int nval = M, double pad = 0.0) {
    const int lane = threadIdx.x & 63, l = lane < M ? lane : M - 1;
    double x[M];
    double low = 1.0;
    if (nval < M) {
#pragma unroll
        for (int i = 0; i < M; ++i) x[i] = i == l ? 1.0 : 0.0;
    } else {
    double g[M];
    const double gll = G[l * M + l];
    const double dl = gll > 1e-300 ? rsqrt_f64(gll) : 0.0;
#pragma unroll
    for (int i = 0; i < M; ++i) g[i] = G[i * M + l] * dl * read_lane(dl, i);
    double ir[M];
#pragma unroll
    for (int j = 0; j < M; ++j) {
        double p = read_lane(g[j], j);
        low = fmin(low, p > 0.0 ? p : 0.0);
        p = p > 1e-12 ? p : 1e-12;
        ir[j] = rsqrt_f64(p);
        g[j] *= ir[j];   // R[j][l], used for l >= j
#pragma unroll
        for (int i = j + 1; i < M; ++i) g[i] -= read_lane(g[j], i) * g[j];
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < M; ++i) x[i] = i == l ? 1.0 : 0.0;
#pragma unroll
    for (int i = M - 1; i >= 0; --i) {
        x[i] *= ir[i];
#pragma unroll
        for (int k = 0; k < i; ++k) x[k] -= read_lane(g[k], i) * x[i];
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < M; ++i) x[i] = i <= l ? x[i] * read_lane(dl, i) : 0.0;
    }
    if (low < min_ritz) {
        if (lane < M) {
#pragma unroll
            for (int i = 0; i < M; ++i) Q[i * M + lane] = x[i];
        }
        wave_sync();
        return low;
    }
    // lane l: column l of H C0, then of C0^T H C0
    double t[M];
#pragma unroll
    for (int i = 0; i < M; ++i) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < M; ++k) s += H[i * M + k] * x[k];
        t[i] = s;
        pin(t[i]);   // formed here: the compiler would load all of H first
    }
    wave_sync();
    if (lane < M) {
#pragma unroll
        for (int i = 0; i < M; ++i) H[i * M + lane] = x[i];
    }
    wave_sync();
#pragma unroll
    for (int m = M - 1; m >= 0; --m) {   // row m needs t[0..m] only
        double s = 0.0;
#pragma unroll
        for (int i = 0; i <= m; ++i) s += H[i * M + m] * t[i];
        t[m] = s;
        pin(t[m]);
    }
    if (lane < M) {
#pragma unroll
        for (int m = 0; m < M; ++m) G[m * M + lane] = m == lane && m >= nval ? pad : t[m];
    }
    wave_sync();
    jacobi_wave<M>(G, Q, th, scr, iscr, rtol);
    {
        const int c = lane < M ? lane : 0;
#pragma unroll
        for (int i = 0; i < M; ++i) t[i] = Q[i * M + c];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < M; ++i) {   // row i needs t[i..M-1] only
        double s = 0.0;
#pragma unroll
        for (int k = i; k < M; ++k) s += H[i * M + k] * t[k];
        t[i] = s;
        pin(t[i]);
    }
    if (lane < M) {
#pragma unroll
        for (int i = 0; i < M; ++i) Q[i * M + lane] = t[i];
    }
    wave_sync();
    return low;
}

// Cluster rule on ascending values th[0..n-1] (n >= target+4 or all values):
// keep `target`, grow to the end of a cluster of equal values up to
// target+3, or shrink before the cluster when it runs past that cap.
__device__ inline int cluster_cut_dev(const double* th, int n, int target, double rtol, double thr) {
    if (thr > 0.0) {
        // threshold rule (strategy 2 of Section 5): the eigenvalues below
        // thr, at least one and at most target, then the cluster rule
        int below = 0;
        for (int j = 0; j < n; ++j) below += th[j] < thr ? 1 : 0;
        target = below < 1 ? 1 : (below < target ? below : target);
    }
    if (target >= n) return n;
    auto same = [&](int k) { return th[k] - th[k - 1] <= rtol * fmax(fabs(th[k]), 1e-12); };
    int k = target;
    const int cap = target + 3 < n ? target + 3 : n;
    while (k < cap && same(k)) ++k;
    if (k == cap && k < n && same(k)) {
        k = target;
        while (k > 1 && same(k)) --k;
    }
    return k;
}

// whether every vector that decides the kept space has converged (see chefsi)
__device__ __forceinline__ bool chefsi_done(const double* th, const double* nrm, int M, int need, double tol,
                                            double bnd, int target, double crtol, double thr, int cyc) {
    const int nk = cluster_cut_dev(th, M, target, crtol, thr);
    bool ok = true;
    for (int j = 0; j < need; ++j) {
        const double rj = sqrt(nrm[j]);
        // under the threshold rule the 5 % separation counts only after
        // a filter cycle: an eigenvalue below the threshold that the start
        // block misses has not been amplified yet and would change the count
        const bool sep = (thr <= 0.0 || cyc > 0) && j >= nk && nk > 0 && th[j] - th[nk - 1] > 0.05 * fabs(th[j]);
        ok = ok && (rj <= (j < nk ? tol : sqrt(tol)) * bnd || sep);
    }
    return ok;
}

}  // namespace specmg
