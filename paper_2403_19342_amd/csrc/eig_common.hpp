// Pieces shared by the local eigensolvers of the set-up phase: the start
// blocks' noise and modes, the small dense steps (one wavefront, LDS and
// registers), the cluster rule and the stopping test.
//
// The order of every sum here and in the eigensolvers is part of the result:
// the local eigenvectors are accurate to the tolerance over the spectral gaps,
// and on media of contrast 1e6 what rounding leaves in them shows in the face
// fluxes of a solve.  Where the compiler would be free to contract a product with
// one of two sums, the fused operation is written out.
#pragma once

#include "common.hpp"

namespace specmg {

constexpr int kDeg = 20;          // Chebyshev degree per cycle of a relaxed, warm-started solve
constexpr int kDegExact = 40;     // ... of an exact solve (fewer cycles, so fewer orthonormalisations
                                  //     and Rayleigh-Ritz steps per filtered vector)
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

// An empty asm statement that takes v as an operand: the arithmetic producing v
// is done before it, and is not contracted with what follows.
__device__ __forceinline__ void pin_value(double& v) { asm volatile("" : "+v"(v)); }
// the same, and no memory access moves across it
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)::"memory"); }

// pointers to LDS that stay LDS pointers across a call
typedef __attribute__((address_space(3))) double lds_double;
typedef __attribute__((address_space(3))) int lds_int;

// ---------------------------------------------------------------------------
// sums over the wavefront

// Sums of 16 values over each 64-lane group of rows, in the order of wave_sum
// (lanes 1, 2, 4 and 8 apart, then the four 16-lane rows pairwise), value i
// returned by the lanes whose low bits name it (sum16_index).  Each of the first
// four steps halves the values that a lane carries: it keeps the half that its
// lane bit names and receives the partner's part of it: 111 instructions for 16
// sums against 22 each.
__device__ __forceinline__ int sum16_index(int lane) {
    return (lane & 1) << 3 | (lane & 2) << 1 | (lane & 4) >> 1 | (lane & 8) >> 3;
}
__device__ __forceinline__ double sum16(double (&p)[16], int lane) {
    auto step = [&](auto exchange, int bit, int half) {
        const bool up = (lane & bit) != 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < half) {
                const double keep = up ? p[i + half] : p[i], send = up ? p[i] : p[i + half];
                p[i] = keep + exchange(send);
            }
        }
    };
    step([](double v) { return dpp_move<0xB1>(v); }, 1, 8);                    // quad_perm [1,0,3,2]
    step([](double v) { return dpp_move<0x4E>(v); }, 2, 4);                    // quad_perm [2,3,0,1]
    step([](double v) { return dpp_move<0x141>(dpp_move<0x1B>(v)); }, 4, 2);   // lane ^ 3, then lane ^ 7
    step([](double v) { return dpp_move<0x128>(v); }, 8, 1);                   // row_ror:8
    double v = p[0];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// sums over the wavefront's rows of value(e), e < NE, to red[e]
template <int NE, class V>
__device__ __forceinline__ void tile_sums(double* red, int lane, V value) {
#pragma unroll
    for (int g = 0; g < (NE + 15) / 16; ++g) {
        double p[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) p[i] = 16 * g + i < NE ? value(16 * g + i) : 0.0;
        const double v = sum16(p, lane);
        const int e = 16 * g + sum16_index(lane);
        if (lane < 16 && e < NE) red[e] = v;
        __builtin_amdgcn_sched_barrier(0);
    }
}

// row and column of entry e of the upper triangle, row by row
template <int M>
struct Triangle {
    unsigned char i[M * (M + 1) / 2], j[M * (M + 1) / 2];
    constexpr Triangle() : i(), j() {
        int e = 0;
        for (int a = 0; a < M; ++a)
            for (int b = a; b < M; ++b) {
                i[e] = (unsigned char)a;
                j[e++] = (unsigned char)b;
            }
    }
};

// the factors of the scaled Chebyshev recurrence (wanted spectrum below a, damped
// interval [a, b], a0 below the whole spectrum): X_1 = (A X - c X) fc[0],
// X_k+1 = (A X_k - c X_k) fc[2k] - fc[2k+1] X_k-1
__device__ __forceinline__ void filter_factors(double* fc, double a, double b, double a0, int deg) {
    const double e = 0.5 * (b - a), cc = 0.5 * (b + a);
    double sigma = e / (a0 - cc);
    const double tau = 2.0 / sigma;
    fc[0] = sigma / e;
    fc[1] = 0.0;
#pragma unroll 1
    for (int it = 1; it < deg; ++it) {
        const double sn = 1.0 / (tau - sigma);
        fc[2 * it] = 2.0 * sn / e;
        fc[2 * it + 1] = sigma * sn;
        sigma = sn;
    }
}

// ---------------------------------------------------------------------------
// small dense steps of one wavefront (every lane calls them)

// Rotation (c, s) that annihilates hpq: the rotated rows are p' = c p - s q and
// q' = s p + c q.
__device__ __forceinline__ void jac_rot(double hpp, double hqq, double hpq, double& c, double& s) {
    c = 1.0;
    s = 0.0;
    if (hpq != 0.0) {
        const double tt = (hqq - hpp) / (2.0 * hpq);
        const double t = (tt >= 0.0 ? 1.0 : -1.0) / (fabs(tt) + sqrt(fma(tt, tt, 1.0)));
        c = 1.0 / sqrt(fma(t, t, 1.0));
        s = t * c;
    }
}

// Symmetric eigendecomposition H = Q diag(th) Q^T, eigenvalues ascending, by
// parallel cyclic Jacobi.  Circle-method round robin on M players (M even): in
// round r player M-1 meets player r and every other pair (i, j) has i + j = 2r
// modulo M-1.  A lane owns the 2 x 2 block of H and of Q where a pair's rows meet a
// pair's columns; the lanes of the diagonal blocks derive the rotations (scr), which
// is most of a round (three divisions and two roots, one after the other).  Stops when the largest off-diagonal entry is
// below 1e-15 times the largest diagonal entry, or after 30 sweeps.  H (M*M) is
// destroyed; Q (M*M) receives the eigenvectors as columns; scr holds 2 M values.
template <int M>
__device__ __forceinline__ void jacobi_wave(lds_double* H, lds_double* Q, lds_double* th, lds_double* scr, lds_int* iscr) {
    static_assert(M % 2 == 0 && M <= 26, "Jacobi block size");
    constexpr int N = M / 2, K = M - 1, PER = (N * N + 63) / 64, MM = M * M, QPER = (MM + 63) / 64;
    const int lane = threadIdx.x & 63;
    int bp[PER], bq[PER];
    bool on[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int t = lane + 64 * u;
        on[u] = t < N * N;
        bp[u] = on[u] ? t / N : 0;
        bq[u] = on[u] ? t % N : 0;
    }
#pragma unroll
    for (int u = 0; u < QPER; ++u) {
        const int t = lane + 64 * u;
        if (t < MM) Q[t] = t / M == t % M ? 1.0 : 0.0;
    }
    wave_sync();
    // players of pair k in round r, the smaller first
    auto players = [](int k, int r, int& a, int& b) {
        int i = r + k, j = r - k;
        i = i >= K ? i - K : i;
        j = k == 0 ? K : (j < 0 ? j + K : j);
        a = min(i, j);
        b = max(i, j);
    };
#pragma unroll 1
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0, dg = 0.0;
#pragma unroll
        for (int u = 0; u < QPER; ++u) {
            const int t = lane + 64 * u;
            const double h = t < MM ? fabs(H[t]) : 0.0;
            if (t / M != t % M) off = fmax(off, h);
            else dg = fmax(dg, h);
        }
        off = wave_max(off);
        dg = wave_max(dg);
        if (off <= 1e-15 * dg || off == 0.0) break;
#pragma unroll 1
        for (int r = 0; r < K; ++r) {
            int ai[PER], bi[PER], aj[PER], bj[PER];
            double h[PER][4], q[PER][4];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                players(bp[u], r, ai[u], bi[u]);
                players(bq[u], r, aj[u], bj[u]);
                h[u][0] = H[ai[u] * M + aj[u]];
                h[u][1] = H[ai[u] * M + bj[u]];
                h[u][2] = H[bi[u] * M + aj[u]];
                h[u][3] = H[bi[u] * M + bj[u]];
                q[u][0] = Q[ai[u] * M + aj[u]];
                q[u][1] = Q[ai[u] * M + bj[u]];
                q[u][2] = Q[bi[u] * M + aj[u]];
                q[u][3] = Q[bi[u] * M + bj[u]];
            }
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (on[u] && bp[u] == bq[u]) {
                    double c, s;
                    jac_rot(h[u][0], h[u][3], h[u][1], c, s);
                    scr[2 * bp[u]] = c;
                    scr[2 * bp[u] + 1] = s;
                }
            wave_sync();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const double ci = scr[2 * bp[u]], si = scr[2 * bp[u] + 1], cj = scr[2 * bq[u]], sj = scr[2 * bq[u] + 1];
                // columns, then rows
                const double a0 = fma(cj, h[u][0], -(sj * h[u][1])), a1 = fma(sj, h[u][0], cj * h[u][1]);
                const double b0 = fma(cj, h[u][2], -(sj * h[u][3])), b1 = fma(sj, h[u][2], cj * h[u][3]);
                const bool dia = bp[u] == bq[u];   // the annihilated entries are zero exactly
                if (on[u]) {
                    H[ai[u] * M + aj[u]] = fma(ci, a0, -(si * b0));
                    H[ai[u] * M + bj[u]] = dia ? 0.0 : fma(ci, a1, -(si * b1));
                    H[bi[u] * M + aj[u]] = dia ? 0.0 : fma(si, a0, ci * b0);
                    H[bi[u] * M + bj[u]] = fma(si, a1, ci * b1);
                    Q[ai[u] * M + aj[u]] = fma(cj, q[u][0], -(sj * q[u][1]));
                    Q[ai[u] * M + bj[u]] = fma(sj, q[u][0], cj * q[u][1]);
                    Q[bi[u] * M + aj[u]] = fma(cj, q[u][2], -(sj * q[u][3]));
                    Q[bi[u] * M + bj[u]] = fma(sj, q[u][2], cj * q[u][3]);
                }
            }
            wave_sync();
        }
    }
    // ascending order: lane k < M finds the rank of H[k][k]
    if (lane < M) {
        const double hk = H[lane * M + lane];
        int rank = 0;
#pragma unroll
        for (int l = 0; l < M; ++l) {
            const double hl = H[l * M + l];
            rank += (hl < hk || (hl == hk && l < lane)) ? 1 : 0;
        }
        iscr[rank] = lane;
        th[rank] = hk;
    }
    wave_sync();
    double nq[QPER];
#pragma unroll
    for (int u = 0; u < QPER; ++u) {
        const int t = lane + 64 * u < MM ? lane + 64 * u : 0;
        nq[u] = Q[t - t % M + iscr[t % M]];
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < QPER; ++u)
        if (lane + 64 * u < MM) Q[lane + 64 * u] = nq[u];
    wave_sync();
}

// Cholesky-QR's small step: C = R^-1 (into C, M*M, upper triangular) with
// G = R^T R.  Lane l holds column l of R, then of R^-1, in registers; rows and
// pivots travel by readlane.  Where G is not numerically positive definite (a
// rank-deficient block) a tiny diagonal shift keeps the factor finite; the next
// Chebyshev cycle restores the lost directions.
template <int M>
__device__ __forceinline__ void cholesky_inverse_wave(const lds_double* G, lds_double* C) {
    const int lane = threadIdx.x & 63, l = lane < M ? lane : M - 1;
    double g[M], dinv[M], shift = 0.0;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < M; ++i) g[i] = G[i * M + l];
        if (attempt) {
            double mx = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) mx = fmax(mx, G[i * M + i]);
            shift = fma(1e-12, mx, 1e-300);
#pragma unroll
            for (int i = 0; i < M; ++i) g[i] = i == l ? g[i] + shift : g[i];
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            double d = read_lane(g[j], j);
            if (!(d > 0.0)) {
                ok = false;
                d = 1.0;
            }
            const double inv_d = 1.0 / d;
            // trailing update of the upper triangle with the unscaled row j
#pragma unroll
            for (int i = j + 1; i < M; ++i) {
                double p = read_lane(g[j], i) * g[j];
                g[i] = fma(-p, inv_d, g[i]);
            }
            const double root = sqrt(d);
            dinv[j] = 1.0 / root;
            g[j] = l == j ? root : g[j] * dinv[j];
            __builtin_amdgcn_sched_barrier(0);
        }
        if (ok) break;
    }
    double x[M];
#pragma unroll
    for (int i = M - 1; i >= 0; --i) {
        double v = l == i ? 1.0 : 0.0;
#pragma unroll
        for (int k = i + 1; k < M; ++k) v = fma(-read_lane(g[i], k), x[k], v);
        x[i] = l >= i ? v * dinv[i] : 0.0;
        __builtin_amdgcn_sched_barrier(0);
    }
    if (lane < M) {
#pragma unroll
        for (int i = 0; i < M; ++i) C[i * M + lane] = x[i];
    }
    wave_sync();
}

// Both as calls of their own: inlined, their registers push the caller's operator
// to scratch.
template <int M>
__device__ __attribute__((noinline)) void jacobi_call(lds_double* H, lds_double* Q, lds_double* th, lds_double* scr,
                                                      lds_int* iscr) {
    jacobi_wave<M>(H, Q, th, scr, iscr);
}
template <int M>
__device__ __attribute__((noinline)) void cholesky_call(const lds_double* G, lds_double* C) {
    cholesky_inverse_wave<M>(G, C);
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

// Whether every vector that decides the kept space has converged: vectors that
// the cluster rule keeps need residual <= tol*bnd; the remaining ones up to index
// need-1 only feed the cluster decision through their eigenvalues (error <=
// residual^2 / gap), so sqrt(tol)*bnd, unless their Ritz value already lies 5 %
// above the last kept one: then the decision cannot change (a partner of a kept
// eigenvalue would have been amplified like the kept vectors, which have
// converged; under the threshold rule this needs at least one filter cycle).
// Without that exception a degenerate cluster straddling the block's end (the
// Laplace ladder of a homogeneous element) is never resolved: the filter's cut
// sits on the cluster.
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
