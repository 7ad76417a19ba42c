// Local eigensolves of the levels >= 3 (Section 3, eq. spectral cc): on every
// parent element E the restricted problem H_E v = lambda v with
// H_E = B_E^T A_E B_E assembled from the level below (its Gram is the identity
// for S-normalised bases), a block 7-point matrix over the kept slots of the
// agg^3 children.
//
// Method: subspace iteration with a Chebyshev filter in the shifted inverse.
// The wanted eigenvalues lie at the bottom of a spectrum of several decades,
// where a polynomial in H_E separates them by sqrt((a - lambda) / b) per degree
// (300 to 700 applications per element at 128^3, contrast 1e6); a polynomial in
// (H_E + sigma)^-1 separates them by sqrt((a - lambda) / (lambda + sigma)): about 22
// solves and 3 factorisations per element, in 3 to 4 cycles.  sigma is a tenth of
// the block's largest Ritz value (at least 1e-7 of the spectral bound), so the
// inverse stays well conditioned and is applied explicitly.
//
// The inverse is kept in block form over the planes of children in z
// (agg = 4: four planes of up to 16 children; agg = 2: one block when its rows
// fit, else two planes): T_p = S_p^-1 with S_p = D_p + sigma -
// C_{p-1}^T T_{p-1} C_{p-1}, D_p the plane's block of H_E and C_p its couplings
// to the next plane (one child each).  A solve is 2 P - 1 dense products
// T_p (m x m) times (m x M) on the FP64 matrix cores.
//
// One workgroup per parent; the block (rows x M) lives in LDS, the planes'
// inverses and the filter's second iterate in a workspace slot of the
// workgroup (read through L2).  Rows are compact: kept slots only.
#include <algorithm>

#include "eig_common.hpp"

namespace specmg {

constexpr int kMaxLP = 23;        // lower-level widths up to target 20 + 3
constexpr int kUpSingle = 112;    // rows up to which the children form one block (agg = 2)

// Hd[c] = Aint[c] + sum of D[c][d] over the faces of c interior to its parent
__global__ void k_build_hd(CoarseGeom lo, const double* __restrict__ Aint, const double* __restrict__ D,
                           double* __restrict__ Hd) {
    const int c = blockIdx.x;
    const int L = lo.L;
    const int cx = c % lo.mx, cy = (c / lo.mx) % lo.my, cz = c / (lo.mx * lo.my);
    const int q0 = cx % lo.agg, q1 = cy % lo.agg, q2 = cz % lo.agg;
    for (int t = threadIdx.x; t < L * L; t += blockDim.x) {
        double v = Aint[(size_t)c * L * L + t];
        for (int d = 0; d < 6; ++d) {
            const int ax = d >> 1;
            const int q = ax == 0 ? q0 : (ax == 1 ? q1 : q2);
            const bool interior = (d & 1) ? (q < lo.agg - 1) : (q > 0);
            if (interior) v += D[((size_t)c * 6 + d) * L * L + t];
        }
        Hd[(size_t)c * L * L + t] = v;
    }
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) double gl_double;
typedef __attribute__((address_space(3))) unsigned short lds_ushort;

__device__ __forceinline__ unsigned uniform32(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v) {
    return (unsigned long long)uniform32((unsigned)v) | ((unsigned long long)uniform32((unsigned)(v >> 32)) << 32);
}

__device__ __forceinline__ int ceil16(int m) { return (m + 15) & ~15; }

// 1 / x: the hardware estimate and one third-order correction
__device__ __forceinline__ double rcp_f64(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// In-place inverse of the symmetric positive definite m x m matrix at T (leading
// dimension ld) by symmetric sweeps over pairs of pivots, the matrix in the
// registers of the NT threads (thread (ty, tx) of a TY x TX grid owns elements
// (ty + TY a, tx + TX b)).  A sweep publishes its two pivot rows (by symmetry
// also the columns) through one of two LDS buffers in turn, so a pair costs one
// barrier; the latency of that exchange and of the pivots' reciprocals is what
// bounds it.  Entries beyond m come out zero.  rows: 4 x 192 doubles.
constexpr int kSweepRow = 192;
template <int NT, int A, int B>
__device__ __attribute__((noinline)) void sweep_inverse(gl_double* Tv, int mv, int ldv, lds_double* rowsv) {
    gl_double* const T = (gl_double*)uniform64((unsigned long long)Tv);
    lds_double* const rows = (lds_double*)uniform32((unsigned)(size_t)rowsv);
    const int m = (int)uniform32((unsigned)mv), ld = (int)uniform32((unsigned)ldv);
    constexpr int TY = 16, TX = NT / TY;
    static_assert(TX == TY || TX == 2 * TY, "pivot columns in a static register");
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    double v[A][B];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = ty + TY * a, j = tx + TX * b;
            v[a][b] = i < m && j < m ? T[(size_t)i * ld + j] : 0.0;
        }
#pragma unroll
    for (int a = 0; a < A; ++a) {
        constexpr int step = TX / TY;
        const int bk = a / step;   // register column of the pivots
#pragma unroll 1
        for (int s = 0; s < TY; s += 2) {
            const int k = TY * a + s;
            if (k >= m) break;
            lds_double* r0 = rows + 2 * kSweepRow * ((k >> 1) & 1);
            lds_double* r1 = r0 + kSweepRow;
            if ((ty & ~1) == s) {
                lds_double* r = ty == s ? r0 : r1;
#pragma unroll
                for (int b = 0; b < B; ++b) r[tx + TX * b] = v[a][b];
            }
            __syncthreads();
            // inverse of the pivot block; a row k + 1 beyond m is zero
            const bool two = k + 1 < m;
            const double a00 = r0[k], a01 = r0[k + 1], a11 = r1[k + 1];
            const double i0 = rcp_f64(a00), l = a01 * i0;
            const double i1 = rcp_f64(two ? a11 - l * a01 : 1.0);
            const double p01 = -l * i1, p00 = i0 - l * p01, p11 = two ? i1 : 0.0;
            double c0[B], c1[B], w0[A], w1[A];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const double x = r0[tx + TX * b], y = r1[tx + TX * b];
                c0[b] = p00 * x + p01 * y;
                c1[b] = p01 * x + p11 * y;
            }
#pragma unroll
            for (int i = 0; i < A; ++i) {
                w0[i] = r0[ty + TY * i];
                w1[i] = r1[ty + TY * i];
            }
#pragma unroll
            for (int i = 0; i < A; ++i)
#pragma unroll
                for (int b = 0; b < B; ++b) v[i][b] -= w0[i] * c0[b] + w1[i] * c1[b];
            const bool row0 = ty == s, row1 = ty == s + 1, col0 = tx == k % TX, col1 = tx == k % TX + 1;
            if (row0 || row1) {
#pragma unroll
                for (int b = 0; b < B; ++b) v[a][b] = row0 ? c0[b] : c1[b];
            }
            if (col0 || col1) {
#pragma unroll
                for (int i = 0; i < A; ++i) v[i][bk] = col0 ? p00 * w0[i] + p01 * w1[i] : p01 * w0[i] + p11 * w1[i];
                if (row0) v[a][bk] = col0 ? -p00 : -p01;
                if (row1) v[a][bk] = col0 ? -p01 : -p11;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = ty + TY * a, j = tx + TX * b;
            if (i < ld && j < ld) T[(size_t)i * ld + j] = -v[a][b];
        }
    __syncthreads();
}

template <int NT>
__device__ __forceinline__ void invert_block(gl_double* T, int m, int ld, lds_double* rows) {
    if constexpr (NT == 256) {
        if (m <= 48) sweep_inverse<NT, 3, 3>(T, m, ld, rows);
        else if (m <= 64) sweep_inverse<NT, 4, 4>(T, m, ld, rows);
        else if (m <= 80) sweep_inverse<NT, 5, 5>(T, m, ld, rows);
        else sweep_inverse<NT, 7, 7>(T, m, ld, rows);
    } else {
        if (m <= 96) sweep_inverse<NT, 6, 3>(T, m, ld, rows);
        else if (m <= 128) sweep_inverse<NT, 8, 4>(T, m, ld, rows);
        else sweep_inverse<NT, 12, 6>(T, m, ld, rows);
    }
}

// Cycles with the inverse filter: up to 10 were seen to suffice, all but one
// of some 36,000 elements a field; what is left converges by the filter in
// H_E, of kDampDeg applications.
constexpr int kInverseCycles = 14;
constexpr int kDampDeg = 40;

template <int M, int NT>
struct UpShared {
    double G[M * M];
    double H[M * M];
    double Q[M * M];
    double th[M], nrm[M], scr[M];
    double red[NT];
    double rows[4 * kSweepRow];
    double misc[NT / 64];
    double ct[3 * 4];
    double low;
    int iscr[M];
    int koff[65];     // first compact row of child p (65: the number of rows)
    int elem[64];     // lower-level element of child p
};

// the parent's operator and block, shared by the kernel's phases
template <int M, int NT>
struct UpProblem {
    static constexpr int NW = NT / 64;
    static constexpr int NCT = (M + 15) / 16;       // column tiles of the matrix cores
    static constexpr int PT = M <= 16 ? 18 : M + 2;  // row pitch of the LDS blocks
    static constexpr int PG = 16 * NCT;             // row pitch of the workspace blocks
    // address spaces are spelled out: the phases are calls of their own, and
    // through plain pointers their accesses would be flat ones
    typedef __attribute__((address_space(3))) UpShared<M, NT> lds_shared;
    lds_shared* sh;
    lds_double* Y;         // rows x PT: the block (the solve's result while filtering)
    lds_double* U;         // a plane's right-hand side
    lds_ushort* row;       // child position << 8 | slot of a compact row
    gl_double* T;          // workspace: the planes' inverses, mp^2 each
    gl_double *Wk, *Yg, *Xg, *AYg;
    const gl_double *Hd, *Aoff;
    int LP, agg, n, planes, mpmax;
    int w, lane;

    __device__ __forceinline__ int plane_row(int p) const {
        return (int)uniform32((unsigned)sh->koff[planes == 1 ? p * 64 : p * agg * agg]);
    }
    __device__ __forceinline__ int plane_end(int p) const {
        return planes == 1 ? n : (int)uniform32((unsigned)sh->koff[(p + 1) * agg * agg]);
    }

    // entry (i, j) of H_E for rows of children that are equal or neighbours
    // along axis ax (ax < 0: the same child); up: the child of j lies above
    __device__ __forceinline__ double entry(int ci, int ai, int cj, int bj, int ax, bool up) const {
        if (ax < 0) return Hd[((size_t)ci * LP + ai) * LP + bj];
        return up ? Aoff[(((size_t)ci * 3 + ax) * LP + ai) * LP + bj] : Aoff[(((size_t)cj * 3 + ax) * LP + bj) * LP + ai];
    }

    // coordinates of child p (agg is 2 or 4: shifts)
    __device__ __forceinline__ int lg() const { return agg == 4 ? 2 : 1; }
    __device__ __forceinline__ int child_x(int p) const { return p & (agg - 1); }
    __device__ __forceinline__ int child_y(int p) const { return (p >> lg()) & (agg - 1); }
    __device__ __forceinline__ int child_z(int p) const { return p >> (2 * lg()); }

    // sum_k c[k cs] x[k xs], k < kn (kn >= 1): eight of each in flight (beyond kn
    // the last one again, with weight zero, so that no load is conditional)
    template <class PC, class PX>
    static __device__ __forceinline__ double coupled(PC c, int cs, PX x, int xs, int kn) {
        double s = 0.0;
#pragma unroll 1
        for (int k0 = 0; k0 < kn; k0 += 8) {
            double h[8], y[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) h[u] = c[min(k0 + u, kn - 1) * cs];
#pragma unroll
            for (int u = 0; u < 8; ++u) y[u] = x[min(k0 + u, kn - 1) * xs];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (k0 + u < kn ? h[u] : 0.0) * y[u];
        }
        return s;
    }

    // AYg = H_E Y, one row per thread
    __device__ __forceinline__ void apply() const {
        const int a2 = agg * agg;
#pragma unroll 1
        for (int r = threadIdx.x; r < n; r += NT) {
            const int p = row[r] >> 8, a = row[r] & 255;
            const int qx = child_x(p), qy = child_y(p), qz = child_z(p);
            const int c = sh->elem[p];
            double acc[M];
#pragma unroll
            for (int j = 0; j < M; ++j) acc[j] = 0.0;
#pragma unroll 1
            for (int d = -1; d < 6; ++d) {
                const int ax = d < 0 ? -1 : d >> 1;
                const int q = ax <= 0 ? qx : (ax == 1 ? qy : qz);
                const bool up = d & 1;
                if (d >= 0 && (up ? q >= agg - 1 : q <= 0)) continue;
                const int st = ax <= 0 ? 1 : (ax == 1 ? agg : a2);
                const int pn = d < 0 ? p : (up ? p + st : p - st);
                const int cn = sh->elem[pn], k0 = sh->koff[pn], kn = sh->koff[pn + 1] - k0;
#pragma unroll 4
                for (int b = 0; b < kn; ++b) {
                    const double h = entry(c, a, cn, b, ax, up);
                    const lds_double* y = Y + (k0 + b) * PT;
#pragma unroll
                    for (int j = 0; j < M; ++j) acc[j] += h * y[j];
                }
            }
#pragma unroll
            for (int j = 0; j < M; ++j) AYg[(size_t)r * PG + j] = acc[j];
        }
    }

    // sh->G = Y^T Y, sh->H = Y^T AYg on the matrix cores: the two operands of a
    // Gram product are the same registers.  The wavefronts' sums are added in
    // wavefront order.
    __device__ __forceinline__ void grams() const {
        v4d g[NCT][NCT], h[NCT][NCT];
#pragma unroll
        for (int a = 0; a < NCT; ++a)
#pragma unroll
            for (int b = 0; b < NCT; ++b) g[a][b] = h[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
        const int li = lane & 15, lk = lane >> 4;
#pragma unroll 2
        for (int t = w; 4 * t < n; t += NW) {
            const int r = 4 * t + lk;
            double y[NCT], z[NCT];
#pragma unroll
            for (int a = 0; a < NCT; ++a) {
                const int j = 16 * a + li;
                const bool in = r < n && j < M;
                y[a] = in ? Y[r * PT + j] : 0.0;
                z[a] = in ? AYg[(size_t)r * PG + j] : 0.0;
            }
#pragma unroll
            for (int a = 0; a < NCT; ++a)
#pragma unroll
                for (int b = 0; b < NCT; ++b) {
                    g[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[a], y[b], g[a][b], 0, 0, 0);
                    h[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(y[a], z[b], h[a][b], 0, 0, 0);
                }
        }
#pragma unroll 1
        for (int ww = 0; ww < NW; ++ww) {
            if (w == ww) {
#pragma unroll
                for (int a = 0; a < NCT; ++a)
#pragma unroll
                    for (int b = 0; b < NCT; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int i = 16 * a + lk + 4 * r, j = 16 * b + li;
                            if (i < M && j < M) {
                                sh->G[i * M + j] = (ww ? sh->G[i * M + j] : 0.0) + g[a][b][r];
                                sh->H[i * M + j] = (ww ? sh->H[i * M + j] : 0.0) + h[a][b][r];
                            }
                        }
            }
            __syncthreads();
        }
    }

    // rows of X (pitch px) times the M x M matrix sh->Q, in place; a wavefront
    // owns whole 16-row tiles
    template <class P>
    __device__ __forceinline__ void mul(P X, int px) const {
        const int li = lane & 15, lk = lane >> 4;
        double q[NCT][(M + 3) / 4];
#pragma unroll
        for (int t = 0; t < (M + 3) / 4; ++t)
#pragma unroll
            for (int b = 0; b < NCT; ++b) {
                const int k = 4 * t + lk, j = 16 * b + li;
                q[b][t] = k < M && j < M ? sh->Q[k * M + j] : 0.0;
            }
#pragma unroll 1
        for (int r0 = 16 * w; r0 < n; r0 += 16 * NW) {
            v4d acc[NCT];
#pragma unroll
            for (int b = 0; b < NCT; ++b) acc[b] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t = 0; t < (M + 3) / 4; ++t) {
                const int k = 4 * t + lk;
                const double x = k < M && r0 + li < n ? X[(size_t)(r0 + li) * px + k] : 0.0;
#pragma unroll
                for (int b = 0; b < NCT; ++b) acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, q[b][t], acc[b], 0, 0, 0);
            }
#pragma unroll
            for (int b = 0; b < NCT; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = r0 + lk + 4 * r, j = 16 * b + li;
                    if (i < n && j < M) X[(size_t)i * px + j] = acc[b][r];
                }
        }
    }

    // sums over all rows of f(row, column) into out[0..M-1]
    template <class F>
    __device__ __forceinline__ void column_sums(lds_double* out, F f) const {
        const int j = threadIdx.x % PG;
        double s = 0.0;
        if (j < M)
            for (int r = threadIdx.x / PG; r < n; r += NT / PG) s += f(r, j);
        sh->red[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x < M) {
            double t = 0.0;
            for (int k = 0; k < NT / PG; ++k) t += sh->red[k * PG + threadIdx.x];
            out[threadIdx.x] = t;
        }
        __syncthreads();
    }

    // Rayleigh-Ritz of the LDS block: Y and AYg become the Ritz vectors and their
    // images, sh->th the values, sh->nrm the squared residual norms; nval < M: only
    // the first nval columns exist.  Returns the smallest scaled pivot.
    __device__ __forceinline__ double rayleigh_ritz_inl(bool rough, int nval, double pad) const {
        const double min_ritz = rough ? 1e-9 : 1e-5;
        double low = 0.0;
#pragma unroll 1
        for (int pass = 0; pass < 4; ++pass) {
            apply();
            __syncthreads();
            grams();
            if (threadIdx.x < 64) {
                const double lw = ritz_wave<M>(sh->G, sh->H, sh->Q, sh->scr, sh->th, sh->iscr,
                                               pass < 3 ? min_ritz : 0.0, rough ? 1e-6 : 1e-15, nval, pad);
                if (threadIdx.x == 0) sh->low = lw;
            }
            __syncthreads();
            low = sh->low;
            mul(Y, PT);
            if (low >= min_ritz || pass == 3) break;
            __syncthreads();
        }
        mul(AYg, PG);
        __syncthreads();
        column_sums(sh->nrm, [&](int r, int j) {
            const double d = AYg[(size_t)r * PG + j] - sh->th[j] * Y[r * PT + j];
            return d * d;
        });
        return low;
    }

    // T_p = (S_p)^-1 for every plane
    __device__ __forceinline__ void factor_inl(double sigma) const {
        const int a2 = agg * agg;
#pragma unroll 1
        for (int p = 0; p < planes; ++p) {
            const int r0 = plane_row(p), m = plane_end(p) - r0, ld = ceil16(m);
            gl_double* Tp = T + (size_t)p * mpmax * mpmax;
            const int q0 = p ? plane_row(p - 1) : 0, mq = r0 - q0, ldq = ceil16(mq);
            const gl_double* Tq = T + (size_t)(p - 1) * mpmax * mpmax;
            const int c0 = planes == 1 ? 0 : p * a2, nch = planes == 1 ? a2 * agg : a2;
            if (p) {
                // Wk[j][i] = (T_{p-1} C_{p-1})[i][j]: a wavefront takes a child of this
                // plane, a lane a row i of the plane below; the child's couplings are
                // the same for every lane
#pragma unroll 1
                for (int q = w; q < nch; q += NW) {
                    const int pj = (int)uniform32((unsigned)(c0 + q)), pb = pj - a2;
                    const int kb = (int)uniform32((unsigned)sh->koff[pb]), kn = (int)uniform32((unsigned)sh->koff[pb + 1]) - kb;
                    const int jb = (int)uniform32((unsigned)sh->koff[pj]), jn = (int)uniform32((unsigned)sh->koff[pj + 1]) - jb;
                    const gl_double* C = Aoff + ((size_t)uniform32((unsigned)sh->elem[pb]) * 3 + 2) * LP * LP;
                    for (int i = lane; i < mq; i += 64) {
                        const gl_double* t = Tq + (size_t)(kb - q0) * ldq + i;
#pragma unroll 1
                        for (int k0 = 0; k0 < kn; k0 += 8) {
                            double x[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) x[u] = t[min(k0 + u, kn - 1) * ldq];
#pragma unroll
                            for (int u = 0; u < 8; ++u) x[u] = k0 + u < kn ? x[u] : 0.0;
#pragma unroll 2
                            for (int b = 0; b < jn; ++b) {
                                gl_double* o = Wk + (size_t)(jb - r0 + b) * mpmax + i;
                                double v = k0 ? *o : 0.0;
#pragma unroll
                                for (int u = 0; u < 8; ++u) v += x[u] * C[min(k0 + u, kn - 1) * LP + b];
                                *o = v;
                            }
                        }
                    }
                }
                __syncthreads();
            }
            // S_p row by row of a child: a lane takes a column j
#pragma unroll 1
            for (int q = w; q < nch; q += NW) {
                const int pi = (int)uniform32((unsigned)(c0 + q)), ci = (int)uniform32((unsigned)sh->elem[pi]);
                const int ib = (int)uniform32((unsigned)sh->koff[pi]), in = (int)uniform32((unsigned)sh->koff[pi + 1]) - ib;
                const int xi = child_x(pi), yi = child_y(pi), zi = child_z(pi);
                const int pb = p ? pi - a2 : pi;
                const int kb = (int)uniform32((unsigned)sh->koff[pb]), kn = p ? (int)uniform32((unsigned)sh->koff[pb + 1]) - kb : 0;
                const gl_double* C = Aoff + ((size_t)uniform32((unsigned)sh->elem[pb]) * 3 + 2) * LP * LP;
                for (int j = lane; j < m; j += 64) {
                    const int pj = row[r0 + j] >> 8, bj = row[r0 + j] & 255, cj = sh->elem[pj];
                    const int dx = child_x(pj) - xi, dy = child_y(pj) - yi, dz = child_z(pj) - zi;
                    const int dist = abs(dx) + abs(dy) + abs(dz);
                    const bool up = dx + dy + dz > 0;
                    const int ax = dx ? 0 : (dy ? 1 : 2);
                    // entries of the lane's column: e[a es]
                    const gl_double* e = dist == 0 ? Hd + (size_t)ci * LP * LP + bj
                                                   : Aoff + ((size_t)(up ? ci : cj) * 3 + ax) * LP * LP + (up ? bj : bj * LP);
                    const int es = dist == 0 || up ? LP : 1;
                    const double we = dist <= 1 ? 1.0 : 0.0;
                    if (dist > 1) e = Hd;   // any valid entry, weight zero
                    const gl_double* x0 = Wk + (size_t)j * mpmax + (p ? kb - q0 : 0);
#pragma unroll 1
                    for (int a0 = 0; a0 < in; a0 += 4) {
                        double v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = e[dist <= 1 ? min(a0 + u, in - 1) * es : 0];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            v[u] = we * v[u] + (dist == 0 && a0 + u == bj ? sigma : 0.0);
#pragma unroll 1
                        for (int k0 = 0; k0 < kn; k0 += 8) {
                            double x[8];
#pragma unroll
                            for (int k = 0; k < 8; ++k) x[k] = x0[min(k0 + k, kn - 1)];
#pragma unroll
                            for (int k = 0; k < 8; ++k) x[k] = k0 + k < kn ? x[k] : 0.0;
#pragma unroll
                            for (int u = 0; u < 4; ++u)
#pragma unroll
                                for (int k = 0; k < 8; ++k)
                                    v[u] -= C[min(k0 + k, kn - 1) * LP + min(a0 + u, in - 1)] * x[k];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (a0 + u < in) Tp[(size_t)(ib - r0 + a0 + u) * ld + j] = v[u];
                    }
                }
            }
            __syncthreads();
            invert_block<NT>(Tp, m, ld, sh->rows);
        }
    }

    // acc = T_p U on the rows of the plane: V rows = acc (sub: V -= acc).  The
    // symmetric T_p is read by its columns, 128 contiguous bytes per 16 lanes,
    // in groups of four k-steps, three groups in flight (the last group again
    // past the end, so that no load is conditional); the first ones are
    // loaded by the caller ahead of U's barrier.  Columns of U beyond M only reach
    // columns of the result that are not stored.
    struct Ahead {
        double a[3][4];
    };
    __device__ __forceinline__ void load_group(const gl_double* tc, int ld, int g, double (&a)[4]) const {
        const gl_double* t = tc + (size_t)(16 * min(g, ld / 16 - 1)) * ld;
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = t[(size_t)(4 * u) * ld];
    }
    __device__ __forceinline__ const gl_double* tile_column(int p, int ld, int t0) const {
        return T + (size_t)p * mpmax * mpmax + (size_t)(lane >> 4) * ld + min(t0, ld - 16) + (lane & 15);
    }
    __device__ __forceinline__ void product_first(int p, Ahead& f) const {
        const int ld = ceil16(plane_end(p) - plane_row(p));
        const gl_double* tc = tile_column(p, ld, 16 * w);
#pragma unroll
        for (int g = 0; g < 3; ++g) load_group(tc, ld, g, f.a[g]);
    }
    __device__ __forceinline__ void product(int p, bool sub, Ahead& f) const {
        const int r0 = plane_row(p), m = plane_end(p) - r0, ld = ceil16(m), ng = ld / 16;
        const int li = lane & 15, lk = lane >> 4;
#pragma unroll 1
        for (int t0 = 16 * w; t0 < ld; t0 += 16 * NW) {
            v4d acc[NCT];
#pragma unroll
            for (int b = 0; b < NCT; ++b) acc[b] = v4d{0.0, 0.0, 0.0, 0.0};
            const gl_double* tc = tile_column(p, ld, t0);
            if (t0 != 16 * w) {
#pragma unroll
                for (int g = 0; g < 3; ++g) load_group(tc, ld, g, f.a[g]);
            }
#pragma unroll 1
            for (int g0 = 0; g0 < ng; g0 += 3) {
#pragma unroll
                for (int g = 0; g < 3; ++g) {
                    if (g0 + g < ng) {
                        double x[NCT][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int b = 0; b < NCT; ++b)
                                x[b][u] = U[(16 * (g0 + g) + 4 * u + lk) * PT + min(16 * b + li, PT - 1)];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int b = 0; b < NCT; ++b)
                                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[g][u], x[b][u], acc[b], 0, 0, 0);
                        load_group(tc, ld, g0 + g + 3, f.a[g]);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < NCT; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = t0 + lk + 4 * r, j = 16 * b + li;
                    if (i < m && j < M) {
                        lds_double* v = Y + (r0 + i) * PT + j;
                        *v = sub ? *v - acc[b][r] : acc[b][r];
                    }
                }
        }
    }

    // Y = (H_E + sigma)^-1 Yg by the planes' inverses
    __device__ __forceinline__ void solve() const {
        const int a2 = agg * agg;
#pragma unroll 1
        for (int s = 0; s < 2 * planes - 1; ++s) {
            const bool back = s >= planes;
            const int p = back ? 2 * planes - 2 - s : s;
            const int r0 = plane_row(p), m = plane_end(p) - r0, ld = ceil16(m);
            Ahead first;
            product_first(p, first);
            const int j = min((int)threadIdx.x % PG, M - 1);
#pragma unroll 1
            for (int i = threadIdx.x / PG; i < ld; i += NT / PG) {
                const int r = r0 + min(i, m - 1);
                double v = back ? 0.0 : Yg[(size_t)r * PG + j];
                if (s) {
                    // the coupled child: below on the way up, above on the way down
                    const int pi = row[r] >> 8, ai = row[r] & 255;
                    const int pn = back ? pi + a2 : pi - a2, k0 = sh->koff[pn], kn = sh->koff[pn + 1] - k0;
                    const gl_double* h =
                        Aoff + ((size_t)sh->elem[back ? pi : pn] * 3 + 2) * LP * LP + (back ? ai * LP : ai);
                    const double q = coupled(h, back ? 1 : LP, Y + k0 * PT + j, PT, kn);
                    v = back ? q : v - q;
                }
                if (threadIdx.x % PG < M) U[i * PT + j] = i < m ? v : 0.0;
            }
            __syncthreads();
            product(p, back, first);
            __syncthreads();
        }
    }

    // T_deg of the inverse mapped from [0, 1 / (a + sigma)] to [-1, 1], applied
    // to the block (left unscaled, see the level-2 filter)
    __device__ __forceinline__ void filter_inl(double a, double sigma, int deg) const {
        const double f = 2.0 * (a + sigma);
        for (int t = threadIdx.x; t < n * PG; t += NT) {
            const int i = t / PG, j = t % PG;
            if (j < M) Yg[t] = Y[i * PT + j];
        }
        __syncthreads();
#pragma unroll 1
        for (int d = 1; d <= deg; ++d) {
            solve();
            for (int t = threadIdx.x; t < n * PG; t += NT) {
                const int i = t / PG, j = t % PG;
                if (j >= M) continue;
                const double y = Yg[t];
                const double z = f * Y[i * PT + j] - y;
                const double v = d == 1 ? z : 2.0 * z - Xg[t];
                Xg[t] = y;
                Yg[t] = v;
                if (d == deg) Y[i * PT + j] = v;
            }
            __syncthreads();
        }
    }

    // The Chebyshev polynomial of H_E itself that damps [a, b], for blocks on
    // which the inverses' rounding (their error times |H_E|) stays above the
    // tolerance: Y <- T_deg((H_E - c) / e) Y
    __device__ __forceinline__ void damp_inl(double a, double b, int deg) const {
        const double c = 0.5 * (a + b), ie = 2.0 / (b - a);
#pragma unroll 1
        for (int d = 1; d <= deg; ++d) {
            apply();
            __syncthreads();
            for (int t = threadIdx.x; t < n * PG; t += NT) {
                const int i = t / PG, j = t % PG;
                if (j >= M) continue;
                const double y = Y[i * PT + j];
                const double z = (AYg[t] - c * y) * ie;
                const double v = d == 1 ? z : 2.0 * z - Xg[t];
                Xg[t] = y;
                Y[i * PT + j] = v;
            }
            __syncthreads();
        }
    }

    // The phases as calls of their own (inlined together they exceed the
    // registers and the instruction cache), each on a copy of the problem in scalar
    // registers.
    __device__ __forceinline__ UpProblem scalar() const {
        UpProblem l = *this;
        l.sh = (lds_shared*)uniform32((unsigned)(size_t)sh);
        l.Y = (lds_double*)uniform32((unsigned)(size_t)Y);
        l.U = (lds_double*)uniform32((unsigned)(size_t)U);
        l.row = (lds_ushort*)uniform32((unsigned)(size_t)row);
        l.T = (gl_double*)uniform64((unsigned long long)T);
        l.Wk = (gl_double*)uniform64((unsigned long long)Wk);
        l.Yg = (gl_double*)uniform64((unsigned long long)Yg);
        l.Xg = (gl_double*)uniform64((unsigned long long)Xg);
        l.AYg = (gl_double*)uniform64((unsigned long long)AYg);
        l.Hd = (const gl_double*)uniform64((unsigned long long)Hd);
        l.Aoff = (const gl_double*)uniform64((unsigned long long)Aoff);
        l.LP = (int)uniform32((unsigned)LP);
        l.agg = (int)uniform32((unsigned)agg);
        l.n = (int)uniform32((unsigned)n);
        l.planes = (int)uniform32((unsigned)planes);
        l.mpmax = (int)uniform32((unsigned)mpmax);
        l.w = (int)uniform32((unsigned)w);
        l.lane = (int)(threadIdx.x & 63);
        return l;
    }
    __device__ __attribute__((noinline)) double rayleigh_ritz(bool rough, int nval, double pad) const {
        return scalar().rayleigh_ritz_inl(rough, nval, pad);
    }
    __device__ __attribute__((noinline)) void factor(double sigma) const { scalar().factor_inl(sigma); }
    __device__ __attribute__((noinline)) void damp(double a, double b) const { scalar().damp_inl(a, b, kDampDeg); }
    __device__ __attribute__((noinline)) void filter(double a, double sigma, int deg) const {
        scalar().filter_inl(a, sigma, (int)uniform32((unsigned)deg));
    }
};

// Degree of the next filter (see the level-2 solver's): the residual of the
// slowest vector that still has to converge shrinks by exp(-acosh t) per degree,
// t its image in the damped interval's coordinate.  At most 4 in the first
// cycle (its cut is far too high), 8 in the next two (the block's columns
// must stay independent), 20 later.
__device__ __forceinline__ int inverse_degree(const double* th, const double* nrm, int lane, int need, double tol,
                                              double bnd, int nk, double a, double sigma, int cyc) {
    const int cap = cyc == 0 ? 4 : (cyc < 3 ? 8 : 20);
    double d = 2.0;
    if (lane < need) {
        const double rho = sqrt(nrm[lane]) / ((lane < nk ? tol : sqrt(tol)) * bnd);
        const bool sep = lane >= nk && nk > 0 && th[lane] - th[nk - 1] > 0.05 * fabs(th[lane]);
        if (rho > 1.0 && !sep) {
            const double t = 2.0 * (a + sigma) / (th[lane] + sigma) - 1.0;
            d = t > 1.0001 ? fmin((double)cap, log(10.0 * rho) / log(t + sqrt(t * t - 1.0)) + 2.0) : (double)cap;
        }
    }
    return (int)wave_max(fmax(d, 2.0));
}

__host__ __device__ inline int up_planes(int agg, int lp) { return agg * agg * agg * lp <= kUpSingle ? 1 : agg; }
// rows of a plane, rounded up to whole tiles
__host__ __device__ inline int up_plane_rows(int agg, int lp) {
    const int m = (up_planes(agg, lp) == 1 ? agg * agg * agg : agg * agg) * lp;
    return (m + 15) & ~15;
}
// doubles of one workspace slot: the planes' inverses and one product, three blocks
static size_t up_slot_doubles(int agg, int lp, int M) {
    const size_t mp = up_plane_rows(agg, lp), n = (size_t)agg * agg * agg * lp, pg = M <= 16 ? 16 : 32;
    return (up_planes(agg, lp) + 1) * mp * mp + 3 * n * pg;
}

template <int M, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_eig_up(CoarseGeom lo, CoarseGeom up, const double* __restrict__ Hd,
                                               const double* __restrict__ Aoff, const int* __restrict__ nkeep_lo,
                                               const double* __restrict__ zlo, int target, double tol, double crtol,
                                               double thr, double* __restrict__ V, double* __restrict__ lam,
                                               int* __restrict__ nkeep, double* __restrict__ Aint,
                                               double* __restrict__ zup, int* __restrict__ status,
                                               double* __restrict__ work, size_t slot) {
    extern __shared__ __align__(16) double dyn[];
    __shared__ UpShared<M, NT> sh;
    typedef UpProblem<M, NT> UP;
    constexpr int PT = UP::PT;
    const int agg = lo.agg, Lu = up.L, LP = lo.L, nch = agg * agg * agg, npad = nch * LP;
    const int planes = up_planes(agg, LP), mpmax = up_plane_rows(agg, LP);
    const int lane = threadIdx.x & 63;
    double* ws = work + (size_t)blockIdx.x * slot;
    double* Ub = dyn + (size_t)npad * PT;
    UP pr{(typename UP::lds_shared*)&sh, (lds_double*)dyn, (lds_double*)Ub, (lds_ushort*)(Ub + (size_t)mpmax * PT),
          (gl_double*)ws, (gl_double*)(ws + (size_t)planes * mpmax * mpmax), nullptr, nullptr, nullptr,
          (const gl_double*)Hd, (const gl_double*)Aoff, LP, agg, 0, planes, mpmax, (int)(threadIdx.x >> 6), lane};
    pr.Yg = pr.Wk + (size_t)mpmax * mpmax;
    pr.Xg = pr.Yg + (size_t)npad * UP::PG;
    pr.AYg = pr.Xg + (size_t)npad * UP::PG;
    // one-dimensional factors cos(pi p (q + 1/2) / agg) of the start modes
    if (threadIdx.x < 12)
        sh.ct[threadIdx.x] =
            cos(3.14159265358979323846 / agg * (double)(threadIdx.x >> 2) * ((threadIdx.x & 3) + 0.5));
#pragma unroll 1
    for (int E = blockIdx.x; E < up.m; E += gridDim.x) {
        const int Ex = E % up.mx, Ey = (E / up.mx) % up.my, Ez = E / (up.mx * up.my);
        __syncthreads();
        if (threadIdx.x < 64) {
            // children and the prefix sums of their kept slots, one child per lane
            int k = 0;
            if (lane < nch) {
                const int c = (Ex * agg + lane % agg) +
                              lo.mx * ((Ey * agg + (lane / agg) % agg) + lo.my * (Ez * agg + lane / (agg * agg)));
                sh.elem[lane] = c;
                k = nkeep_lo[c];
            }
            int s = k;
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(s, off, 64);
                if (lane >= off) s += o;
            }
            if (lane < nch) sh.koff[lane] = s - k;
            if (lane == 63) {
                for (int p = nch; p <= 64; ++p) sh.koff[p] = s;
            }
        }
        __syncthreads();
        const int nval = sh.koff[nch];
        pr.n = nval;
        for (int t = threadIdx.x; t < npad; t += NT) {
            const int p = t / LP, a = t % LP;
            if (a < sh.koff[p + 1] - sh.koff[p]) pr.row[sh.koff[p] + a] = (unsigned short)(p << 8 | a);
        }
        __syncthreads();
        // Gershgorin bound (absolute row sums) and the largest constant coefficient
        double rs = 0.0, az = 0.0;
        for (int r = threadIdx.x; r < nval; r += NT) {
            const int p = pr.row[r] >> 8, a = pr.row[r] & 255, c = sh.elem[p];
            const int q[3] = {pr.child_x(p), pr.child_y(p), pr.child_z(p)}, st[3] = {1, agg, agg * agg};
            double s = 0.0;
            for (int b = 0; b < sh.koff[p + 1] - sh.koff[p]; ++b) s += fabs(pr.entry(c, a, c, b, -1, false));
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                const bool in = (d & 1) ? q[d >> 1] < agg - 1 : q[d >> 1] > 0;
                if (!in) continue;
                const int pn = (d & 1) ? p + st[d >> 1] : p - st[d >> 1], cn = sh.elem[pn];
                for (int b = 0; b < sh.koff[pn + 1] - sh.koff[pn]; ++b)
                    s += fabs(pr.entry(c, a, cn, b, d >> 1, d & 1));
            }
            rs = fmax(rs, s);
            az = fmax(az, fabs(zlo[(size_t)c * LP + a]));
        }
        auto block_max = [&](double v) {
            v = wave_max(v);
            __syncthreads();
            if (lane == 0) sh.misc[threadIdx.x >> 6] = v;
            __syncthreads();
            double t = sh.misc[0];
            for (int i = 1; i < NT / 64; ++i) t = fmax(t, sh.misc[i]);
            return t;
        };
        const double bnd = block_max(rs);
        az = block_max(az) + 1e-300;
        // Start block: unit vectors when they span the whole space (one
        // Rayleigh-Ritz step is then exact); else the constant function, smooth
        // weights of the children's constant modes, and noise on every kept
        // slot.  The noise has one amplitude for the whole element: the constant
        // function's coefficient vanishes on the children's non-constant slots,
        // and noise scaled by it would leave the block without those
        // directions, which a filter cannot restore.
        const bool whole = nval <= M;
        for (int t = threadIdx.x; t < nval * M; t += NT) {
            const int r = t / M, j = t % M;
            const int p = pr.row[r] >> 8, a = pr.row[r] & 255;
            double v;
            if (whole) {
                v = r == j ? 1.0 : 0.0;
            } else {
                const double z = zlo[(size_t)sh.elem[p] * LP + a];
                v = 0.05 * az * hash_noise((unsigned)E + 77u, (unsigned)j, (unsigned)(p * LP + a));
                if (j == 0) v = z;
                else if (a == 0) {
                    const unsigned char* md = kModes[j & 15];
                    v += z * sh.ct[4 * md[0] + pr.child_x(p)] * sh.ct[4 * md[1] + pr.child_y(p)] *
                         sh.ct[4 * md[2] + pr.child_z(p)];
                }
            }
            pr.Y[r * PT + j] = v;
        }
        __syncthreads();
        int cyc = 0;
        if (whole) {
            pr.rayleigh_ritz(false, nval, 2.0 * bnd + 1.0);
        } else {
            const int need = (target + 4 < M - 2) ? target + 4 : M - 2;
            double sigma = -1.0;
            bool clean = false;
#pragma unroll 1
            for (;;) {
                const double low = pr.rayleigh_ritz(cyc == 0 && !clean, M, 0.0);
                if (clean) break;
                if (chefsi_done(sh.th, sh.nrm, M, need, tol, bnd, target, crtol, thr, cyc)) {
                    // once more where the block was far from orthonormal
                    if (low >= 0.1) break;
                    clean = true;
                    __syncthreads();
                    continue;
                }
                if (cyc >= kMaxCycles) {
                    cyc = -1;
                    break;
                }
                const double a = sh.th[M - 1], want = fmax(0.1 * a, 1e-7 * bnd);
                const int nk = cluster_cut_dev(sh.th, M, target, crtol, thr);
                __syncthreads();
                if (cyc >= kInverseCycles) {
                    pr.damp(a, bnd);
                    ++cyc;
                    continue;
                }
                if (sigma < 0.0 || want < 0.7 * sigma || want > sigma) {
                    sigma = want;
                    pr.factor(sigma);
                }
                pr.filter(a, sigma, inverse_degree(sh.th, sh.nrm, lane, need, tol, bnd, nk, a, sigma, cyc));
                ++cyc;
            }
        }
        const int nk = cluster_cut_dev(sh.th, whole ? nval : M, target, crtol, thr);
        if (threadIdx.x == 0) {
            nkeep[E] = nk;
            status[E] = cyc;
            for (int b = 0; b < Lu; ++b) lam[(size_t)E * Lu + b] = b < nval && b < M ? sh.th[b] : 0.0;
        }
        // V^T H_E V on the kept vectors, the constant function's coefficients, V
        __syncthreads();
        pr.grams();
        for (int t = threadIdx.x; t < Lu * Lu; t += NT) {
            const int i = t / Lu, j = t % Lu;
            Aint[(size_t)E * Lu * Lu + t] = (i < nk && j < nk) ? 0.5 * (sh.H[i * M + j] + sh.H[j * M + i]) : 0.0;
        }
        pr.column_sums((lds_double*)sh.nrm, [&](int r, int j) {
            const int p = pr.row[r] >> 8, a = pr.row[r] & 255;
            return pr.Y[r * PT + j] * zlo[(size_t)sh.elem[p] * LP + a];
        });
        for (int j = threadIdx.x; j < Lu; j += NT) zup[(size_t)E * Lu + j] = j < nk ? sh.nrm[j] : 0.0;
        for (int t = threadIdx.x; t < Lu * npad; t += NT) {
            const int j = t / npad, r = t % npad, p = r / LP, a = r % LP;
            const bool in = j < nk && a < sh.koff[p + 1] - sh.koff[p];
            V[((size_t)E * Lu + j) * npad + r] = in ? pr.Y[(sh.koff[p] + a) * PT + j] : 0.0;
        }
    }
}

// ---------------------------------------------------------------------------
// launcher

// workgroups of one launch, each with its own workspace slot: one per parent up to
// what the chip holds (LDS: one workgroup of 4^3 children per CU, up to four of 2^3)
static int up_slots(const CoarseGeom& up, int agg) { return std::min(up.m, agg == 4 ? 256 : 1024); }

size_t eig_up_work_doubles(const CoarseGeom& lo, const CoarseGeom& up, int nvec) {
    return (size_t)up_slots(up, lo.agg) * up_slot_doubles(lo.agg, lo.L, nvec);
}

void launch_eig_up(const CoarseGeom& lo, const CoarseGeom& up, const double* Aint_lo, const double* Dlo,
                   const double* Aofflo, const int* nkeep_lo, const double* zlo, double* Hd_work, double* work,
                   int target, int nvec, double tol, double crtol, double thr, double* V, double* lam, int* nkeep,
                   double* Aint, double* zup, int* status, hipStream_t s) {
    hipLaunchKernelGGL(k_build_hd, dim3(lo.m), dim3(128), 0, s, lo, Aint_lo, Dlo, Hd_work);
    const int n = lo.agg * lo.agg * lo.agg * lo.L;
    if (up.L != target + 3 || lo.L > kMaxLP || n > 768 || target < 1 || target > 20 || nvec < target + 6 ||
        (lo.agg != 2 && lo.agg != 4))
        throw HipError{hipErrorInvalidValue, "eig_up shape"};
    const size_t slot = up_slot_doubles(lo.agg, lo.L, nvec);
    const int mp = up_plane_rows(lo.agg, lo.L);
#define SPECMG_EIG_UP_NT(MV, NTV)                                                                                   \
    {                                                                                                               \
        const size_t shmem = ((size_t)n + mp) * UpProblem<MV, NTV>::PT * sizeof(double) + ((size_t)n + 3) / 4 * 8;   \
        hipFuncSetAttribute((const void*)k_eig_up<MV, NTV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem); \
        hipLaunchKernelGGL((k_eig_up<MV, NTV>), dim3(up_slots(up, lo.agg)), dim3(NTV), shmem, s, lo, up, Hd_work,    \
                           Aofflo, nkeep_lo, zlo, target, tol, crtol, thr, V, lam, nkeep, Aint, zup, status, work,   \
                           slot);                                                                                   \
        const hipError_t e = hipGetLastError();                                                                      \
        if (e != hipSuccess) throw HipError{e, "eig_up launch"};                                                     \
        return;                                                                                                     \
    }
#define SPECMG_EIG_UP(MV)                     \
    case MV:                                  \
        if (lo.agg == 4) SPECMG_EIG_UP_NT(MV, 512) \
        else SPECMG_EIG_UP_NT(MV, 256)
    switch (nvec) {
        SPECMG_EIG_UP(10)
        SPECMG_EIG_UP(12)
        SPECMG_EIG_UP(14)
        SPECMG_EIG_UP(16)
        SPECMG_EIG_UP(20)
        SPECMG_EIG_UP(26)
        default: break;
    }
#undef SPECMG_EIG_UP
#undef SPECMG_EIG_UP_NT
    throw HipError{hipErrorInvalidValue, "eig_up block size"};
}

}  // namespace specmg
