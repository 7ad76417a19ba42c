// Coarsest level (Algorithm 1, step 5): the dense inverse of the regularised
// coarsest matrix A_L + alpha z z^T, which the V-cycle applies as one dense
// matrix-vector product.
//
// Matrices are row-major np x np with np a multiple of 32 (padding rows and
// columns carry an identity).  Up to kElimMax rows, which is every matrix that
// is kept dense, k_elim_* eliminate by blocks of 64 (second half of this file).
// Above, Cholesky A = L L^T is right-looking in panels of KB = 256 columns: inside a panel, 32 x 32 diagonal tiles in LDS, a panel
// solve and rank-32 updates restricted to the panel; after the panel, one
// rank-KB update of the trailing lower triangle.  W = L^{-1}: every KB x KB
// diagonal block inverted at once, then halves joined bottom-up,
// W21 = -W22 (L21 W11).  Finally A^{-1} = W^T W.  The rank-KB updates and
// the products run on the FP64 matrix cores (k_gemm).
#include "common.hpp"

namespace specmg {

constexpr int NB = 32;
constexpr int KB = 256;   // panel width of the Cholesky factorisation, leaf of the triangular inverse

__global__ __launch_bounds__(256) void k_potrf_diag(double* A, int np, int k0, int* bad) {
    __shared__ double T[NB][NB + 1];
    for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
        const int i = t / NB, j = t % NB;
        T[i][j] = A[(size_t)(k0 + i) * np + k0 + j];
    }
    __syncthreads();
    for (int j = 0; j < NB; ++j) {
        if (threadIdx.x == 0) {
            double d = T[j][j];
            if (!(d > 0.0)) {
                atomicOr(bad, 4);
                d = 1.0;
            }
            T[j][j] = sqrt(d);
        }
        __syncthreads();
        const double ljj = T[j][j];
        for (int i = j + 1 + threadIdx.x; i < NB; i += blockDim.x) T[i][j] /= ljj;
        __syncthreads();
        for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
            const int i = t / NB, c = t % NB;
            if (c > j && i >= c) T[i][c] -= T[i][j] * T[c][j];
        }
        __syncthreads();
    }
    for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
        const int i = t / NB, j = t % NB;
        A[(size_t)(k0 + i) * np + k0 + j] = (j <= i) ? T[i][j] : 0.0;
    }
}

// rows i >= k0+NB: A[i, k0:k0+NB] <- A[i, k0:k0+NB] L_kk^{-T}
__global__ __launch_bounds__(64) void k_trsm_panel(double* A, int np, int k0) {
    __shared__ double Lk[NB][NB + 1];
    for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
        const int i = t / NB, j = t % NB;
        Lk[i][j] = A[(size_t)(k0 + i) * np + k0 + j];
    }
    __syncthreads();
    const int i = k0 + NB + blockIdx.x * 64 + threadIdx.x;
    if (i >= np) return;
    double x[NB];
    double* row = A + (size_t)i * np + k0;
#pragma unroll
    for (int j = 0; j < NB; ++j) x[j] = row[j];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        double v = x[j];
#pragma unroll
        for (int k = 0; k < j; ++k) v -= x[k] * Lk[j][k];
        x[j] = v / Lk[j][j];
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) row[j] = x[j];
}

// inside a panel: A[i][j] -= sum_{k < 32} A[i][kk+k] A[j][kk+k] for the lower
// 32 x 32 tiles (ti >= tj) of rows >= kk+32 whose column tile tj < ntc
__global__ __launch_bounds__(256) void k_syrk_panel(double* A, int np, int kk, int T) {
    __shared__ double Pi[NB][NB + 1], Pj[NB][NB + 1];
    int b = blockIdx.x, tj = 0;
    while (b >= T - tj) {
        b -= T - tj;
        ++tj;
    }
    const int ti = tj + b;
    const int base = kk + NB;
    const int r0 = base + ti * NB, c0 = base + tj * NB;
    for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
        const int i = t / NB, k = t % NB;
        Pi[i][k] = A[(size_t)(r0 + i) * np + kk + k];
        Pj[i][k] = A[(size_t)(c0 + i) * np + kk + k];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
        const int i = t / NB, j = t % NB;
        if (ti == tj && j > i) continue;
        double s = 0.0;
#pragma unroll 8
        for (int k = 0; k < NB; ++k) s += Pi[i][k] * Pj[j][k];
        A[(size_t)(r0 + i) * np + c0 + j] -= s;
    }
}

enum { OPN = 0, OPT = 1 };
typedef double dbl4 __attribute__((ext_vector_type(4)));

// lower tile (ti >= tj) of a T x T tile grid from a linear block index
__device__ __forceinline__ void lower_tile(int b, int& ti, int& tj) {
    int i = (int)((sqrt(8.0 * (double)b + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= b) ++i;
    while (i * (i + 1) / 2 > b) --i;
    ti = i;
    tj = b - i * (i + 1) / 2;
}

// W_JJ = L_JJ^{-1} for every KB x KB diagonal block (blockIdx.y; the last
// one may be narrower): one workgroup per 32-column strip of the block, rows
// marched downwards
__global__ __launch_bounds__(256) void k_trtri_diag(const double* __restrict__ Lm, double* W, int np) {
    __shared__ double Lii[NB][NB + 1];
    __shared__ double R[NB][NB + 1];
    const int o = blockIdx.y * KB;
    const int nbk = min(KB, np - o) / NB;
    const int J = blockIdx.x;
    if (J >= nbk) return;   // whole workgroup
    const int j0 = o + J * NB;
    for (int I = J; I < nbk; ++I) {
        const int i0 = o + I * NB;
        for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
            const int i = t / NB, j = t % NB;
            Lii[i][j] = Lm[(size_t)(i0 + i) * np + i0 + j];
            double s = (I == J && i == j) ? 1.0 : 0.0;
            for (int k = j0; k < i0; ++k) s -= Lm[(size_t)(i0 + i) * np + k] * W[(size_t)k * np + j0 + j];
            R[i][j] = s;
        }
        __syncthreads();
        if (threadIdx.x < NB) {
            const int j = threadIdx.x;
            for (int i = 0; i < NB; ++i) {
                double v = R[i][j];
                for (int k = 0; k < i; ++k) v -= Lii[i][k] * R[k][j];
                R[i][j] = v / Lii[i][i];
            }
        }
        __syncthreads();
        for (int t = threadIdx.x; t < NB * NB; t += blockDim.x) {
            const int i = t / NB, j = t % NB;
            W[(size_t)(i0 + i) * np + j0 + j] = R[i][j];
        }
        __threadfence_block();
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// FP64 matrix-core GEMM: C (M x N) = alpha op(A) op(B) over k in [kbeg, kend),
// a 128 x 128 tile per 256-thread workgroup, wave w owning the 64 x 64
// quarter (rows 64 (w >> 1), columns 64 (w & 1)) as 4 x 4 blocks of
// v_mfma_f64_16x16x4f64.  Operand lanes: A(i, k) with i = lane % 16,
// k = lane / 16; B(k, j) with j = lane % 16, k = lane / 16; result element r
// of a block in lane l is (l / 16 + 4 r, l % 16) of the block.  k chunks of
// 16 are staged through LDS; the next chunk's loads are issued before the
// current chunk's products.
//   kb_mode: 0 kbeg = 0; 1 kbeg = j0 (B lower triangular); 2 kbeg = i0 (A^T
//            of a lower triangular matrix)
//   ke_mode: 0 kend = K; 1 kend = min(i0 + 128, K) (A lower triangular)
//   lower:   the grid enumerates the lower tiles (ti >= tj) of a square C
//   EPI 0: C = alpha acc;  1: C -= acc on i >= j;  2: C = acc on i >= j, mirrored
constexpr int GT = 128;
constexpr int GK = 16;

struct GemmArgs {
    const double* A;
    const double* B;
    double* C;
    int lda, ldb, ldc;
    int M, N, K;
    double alpha;
    int kb_mode, ke_mode, lower;
};

template <int AOP, int BOP, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm(GemmArgs g) {
    __shared__ double As[GK][GT + 1], Bs[GK][GT + 1];
    int ti, tj;
    if (g.lower) {
        lower_tile(blockIdx.x, ti, tj);
    } else {
        ti = blockIdx.x;
        tj = blockIdx.y;
    }
    const int i0 = ti * GT, j0 = tj * GT;
    const int kbeg = g.kb_mode == 1 ? j0 : (g.kb_mode == 2 ? i0 : 0);
    const int kend = g.ke_mode == 1 ? min(i0 + GT, g.K) : g.K;
    const int t = threadIdx.x, l = t & 63, w = t >> 6;
    const int wr = 64 * (w >> 1), wc = 64 * (w & 1);
    const int li = l & 15, lk = l >> 4;
    dbl4 acc[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[m][n] = dbl4{0.0, 0.0, 0.0, 0.0};
    // staging: 4 pairs of A and 4 of B per thread and chunk, each pair two
    // elements adjacent in memory (along k for OPN A / OPT B, along i or j
    // otherwise); K bounds are multiples of 16, so a pair never straddles kend
    double2 ra[4], rb[4];
    auto a_slot = [&](int u, int& ia, int& ka) {
        const int e = t + 256 * u;
        if (AOP == OPN) { ia = e >> 3; ka = 2 * (e & 7); }
        else { ia = 2 * (e & 63); ka = e >> 6; }
    };
    auto b_slot = [&](int u, int& jb, int& kb) {
        const int e = t + 256 * u;
        if (BOP == OPN) { jb = 2 * (e & 63); kb = e >> 6; }
        else { jb = e >> 3; kb = 2 * (e & 7); }
    };
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ia, ka, jb, kb;
            a_slot(u, ia, ka);
            b_slot(u, jb, kb);
            const int gi = i0 + ia, gka = k0 + ka;
            const bool va = gi < g.M && gka < kend;
            ra[u] = va ? *reinterpret_cast<const double2*>(AOP == OPN ? g.A + (size_t)gi * g.lda + gka
                                                                      : g.A + (size_t)gka * g.lda + gi)
                       : double2{0.0, 0.0};
            const int gj = j0 + jb, gkb = k0 + kb;
            const bool vb = gj < g.N && gkb < kend;
            rb[u] = vb ? *reinterpret_cast<const double2*>(BOP == OPN ? g.B + (size_t)gkb * g.ldb + gj
                                                                      : g.B + (size_t)gj * g.ldb + gkb)
                       : double2{0.0, 0.0};
        }
    };
    if (kbeg < kend) load(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += GK) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ia, ka, jb, kb;
            a_slot(u, ia, ka);
            b_slot(u, jb, kb);
            if (AOP == OPN) {
                As[ka][ia] = ra[u].x;
                As[ka + 1][ia] = ra[u].y;
            } else {
                As[ka][ia] = ra[u].x;
                As[ka][ia + 1] = ra[u].y;
            }
            if (BOP == OPN) {
                Bs[kb][jb] = rb[u].x;
                Bs[kb][jb + 1] = rb[u].y;
            } else {
                Bs[kb][jb] = rb[u].x;
                Bs[kb + 1][jb] = rb[u].y;
            }
        }
        __syncthreads();
        if (k0 + GK < kend) load(k0 + GK);
#pragma unroll
        for (int kk = 0; kk < GK / 4; ++kk) {
            const int k = 4 * kk + lk;
            double a[4], b[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) a[m] = As[k][wr + 16 * m + li];
#pragma unroll
            for (int n = 0; n < 4; ++n) b[n] = Bs[k][wc + 16 * n + li];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int n = 0; n < 4; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], b[n], acc[m][n], 0, 0, 0);
        }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + wr + 16 * m + lk + 4 * r, j = j0 + wc + 16 * n + li;
                if (i >= g.M || j >= g.N) continue;
                const double v = acc[m][n][r];
                if (EPI == 0) {
                    g.C[(size_t)i * g.ldc + j] = g.alpha * v;
                } else if (EPI == 1) {
                    if (i >= j) g.C[(size_t)i * g.ldc + j] -= v;
                } else {
                    if (i >= j) {
                        g.C[(size_t)i * g.ldc + j] = v;
                        g.C[(size_t)j * g.ldc + i] = v;
                    }
                }
            }
}

template <int AOP, int BOP, int EPI>
static void launch_gemm(const GemmArgs& g, hipStream_t s) {
    const int tm = (g.M + GT - 1) / GT, tn = (g.N + GT - 1) / GT;
    const dim3 grid = g.lower ? dim3(tm * (tm + 1) / 2) : dim3(tm, tn);
    if (tm > 0 && tn > 0) hipLaunchKernelGGL((k_gemm<AOP, BOP, EPI>), grid, dim3(256), 0, s, g);
}

__global__ void k_rank1(double* A, int np, int n, const double* __restrict__ z, double alpha) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < (int64_t)n * n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(t / n), j = (int)(t % n);
        A[(size_t)i * np + j] += alpha * z[i] * z[j];
    }
}

__global__ void k_pad_identity(double* A, int np, int n) {
    const int i = n + blockIdx.x * blockDim.x + threadIdx.x;
    if (i < np) A[(size_t)i * np + i] = 1.0;
}

void launch_pad_identity(double* a, int np, int n, hipStream_t s) {
    if (np > n) hipLaunchKernelGGL(k_pad_identity, dim3((np - n + 63) / 64), dim3(64), 0, s, a, np, n);
}

// W[o:e, o:e] = L[o:e, o:e]^{-1} for the KB-blocks [b0, b1) (o = KB b0,
// e = min(KB b1, np)), leaves already inverted: inv([L11 0; L21 L22]) =
// [W11 0; -W22 L21 W11  W22], the two halves first (post-order), then
// P = L21 W11 (W11 lower triangular: k >= j) and W21 = -W22 P (W22 lower
// triangular: k <= i) as matrix-core GEMMs; P lives in tbuf.
static void trtri_node(const double* Lm, double* W, double* P, int np, int b0, int b1, hipStream_t s) {
    if (b1 - b0 < 2) return;
    const int bm = (b0 + b1) / 2;
    trtri_node(Lm, W, P, np, b0, bm, s);
    trtri_node(Lm, W, P, np, bm, b1, s);
    const int o = KB * b0, h = KB * (bm - b0), n = std::min(KB * b1, np) - o;
    GemmArgs g{};
    g.A = Lm + (size_t)(o + h) * np + o;
    g.lda = np;
    g.B = W + (size_t)o * np + o;
    g.ldb = np;
    g.C = P;
    g.ldc = h;
    g.M = n - h;
    g.N = h;
    g.K = h;
    g.alpha = 1.0;
    g.kb_mode = 1;
    launch_gemm<OPN, OPN, 0>(g, s);
    GemmArgs q{};
    q.A = W + (size_t)(o + h) * np + o + h;
    q.lda = np;
    q.B = P;
    q.ldb = h;
    q.C = W + (size_t)(o + h) * np + o;
    q.ldc = np;
    q.M = n - h;
    q.N = h;
    q.K = n - h;
    q.alpha = -1.0;
    q.ke_mode = 1;
    launch_gemm<OPN, OPN, 0>(q, s);
}

// ---------------------------------------------------------------------------
// Spaces of up to kElimMax unknowns: A = L L^T and W = L^{-1} in one forward
// elimination of [A | I] by blocks of 64, two launches a block.
//
// The lower tiles of the working matrix V hold, at step k, the rows of
// L^{-1} applied so far in the columns j <= k (I starts implicitly: column k
// enters at step k) and the remaining A in the columns j > k.  Step k, with
// W_kk = L_kk^{-1} already in V_kk:
//   k_elim_panel   Y_i = A_ik W_kk^T for i > k (kept as Y^T, 64 x nw), and
//                  row k: W_kj = W_kk V_kj for j < k
//   k_elim_update  rows i > k: V_ij -= Y_i W_kj (j <= k, V_ik from zero),
//                  V_ij -= Y_i Y_j^T (j > k); the workgroup of the next
//                  diagonal tile goes on to factor and invert it, which the
//                  other tiles hide
// and at the end A^{-1} = W^T W (k_elim_wtw).  The arithmetic is that of
// the factorisation by panels; what it saves is the serial part (there
// 3 launches for 32 columns, 45 us at any size, and 0.46 to 0.66 ms for the
// inverses of the diagonal blocks).  All products are wavefront tiles of 32 x
// 32 on v_mfma_f64_16x16x4f64 whose operands are read from the caches in
// operand order: rows of V and of Y^T, 16 consecutive columns a lane group,
// so nothing is staged and nothing waits.  Measured, panels of 256 columns
// against this: 0.066 / 0.031 ms at 32 rows, 1.23 / 0.164 at 384, 2.57 / 0.42
// at 1024, 10.4 / 2.8 at 4096, 14.2 / 4.7 at 5120, 29.4 / 17.0 at 8192.  The
// rank-64 updates read and write their whole range, np^3 / 12 bytes in all,
// four times what panels of 256 do, and pass the caches by then: hence
// kElimMax.  A step below 2000 rows is the launch of the panel (5 us) and the
// 18 us of the update's diagonal tile.
constexpr int EB = 64;
constexpr int kElimMax = 8192;
constexpr int ELD = EB + 2, EYD = 18;

static int elim_ld(int np) { return (np + EB - 1) / EB * EB; }

__device__ __forceinline__ double rcp_f64(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

union F64Words {
    double d;
    unsigned w[2];
};

// lane l of x, for a compile-time l
template <int LANE>
__device__ __forceinline__ double lane_value(double x) {
    F64Words u{x};
    u.w[0] = __builtin_amdgcn_readlane(u.w[0], LANE);
    u.w[1] = __builtin_amdgcn_readlane(u.w[1], LANE);
    return u.d;
}

// lane J of every group of 16 lanes, to its group
template <int J>
__device__ __forceinline__ double group_lane(double x) {
    F64Words u{x};
#pragma unroll
    for (int h = 0; h < 2; ++h) u.w[h] = __builtin_amdgcn_update_dpp(0, (int)u.w[h], 0x150 + J, 0xf, 0xf, true);
    return u.d;
}

// group G of 16 lanes, to all four groups
template <int G>
__device__ __forceinline__ double group_bcast(double x) {
    F64Words u{x};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const auto y = __builtin_amdgcn_permlane32_swap(u.w[h], u.w[h], false, false);
        const unsigned z = G < 2 ? y[0] : y[1];
        const auto v = __builtin_amdgcn_permlane16_swap(z, z, false, false);
        u.w[h] = G % 2 == 0 ? v[0] : v[1];
    }
    return u.d;
}

// pivot J of elim_diag16
template <int J>
__device__ __forceinline__ void elim_pivot(double (&a)[4], int g, int i, double& dsave, bool& ok) {
    constexpr int G = J / 4, E = J % 4;
    double d = lane_value<16 * G + J>(a[E]);
    if (!(d > 0.0)) {
        ok = false;
        d = 1.0;
    }
    if (i == J) dsave = d;
    const double q = group_bcast<G>(a[E]) * rcp_f64(d);
    const double lf = i > J ? -q : 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double t = fma(lf, group_lane<J>(a[e]), a[e]);
        a[e] = e == E && g == G ? (i == J ? 1.0 : lf) : t;
    }
    if constexpr (J < 15) elim_pivot<J + 1>(a, g, i, dsave, ok);
}

// The 16 x 16 tile of S at (r0, r0), symmetric, becomes the inverse of its
// Cholesky factor: [A | I] eliminated pivot by pivot in one wavefront, lane
// 16 g + i holding row i, columns 4 g to 4 g + 3; column j of I takes the
// place that column j of A leaves.  Returns false if a pivot is not positive.
__device__ __forceinline__ bool elim_diag16(double* S, int r0) {
    const int i = threadIdx.x & 15, g = (threadIdx.x >> 4) & 3;
    double* T = S + (r0 + i) * ELD + r0 + 4 * g;
    double a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = T[e];
    double dsave = 1.0;
    bool ok = true;
    elim_pivot<0>(a, g, i, dsave, ok);
    const double rs = 1.0 / sqrt(dsave);
#pragma unroll
    for (int e = 0; e < 4; ++e) T[e] = 4 * g + e <= i ? a[e] * rs : 0.0;
    return ok;
}

// acc += sum over 16 values of k of A(i, k) B(k, j); A(i, k) at a[i * ai + k * ak]
__device__ __forceinline__ dbl4 elim_mul16(const double* a, int ai, int ak, const double* b, int bk, int bj,
                                           dbl4 acc) {
    const int li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double x = a[li * ai + (4 * q + lk) * ak], y = b[(4 * q + lk) * bk + li * bj];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc, 0, 0, 0);
    }
    return acc;
}

// the 64 x 64 tile in S becomes the inverse of its Cholesky factor (lower; the
// tiles above the diagonal are left as they are): the same elimination by
// blocks of 16, one workgroup of four wavefronts.  About 13 us (23 with lane i
// holding all of row i: 16 columns a lane, read lane by lane), a serial chain.
__device__ bool elim_diag64(double* S, double* Y) {
    const int w = threadIdx.x >> 6, li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
    bool ok = true;
#pragma nounroll
    for (int b = 0; b < 4; ++b) {
        const int r0 = 16 * b;
        if (w == 0) ok &= elim_diag16(S, r0);
        __syncthreads();
        if (w < 3) {
            const int t = w < b ? w : w + 1;
            const double* Wb = S + r0 * ELD + r0;
            dbl4 c{0.0, 0.0, 0.0, 0.0};
            if (t > b) {
                c = elim_mul16(S + 16 * t * ELD + r0, ELD, 1, Wb, 1, ELD, c);
#pragma unroll
                for (int r = 0; r < 4; ++r) Y[(16 * t + lk + 4 * r) * EYD + li] = c[r];
            } else {
                c = elim_mul16(Wb, ELD, 1, S + r0 * ELD + 16 * t, ELD, 1, c);
#pragma unroll
                for (int r = 0; r < 4; ++r) S[(r0 + lk + 4 * r) * ELD + 16 * t + li] = c[r];
            }
        }
        __syncthreads();
        int e = w;
        for (int i = b + 1; i < 4; ++i) {
            for (; e <= i; e += 4) {
                const int j = e;
                double* C = S + 16 * i * ELD + 16 * j;
                dbl4 old{0.0, 0.0, 0.0, 0.0}, c{0.0, 0.0, 0.0, 0.0};
                if (j != b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) old[r] = C[(lk + 4 * r) * ELD + li];
                const bool w_row = j <= b;
                const double* B = w_row ? S + r0 * ELD + 16 * j : Y + 16 * j * EYD;
                c = elim_mul16(Y + 16 * i * EYD, EYD, 1, B, w_row ? ELD : 1, w_row ? 1 : EYD, c);
#pragma unroll
                for (int r = 0; r < 4; ++r) C[(lk + 4 * r) * ELD + li] = old[r] - c[r];
            }
            e -= i + 1;
        }
        __syncthreads();
    }
    return ok;
}

// the tile in S to V_kk (zero above the diagonal), after elim_diag64
__device__ __forceinline__ void elim_store_diag(double* S, double* Y, double* Vkk, int nw, int* bad) {
    if (!elim_diag64(S, Y) && threadIdx.x == 0) atomicOr(bad, 4);
    for (int t = threadIdx.x; t < EB * EB; t += 256) {
        const int i = t / EB, j = t % EB;
        Vkk[(size_t)i * nw + j] = j <= i ? S[i * ELD + j] : 0.0;
    }
}

// V <- lower tiles of A (the identity beyond np), and the first diagonal tile
__global__ __launch_bounds__(256) void k_elim_begin(const double* __restrict__ A, int np, double* V, int nw, int* bad) {
    __shared__ double S[EB * ELD], Y[EB * EYD];
    int ti, tj;
    lower_tile(blockIdx.x, ti, tj);
    for (int t = threadIdx.x; t < EB * EB; t += 256) {
        const int i = EB * ti + t / EB, j = EB * tj + t % EB;
        const int hi = max(i, j), lo = min(i, j);   // only the lower triangle of A is read
        const double v = hi < np ? A[(size_t)hi * np + lo] : (i == j ? 1.0 : 0.0);
        if (blockIdx.x == 0) S[(t / EB) * ELD + t % EB] = v;
        else V[(size_t)i * nw + j] = v;
    }
    if (blockIdx.x == 0) {
        __syncthreads();
        elim_store_diag(S, Y, V, nw, bad);
    }
}

// acc (32 x 32 of a wavefront) += sum over 64 values of k of A(i, k) B(k, j),
// A(i, k) at a[k * ld + i], B(k, j) at b[k * ld + j]
__device__ __forceinline__ void elim_mul64(const double* a, const double* b, size_t ld, dbl4 (&acc)[2][2]) {
    const int li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
    a += lk * ld + li;
    b += lk * ld + li;
#pragma unroll 8
    for (int q = 0; q < EB / 4; ++q) {
        double x[2], y[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            x[u] = a[16 * u + 4 * q * ld];
            y[u] = b[16 * u + 4 * q * ld];
        }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m], y[n], acc[m][n], 0, 0, 0);
    }
}

// both factors are staged: read from the caches in operand order, 32 bytes of
// a row at a time, the same products take 10 us
__global__ __launch_bounds__(512) void k_elim_panel(double* V, int nw, double* YT, int k) {
    __shared__ double Ws[EB * ELD], Bs[EB * ELD];
    const int j = (int)blockIdx.x < k ? blockIdx.x : blockIdx.x + 1;
    const size_t ld = nw;
    const double* Wkk = V + (size_t)EB * k * ld + EB * k;
    const double* B = j < k ? V + (size_t)EB * k * ld + EB * j : V + (size_t)EB * j * ld + EB * k;
    double wv[8], bv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int r = (threadIdx.x >> 6) + 8 * u, c = threadIdx.x & 63;
        wv[u] = Wkk[r * ld + c];
        bv[u] = B[r * ld + c];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int r = (threadIdx.x >> 6) + 8 * u, c = threadIdx.x & 63;
        Ws[r * ELD + c] = wv[u];
        Bs[r * ELD + c] = bv[u];
    }
    __syncthreads();
    // wavefront w: rows 32 (w / 4), columns 16 (w % 4)
    const int w = threadIdx.x >> 6, li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
    const int wr = 32 * (w >> 2), wc = 16 * (w & 3);
    const int bk = j < k ? ELD : 1, bj = j < k ? 1 : ELD;   // B(m, x), or its transpose
    const double* a = Ws + (wr + li) * ELD + lk;
    const double* b = Bs + lk * bk + (wc + li) * bj;
    dbl4 acc[2] = {};
#pragma unroll
    for (int q = 0; q < EB / 4; ++q)
#pragma unroll
        for (int m = 0; m < 2; ++m)
            acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * m * ELD + 4 * q], b[4 * q * bk], acc[m], 0, 0, 0);
    double* out = j < k ? V + (size_t)EB * k * ld + EB * j : YT + EB * j;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(size_t)(wr + 16 * m + lk + 4 * r) * ld + wc + li] = acc[m][r];
}

// block 0 is the tile (k + 1, k + 1)
__global__ __launch_bounds__(256) void k_elim_update(double* V, int nw, const double* __restrict__ YT, int k, int* bad) {
    __shared__ double S[EB * ELD], Y[EB * EYD];
    const int w = threadIdx.x >> 6, li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
    const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
    int i, j;
    lower_tile(blockIdx.x + (k + 1) * (k + 2) / 2, i, j);
    j = i - j;
    const size_t ld = nw;
    double* C = V + ((size_t)EB * i + wr + lk) * ld + EB * j + wc + li;
    dbl4 acc[2][2] = {}, old[2][2] = {};   // the sum is taken off at once: one rounding at the size of V_ij
    if (j != k)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) old[m][n][r] = C[(size_t)(16 * m + 4 * r) * ld + 16 * n];
    const double* Z = (j <= k ? V + (size_t)EB * k * ld : YT) + EB * j + wc;
    elim_mul64(YT + EB * i + wr, Z, ld, acc);
    if (blockIdx.x == 0) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    S[(wr + 16 * m + lk + 4 * r) * ELD + wc + 16 * n + li] = old[m][n][r] - acc[m][n][r];
        __syncthreads();
        elim_store_diag(S, Y, V + (size_t)EB * i * ld + EB * j, nw, bad);
        return;
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) C[(size_t)(16 * m + 4 * r) * ld + 16 * n] = old[m][n][r] - acc[m][n][r];
}

// A <- W^T W, lower tiles and their mirror images (W_kj = 0 for k < j)
__global__ __launch_bounds__(256) void k_elim_wtw(const double* __restrict__ V, int nw, double* A, int np) {
    const int w = threadIdx.x >> 6, li = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
    const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
    int ti, tj;
    lower_tile(blockIdx.x, ti, tj);
    const size_t ld = nw;
    dbl4 acc[2][2] = {};
    for (int k = ti; k < nw / EB; ++k)
        elim_mul64(V + (size_t)EB * k * ld + EB * ti + wr, V + (size_t)EB * k * ld + EB * tj + wc, ld, acc);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = EB * ti + wr + 16 * m + lk + 4 * r, j = EB * tj + wc + 16 * n + li;
                if (i >= np || j >= np) continue;
                A[(size_t)i * np + j] = acc[m][n][r];
                if (ti != tj) A[(size_t)j * np + i] = acc[m][n][r];
            }
}

static int elim_inverse(double* a, int np, double* V, double* YT, int* bad, hipStream_t s) {
    const int nw = elim_ld(np), nb = nw / EB, lower = nb * (nb + 1) / 2;
    hipLaunchKernelGGL(k_elim_begin, dim3(lower), dim3(256), 0, s, a, np, V, nw, bad);
    for (int k = 0; k < nb; ++k) {
        if (nb > 1) hipLaunchKernelGGL(k_elim_panel, dim3(nb - 1), dim3(512), 0, s, V, nw, YT, k);
        const int tiles = lower - (k + 1) * (k + 2) / 2;
        if (tiles > 0) hipLaunchKernelGGL(k_elim_update, dim3(tiles), dim3(256), 0, s, V, nw, YT, k, bad);
    }
    hipLaunchKernelGGL(k_elim_wtw, dim3(lower), dim3(256), 0, s, V, nw, a, np);
    return (int)hipGetLastError();
}

size_t dense_spd_inverse_work_doubles(int np) {
    const size_t n = np <= kElimMax ? elim_ld(np) : np;
    return n * n;
}

size_t dense_spd_inverse_tbuf_doubles(int np) {
    if (np <= kElimMax) return (size_t)EB * elim_ld(np);   // Y^T
    // P of the root node of trtri_node, the largest
    const int nb = (np + KB - 1) / KB;
    const size_t h = (size_t)KB * (nb / 2);
    return nb < 2 ? 1 : (size_t)(np - h) * h;
}

int dense_spd_inverse(double* a, int np, double* work, double* tbuf, int* bad, hipStream_t s) {
    if (np % NB) return (int)hipErrorInvalidValue;
    if (np <= kElimMax) {
        const int r = elim_inverse(a, np, work, tbuf, bad, s);
        const hipError_t e = hipStreamSynchronize(s);
        return r != 0 ? r : (int)e;
    }
    // ---- Cholesky, panels of KB columns; the trailing update on the matrix cores
    for (int k0 = 0; k0 < np; k0 += KB) {
        const int kw = std::min(KB, np - k0);
        for (int kk = k0; kk < k0 + kw; kk += NB) {
            hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, s, a, np, kk, bad);
            const int rest = np - kk - NB;
            if (rest > 0) {
                hipLaunchKernelGGL(k_trsm_panel, dim3((rest + 63) / 64), dim3(64), 0, s, a, np, kk);
                const int T = rest / NB, ntc = (k0 + kw - kk - NB) / NB;
                const int blocks = ntc * T - ntc * (ntc - 1) / 2;
                if (blocks > 0) hipLaunchKernelGGL(k_syrk_panel, dim3(blocks), dim3(256), 0, s, a, np, kk, T);
            }
        }
        const int j0 = k0 + kw;
        if (j0 < np) {
            // A[i][j] -= sum_{k in panel} A[i][k] A[j][k], i >= j >= j0
            GemmArgs g{};
            g.A = a + (size_t)j0 * np + k0;
            g.lda = np;
            g.B = g.A;
            g.ldb = np;
            g.C = a + (size_t)j0 * np + j0;
            g.ldc = np;
            g.M = g.N = np - j0;
            g.K = kw;
            g.alpha = 1.0;
            g.lower = 1;
            launch_gemm<OPN, OPT, 1>(g, s);
        }
    }
    // ---- W = L^{-1}: the KB x KB diagonal blocks, then the recursive halves
    hipError_t e = hipMemsetAsync(work, 0, (size_t)np * np * sizeof(double), s);
    if (e != hipSuccess) return (int)e;
    const int nb = (np + KB - 1) / KB;
    hipLaunchKernelGGL(k_trtri_diag, dim3(KB / NB, nb), dim3(256), 0, s, a, work, np);
    trtri_node(a, work, tbuf, np, 0, nb, s);
    // ---- A^{-1} = W^T W (lower tiles, mirrored; W[k][i] = 0 for k < i)
    {
        GemmArgs g{};
        g.A = work;
        g.lda = np;
        g.B = work;
        g.ldb = np;
        g.C = a;
        g.ldc = np;
        g.M = g.N = g.K = np;
        g.alpha = 1.0;
        g.kb_mode = 2;
        g.lower = 1;
        launch_gemm<OPT, OPN, 2>(g, s);
    }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return (int)e;
    return (int)hipGetLastError();
}

void launch_add_rank1(double* a, int np, int n, const double* z, double alpha, hipStream_t s) {
    hipLaunchKernelGGL(k_rank1, dim3(1024), dim3(256), 0, s, a, np, n, z, alpha);
}


}  // namespace specmg
