// Flexible GMRES, the outer Krylov solver of the paper's experiments
// (Section 5, with restarts; right preconditioning by the V-cycle).  The
// Arnoldi basis V (restart + 1 vectors) and the preconditioned directions Z
// (restart vectors) are stored as consecutive vectors of n entries.  Each
// Arnoldi step orthogonalises w = A z_j by classical Gram-Schmidt applied
// twice, h = V^T w and w -= V h, in three streaming passes over the basis: the
// first subtraction forms the second one's products as it goes, and the second
// the norm.  At 96 x 64 x 128 (6.3 MB a vector) a step's orthogonalisation took
// 130 us in five passes, and 85 in these, the basis read at 3.7 to 4.8 TB/s.  The (restart+1) x restart Hessenberg problem lives in device memory
// and is reduced by Givens rotations there, so the host reads back only the
// convergence flag.
#include <algorithm>

#include "common.hpp"

namespace specmg {

constexpr int kDotChunk = 16;      // basis vectors per pass of the multi-dot, narrow and
constexpr int kDotWide = 32;       // wide (up to 32 vectors in one pass)
constexpr int kKryThreads = 256;
constexpr int kKryBlocks = 1024;   // grid of the streaming kernels (4 x 256 CUs)

// block sums of acc to part[block][i], i < cnt <= C
template <int C>
__device__ __forceinline__ void block_parts(const double (&acc)[C], int cnt, double* __restrict__ part) {
    __shared__ double red[kKryThreads / 64][C];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const double s = wave_sum(acc[i]);
        if (lane == 0) red[wid][i] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < cnt) {
        double s = 0.0;
        for (int k = 0; k < kKryThreads / 64; ++k) s += red[k][threadIdx.x];
        part[(size_t)blockIdx.x * C + threadIdx.x] = s;
    }
}

// part[b][i] = sum over the rows of block b of V_i . w, i < cnt <= C
template <int C>
__global__ __launch_bounds__(kKryThreads) void k_mdot_part(const double* __restrict__ V, int64_t pitch, int cnt,
                                                           const double* __restrict__ w, int64_t n,
                                                           double* __restrict__ part) {
    double acc[C];
#pragma unroll
    for (int i = 0; i < C; ++i) acc[i] = 0.0;
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n;
         row += (int64_t)gridDim.x * blockDim.x) {
        const double wv = w[row];
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i < cnt) acc[i] += V[i * pitch + row] * wv;
    }
    block_parts<C>(acc, cnt, part);
}

// out[i] = sum_b part[b * C + i] (block i; fixed summation order)
__global__ __launch_bounds__(kKryThreads) void k_mdot_final(const double* __restrict__ part, int nb, int C,
                                                            double* __restrict__ out) {
    __shared__ double red[kKryThreads / 64];
    const int i = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) s += part[(size_t)b * C + i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < kKryThreads / 64; ++k) t += red[k];
        out[i] = t;
    }
}

// w += sign * sum_{i < cnt} coef[i] V_i (coefficients in device memory); NORM:
// and the block sums of the new w's squares to part
template <bool NORM>
__global__ __launch_bounds__(kKryThreads) void k_maxpy(const double* __restrict__ V, int64_t pitch, int cnt,
                                                       const double* __restrict__ coef, double sign,
                                                       double* __restrict__ w, int64_t n, double* __restrict__ part) {
    double acc[1] = {0.0};
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n;
         row += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
#pragma unroll 8
        for (int i = 0; i < cnt; ++i) s += coef[i] * V[i * pitch + row];
        const double wn = w[row] + sign * s;
        w[row] = wn;
        if (NORM) acc[0] += wn * wn;
    }
    if (NORM) block_parts<1>(acc, 1, part);
}

// The first projection and the second one's products in one pass over the
// basis: w -= sum coef[i] V_i, part[b][i] = sum of V_i . w with the new w; a
// row's entries of up to C vectors stay in registers between the two.
template <int C>
__global__ __launch_bounds__(kKryThreads) void k_project_dot(const double* __restrict__ V, int64_t pitch, int cnt,
                                                             const double* __restrict__ coef, double* __restrict__ w,
                                                             int64_t n, double* __restrict__ part) {
    double acc[C];
#pragma unroll
    for (int i = 0; i < C; ++i) acc[i] = 0.0;
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n;
         row += (int64_t)gridDim.x * blockDim.x) {
        double v[C], s = 0.0;
        const double wv = w[row];
#pragma unroll
        for (int i = 0; i < C; ++i) v[i] = i < cnt ? V[i * pitch + row] : 0.0;
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i < cnt) s += coef[i] * v[i];
        const double wn = wv - s;
        w[row] = wn;
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i < cnt) acc[i] += v[i] * wn;
    }
    block_parts<C>(acc, cnt, part);
}

// dst = src * (*factor)
__global__ __launch_bounds__(kKryThreads) void k_scale_dev(double* __restrict__ dst, const double* __restrict__ src,
                                                           const double* __restrict__ factor, int64_t n) {
    const double f = *factor;
    for (int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; row < n;
         row += (int64_t)gridDim.x * blockDim.x)
        dst[row] = src[row] * f;
}

// (re)start: beta = ||r|| from nrm2, g = beta e_1, inv = 1 / beta
__global__ void k_gmres_begin(GmresState* st, Scalars* sc, double thr) {
    const double beta = sqrt(st->nrm2);
    st->tail.beta = beta;
    for (int i = 0; i <= kMaxRestart; ++i) st->g[i] = 0.0;
    st->g[0] = beta;
    st->inv = beta > 0.0 ? 1.0 / beta : 0.0;
    st->tail.res = beta;
    st->tail.done = beta <= thr ? 1 : 0;
    sc->done = st->tail.done;
}

// Arnoldi step j: ||w||^2 from its block sums; column j of H from the two
// Gram-Schmidt passes and ||w||; earlier rotations, the new rotation, g; done
// when |g_{j+1}| <= thr or w vanished (the Krylov space is invariant: the
// iterate is exact).  One block: all that is read comes in at once, the
// rotations run on LDS.
__global__ __launch_bounds__(kKryThreads) void k_gmres_step(GmresState* st, Scalars* sc, int j, double thr,
                                                            const double* __restrict__ part, int nb) {
    constexpr int ld = kMaxRestart + 1;
    __shared__ double red[kKryThreads / 64], col[kMaxRestart + 2], cs[kMaxRestart], sn[kMaxRestart];
    const int t = threadIdx.x;
    double s2 = 0.0;
    for (int b = t; b < nb; b += blockDim.x) s2 += part[b];
    if (t <= j) col[t] = st->h[t] + st->h2[t];
    if (t < j) {
        cs[t] = st->cs[t];
        sn[t] = st->sn[t];
    }
    const double gj = st->g[j];
    s2 = wave_sum(s2);
    if ((t & 63) == 0) red[t >> 6] = s2;
    __syncthreads();
    if (t == 0) {
        double nrm2 = 0.0;
        for (int k = 0; k < kKryThreads / 64; ++k) nrm2 += red[k];
        st->nrm2 = nrm2;
        const double hn = sqrt(nrm2);
        double x = col[0];
        for (int i = 0; i < j; ++i) {
            const double y = col[i + 1];
            col[i] = cs[i] * x + sn[i] * y;
            x = -sn[i] * x + cs[i] * y;
        }
        const double d = hypot(x, hn);
        const double c = d > 0.0 ? x / d : 1.0, s = d > 0.0 ? hn / d : 0.0;
        st->cs[j] = c;
        st->sn[j] = s;
        col[j] = d;
        col[j + 1] = 0.0;
        st->g[j + 1] = -s * gj;
        st->g[j] = c * gj;
        const double res = fabs(-s * gj);
        st->inv = hn > 0.0 ? 1.0 / hn : 0.0;
        st->tail.res = res;
        // 2: singular Hessenberg column, breakdown
        const int done = !(d > 0.0) ? 2 : ((res <= thr || !(hn > 0.0)) ? 1 : 0);
        st->tail.done = done;
        sc->done = done;   // the V-cycle queued next returns at once
    }
    __syncthreads();
    if (t <= j + 1) st->H[(size_t)j * ld + t] = col[t];
}

// y = R_k^{-1} g_k (R: the rotated, upper triangular H), column by column from
// LDS: lane i holds row i's right-hand side
__global__ __launch_bounds__(kKryThreads) void k_gmres_lsq(GmresState* st, int k) {
    constexpr int ld = kMaxRestart + 1;
    __shared__ double R[kMaxRestart * ld];
    for (int t = threadIdx.x; t < k * ld; t += blockDim.x) R[t] = st->H[t];
    __syncthreads();
    const int i = threadIdx.x;
    if (i >= 64) return;
    double v = i < k ? st->g[i] : 0.0;
    const double d = i < k ? R[i * ld + i] : 1.0;
    for (int l = k - 1; l >= 0; --l) {
        const double y = __shfl(v / d, l);
        if (i == l) st->y[l] = y;
        if (i < l) v -= R[l * ld + i] * y;
    }
}

// ---------------------------------------------------------------------------
// launchers

static int kry_blocks(int64_t n) {
    const int64_t b = (n + kKryThreads - 1) / kKryThreads;
    return (int)(b < kKryBlocks ? (b < 1 ? 1 : b) : kKryBlocks);
}

size_t mdot_part_doubles() { return (size_t)kKryBlocks * kDotWide; }

template <int C>
static void mdot_pass(const double* V, int64_t pitch, int cnt, const double* w, int64_t n, double* part, double* out,
                      hipStream_t s) {
    const int nb = kry_blocks(n);
    hipLaunchKernelGGL(k_mdot_part<C>, dim3(nb), dim3(kKryThreads), 0, s, V, pitch, cnt, w, n, part);
    hipLaunchKernelGGL(k_mdot_final, dim3(cnt), dim3(kKryThreads), 0, s, part, nb, C, out);
}

void launch_mdot(const double* V, int64_t pitch, int cnt, const double* w, int64_t n, double* part, double* out,
                 hipStream_t s) {
    for (int i0 = 0; i0 < cnt; i0 += kDotWide) {
        const int c = std::min(cnt - i0, kDotWide);
        const double* Vi = V + (size_t)i0 * pitch;
        if (c <= kDotChunk) mdot_pass<kDotChunk>(Vi, pitch, c, w, n, part, out + i0, s);
        else mdot_pass<kDotWide>(Vi, pitch, c, w, n, part, out + i0, s);
    }
}

void launch_maxpy(const double* V, int64_t pitch, int cnt, const double* coef, double sign, double* w, int64_t n,
                  hipStream_t s) {
    hipLaunchKernelGGL(k_maxpy<false>, dim3(kry_blocks(n)), dim3(kKryThreads), 0, s, V, pitch, cnt, coef, sign, w, n,
                       (double*)nullptr);
}

// w -= V h, h2 = V^T w (new w), w -= V h2, ||w||^2 and Arnoldi step j, h given
void launch_gmres_orthogonalise(const double* V, int64_t n, int j, double* w, double* part, GmresState* st, Scalars* sc,
                                double thr, hipStream_t s) {
    const int cnt = j + 1, nb = kry_blocks(n);
    if (cnt <= kDotChunk) {
        hipLaunchKernelGGL(k_project_dot<kDotChunk>, dim3(nb), dim3(kKryThreads), 0, s, V, n, cnt, st->h, w, n, part);
        hipLaunchKernelGGL(k_mdot_final, dim3(cnt), dim3(kKryThreads), 0, s, part, nb, kDotChunk, st->h2);
    } else if (cnt <= kDotWide) {
        hipLaunchKernelGGL(k_project_dot<kDotWide>, dim3(nb), dim3(kKryThreads), 0, s, V, n, cnt, st->h, w, n, part);
        hipLaunchKernelGGL(k_mdot_final, dim3(cnt), dim3(kKryThreads), 0, s, part, nb, kDotWide, st->h2);
    } else {   // more vectors than the registers hold: a pass for each
        launch_maxpy(V, n, cnt, st->h, -1.0, w, n, s);
        launch_mdot(V, n, cnt, w, n, part, st->h2, s);
    }
    hipLaunchKernelGGL(k_maxpy<true>, dim3(nb), dim3(kKryThreads), 0, s, V, n, cnt, st->h2, -1.0, w, n, part);
    hipLaunchKernelGGL(k_gmres_step, dim3(1), dim3(kKryThreads), 0, s, st, sc, j, thr, part, nb);
}

void launch_scale_dev(double* dst, const double* src, const double* factor, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_scale_dev, dim3(kry_blocks(n)), dim3(kKryThreads), 0, s, dst, src, factor, n);
}

void launch_gmres_begin(GmresState* st, Scalars* sc, double thr, hipStream_t s) {
    hipLaunchKernelGGL(k_gmres_begin, dim3(1), dim3(1), 0, s, st, sc, thr);
}

void launch_gmres_lsq(GmresState* st, int k, hipStream_t s) {
    hipLaunchKernelGGL(k_gmres_lsq, dim3(1), dim3(kKryThreads), 0, s, st, k);
}

}  // namespace specmg
