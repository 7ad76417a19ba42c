// Level-2 eigensolves of the set-up phase (eq. spepb): on every 8^3 element K
// the smallest eigenpairs of A_K phi = lambda S_K phi, S_K = diag(tr kappa~),
// in the symmetric form A~ x = lambda x with A~ = S^-1/2 A_K S^-1/2,
// phi = S^-1/2 x (so phi^T S phi = 1, the normalisation of Section 3), by
// Chebyshev-filtered subspace iteration: each cycle applies a polynomial that
// damps the unwanted interval [a, b] (b: Gershgorin bound, a: the largest Ritz
// value of the block), re-orthonormalises by Cholesky-QR (twice) and performs
// Rayleigh-Ritz.
//
// One workgroup of four wavefronts per element, the block of M columns in LDS
// (cells x + 8 (y + 8 z)), in two layouts of work:
//   The filter acts on every column by itself, so a wavefront takes a column and
//   keeps the two iterates of the three-term recurrence in registers: a lane holds
//   a 2 x 2 x 2 cube of cells, 4 x 4 x 4 lanes, so 24 of the 48 neighbour values
//   come from other lanes (x by DPP quad_perm, y by DPP row shifts, z by bpermute),
//   and all degrees run without a barrier or an LDS access.
//   Everything else takes two cells a thread, cells threadIdx and threadIdx + 256:
//   a wavefront then holds whole z planes, and the Gram sums are those of the eight
//   planes (sum16), added in plane order.
// Two workgroups a CU (256 registers), so that one's serial phases (Cholesky,
// Jacobi, one wavefront each) overlap the other's filter.  Every sum keeps the order
// of a cell-a-thread form (LDS and a barrier for each degree), so that all results are
// the same to the last bit; that form took 11.6 ms for 4,096 elements of 12 vectors
// (128^3), 109 for 32,768 of 14 and 73.6 for 32,768 of 12 (256^3): now 4.5, 33.8 and
// 28.4.  Bound by FP64 vector issue in the filter and by the latency of the serial
// phases.
#include "eig_common.hpp"

namespace specmg {

constexpr int kEigWaves = 4;

// lane <- the value of the lane one step down (up) the axis; lanes at the
// element's boundary get some finite value, which meets a zero coupling
template <int CTRL>
__device__ __forceinline__ double dpp_take(double v) {   // bound_ctrl: lanes without a source read zero
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo);
}
template <int AX, bool UP>
__device__ __forceinline__ double from_lane(double v) {
    if constexpr (AX == 0) return UP ? dpp_take<0xF9>(v) : dpp_take<0x90>(v);        // quad_perm [1,2,3,3], [0,0,1,2]
    else if constexpr (AX == 1) return UP ? dpp_take<0x104>(v) : dpp_take<0x114>(v);   // row_shl:4, row_shr:4
    else return UP ? __shfl_down(v, 16, 64) : __shfl_up(v, 16, 64);
}

// The couplings of a cell (negated) and its diagonal, in the axis order of every
// application: -x, +x, -y, +y, -z, +z.
struct CellOp {
    double dg, off[6];
};

template <int M>
struct CubeShared {
    alignas(16) double Y[M * 512];
    double red[8 * M * M];
    double G[M * M];
    double Q[M * M];
    double th[M], nrm[M], scr[2 * M];
    double fc[2 * kDegExact];   // the filter's two factors of each degree
    double bound[kEigWaves];
    int iscr[M];
};

// A~ on the lane's cube: slot q = x + 2 y + 4 z (parities of the cell)
struct CubeOp {
    double dg[8];
    double ix[4], iy[4], iz[4];    // negated couplings inside the cube (index: the other two bits)
    double ox[8], oy[8], oz[8];    // ... of slot q to the next lane
    // out = A v, then f(q, out)
    template <class F>
    __device__ __forceinline__ void apply(const double (&v)[8], F f) const {
        double nz[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) nz[q] = from_lane<2, false>(v[q + 4]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q == 2) {   // the z exchanges go through LDS: ahead of their use
#pragma unroll
                for (int i = 4; i < 8; ++i) nz[i] = from_lane<2, true>(v[i - 4]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const double kx = ix[q >> 1], ky = iy[(q & 1) | ((q >> 1) & 2)], kz = iz[q & 3];
            double s;   // the diagonal's product fused onto the rounded one of -x, then the others in turn
            if (q & 1) {
                s = fma(dg[q], v[q], kx * v[q ^ 1]);
                s = fma(ox[q], from_lane<0, true>(v[q ^ 1]), s);
            } else {
                s = fma(dg[q], v[q], ox[q] * from_lane<0, false>(v[q ^ 1]));
                s = fma(kx, v[q ^ 1], s);
            }
            if (q & 2) {
                s = fma(ky, v[q ^ 2], s);
                s = fma(oy[q], from_lane<1, true>(v[q ^ 2]), s);
            } else {
                s = fma(oy[q], from_lane<1, false>(v[q ^ 2]), s);
                s = fma(ky, v[q ^ 2], s);
            }
            if (q & 4) {
                s = fma(kz, v[q ^ 4], s);
                s = fma(oz[q], nz[q], s);
            } else {
                s = fma(oz[q], nz[q], s);
                s = fma(kz, v[q ^ 4], s);
            }
            f(q, s);
            if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// first cell of the lane's cube
__device__ __forceinline__ int cube_cell(int lane) {
    return 2 * (lane & 3) + 16 * ((lane >> 2) & 3) + 128 * (lane >> 4);
}
__device__ __forceinline__ void cube_load(const double* y, double (&v)[8]) {
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
        const double2 d = *reinterpret_cast<const double2*>(y + 8 * ((q >> 1) & 1) + 64 * (q >> 2));
        v[q] = d.x;
        v[q + 1] = d.y;
    }
}
__device__ __forceinline__ void cube_store(double* y, const double (&v)[8]) {
#pragma unroll
    for (int q = 0; q < 8; q += 2)
        *reinterpret_cast<double2*>(y + 8 * ((q >> 1) & 1) + 64 * (q >> 2)) = make_double2(v[q], v[q + 1]);
}

// Chebyshev filter of the wavefront's columns in place
template <int M>
__device__ __forceinline__ void cube_filter(const CubeOp& op, double* Y, const double* fc, int w, int lane, double cc,
                                            int deg) {
#pragma unroll 1
    for (int j = w; j < M; j += kEigWaves) {
        double x[8], y[8];
        double* col = Y + j * 512 + cube_cell(lane);
        cube_load(col, x);
        const double f0 = fc[0];
        op.apply(x, [&](int q, double s) { y[q] = fma(-cc, x[q], s) * f0; });
        // u <- (A v - c v) f - g u
        auto step = [&](double (&u)[8], const double (&v)[8], int k) {
            const double2 f = *reinterpret_cast<const double2*>(fc + 2 * k);
            op.apply(v, [&](int q, double s) { u[q] = fma(fma(-cc, v[q], s), f.x, -(f.y * u[q])); });
        };
        int it = 2;
#pragma unroll 1
        for (; it + 1 <= deg; it += 2) {
            step(x, y, it - 1);
            step(y, x, it);
        }
        if (it <= deg) {
            step(x, y, it - 1);
            cube_store(col, x);
        } else {
            cube_store(col, y);
        }
    }
}

// (A~ Y) of the thread's cell c, column y
__device__ __forceinline__ double cell_apply(const CellOp& o, const double* y, int c) {
    const int i = c & 7, j = (c >> 3) & 7, k = c >> 6;
    double s = fma(o.dg, y[c], o.off[0] * y[i > 0 ? c - 1 : c]);
    s = fma(o.off[1], y[i < 7 ? c + 1 : c], s);
    s = fma(o.off[2], y[j > 0 ? c - 8 : c], s);
    s = fma(o.off[3], y[j < 7 ? c + 8 : c], s);
    s = fma(o.off[4], y[k > 0 ? c - 64 : c], s);
    s = fma(o.off[5], y[k < 7 ? c + 64 : c], s);
    return s;
}

// G = Y^T Y
template <int M>
__device__ __forceinline__ void gram(CubeShared<M>& sh, int lane) {
    constexpr int NE = M * (M + 1) / 2;
    constexpr Triangle<M> tri{};
#pragma unroll 1
    for (int pl = threadIdx.x >> 6; pl < 8; pl += kEigWaves) {
        double y[M];
#pragma unroll
        for (int j = 0; j < M; ++j) y[j] = sh.Y[j * 512 + 64 * pl + lane];
        tile_sums<NE>(sh.red + pl * NE, lane, [&](int e) { return fma(y[tri.i[e]], y[tri.j[e]], 0.0); });
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NE; e += 64 * kEigWaves) {
        double x = 0.0;
#pragma unroll
        for (int pl = 0; pl < 8; ++pl) x += sh.red[pl * NE + e];
        int i = 0, r = e;   // row of entry e
        while (r >= M - i) r -= M - i++;
        sh.G[i * M + i + r] = x;
        sh.G[(i + r) * M + i] = x;
    }
    __syncthreads();
}

// G = the symmetric part of Y^T A~ Y
template <int M>
__device__ __forceinline__ void projected(const CellOp (&op)[2], CubeShared<M>& sh, int lane) {
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
        const int c = threadIdx.x + 256 * h, pl = c >> 6;
        const CellOp o = h ? op[1] : op[0];
#pragma unroll 1
        for (int j0 = 0; j0 < M; j0 += M / 2) {   // half the columns of A~ Y at a time
            double b[M / 2];
#pragma unroll
            for (int j = 0; j < M / 2; ++j) {
                b[j] = cell_apply(o, sh.Y + (j0 + j) * 512, c);
                pin(b[j]);
            }
            double y[M];
#pragma unroll
            for (int i = 0; i < M; ++i) y[i] = sh.Y[i * 512 + c];
            tile_sums<M * M / 2>(sh.red + pl * M * M + j0 * M, lane,
                                  [&](int e) { return fma(y[e % M], b[e / M], 0.0); });
        }
    }
    __syncthreads();
    // red: column-major, entry (i, j) at j M + i
    for (int t = threadIdx.x; t < M * M; t += 64 * kEigWaves) {
        const int i = t / M, j = t % M;
        if (i > j) continue;
        double x = 0.0, y = 0.0;
#pragma unroll
        for (int pl = 0; pl < 8; ++pl) {
            x += sh.red[pl * M * M + j * M + i];
            y += sh.red[pl * M * M + i * M + j];
        }
        const double v = 0.5 * (x + y);
        sh.G[i * M + j] = v;
        sh.G[j * M + i] = v;
    }
    __syncthreads();
}

// Y <- Y C, every thread its own cells (TRI: C upper triangular)
template <int M, bool TRI>
__device__ __forceinline__ void multiply(CubeShared<M>& sh, const double* C) {
    double t[2][M];
#pragma unroll
    for (int j = 0; j < M; ++j) t[0][j] = t[1][j] = 0.0;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        const double a0 = sh.Y[i * 512 + threadIdx.x], a1 = sh.Y[i * 512 + threadIdx.x + 256];
#pragma unroll
        for (int j = TRI ? i : 0; j < M; ++j) {
            const double f = C[i * M + j];
            t[0][j] = fma(a0, f, t[0][j]);
            t[1][j] = fma(a1, f, t[1][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < M; ++j) {
        sh.Y[j * 512 + threadIdx.x] = t[0][j];
        sh.Y[j * 512 + threadIdx.x + 256] = t[1][j];
    }
}

// Y <- an orthonormal basis of its columns (Cholesky-QR, twice)
template <int M>
__device__ __forceinline__ void orthonormalise(CubeShared<M>& sh, int lane) {
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        gram<M>(sh, lane);
        if (threadIdx.x < 64) cholesky_call<M>((lds_double*)sh.G, (lds_double*)sh.Q);
        __syncthreads();
        multiply<M, true>(sh, sh.Q);
        __syncthreads();
    }
}

// CheFSI on the LDS block (start block on entry, Ritz vectors on exit); the
// cycles taken, or -1 when max_cycles did not suffice.
template <int M>
__device__ __forceinline__ int cube_chefsi(const CubeOp& cube, const CellOp (&op)[2], CubeShared<M>& sh, int w,
                                           int lane, double bnd, int need, double tol, int target, double crtol,
                                           double thr, int max_cycles, int deg) {
    double below = 1e-3 * bnd;
    pin_value(below);
    orthonormalise<M>(sh, lane);
#pragma unroll 1
    for (int cyc = 0;; ++cyc) {
        // Rayleigh-Ritz: Y becomes the Ritz vectors, th the values
        projected<M>(op, sh, lane);
        if (threadIdx.x < 64) jacobi_call<M>((lds_double*)sh.G, (lds_double*)sh.Q, (lds_double*)sh.th, (lds_double*)sh.scr, (lds_int*)sh.iscr);
        __syncthreads();
        multiply<M, false>(sh, sh.Q);
        const double a = fmin(sh.th[M - 1], 0.5 * bnd);
        const double a0 = fmin(sh.th[0], 0.0) - below;
        __syncthreads();
        // squared residual norms, one plane of sums at a time; the last wavefront's
        // first lane forms the next filter's factors meanwhile
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const int c = threadIdx.x + 256 * h;
            const CellOp o = h ? op[1] : op[0];
            double p[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                p[j] = 0.0;
                if (j < M) {
                    double s = cell_apply(o, sh.Y + j * 512, c);
                    pin(s);
                    const double r = fma(-sh.th[j], sh.Y[j * 512 + c], s);
                    p[j] = fma(r, r, 0.0);
                }
            }
            const double v = sum16(p, lane);
            if (lane < 16) sh.red[(c >> 6) * 16 + sum16_index(lane)] = v;
        }
        if (threadIdx.x == 64 * kEigWaves - 1) filter_factors(sh.fc, a, bnd, a0, deg);
        __syncthreads();
        if (threadIdx.x < M) {
            double s = 0.0;
#pragma unroll
            for (int pl = 0; pl < 8; ++pl) s += sh.red[pl * 16 + threadIdx.x];
            sh.nrm[threadIdx.x] = s;
        }
        __syncthreads();
        if (chefsi_done(sh.th, sh.nrm, M, need, tol, bnd, target, crtol, thr, cyc)) return cyc;
        if (cyc >= max_cycles) return -1;
        cube_filter<M>(cube, sh.Y, sh.fc, w, lane, 0.5 * (bnd + a), deg);
        __syncthreads();
        orthonormalise<M>(sh, lane);
    }
}

// Learned start (warm != null): the first kw columns of the start block are
// the predicted cell vectors warm[blockIdx.x][0..kw-1][512] (row pitch kp),
// the rest the next cosine modes.  From that block the eigensolve runs to
// the relaxed residual ws_tol (times the spectral bound) within
// kWarmCycles cycles; an element that does not get there falls back to the
// exact solve (tolerance tol) from the cold start, and ws_fb[e] = 1.
// status[e] counts the cycles of both attempts.
template <int M>
__global__ __launch_bounds__(64 * kEigWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_eig2(
    FineGeom g, const double* __restrict__ kt, int target, int L, double tol, double crtol,
    double* __restrict__ phi, double* __restrict__ lam, int* __restrict__ nkeep, double* __restrict__ Aint,
    double* __restrict__ zc, int* __restrict__ status, int e0, const float* __restrict__ warm, int kp, int kw,
    double ws_tol, int* __restrict__ ws_fb, double thr) {
    __shared__ CubeShared<M> sh;
    const int e = e0 + blockIdx.x;
    const int lane = threadIdx.x & 63;
    // the wavefronts that filter one column more sit on another SIMD in the
    // next workgroup
    const int w = (int)((threadIdx.x >> 6) + blockIdx.x) % kEigWaves;
    // kappa~ per face direction: one array (isotropic) or three (orthotropic);
    // weight tr K~: kappa~ (1 + cy + cz) with the y and z faces carrying cy
    // and cz, or the sum of the three components
    const size_t N = g.ortho ? g.ncell() : 0;
    const double* ke = kt + (size_t)e * 512;
    const double wsum = 1.0 + g.cy + g.cz;
    auto weight = [&](int c) {
        const int p = phi_pos(c);
        return g.ortho ? ke[p] + ke[N + p] + ke[2 * N + p] : wsum * ke[p];
    };
    // one-dimensional factors cos(pi p (i + 1/2) / 8), p = 0, 1, 2, of the cosine modes
    double* ctab = sh.fc;
    if (threadIdx.x < 24)
        ctab[threadIdx.x] = cos(3.14159265358979323846 / 8.0 * (double)(threadIdx.x >> 3) * ((threadIdx.x & 7) + 0.5));
    // the operator of the thread's two cells, and through LDS that of the lane's cube
    CellOp op[2];
    double bnd;
    {
        double* S = sh.Y;   // weights, then the cells' operators
        for (int c = threadIdx.x; c < 512; c += 64 * kEigWaves) S[c] = weight(c);
        __syncthreads();
        double mx = 0.0;
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const int c = threadIdx.x + 256 * h;
            const double sq = sqrt(S[c]);
            double diag = 0.0, rowsum = 0.0;
            CellOp o;
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                const int ax = d >> 1, st = ax == 0 ? 1 : (ax == 1 ? 8 : 64), x = (c / st) & 7;
                o.off[d] = 0.0;
                if ((d & 1) ? x < 7 : x > 0) {
                    const int cn = (d & 1) ? c + st : c - st;
                    const double k = harm_e(ke[ax * N + phi_pos(c)], ke[ax * N + phi_pos(cn)]);
                    const double f = ax == 0 ? 1.0 : (ax == 1 ? g.cy : g.cz), T = k * f;
                    diag = fma(k, f, diag);
                    const double v = T / (sq * sqrt(S[cn]));
                    rowsum += v;
                    o.off[d] = -v;
                }
            }
            o.dg = diag / S[c];
            mx = fmax(mx, o.dg + rowsum);
            if (h) op[1] = o;
            else op[0] = o;
        }
        mx = wave_max(mx);
        if (lane == 0) sh.bound[threadIdx.x >> 6] = mx;
        __syncthreads();
        bnd = fmax(fmax(sh.bound[0], sh.bound[1]), fmax(sh.bound[2], sh.bound[3]));
    }
    CubeOp cube;
    {
        double* A = sh.Y;   // diagonal, then the six couplings, 512 each
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = threadIdx.x + 256 * h;
            A[c] = op[h].dg;
#pragma unroll
            for (int d = 0; d < 6; ++d) A[(1 + d) * 512 + c] = op[h].off[d];
        }
        __syncthreads();
        const int c0 = cube_cell(lane);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = c0 + (q & 1) + 8 * ((q >> 1) & 1) + 64 * (q >> 2);
            cube.dg[q] = A[c];
            cube.ox[q] = A[((q & 1) ? 2 : 1) * 512 + c];
            cube.oy[q] = A[((q & 2) ? 4 : 3) * 512 + c];
            cube.oz[q] = A[((q & 4) ? 6 : 5) * 512 + c];
            if (!(q & 1)) cube.ix[q >> 1] = A[2 * 512 + c];
            if (!(q & 2)) cube.iy[(q & 1) | ((q >> 1) & 2)] = A[4 * 512 + c];
            if (!(q & 4)) cube.iz[q & 3] = A[6 * 512 + c];
        }
        __syncthreads();
    }
    const int need = (target + 4 < M - 2) ? target + 4 : M - 2;
    int cyc = -1, spent = 0;
    // one pass from the predicted start, one from the cold start
#pragma unroll 1
    for (int att = warm ? 0 : 1; att < 2 && cyc < 0; ++att) {
        if (att == 1 && warm) {
            spent = kWarmCycles + 1;
            __syncthreads();
            if (threadIdx.x < 24)
                ctab[threadIdx.x] =
                    cos(3.14159265358979323846 / 8.0 * (double)(threadIdx.x >> 3) * ((threadIdx.x & 7) + 0.5));
            __syncthreads();
        }
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            const int c = threadIdx.x + 256 * h;
            const double sq = sqrt(weight(c));
#pragma unroll 1
            for (int jj = 0; jj < M; ++jj) {
                const unsigned char* md = kModes[jj];
                double v;
                if (att == 0 && jj < kw) {
                    v = sq * (double)warm[((size_t)blockIdx.x * kp + jj) * 512 + c];
                } else {
                    double m = ctab[8 * md[0] + (c & 7)] * ctab[8 * md[1] + ((c >> 3) & 7)] * ctab[8 * md[2] + (c >> 6)];
                    pin_value(m);
                    v = sq * fma(0.05, hash_noise((unsigned)e, (unsigned)jj, (unsigned)c), m);
                }
                sh.Y[jj * 512 + c] = v;
            }
        }
        __syncthreads();
        cyc = cube_chefsi<M>(cube, op, sh, w, lane, bnd, need, att == 0 ? ws_tol : tol, target, crtol, thr,
                             att == 0 ? kWarmCycles : kMaxCycles, att == 0 ? kDeg : kDegExact);
        if (warm && att == 0 && threadIdx.x == 0) ws_fb[e] = cyc < 0 ? 1 : 0;
    }
    if (cyc >= 0) cyc += spent;

    const int nk = cluster_cut_dev(sh.th, M, target, crtol, thr);
    if (threadIdx.x == 0) {
        nkeep[e] = nk;
        status[e] = cyc;
        for (int a = 0; a < L; ++a) lam[(size_t)e * L + a] = sh.th[a];
    }
    // interior block X^T A~ X on the kept vectors (= Phi^T A_K Phi), the
    // coefficients of the constant function Phi^T S 1 = X^T S^1/2 1, and Phi
    projected<M>(op, sh, lane);
    for (int t = threadIdx.x; t < L * L; t += 64 * kEigWaves) {
        const int a = t / L, b = t % L;
        Aint[(size_t)e * L * L + t] = (a < nk && b < nk) ? sh.G[a * M + b] : 0.0;
    }
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
        const int c = threadIdx.x + 256 * h;
        const double sq = sqrt(weight(c));
        double p[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] = j < M ? fma(sh.Y[j * 512 + c], sq, 0.0) : 0.0;
        const double v = sum16(p, lane);
        if (lane < 16) sh.red[(c >> 6) * 16 + sum16_index(lane)] = v;
#pragma unroll 1
        for (int j = 0; j < L; ++j)
            phi[((size_t)e * L + j) * 512 + phi_pos(c)] = j < nk ? sh.Y[j * 512 + c] / sq : 0.0;
    }
    __syncthreads();
    if ((int)threadIdx.x < L) {
        double s = 0.0;
#pragma unroll
        for (int pl = 0; pl < 8; ++pl) s += sh.red[pl * 16 + threadIdx.x];
        zc[(size_t)e * L + threadIdx.x] = (int)threadIdx.x < nk ? s : 0.0;
    }
}

// ---------------------------------------------------------------------------
// launcher

#define SPECMG_M_DISPATCH(MV, ...)                   \
    switch (MV) {                                    \
        case 10: {                                   \
            constexpr int M = 10;                    \
            __VA_ARGS__;                             \
        } break;                                     \
        case 12: {                                   \
            constexpr int M = 12;                    \
            __VA_ARGS__;                             \
        } break;                                     \
        default: {                                   \
            constexpr int M = 14;                    \
            __VA_ARGS__;                             \
        } break;                                     \
    }

void launch_eig2(const FineGeom& g, const double* kt, int target, int nvec, double tol, double crtol,
                 double* phi, double* lam, int* nkeep, double* Aint, int* status, double* zc, int e0, int count,
                 const float* warm, int kp, int kw, double ws_tol, int* ws_fb, double thr, hipStream_t s) {
    const int L = target + 3;
    SPECMG_M_DISPATCH(nvec, hipLaunchKernelGGL((k_eig2<M>), dim3(count), dim3(64 * kEigWaves), 0, s, g, kt, target, L,
                                               tol, crtol, phi, lam, nkeep, Aint, zc, status, e0, warm, kp, kw,
                                               ws_tol, ws_fb, thr));
}

}  // namespace specmg
