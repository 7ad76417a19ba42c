// Level-2 eigensolves of the set-up phase (eq. spepb): on every 8^3 element K
// the smallest eigenpairs of A_K phi = lambda S_K phi, S_K = diag(tr kappa~),
// in the symmetric form A~ x = lambda x with A~ = S^-1/2 A_K S^-1/2,
// phi = S^-1/2 x (so phi^T S phi = 1, the normalisation of Section 3), by
// Chebyshev-filtered subspace iteration: each cycle applies a polynomial that
// damps the unwanted interval [a, b] (b: Gershgorin bound, a: the largest Ritz
// value of the block) and performs Rayleigh-Ritz on the filtered block, with
// a one-wavefront Cholesky factor and parallel cyclic Jacobi eigensolver.
#include <type_traits>

#include "eig_common.hpp"

namespace specmg {

// One workgroup of NW wavefronts per 8^3 element, whole
// columns in the registers of one wavefront.
//
// The filter is 80 % of the floating-point work and acts on every column by
// itself, so a wavefront takes a column, keeps the two iterates of the
// three-term recurrence in registers (8 cells per lane) and runs all degrees
// without a barrier or an LDS access.  Lane cells: a 2 x 2 x 2 cube, 4 x 4 x 4
// lanes, so 24 of the 48 neighbour values come from other lanes (an x-pencil
// per lane needs 32).  Along each axis the four lane positions are numbered
// by a Gray code and odd positions hold their cube mirrored: slot bit 0 of an
// axis always faces the partner whose first code bit differs, slot bit 1 the
// one whose second differs, and an exchange is one lane permutation for every
// lane: x by DPP quad_perm (lane ^ 1, lane ^ 2), y by DPP half-row mirror and
// row rotation (lane ^ 7, lane ^ 8), z by bpermute (lane ^ 16, lane ^ 32).
// Couplings that leave the element are zero.
//
// The LDS holds one block of M columns (4 KB each, 16-byte pairs of slots
// across the lanes) for the Gram matrices and the small products only.

// lane ^ MASK for the six exchanges above.  Every source lane is valid, so
// the DPP moves carry bound_ctrl: without it the compiler zeroes each
// destination first (32 moves more per operator application).
template <int CTRL>
__device__ __forceinline__ double dpp_perm(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned long long)(unsigned)lo);
}
template <int MASK>
__device__ __forceinline__ double lane_xor(double v) {
    if constexpr (MASK == 1) return dpp_perm<0xB1>(v);         // quad_perm [1,0,3,2]
    else if constexpr (MASK == 2) return dpp_perm<0x4E>(v);    // quad_perm [2,3,0,1]
    else if constexpr (MASK == 7) return dpp_perm<0x141>(v);   // row_half_mirror
    else if constexpr (MASK == 8) return dpp_perm<0x128>(v);   // row_ror:8
    else return __shfl_xor(v, MASK, 64);
}

// position 0..3 of the lane along an axis from its two Gray code bits
__device__ __forceinline__ int gray_pos(int b1, int b2) { return 2 * b2 + (b1 ^ b2); }
// cell coordinate of slot bit s at position pos: the odd cell first at even positions
__device__ __forceinline__ int slot_cell(int pos, int s) { return 2 * pos + (s ^ 1 ^ (pos & 1)); }

// the lane's place in the element
struct CubePos {
    int px, py, pz;
    __device__ __forceinline__ explicit CubePos(int lane) {
        const int b0 = lane & 1, b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
        px = gray_pos(b0 ^ b2, b1 ^ b2);
        py = gray_pos(b2, b3);
        pz = gray_pos((lane >> 4) & 1, lane >> 5);
    }
    // x + 8 (y + 8 z) of slot q
    __device__ __forceinline__ int cell(int q) const {
        return slot_cell(px, q & 1) + 8 * (slot_cell(py, (q >> 1) & 1) + 8 * slot_cell(pz, q >> 2));
    }
};

// the same value, formed anew by the compiler (nothing derived from it is
// kept in registers across the solver's loops)
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

template <int M>
struct CubeShared {
    double Y[M * 512];
    double G[M * M];
    double H[M * M];
    double Q[M * M];
    double th[M], nrm[M], scr[M];
    double low;
    int iscr[M];
};

// A~ on the lane's cube: slot q = ax + 2 ay + 4 az (slot bits of the axes)
struct CubeOp {
    double dg[8];                  // diagonal
    double ix[4], iy[4], iz[4];    // couplings inside the cube (index: the other two slot bits)
    double ox[8], oy[8], oz[8];    // couplings of slot q to the lane its slot bit faces
    // scale (A - shift), made of new values: the solver's other phases need the registers,
    // so the couplings go to scratch between them, and without the copy the
    // compiler reloads them from there inside the filter's loop.
    __device__ __forceinline__ CubeOp fresh(double scale, double shift) const {
        CubeOp o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            o.dg[i] = (dg[i] - shift) * scale;
            o.ox[i] = ox[i] * scale;
            o.oy[i] = oy[i] * scale;
            o.oz[i] = oz[i] * scale;
            pin_value(o.dg[i]);
            pin_value(o.ox[i]);
            pin_value(o.oy[i]);
            pin_value(o.oz[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o.ix[i] = ix[i] * scale;
            o.iy[i] = iy[i] * scale;
            o.iz[i] = iz[i] * scale;
            pin_value(o.ix[i]);
            pin_value(o.iy[i]);
            pin_value(o.iz[i]);
        }
        return o;
    }
    // calls f(q, init(q) + (A v)_q) slot by slot.  The z exchanges (LDS crossbar) are
    // issued four at a time ahead of their use; the barriers keep the compiler from hoisting the x and y
    // exchanges of all slots ahead of the arithmetic (16 registers each).
    template <class I, class F>
    __device__ __forceinline__ void for_each(const double (&v)[8], I init, F f) const {
        double nz[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) nz[q] = lane_xor<16>(v[q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q == 2) {
#pragma unroll
                for (int i = 4; i < 8; ++i) nz[i] = lane_xor<32>(v[i]);
                __builtin_amdgcn_sched_barrier(0);
            }
            const double nx = q & 1 ? lane_xor<2>(v[q]) : lane_xor<1>(v[q]);
            const double ny = q & 2 ? lane_xor<8>(v[q]) : lane_xor<7>(v[q]);
            double s = fma(dg[q], v[q], init(q));
            s -= ix[q >> 1] * v[q ^ 1];
            s -= iy[(q & 1) | ((q >> 1) & 2)] * v[q ^ 2];
            s -= iz[q & 3] * v[q ^ 4];
            s -= ox[q] * nx;
            s -= oy[q] * ny;
            s -= oz[q] * nz[q];
            f(q, s);
            if (q % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    // out = A v
    __device__ __forceinline__ void apply(const double (&v)[8], double (&out)[8]) const {
        for_each(v, [](int) { return 0.0; }, [&](int q, double s) { out[q] = s; });
    }
};

__device__ __forceinline__ void cube_load(const double* Y, int j, int lane, double (&v)[8]) {
    const double2* p = reinterpret_cast<const double2*>(Y + j * 512) + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const double2 d = p[64 * i];
        v[2 * i] = d.x;
        v[2 * i + 1] = d.y;
    }
}
__device__ __forceinline__ void cube_store(double* Y, int j, int lane, const double (&v)[8]) {
    double2* p = reinterpret_cast<double2*>(Y + j * 512) + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[64 * i] = make_double2(v[2 * i], v[2 * i + 1]);
}

// Sums of 16 values over the wavefront, value i in lane i (and i + 16, ...):
// each of the four steps inside a 16-lane row halves the values a lane
// carries (it keeps the half its lane bit names and receives the partner's),
// 105 instructions for up to 16 sums instead of 22 each.  Fixed order.
__device__ __forceinline__ double sum16(double (&p)[16], int lane) {
    auto step = [&](auto mask, int bit, int half) {
        const bool up = (lane & bit) != 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < half) {
                const double keep = up ? p[i + half] : p[i], send = up ? p[i] : p[i + half];
                p[i] = keep + lane_xor<decltype(mask)::value>(send);
            }
        }
    };
    step(std::integral_constant<int, 8>{}, 8, 8);
    step(std::integral_constant<int, 7>{}, 4, 4);
    step(std::integral_constant<int, 2>{}, 2, 2);
    step(std::integral_constant<int, 1>{}, 1, 1);
    double v = p[0];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// rows i >= j of column j of G = Y^T B, mirrored (b: column j of B in
// registers; Y the LDS block)
template <int M>
__device__ __forceinline__ void cube_dots(const double* Y, int j, int lane, const double (&b)[8], double* G) {
    double p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = 0.0;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        if (i >= j) {   // uniform over the wavefront
            double y[8];
            cube_load(Y, i, lane, y);
            double s = y[0] * b[0];
#pragma unroll
            for (int q = 1; q < 8; ++q) s += y[q] * b[q];
            p[i] = s;
        }
        if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    const double v = sum16(p, lane);
    if (lane >= j && lane < M) {
        G[lane * M + j] = v;
        G[j * M + lane] = v;
    }
}

// b = sum_i Y_i Cm[i][j] for this wavefront's columns
template <int M, int NW, int CW>
__device__ __forceinline__ void cube_mul(const double* Y, const double* Cm, int w, int lane, double (&b)[CW][8]) {
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int q = 0; q < 8; ++q) b[c][q] = 0.0;
#pragma unroll 1
    for (int i = 0; i < M; ++i) {
        double y[8];
        cube_load(Y, i, lane, y);
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const int j = w + NW * c;
            const double f = j < M ? Cm[i * M + j] : 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) b[c][q] += y[q] * f;
        }
    }
}

// Chebyshev filter of the wavefront's columns in place: T_deg of the operator
// mapped from the damped interval [a, b] to [-1, 1].  The recurrence
// u <- 2 A' v - u is left unscaled (an operator application and one negated
// addend, 56 multiply-adds per column and step against 80 with the usual
// scaling by T_deg(a0)): at degree 60 the values stay below 1e50, and the
// Cholesky factor that follows scales the columns.
template <int M, int NW>
__device__ __forceinline__ void cube_filter(const CubeOp& kept, double* Y, int w, int lane, double a, double b,
                                            int deg) {
    const double e = 0.5 * (b - a), cc = 0.5 * (b + a);
    CubeOp op = kept.fresh(2.0 / e, cc);
#pragma unroll 1
    for (int j = w; j < M; j += NW) {
        double x[8], y[8];
        cube_load(Y, j, lane, x);
        op.for_each(x, [](int) { return 0.0; }, [&](int q, double s) { y[q] = 0.5 * s; });
        // u <- 2 A' v - u
        auto step = [&](double (&u)[8], const double (&v)[8]) {
            op.for_each(v, [&](int q) { return -u[q]; }, [&](int q, double s) { u[q] = s; });
        };
        int it = 2;
#pragma unroll 1
        for (; it + 1 <= deg; it += 2) {
            step(x, y);
            step(y, x);
        }
        if (it <= deg) {
            step(x, y);
            cube_store(Y, j, lane, x);
        } else {
            cube_store(Y, j, lane, y);
        }
    }
}

// Rayleigh-Ritz on the LDS block: its Ritz vectors replace it, sh.th holds
// the values (ascending), sh.nrm the squared residual norms.  The small
// problem is solved in its generalised form (Gram and projected matrix), so a cycle needs no
// orthonormalisation of its own: after the first cycle the filtered Ritz
// vectors are orthogonal but for their lengths (a smallest scaled pivot of
// 0.5 and more).  A block whose scaled pivots fall below min_ritz is
// orthonormalised first, at most three times (start blocks of high-contrast
// elements).  The start block's Ritz vectors only have to be good enough to
// filter, so its bounds are looser (rough).  Returns the smallest scaled
// pivot.
template <int M, int NW>
__device__ __forceinline__ double cube_rayleigh_ritz(const CubeOp& op, CubeShared<M>& sh, int w, int lane,
                                                     bool rough) {
    constexpr int CW = (M + NW - 1) / NW;
    const double min_ritz = rough ? 1e-9 : 1e-5;
    double low = 0.0;
#pragma unroll 1
    for (int pass = 0; pass < 4; ++pass) {
#pragma unroll 1
        for (int j = w; j < M; j += NW) {
            // first column j of the Gram matrix, then of the projected one
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                double y[8];
                cube_load(sh.Y, j, lane, y);
                if (h) {
                    double ay[8];
                    op.apply(y, ay);
#pragma unroll
                    for (int q = 0; q < 8; ++q) y[q] = ay[q];
                }
                cube_dots<M>(sh.Y, j, lane, y, h ? sh.H : sh.G);
            }
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            const double lw = ritz_wave<M>((lds_double*)sh.G, (lds_double*)sh.H, (lds_double*)sh.Q, (lds_double*)sh.scr,
                                           (lds_double*)sh.th, (lds_int*)sh.iscr, pass < 3 ? min_ritz : 0.0,
                                           rough ? 1e-6 : 1e-15);
            if (threadIdx.x == 0) sh.low = lw;
        }
        __syncthreads();
        low = sh.low;
        double b[CW][8];
        cube_mul<M, NW, CW>(sh.Y, sh.Q, w, lane, b);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < CW; ++c)
            if (w + NW * c < M) cube_store(sh.Y, w + NW * c, lane, b[c]);
        __syncthreads();
        if (low >= min_ritz) break;
    }
#pragma unroll 1
    for (int j = w; j < M; j += NW) {
        double x[8];
        cube_load(sh.Y, j, lane, x);
        const double tj = sh.th[j];
        double s = 0.0;
        op.for_each(x, [](int) { return 0.0; }, [&](int q, double a) {
            const double r = a - tj * x[q];
            s += r * r;
        });
        s = wave_sum(s);
        if (lane == 0) sh.nrm[j] = s;
    }
    __syncthreads();
    return low;
}

// Degree of the next filter: what the slowest of the vectors that still have
// to converge needs for a tenth of its tolerance (its residual shrinks by
// exp(-acosh x) per degree, x its Ritz value in the damped interval's
// coordinate), at most kDegMax; the first cycle, whose cut a is far too
// high, takes kDegFirst.  Against a fixed degree of 40 this saves a tenth of
// the applications and of the cycles (3.4 -> 3.0 cycles, 138 -> 127
// applications on Gaussian elements of contrast 1e6).
constexpr int kDegFirst = 30;
constexpr int kDegMax = 60;
template <int M>
__device__ __forceinline__ int filter_degree(const double* th, const double* nrm, int lane, int need, double tol,
                                             double bnd, int nk, double a) {
    const double e = 0.5 * (bnd - a), cc = 0.5 * (bnd + a);
    double d = 8.0;
    if (lane < need) {
        const double rho = sqrt(nrm[lane]) / ((lane < nk ? tol : sqrt(tol)) * bnd);
        const bool sep = lane >= nk && nk > 0 && th[lane] - th[nk - 1] > 0.05 * fabs(th[lane]);
        if (rho > 1.0 && !sep) {
            const double x = (cc - th[lane]) / e;
            d = x > 1.0001 ? fmin((double)kDegMax, log(10.0 * rho) / log(x + sqrt(x * x - 1.0)) + 2.0) : (double)kDegMax;
        }
    }
    return (int)wave_max(fmax(d, 8.0));
}

// CheFSI on the LDS block (start block on entry, Ritz vectors on exit); the
// cycles taken, or -1 when max_cycles did not suffice.  deg: the filter's
// degree, 0: chosen per cycle (filter_degree).
template <int M, int NW>
__device__ __forceinline__ int cube_chefsi(const CubeOp& op, CubeShared<M>& sh, int w, int lane, double bnd, int need,
                                           double tol, int target, double crtol, double thr, int max_cycles, int deg) {
    bool clean = false;
#pragma unroll 1
    for (int cyc = 0;;) {
        const double low = cube_rayleigh_ritz<M, NW>(op, sh, w, lane, cyc == 0 && !clean);
        if (clean) return cyc;
        if (chefsi_done(sh.th, sh.nrm, M, need, tol, bnd, target, crtol, thr, cyc)) {
            // Ritz vectors of a block that was far from orthonormal are
            // orthonormal to rounding over its smallest pivot: once more
            if (low >= 0.1) return cyc;
            clean = true;
            __syncthreads();
            continue;
        }
        if (cyc >= max_cycles) return -1;
        const double a = fmin(sh.th[M - 1], 0.5 * bnd);
        const int nk = cluster_cut_dev(sh.th, M, target, crtol, thr);
        const int dg = deg > 0 ? deg : (cyc == 0 ? kDegFirst
                                                 : filter_degree<M>(sh.th, sh.nrm, lane, need, tol, bnd, nk, a));
        cube_filter<M, NW>(op, sh.Y, w, lane, a, bnd, dg);
        ++cyc;
        __syncthreads();
    }
}

// Learned start (warm != null): the first kw columns of the start block are
// the predicted cell vectors warm[blockIdx.x][0..kw-1][512] (row pitch kp),
// the rest the next cosine modes.  From that block the eigensolve runs to
// the relaxed residual ws_tol (times the spectral bound) within
// kWarmCycles cycles; an element that does not get there falls back to the
// exact solve (tolerance tol) from the cold start, and ws_fb[e] = 1.
// status[e] counts the cycles of both attempts.
// Three wavefronts per SIMD (at most 168 VGPRs) and, up to M = 12, 53 KB of
// LDS: three elements share a CU, so that the serial phases of one (Jacobi,
// Cholesky, one wavefront each) overlap the filters of the others.
template <int M, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void k_eig2(
    FineGeom g, const double* __restrict__ kt, int target, int L, double tol, double crtol,
    double* __restrict__ phi, double* __restrict__ lam, int* __restrict__ nkeep, double* __restrict__ Aint,
    double* __restrict__ zc, int* __restrict__ status, int e0, const float* __restrict__ warm, int kp, int kw,
    double ws_tol, int* __restrict__ ws_fb, double thr) {
    __shared__ CubeShared<M> sh;
    const int e = e0 + blockIdx.x;
    const int lane = threadIdx.x & 63;
    // the wavefronts that carry one column more sit on another SIMD in the
    // next workgroup
    const int w = (int)((threadIdx.x >> 6) + blockIdx.x) % NW;
    // kappa~ per face direction: one array (isotropic) or three (orthotropic);
    // weight tr K~: kappa~ (1 + cy + cz) with the y and z faces carrying cy
    // and cz, or the sum of the three components
    const size_t N = g.ortho ? g.ncell() : 0;
    const double* ke = kt + (size_t)e * 512;
    auto weight = [&](double kx, double ky, double kz) { return g.ortho ? kx + ky + kz : (1.0 + g.cy + g.cz) * kx; };
    // one-dimensional factors cos(pi p (i + 1/2) / 8), p = 0, 1, 2, of the cosine modes
    double* ctab = sh.H;
    if (threadIdx.x < 24)
        ctab[threadIdx.x] = cos(3.14159265358979323846 / 8.0 * (double)(threadIdx.x >> 3) * ((threadIdx.x & 7) + 0.5));
    CubeOp op;
    double bnd;
    {
        const CubePos cp(lane);
        const int px = cp.px, py = cp.py, pz = cp.pz;
        double kx[8], ky[8], kz[8], S[8], sq[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = phi_pos(cp.cell(q));
            kx[q] = ke[c];
            ky[q] = ke[N + c];
            kz[q] = ke[2 * N + c];
            S[q] = weight(kx[q], ky[q], kz[q]);
            sq[q] = sqrt(S[q]);
        }
        double rs = 0.0;
        double mx = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            double diag = 0.0, row = 0.0;
            auto face = [&](double a, double b, double f, double sn, bool in) {
                const double T = in ? harm_e(a, b) * f : 0.0;
                diag += T;
                const double o = T / (sq[q] * sn);
                row += o;
                return o;
            };
            // an outward face exists unless it lies on the element's boundary
            // (slot bit 1 at the end positions)
            const bool inx = !((q & 1) && (px == 0 || px == 3)), iny = !((q & 2) && (py == 0 || py == 3)),
                       inz = !((q & 4) && (pz == 0 || pz == 3));
            const double nkx = q & 1 ? lane_xor<2>(kx[q]) : lane_xor<1>(kx[q]);
            const double nky = q & 2 ? lane_xor<8>(ky[q]) : lane_xor<7>(ky[q]);
            const double nkz = q & 4 ? lane_xor<32>(kz[q]) : lane_xor<16>(kz[q]);
            const double nsx = q & 1 ? lane_xor<2>(sq[q]) : lane_xor<1>(sq[q]);
            const double nsy = q & 2 ? lane_xor<8>(sq[q]) : lane_xor<7>(sq[q]);
            const double nsz = q & 4 ? lane_xor<32>(sq[q]) : lane_xor<16>(sq[q]);
            op.ix[q >> 1] = face(kx[q], kx[q ^ 1], 1.0, sq[q ^ 1], true);
            op.iy[(q & 1) | ((q >> 1) & 2)] = face(ky[q], ky[q ^ 2], g.cy, sq[q ^ 2], true);
            op.iz[q & 3] = face(kz[q], kz[q ^ 4], g.cz, sq[q ^ 4], true);
            op.ox[q] = face(kx[q], nkx, 1.0, nsx, inx);
            op.oy[q] = face(ky[q], nky, g.cy, nsy, iny);
            op.oz[q] = face(kz[q], nkz, g.cz, nsz, inz);
            op.dg[q] = diag / S[q];
            rs = op.dg[q] + row;
            mx = fmax(mx, rs);
        }
        bnd = wave_max(mx);   // every wavefront holds the whole element
    }
    __syncthreads();
    // S^1/2 of the lane's cells, formed again where it is needed (16 registers
    // across the filter otherwise)
    auto roots = [&](const CubePos& cp, double (&sq)[8]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = phi_pos(cp.cell(q));
            sq[q] = sqrt(g.ortho ? weight(ke[c], ke[N + c], ke[2 * N + c]) : weight(ke[c], 0.0, 0.0));
        }
    };
    auto start = [&](int jj, bool predicted) {
        double v[8], sq[8];
        const unsigned char* md = kModes[jj];
        const CubePos cp(opaque(lane));
        roots(cp, sq);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = cp.cell(q);
            if (predicted && jj < kw) {
                v[q] = sq[q] * (double)warm[((size_t)blockIdx.x * kp + jj) * 512 + c];
            } else {
                const double m = ctab[8 * md[0] + (c & 7)] * ctab[8 * md[1] + ((c >> 3) & 7)] * ctab[8 * md[2] + (c >> 6)];
                v[q] = sq[q] * (m + 0.05 * hash_noise((unsigned)e, (unsigned)jj, (unsigned)c));
            }
        }
        cube_store(sh.Y, jj, lane, v);
    };
    const int need = (target + 4 < M - 2) ? target + 4 : M - 2;
    int cyc = -1, spent = 0;
    // one pass from the predicted start, one from the cold start
#pragma unroll 1
    for (int att = warm ? 0 : 1; att < 2 && cyc < 0; ++att) {
        if (att == 1 && warm) {
            spent = kWarmCycles + 1;
            if (threadIdx.x < 24)
                ctab[threadIdx.x] =
                    cos(3.14159265358979323846 / 8.0 * (double)(threadIdx.x >> 3) * ((threadIdx.x & 7) + 0.5));
            __syncthreads();
        }
#pragma unroll 1
        for (int j = w; j < M; j += NW) start(j, att == 0);
        __syncthreads();
        cyc = cube_chefsi<M, NW>(op, sh, w, lane, bnd, need, att == 0 ? ws_tol : tol, target, crtol, thr,
                                 att == 0 ? kWarmCycles : kMaxCycles, att == 0 ? kDeg : 0);
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
#pragma unroll 1
    for (int j = w; j < M; j += NW) {
        double x[8], ax[8];
        cube_load(sh.Y, j, lane, x);
        op.apply(x, ax);
        cube_dots<M>(sh.Y, j, lane, ax, sh.H);
        if (j >= L) continue;
        const CubePos cp(opaque(lane));
        double sq[8];
        roots(cp, sq);
        double s = x[0] * sq[0];
#pragma unroll
        for (int q = 1; q < 8; ++q) s += x[q] * sq[q];
        s = wave_sum(s);
        if (lane == 0) zc[(size_t)e * L + j] = j < nk ? s : 0.0;
        double* pj = phi + ((size_t)e * L + j) * 512;
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
            // slots q, q + 1 are the x pair (mirrored at even positions)
            const double va = j < nk ? x[q] / sq[q] : 0.0, vb = j < nk ? x[q + 1] / sq[q + 1] : 0.0;
            const bool flip = (cp.px & 1) == 0;
            *reinterpret_cast<double2*>(pj + phi_pos(cp.cell(q) & ~1)) = flip ? make_double2(vb, va) : make_double2(va, vb);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < L * L; t += blockDim.x) {
        const int a = t / L, b = t % L;
        Aint[(size_t)e * L * L + t] = (a < nk && b < nk) ? sh.H[a * M + b] : 0.0;
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
    constexpr int NW = 4;
    SPECMG_M_DISPATCH(nvec, hipLaunchKernelGGL((k_eig2<M, NW>), dim3(count), dim3(64 * NW), 0, s, g, kt, target, L,
                                               tol, crtol, phi, lam, nkeep, Aint, zc, status, e0, warm, kp, kw,
                                               ws_tol, ws_fb, thr));
}

}  // namespace specmg
