// Local eigensolves of the levels >= 3 (Section 3, eq. spectral cc): on every
// parent element E the restricted problem H_E v = lambda v with
// H_E = B_E^T A_E B_E assembled from the level below (its Gram is the identity
// for S-normalised bases), a block 7-point matrix over the kept slots of the
// agg^3 children, by Chebyshev-filtered subspace iteration (see the level-2
// solver; the filter has degree 40).
//
// One workgroup per parent.  The block of M columns lies in LDS, rows p LP + a
// (slot a of child p, padded slots zero).  An application of H_E, 40 a cycle, runs
// on the FP64 matrix cores, a child's rows a tile: v_mfma_f64_16x16x4 adds its four
// products to the sum one after the other, so a chain of them sums a row's entries
// in the order diagonal block, -x, +x, -y, +y, -z, +z, as a loop would.  A parent's
// operator is packed once, kept slots only, in the order of the products (P, terms
// t of child p: its blocks' kept columns); the wavefronts read it from L2, a child
// ahead, and keep the filter's last two iterates of their children in
// registers.  The Gram sums are those of the 64-row tiles (sum16), added in turn.
// All results equal to the last bit those of a row-a-thread form on the vector units,
// which took 9.1 ms for 64 parents of 576 rows x 12 vectors, 27.1 for 512 of 704 x 14,
// 40 for 4,096 of 72 x 16 and then 512 of 104 x 16, and 45 for 27 of 448 x 14: now
// 5.6, 10.2, 9.7 and 10.6.  Bound by the matrix cores' passes (16 x 16 tiles for some
// 6 x 12) and the latency of one workgroup a CU; up to 64 parents leave three quarters
// of the CUs idle.
#include <algorithm>

#include "eig_common.hpp"

namespace specmg {

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

// nonzero blocks of a parent's operator
__host__ __device__ constexpr int up_blocks(int agg) { return agg == 4 ? 64 + 2 * 144 : 8 + 2 * 12; }

template <int M, int NT, int AGG, int RT>
struct UpProblem {
    static constexpr int NW = NT / 64, NCH = AGG * AGG * AGG, CPW = NCH / NW;
    static constexpr int CT = (M + 15) / 16;      // column tiles of the matrix cores
    static constexpr int PT = M + 1;              // row pitch of the block (odd: rows spread over the banks)
    static constexpr int DR = AGG == 4 ? 3 : 4;   // result registers a tile: rows lk + 4 r (agg 4: widths up to 12)
    static constexpr int NE = M * (M + 1) / 2;
    static constexpr int GU = RT * CT == 1 ? 12 : 6, GX = 4;   // instructions of a child loaded ahead

    struct Shared {
        double G[M * M];
        double Q[M * M];
        double th[M], nrm[M], scr[2 * M];
        double fc[2 * kDegExact];
        double bound[NW];
        double ct[3 * 4];
        int iscr[M];
        int nk[NCH], elem[NCH];   // kept slots, lower-level element of child p
        int nt[NCH], nq[NCH];     // terms (kept columns of its blocks), and in fours
        int tb[NCH], pb[NCH];     // its first term, first entry of P
        int first[NCH + 1];       // compact index of its first row
    };

    Shared& sh;
    double* Y;                 // LDS: rows x PT
    double* red;               // LDS: tiles x NE
    unsigned short* term;      // LDS: row of Y that a term meets
    double* P;                 // workspace: entries, term by term
    double* AY;                // workspace: H_E Y, column by column
    int LP, n, w, lane;

    __device__ __forceinline__ int child(int ci) const { return w + NW * ci; }

    // direction d of child p inside the parent: its neighbour, or -1 (d < 0: the child itself)
    static __device__ __forceinline__ int neighbour(int p, int d) {
        if (d < 0) return p;
        constexpr int sh1 = AGG == 4 ? 2 : 1;
        const int ax = d >> 1, q = (p >> (sh1 * ax)) & (AGG - 1);
        const bool in = (d & 1) ? q < AGG - 1 : q > 0;
        return in ? ((d & 1) ? p + (1 << (sh1 * ax)) : p - (1 << (sh1 * ax))) : -1;
    }

    // the wavefront's children, in scalar registers
    struct Kids {
        int nk[CPW], nq[CPW], pb[CPW], tb[CPW];
    };
    __device__ __forceinline__ Kids kids() const {
        Kids k;
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci) {
            const int p = child(ci);
            k.nk[ci] = __builtin_amdgcn_readfirstlane(sh.nk[p]);
            k.nq[ci] = __builtin_amdgcn_readfirstlane(sh.nq[p]);
            k.pb[ci] = __builtin_amdgcn_readfirstlane(sh.pb[p]);
            k.tb[ci] = __builtin_amdgcn_readfirstlane(sh.tb[p]);
        }
        return k;
    }

    static __device__ __forceinline__ int again(int v) {
        asm volatile("" : "+s"(v));
        return v;
    }

    // use(ci, acc): acc = the rows of H_E Y of the wavefront's child ci (beyond its
    // kept slots: copies of the last one's).  Entries are on their way while the
    // child before is multiplied: GU instructions' of every child, and GX more of
    // those that have more.
    template <class F>
    __device__ __forceinline__ void apply(const Kids& k, F use) const {
        const int li = lane & 15, lk = lane >> 4;
        double a[2][GU][RT];
        // Addresses are formed anew each time (again): kept across the filter's loop they
        // would take all the registers.  Instructions beyond a child's last read what
        // follows (P: the next child or AY; terms: the next child or up_terms' zeros).
        auto fetch = [&](int ci, int q, double (&v)[RT]) {
            const int nk = again(k.nk[ci]);
            const char* e = (const char*)(P + (again(k.pb[ci]) + 4 * nk * q));
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                v[rt] = *(const double*)(e + (unsigned)(8 * (lk * nk + min(li + 16 * rt, nk - 1))));
        };
        auto columns = [&](int ci, int q, double (&y)[CT]) {
            const int row = term[again(k.tb[ci]) + 4 * q + lk];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) y[ct] = Y[row * PT + min(li + 16 * ct, M)];
        };
#pragma unroll
        for (int u = 0; u < GU; ++u) fetch(0, u, a[0][u]);
#pragma unroll
        for (int ci = 0; ci < CPW; ++ci) {
            const int nq = again(k.nq[ci]);
            if (ci + 1 < CPW) {
#pragma unroll
                for (int u = 0; u < GU; ++u) fetch(ci + 1, u, a[(ci + 1) & 1][u]);
            }
            double x[GX][RT];
            if (nq > GU) {
#pragma unroll
                for (int u = 0; u < GX; ++u) fetch(ci, GU + u, x[u]);
            }
            v4d acc[RT][CT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = v4d{0.0, 0.0, 0.0, 0.0};
            auto add = [&](const double (&v)[RT], const double (&y)[CT]) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[rt][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[rt], y[ct], acc[rt][ct], 0, 0, 0);
            };
            double y[GU][CT];
#pragma unroll
            for (int u = 0; u < GU; ++u) columns(ci, u, y[u]);
#pragma unroll
            for (int u = 0; u < GU; ++u)
                if (u < nq) add(a[ci & 1][u], y[u]);
            if (nq > GU) {
#pragma unroll
                for (int u = 0; u < GX; ++u) columns(ci, GU + u, y[u]);
#pragma unroll
                for (int u = 0; u < GX; ++u)
                    if (GU + u < nq) add(x[u], y[u]);
#pragma unroll 1
                for (int q = GU + GX; q < nq; ++q) {
                    fetch(ci, q, x[0]);
                    columns(ci, q, y[0]);
                    add(x[0], y[0]);
                }
            }
            use(ci, acc);
        }
    }

    // AY = H_E Y
    __device__ __forceinline__ void product(const Kids& k) const {
        const int li = lane & 15, lk = lane >> 4;
        apply(k, [&](int ci, const v4d (&acc)[RT][CT]) {
            const int p = child(ci), nk = again(k.nk[ci]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < DR; ++r) {
                        const int i = 16 * rt + lk + 4 * r, j = 16 * ct + li;
                        if (i < nk && j < M) AY[(size_t)j * n + p * LP + i] = acc[rt][ct][r];
                    }
        });
        __syncthreads();
    }

    // Chebyshev filter in place (factors sh.fc)
    __device__ __forceinline__ void filter(const Kids& k, double cc, int deg) const {
        const int li = lane & 15, lk = lane >> 4;
        double x[CPW][RT][CT][DR], y[CPW][RT][CT][DR];   // the last two iterates
        // f(ci, rt, ct, r, row of Y, column) for the lane's entries that exist
        auto entries = [&](auto f) {
            int at0 = (w * LP + lk) * PT + li;
            asm volatile("" : "+v"(at0));
#pragma unroll
            for (int ci = 0; ci < CPW; ++ci)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                        for (int r = 0; r < DR; ++r) {
                            const int i = 16 * rt + lk + 4 * r, j = 16 * ct + li;
                            f(ci, rt, ct, r, i < again(k.nk[ci]) && j < M, at0 + ci * NW * LP * PT + (16 * rt + 4 * r) * PT + 16 * ct);
                        }
        };
        entries([&](int ci, int rt, int ct, int r, bool in, int at) {
            x[ci][rt][ct][r] = 0.0;
            y[ci][rt][ct][r] = in ? Y[at] : 0.0;
        });
#pragma unroll 1
        for (int d = 0; d < deg; ++d) {
            const double f = sh.fc[2 * d], h = sh.fc[2 * d + 1];
            apply(k, [&](int ci, const v4d (&acc)[RT][CT]) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                        for (int r = 0; r < DR; ++r) {
                            const double v = y[ci][rt][ct][r];
                            y[ci][rt][ct][r] = fma(fma(-cc, v, acc[rt][ct][r]), f, -(h * x[ci][rt][ct][r]));
                            x[ci][rt][ct][r] = v;
                        }
            });
            __syncthreads();
            entries([&](int ci, int rt, int ct, int r, bool in, int at) {
                if (in) Y[at] = y[ci][rt][ct][r];
            });
            __syncthreads();
        }
    }

    // G = Y^T Y
    __device__ __forceinline__ void gram() const {
        constexpr Triangle<M> tri{};
#pragma unroll 1
        for (int t = w; 64 * t < n; t += NW) {
            const int row = 64 * t + lane;
            double y[M];
#pragma unroll
            for (int j = 0; j < M; ++j) y[j] = row < n ? Y[row * PT + j] : 0.0;
            tile_sums<NE>(red + t * NE, lane, [&](int e) { return fma(y[tri.i[e]], y[tri.j[e]], 0.0); });
        }
        __syncthreads();
        for (int e = threadIdx.x; e < NE; e += NT) {
            double s = 0.0;
            for (int t = 0; 64 * t < n; ++t) s += red[t * NE + e];
            int i = 0, r = e;   // row of entry e
            while (r >= M - i) r -= M - i++;
            sh.G[i * M + i + r] = s;
            sh.G[(i + r) * M + i] = s;
        }
        __syncthreads();
    }

    // G = the symmetric part of Y^T AY
    __device__ __forceinline__ void projected() const {
        constexpr int H = M / 2, HE = H * M;
#pragma unroll 1
        for (int j0 = 0; j0 < M; j0 += H) {   // half the columns at a time
#pragma unroll 1
            for (int t = w; 64 * t < n; t += NW) {
                const int row = 64 * t + lane;
                double b[H], y[M];
#pragma unroll
                for (int j = 0; j < H; ++j) b[j] = row < n ? AY[(size_t)(j0 + j) * n + row] : 0.0;
#pragma unroll
                for (int i = 0; i < M; ++i) y[i] = row < n ? Y[row * PT + i] : 0.0;
                tile_sums<HE>(red + t * NE, lane, [&](int e) { return fma(y[e % M], b[e / M], 0.0); });
            }
            __syncthreads();
            for (int e = threadIdx.x; e < HE; e += NT) {
                double s = 0.0;
                for (int t = 0; 64 * t < n; ++t) s += red[t * NE + e];
                sh.Q[(e % M) * M + j0 + e / M] = s;
            }
            __syncthreads();
        }
        for (int t = threadIdx.x; t < M * M; t += NT) {
            const int i = t / M, j = t % M;
            if (i > j) continue;
            const double v = 0.5 * (sh.Q[i * M + j] + sh.Q[j * M + i]);
            sh.G[i * M + j] = v;
            sh.G[j * M + i] = v;
        }
        __syncthreads();
    }

    // Y <- Y Q, a row a thread (TRI: Q upper triangular)
    template <bool TRI>
    __device__ __forceinline__ void multiply() const {
#pragma unroll 1
        for (int row = threadIdx.x; row < n; row += NT) {
            double s[M];
#pragma unroll
            for (int j = 0; j < M; ++j) s[j] = 0.0;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const double a = Y[row * PT + i];
#pragma unroll
                for (int j = TRI ? i : 0; j < M; ++j) s[j] = fma(a, sh.Q[i * M + j], s[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < M; ++j) Y[row * PT + j] = s[j];
        }
        __syncthreads();
    }

    // out[j] = the sum over all rows of value(row, j), rows in tiles of 64
    template <class V>
    __device__ __forceinline__ void column_sums(double* out, V value) const {
#pragma unroll 1
        for (int t = w; 64 * t < n; t += NW) {
            const int row = 64 * t + lane;
            tile_sums<M>(red + t * NE, lane, [&](int j) { return row < n ? value(row, j) : 0.0; });
        }
        __syncthreads();
        if (threadIdx.x < M) {
            double s = 0.0;
            for (int t = 0; 64 * t < n; ++t) s += red[t * NE + threadIdx.x];
            out[threadIdx.x] = s;
        }
        __syncthreads();
    }
};

// terms of a parent's children at most (each child's filled up to fours), and 64
// zeros beyond the last one's
__host__ __device__ constexpr int up_terms(int agg, int lp) { return up_blocks(agg) * lp + 3 * agg * agg * agg + 64; }

// doubles of one workspace slot: P and AY
static size_t up_slot_doubles(int agg, int lp, int M) {
    return (size_t)up_terms(agg, lp) * lp + (size_t)M * agg * agg * agg * lp;
}

template <int M, int NT, int AGG, int RT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(AGG == 4 || M > 16 ? 2 : 3))) void k_eig_up(
    CoarseGeom lo, CoarseGeom up, const double* __restrict__ Hd, const double* __restrict__ Aoff,
    const int* __restrict__ nkeep_lo, const double* __restrict__ zlo, int target, double tol, double crtol, double thr,
    double* __restrict__ V, double* __restrict__ lam, int* __restrict__ nkeep, double* __restrict__ Aint,
    double* __restrict__ zup, int* __restrict__ status, double* work, size_t slot) {
    typedef UpProblem<M, NT, AGG, RT> UP;
    constexpr int NCH = UP::NCH, PT = UP::PT;
    extern __shared__ __align__(16) double dyn[];
    __shared__ typename UP::Shared sh;
    const int Lu = up.L, LP = lo.L, n = NCH * LP, tiles = (n + 63) / 64;
    const int lane = threadIdx.x & 63;
    double* red = dyn + (size_t)n * PT;
    double* ws = work + (size_t)blockIdx.x * slot;
    const UP pr{sh, dyn, red, (unsigned short*)(red + (size_t)tiles * UP::NE), ws,
                ws + (size_t)up_terms(AGG, LP) * LP, LP, n, __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane};
    // one-dimensional factors cos(pi p (q + 1/2) / agg) of the start modes
    if (threadIdx.x < 12)
        sh.ct[threadIdx.x] =
            cos(3.14159265358979323846 / AGG * (double)(threadIdx.x >> 2) * ((threadIdx.x & 3) + 0.5));
#pragma unroll 1
    for (int E = blockIdx.x; E < up.m; E += gridDim.x) {
        const int Ex = E % up.mx, Ey = (E / up.mx) % up.my, Ez = E / (up.mx * up.my);
        __syncthreads();
        // children, one per lane: kept slots, terms, and where their entries start
        if (threadIdx.x < 64) {
            int k = 0;
            if (lane < NCH) {
                const int c = (Ex * AGG + lane % AGG) +
                              lo.mx * ((Ey * AGG + (lane / AGG) % AGG) + lo.my * (Ez * AGG + lane / (AGG * AGG)));
                sh.elem[lane] = c;
                k = nkeep_lo[c];
                sh.nk[lane] = k;
            }
            wave_sync();
            int nt = 0;
            if (lane < NCH)
                for (int d = -1; d < 6; ++d) {
                    const int pn = UP::neighbour(lane, d);
                    if (pn >= 0) nt += sh.nk[pn];
                }
            const int nq = (nt + 3) / 4;   // the last four filled up with zeros
            int s0 = k, s1 = 4 * nq, s2 = 4 * nq * k;
            for (int off = 1; off < 64; off <<= 1) {
                const int a = __shfl_up(s0, off, 64), b = __shfl_up(s1, off, 64), c = __shfl_up(s2, off, 64);
                if (lane >= off) {
                    s0 += a;
                    s1 += b;
                    s2 += c;
                }
            }
            if (lane < NCH) {
                sh.nt[lane] = nt;
                sh.nq[lane] = nq;
                sh.first[lane] = s0 - k;
                sh.tb[lane] = s1 - 4 * nq;
                sh.pb[lane] = s2 - 4 * nq * k;
                if (lane == NCH - 1) sh.first[NCH] = s0;
            }
        }
        __syncthreads();
        const int nval = sh.first[NCH];
        // the operator, term by term
#pragma unroll 1
        for (int p = pr.w; p < NCH; p += UP::NW) {
            const int nk = sh.nk[p], c = sh.elem[p];
            double* e = pr.P + sh.pb[p];
            unsigned short* tr = pr.term + sh.tb[p];
            int t0 = 0;
#pragma unroll 1
            for (int d = -1; d < 6; ++d) {
                const int pn = UP::neighbour(p, d);
                if (pn < 0) continue;
                const int kn = sh.nk[pn], cn = sh.elem[pn], ax = d >> 1;
                // + direction: A(c, cn)[a][b] = Aoff[c][ax][a][b]; - direction: Aoff[cn][ax][b][a]
                const double* A = d < 0 ? Hd + (size_t)c * LP * LP
                                        : Aoff + ((size_t)((d & 1) ? c : cn) * 3 + ax) * LP * LP;
                const int sa = d < 0 || (d & 1) ? LP : 1, sb = d < 0 || (d & 1) ? 1 : LP;
                for (int x = lane; x < kn * nk; x += 64) {
                    const int b = x / nk, a = x - b * nk;
                    e[(t0 + b) * nk + a] = A[a * sa + b * sb];
                }
                for (int b = lane; b < kn; b += 64) tr[t0 + b] = (unsigned short)(pn * LP + b);
                t0 += kn;
            }
            for (; t0 < 4 * sh.nq[p]; ++t0) {
                if (lane < nk) e[t0 * nk + lane] = 0.0;
                if (lane == 0) tr[t0] = 0;
            }
        }
        for (int t = threadIdx.x; t < n * M; t += NT) pr.AY[t] = 0.0;
        if (threadIdx.x < 64) pr.term[sh.tb[NCH - 1] + 4 * sh.nq[NCH - 1] + threadIdx.x] = 0;
        __syncthreads();
        const typename UP::Kids kids = pr.kids();
        // Gershgorin bound (absolute row sums) and the largest constant coefficient
        double rs = 0.0, az = 0.0;
        for (int r = threadIdx.x; r < n; r += NT) {
            const int p = r / LP, a = r - p * LP, nk = sh.nk[p];
            if (a >= nk) continue;
            const double* e = pr.P + sh.pb[p] + a;
            double s = 0.0;
            for (int t = 0; t < sh.nt[p]; ++t) s += fabs(e[t * nk]);
            rs = fmax(rs, s);
            az = fmax(az, fabs(zlo[(size_t)sh.elem[p] * LP + a]));
        }
        auto block_max = [&](double v) {
            v = wave_max(v);
            __syncthreads();
            if (lane == 0) sh.bound[threadIdx.x >> 6] = v;
            __syncthreads();
            double t = sh.bound[0];
            for (int i = 1; i < UP::NW; ++i) t = fmax(t, sh.bound[i]);
            return t;
        };
        const double bnd = block_max(rs);
        az = 0.05 * (block_max(az) + 1e-300);
        pin_value(az);
        // Start block: unit vectors when the block can hold the whole space (one
        // Rayleigh-Ritz step is then exact); else the constant function, smooth
        // weights of the children's constant modes, and noise on every kept slot.
        // The noise has one amplitude for the whole element: the constant
        // function's coefficient vanishes on the children's non-constant slots,
        // and noise scaled by it would leave the block without those directions,
        // which a polynomial filter cannot restore.
        const bool whole = nval <= M;
        for (int t = threadIdx.x; t < n * M; t += NT) {
            const int r = t / M, j = t - r * M;
            const int p = r / LP, a = r - p * LP;
            double v = 0.0;
            if (a < sh.nk[p]) {
                if (whole) {
                    v = sh.first[p] + a == j ? 1.0 : 0.0;
                } else {
                    const double z = zlo[(size_t)sh.elem[p] * LP + a];
                    v = az * hash_noise((unsigned)E + 77u, (unsigned)j, (unsigned)r);
                    pin_value(v);
                    if (j == 0) v = z;
                    else if (a == 0) {
                        const unsigned char* md = kModes[j & 15];
                        constexpr int s1 = AGG == 4 ? 2 : 1;
                        const double m = z * sh.ct[4 * md[0] + (p & (AGG - 1))] * sh.ct[4 * md[1] + ((p >> s1) & (AGG - 1))];
                        v = fma(m, sh.ct[4 * md[2] + (p >> (2 * s1))], v);
                    }
                }
            }
            pr.Y[r * PT + j] = v;
            if (j == 0) pr.Y[r * PT + M] = 0.0;   // the pitch's last word meets the unused columns of a tile
        }
        __syncthreads();
        const int need = (target + 4 < M - 2) ? target + 4 : M - 2;
        double below = 1e-3 * bnd;
        pin_value(below);
        int cyc = 0;
#pragma unroll 1
        for (;; ++cyc) {
            // an orthonormal basis (Cholesky-QR, twice)
            if (!whole) {
#pragma unroll 1
                for (int pass = 0; pass < 2; ++pass) {
                    pr.gram();
                    if (threadIdx.x < 64) cholesky_call<M>((lds_double*)sh.G, (lds_double*)sh.Q);
                    __syncthreads();
                    pr.template multiply<true>();
                }
            }
            // Rayleigh-Ritz: Y becomes the Ritz vectors, AY their images, th the values
#pragma unroll 1
            for (int h = 0; h < 2; ++h) {
                pr.product(kids);
                if (h) break;
                pr.projected();
                // the columns of Y beyond the space are zero: their values lie above the
                // spectrum, so that they sort last and their Ritz vectors stay zero
                if (whole && (int)threadIdx.x < M && (int)threadIdx.x >= nval)
                    sh.G[threadIdx.x * M + threadIdx.x] = fma(2.0, bnd, 1.0);
                __syncthreads();
                if (threadIdx.x < 64)
                    jacobi_call<M>((lds_double*)sh.G, (lds_double*)sh.Q, (lds_double*)sh.th, (lds_double*)sh.scr,
                                   (lds_int*)sh.iscr);
                __syncthreads();
                pr.template multiply<false>();
            }
            if (whole) break;
            const double a = fmin(sh.th[M - 1], 0.5 * bnd);
            if (threadIdx.x == NT - 1) filter_factors(sh.fc, a, bnd, fmin(sh.th[0], 0.0) - below, kDegExact);
            pr.column_sums(sh.nrm, [&](int r, int j) {
                const double d = fma(-sh.th[j], pr.Y[r * PT + j], pr.AY[(size_t)j * n + r]);
                return fma(d, d, 0.0);
            });
            if (chefsi_done(sh.th, sh.nrm, M, need, tol, bnd, target, crtol, thr, cyc)) break;
            if (cyc >= kMaxCycles) {
                cyc = -1;
                break;
            }
            pr.filter(kids, 0.5 * (bnd + a), kDegExact);
        }
        const int nk = cluster_cut_dev(sh.th, nval < M ? nval : M, target, crtol, thr);
        if (threadIdx.x == 0) {
            nkeep[E] = nk;
            status[E] = cyc;
            for (int b = 0; b < Lu; ++b) lam[(size_t)E * Lu + b] = b < nval ? sh.th[b] : 0.0;
        }
        // V^T H_E V on the kept vectors, the constant function's coefficients, V
        pr.projected();
        for (int t = threadIdx.x; t < Lu * Lu; t += NT) {
            const int i = t / Lu, j = t % Lu;
            Aint[(size_t)E * Lu * Lu + t] = (i < nk && j < nk) ? sh.G[i * M + j] : 0.0;
        }
        pr.column_sums(sh.nrm, [&](int r, int j) {
            const int p = r / LP, a = r - p * LP;
            const double z = a < sh.nk[p] ? zlo[(size_t)sh.elem[p] * LP + a] : 0.0;
            return fma(pr.Y[r * PT + j], z, 0.0);
        });
        for (int j = threadIdx.x; j < Lu; j += NT) zup[(size_t)E * Lu + j] = j < nk ? sh.nrm[j] : 0.0;
        for (int t = threadIdx.x; t < Lu * n; t += NT) {
            const int j = t / n, r = t - j * n;
            V[((size_t)E * Lu + j) * n + r] = j < nk ? pr.Y[r * PT + j] : 0.0;
        }
    }
}

// ---------------------------------------------------------------------------
// launcher

// workgroups of one launch, each with its own workspace slot: one per parent up to
// what the chip holds (LDS: one workgroup of 4^3 children per CU, up to six of 2^3)
static int up_slots(const CoarseGeom& up, int agg) { return std::min(up.m, agg == 4 ? 256 : 1536); }

size_t eig_up_work_doubles(const CoarseGeom& lo, const CoarseGeom& up, int nvec) {
    return (size_t)up_slots(up, lo.agg) * up_slot_doubles(lo.agg, lo.L, nvec);
}

// bytes of dynamic LDS: the block, the tiles' sums, the terms' rows
constexpr size_t up_lds(int agg, int lp, int M) {
    const size_t n = (size_t)agg * agg * agg * lp, tiles = (n + 63) / 64;
    return (n * (M + 1) + tiles * (M * (M + 1) / 2)) * sizeof(double) + (size_t)up_terms(agg, lp) * 2;
}

// the widest lower levels that set-up lets through, block by block, fit a CU's 160 KB
template <int M, int NT, int AGG, int RT>
constexpr bool up_fits(int lp) {
    return up_lds(AGG, lp, M) + sizeof(typename UpProblem<M, NT, AGG, RT>::Shared) <= 163840;
}
static_assert(up_fits<10, 512, 4, 1>(eig_up_widest(4, 10)) && up_fits<12, 512, 4, 1>(eig_up_widest(4, 12)) &&
              up_fits<14, 512, 4, 1>(eig_up_widest(4, 14)) && up_fits<16, 512, 4, 1>(eig_up_widest(4, 16)) &&
              up_fits<20, 512, 4, 1>(eig_up_widest(4, 20)) && up_fits<26, 512, 4, 1>(eig_up_widest(4, 26)) &&
              up_fits<26, 256, 2, 2>(eig_up_widest(2, 26)), "LDS of the upper levels' eigensolver");

void launch_eig_up(const CoarseGeom& lo, const CoarseGeom& up, const double* Aint_lo, const double* Dlo,
                   const double* Aofflo, const int* nkeep_lo, const double* zlo, double* Hd_work, double* work,
                   int target, int nvec, double tol, double crtol, double thr, double* V, double* lam, int* nkeep,
                   double* Aint, double* zup, int* status, hipStream_t s) {
    hipLaunchKernelGGL(k_build_hd, dim3(lo.m), dim3(128), 0, s, lo, Aint_lo, Dlo, Hd_work);
    if (up.L != target + 3 || (lo.agg != 2 && lo.agg != 4) || lo.L > eig_up_widest(lo.agg, nvec) || target < 1 ||
        target > 20 || nvec < target + 6)
        throw HipError{hipErrorInvalidValue, "eig_up shape"};
    const size_t slot = up_slot_doubles(lo.agg, lo.L, nvec), shmem = up_lds(lo.agg, lo.L, nvec);
#define SPECMG_EIG_UP_AS(MV, NTV, AGGV, RTV)                                                                      \
    {                                                                                                             \
        hipError_t e = hipFuncSetAttribute((const void*)k_eig_up<MV, NTV, AGGV, RTV>,                              \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);               \
        if (e == hipSuccess) {                                                                                    \
            hipLaunchKernelGGL((k_eig_up<MV, NTV, AGGV, RTV>), dim3(up_slots(up, lo.agg)), dim3(NTV), shmem, s, lo, \
                               up, Hd_work, Aofflo, nkeep_lo, zlo, target, tol, crtol, thr, V, lam, nkeep, Aint,   \
                               zup, status, work, slot);                                                          \
            e = hipGetLastError();                                                                                \
        }                                                                                                         \
        if (e != hipSuccess) throw HipError{e, "eig_up launch"};                                                  \
        return;                                                                                                   \
    }
#define SPECMG_EIG_UP(MV)                                                            \
    case MV:                                                                         \
        if (lo.agg == 4) SPECMG_EIG_UP_AS(MV, 512, 4, 1)                             \
        else if (lo.L <= 16) SPECMG_EIG_UP_AS(MV, (MV <= 16 ? 128 : 256), 2, 1)      \
        else SPECMG_EIG_UP_AS((MV <= 16 ? 20 : MV), 256, 2, 2)   /* (blocks up to 16: refused above) */
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
#undef SPECMG_EIG_UP_AS
    throw HipError{hipErrorInvalidValue, "eig_up block size"};
}

}  // namespace specmg
