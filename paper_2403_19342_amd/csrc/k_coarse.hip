// Coarse levels of the V-cycle (Algorithm 1 steps 3-7, applied recursively)
// and their set-up.
//
// A coarse level l >= 2 has one block of L (padded) unknowns per element;
// its Galerkin operator A_l = R_l A_{l-1} R_l^T (text above Algorithm 1) is
// a block 7-point stencil stored as
//   Ad[e]        diagonal block  (L x L)
//   Aoff[e][d]   coupling A_l(e, e + unit vector d), d = x, y, z (L x L)
// The level-l smoother is one block-Jacobi sweep whose blocks are the
// level-(l+1) parent elements, each factored by block IC(0) over its agg^3
// children in lexicographic order (Section 5): pivots
//   D_c = Ad_c - sum_{lower neighbour c'} A(c, c') D_c'^{-1} A(c', c),
// stored inverted in Dinv.  Padded slots carry an identity pivot and zero
// couplings, so they stay zero.  For the substitutions the set-up also forms
//   G[c][2 ax]     = D_c^{-1} A(c, c - e_ax)   (lower neighbour, same parent)
//   G[c][2 ax + 1] = D_c^{-1} A(c, c + e_ax)   (upper neighbour, same parent)
// so that every hyperplane step is a single product:
//   forward   y_c = D_c^{-1} r_c - sum_lower G y_c'
//   backward  z_c = y_c - sum_upper G z_c''.
#include <vector>

#include "common.hpp"

namespace specmg {

__device__ __forceinline__ int log2_agg(int agg) { return agg == 4 ? 2 : 1; }

// level-l index of the child at position p (lexicographic in the parent) of
// parent E; agg is 2 or 4, so positions decode with shifts
__device__ __forceinline__ int child_of(const CoarseGeom& g, int E, int p) {
    const int a = g.agg, sh = log2_agg(a);
    const int Ex = E % g.px, Ey = (E / g.px) % g.py, Ez = E / (g.px * g.py);
    const int qx = p & (a - 1), qy = (p >> sh) & (a - 1), qz = p >> (2 * sh);
    return (Ex * a + qx) + g.mx * ((Ey * a + qy) + g.my * (Ez * a + qz));
}

// children positions sorted by qx+qy+qz for agg = 2 and agg = 4
struct ChildPlanes {
    unsigned char pos2[8], off2[5], rank2[8];
    unsigned char pos4[64], off4[11], rank4[64];
};

constexpr ChildPlanes make_child_planes() {
    ChildPlanes t{};
    int k = 0;
    for (int s = 0; s <= 3; ++s) {
        t.off2[s] = (unsigned char)k;
        for (int p = 0; p < 8; ++p)
            if ((p & 1) + ((p >> 1) & 1) + (p >> 2) == s) t.pos2[k++] = (unsigned char)p;
    }
    t.off2[4] = (unsigned char)k;
    k = 0;
    for (int s = 0; s <= 9; ++s) {
        t.off4[s] = (unsigned char)k;
        for (int p = 0; p < 64; ++p)
            if ((p & 3) + ((p >> 2) & 3) + (p >> 4) == s) t.pos4[k++] = (unsigned char)p;
    }
    t.off4[10] = (unsigned char)k;
    for (int i = 0; i < 8; ++i) t.rank2[t.pos2[i]] = (unsigned char)i;
    for (int i = 0; i < 64; ++i) t.rank4[t.pos4[i]] = (unsigned char)i;
    return t;
}

__constant__ ChildPlanes kCP = make_child_planes();

// positions of the agg^3 children sorted by qx+qy+qz, copied into LDS
__device__ void build_planes(int agg, int* pos, int* off) {
    const int nc = agg * agg * agg, np = 3 * (agg - 1) + 2;
    for (int t = threadIdx.x; t < nc; t += blockDim.x) pos[t] = agg == 4 ? kCP.pos4[t] : kCP.pos2[t];
    for (int t = threadIdx.x; t < np; t += blockDim.x) off[t] = agg == 4 ? kCP.off4[t] : kCP.off2[t];
    __syncthreads();
}

constexpr int kMaxLc = 23;   // padded widths up to target 20 + 3 (levels >= 3)
constexpr int kNarrow = 13;  // widths up to target 10 + 3 get their own instantiations

// y_c = (A_l u)_c for row a of child element c: the diagonal block (its row,
// which neighbouring threads read side by side from the transposed copy AdT),
// then both coupling blocks of each axis (at the domain boundary from valid
// stand-in rows of the element itself, whose sums a select then drops).  The
// order of the sums is part of the result (on media of contrast 1e6 the last bit
// of a pressure shows in the face fluxes): in a sweep (SWEEP) the two sums of an
// axis first; in a residual to be restricted one after the other, at widths above
// 9 entry by entry onto the row's sum.  ALL: every load of the row is in flight at
// once, one wait for memory, for launches that leave the chip idle; otherwise one
// axis at a time, four waits but half the registers.
template <typename T, int LP, bool ALL, bool SWEEP>
__device__ __forceinline__ T block_row_apply(const CoarseGeom& g, const T* __restrict__ AdT,
                                             const T* __restrict__ Aoff, const T* __restrict__ u, int c,
                                             int a) {
    constexpr bool RT = LP == kMaxLc;   // the widest serves every width above kNarrow
    const int W = RT ? g.L : LP;
    const int cx = c % g.mx, cy = (c / g.mx) % g.my, cz = c / (g.mx * g.my);
    T acc = T(0);
    {
        const T* ad = AdT + (size_t)c * W * W + a;
        const T* uc = u + (size_t)c * W;
#pragma unroll
        for (int b = 0; b < LP; ++b)
            if (!RT || b < W) acc += ad[b * W] * uc[b];
    }
    auto axis = [&](int ax) {
        const int cca = ax == 0 ? cx : (ax == 1 ? cy : cz);
        const int exa = ax == 0 ? g.mx : (ax == 1 ? g.my : g.mz);
        const int sta = ax == 0 ? 1 : (ax == 1 ? g.mx : g.mx * g.my);
        const bool hp = cca + 1 < exa, hm = cca > 0;
        const int cp = hp ? c + sta : c, cm = hm ? c - sta : c;
        // A(c, c+e) = Aoff[c][ax]; A(c, c-e) = Aoff[c-e][ax]^T
        const T* op = Aoff + (((size_t)c * 3 + ax) * W + a) * W;
        const T* om = Aoff + ((size_t)cm * 3 + ax) * W * W + a;
        const T* up = u + (size_t)cp * W;
        const T* um = u + (size_t)cm * W;
        if constexpr (SWEEP || LP <= 9) {
            T sp = T(0), sm = T(0);
#pragma unroll
            for (int b = 0; b < LP; ++b) {
                if (RT && b >= W) continue;
                sp += op[b] * up[b];
                sm += om[b * W] * um[b];
            }
            sp = hp ? sp : T(0);
            sm = hm ? sm : T(0);
            if constexpr (SWEEP) {
                acc += sp + sm;
            } else {
                acc += sp;
                acc += sm;
            }
        } else {
            T t = acc;
#pragma unroll
            for (int b = 0; b < LP; ++b)
                if (!RT || b < W) t += op[b] * up[b];
            acc = hp ? t : acc;
            t = acc;
#pragma unroll
            for (int b = 0; b < LP; ++b)
                if (!RT || b < W) t += om[b * W] * um[b];
            acc = hm ? t : acc;
        }
    };
    if constexpr (ALL && !RT) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) axis(ax);
    } else {
#pragma unroll 1
        for (int ax = 0; ax < 3; ++ax) axis(ax);
    }
    return acc;
}

constexpr int kCoarseThreads = 1024;   // upper bound; launches use agg^3 L rounded to waves
constexpr int kMaxChildren = 64;   // agg <= 4
constexpr int kMaxParts = 12;      // parts of a parent's restricted residual (agg 4: up to its width)
constexpr int kMaxL = kMaxLc;      // set-up arrays of the levels >= 3
constexpr int kMaxL2 = 16;         // level 2 (target <= 10)

// ---- the residual's row, u staged in LDS ------------------------------------
// The sweep's workgroup (agg 4) keeps u of its parent's children and of the
// children across the parent's faces in LDS: 64 blocks in hyperplane order (as
// the rows of the sweep), then face d = 2 ax (below) or 2 ax + 1 (above), 16
// blocks each; beyond the domain zeros, so the products need no test.  The
// rows of A are then the only loads of a row from memory.
constexpr int kHaloBlocks = 160;

template <typename T, int LP>
__device__ __forceinline__ void stage_u(const CoarseGeom& g, const T* __restrict__ u, int E, T* sU) {
    const int x0 = E % g.px * 4, y0 = E / g.px % g.py * 4, z0 = E / (g.px * g.py) * 4;
    for (int t = threadIdx.x; t < kHaloBlocks * LP; t += blockDim.x) {
        const int h = t / LP, b = t - h * LP;
        int x, y, z;
        if (h < 64) {
            const int p = kCP.pos4[h];
            x = x0 + (p & 3);
            y = y0 + ((p >> 2) & 3);
            z = z0 + (p >> 4);
        } else {
            const int d = (h - 64) >> 4, ax = d >> 1, i = h & 3, j = (h >> 2) & 3, o = (d & 1) ? 4 : -1;
            x = x0 + (ax == 0 ? o : i);
            y = y0 + (ax == 1 ? o : (ax == 0 ? i : j));
            z = z0 + (ax == 2 ? o : j);
        }
        const bool in = x >= 0 && x < g.mx && y >= 0 && y < g.my && z >= 0 && z < g.mz;
        sU[t] = in ? u[(size_t)(x + g.mx * (y + g.my * z)) * LP + b] : T(0);
    }
}

// Row a of child c at hyperplane rank k, position pos of its parent: the loads
// of A, then (after the barrier that publishes sU) the products.  The diagonal
// block and FIRST axes are loaded at once, as many as the registers of a
// workgroup hold (up to width 8 it has 256 a thread, wider ones 168), the
// other axes in turn.
template <typename T, int LP, int FIRST = LP <= 8 ? 3 : 1>
struct ResidRow {
    T ad[LP], op[FIRST][LP], om[FIRST][LP];

    struct Place {
        int c, a, k, qx, qy, qz, cx, cy, cz;
    };

    __device__ static __forceinline__ Place place(const CoarseGeom& g, int c, int a, int k, int pos) {
        return {c, a, k, pos & 3, (pos >> 2) & 3, pos >> 4, c % g.mx, (c / g.mx) % g.my, c / (g.mx * g.my)};
    }
    // row a of A(c, c) from the transposed copy, where neighbouring rows lie side by
    // side; A(c, c+e) = Aoff[c][ax], A(c, c-e) = Aoff[c-e][ax]^T, beyond the domain
    // any block of the array, against zeros
    __device__ static __forceinline__ const T* above_row(const Place& p, const T* Aoff, int ax) {
        return Aoff + (((size_t)p.c * 3 + ax) * LP + p.a) * LP;
    }
    __device__ static __forceinline__ const T* below_col(const CoarseGeom& g, const Place& p, const T* Aoff, int ax) {
        const int st = ax == 0 ? 1 : (ax == 1 ? g.mx : g.mx * g.my);
        const int x = ax == 0 ? p.cx : (ax == 1 ? p.cy : p.cz);
        return Aoff + ((size_t)(x > 0 ? p.c - st : p.c) * 3 + ax) * LP * LP + p.a;
    }
    // block of sU next to p, above (up) or below along ax
    __device__ static __forceinline__ int block(const Place& p, int ax, bool up) {
        const int x = ax == 0 ? p.qx : (ax == 1 ? p.qy : p.qz);
        const bool in = up ? x < 3 : x > 0;
        const int pos = p.qx | (p.qy << 2) | (p.qz << 4), st = 1 << (2 * ax);
        const int i = ax == 0 ? p.qy : p.qx, j = ax == 2 ? p.qy : p.qz;
        return in ? kCP.rank4[up ? pos + st : pos - st] : 64 + ((2 * ax + (up ? 1 : 0)) << 4) + i + (j << 2);
    }
    __device__ __forceinline__ void load(const CoarseGeom& g, const Place& p, const T* __restrict__ AdT,
                                         const T* __restrict__ Aoff) {
#pragma unroll
        for (int b = 0; b < LP; ++b) ad[b] = AdT[((size_t)p.c * LP + b) * LP + p.a];
#pragma unroll
        for (int ax = 0; ax < FIRST; ++ax) {
            const T* po = above_row(p, Aoff, ax);
            const T* pm = below_col(g, p, Aoff, ax);
#pragma unroll
            for (int b = 0; b < LP; ++b) {
                op[ax][b] = po[b];
                om[ax][b] = pm[b * LP];
            }
        }
    }
    __device__ __forceinline__ T apply(const CoarseGeom& g, const Place& p, const T* __restrict__ Aoff,
                                       const T* sU) const {
        T acc = T(0);
#pragma unroll
        for (int b = 0; b < LP; ++b) acc += ad[b] * sU[p.k * LP + b];
#pragma unroll
        for (int ax = 0; ax < FIRST; ++ax) {
            const T* up = sU + block(p, ax, true) * LP;
            const T* um = sU + block(p, ax, false) * LP;
            T sp = T(0), sm = T(0);
#pragma unroll
            for (int b = 0; b < LP; ++b) {
                sp += op[ax][b] * up[b];
                sm += om[ax][b] * um[b];
            }
            acc += sp + sm;
        }
        if constexpr (FIRST < 3) __builtin_amdgcn_sched_barrier(0);   // the rest's loads stay behind: registers
#pragma unroll 1
        for (int ax = FIRST; ax < 3; ++ax) {
            const T* po = above_row(p, Aoff, ax);
            const T* pm = below_col(g, p, Aoff, ax);
            const T* up = sU + block(p, ax, true) * LP;
            const T* um = sU + block(p, ax, false) * LP;
            T sp = T(0), sm = T(0);
#pragma unroll
            for (int b = 0; b < LP; ++b) {
                sp += po[b] * up[b];
                sm += pm[b * LP] * um[b];
            }
            acc += sp + sm;
        }
        return acc;
    }
};

// value of a level vector that arrives in nparts parts, pstride apart: all loaded
// at once, added in order
template <typename T>
__device__ __forceinline__ T gather_parts(const T* r, int nparts, int64_t pstride) {
    T v = r[0];
    if (nparts > 1) {
        T w[kMaxParts - 1];
#pragma unroll
        for (int i = 1; i < kMaxParts; ++i) w[i - 1] = r[(i < nparts ? i : 0) * pstride];
#pragma unroll
        for (int i = 1; i < kMaxParts; ++i) v = i < nparts ? v + w[i - 1] : v;
    }
    return v;
}

// parents of one sweep workgroup: with 2x aggregation as many as fill about 512
// threads (a parent has 8 W rows), otherwise one
constexpr int sweep_parents(int agg, int W) {
    return agg != 2 ? 1 : (512 / (8 * W) < 1 ? 1 : (512 / (8 * W) > kMaxChildren / 8 ? kMaxChildren / 8 : 512 / (8 * W)));
}

// Level-l smoother on parent E, both substitutions in one kernel:
//   t = r (mode 0) or t = r - A_l u (mode 1)
//   w = D^-1 t per child; y = forward substitution, z = backward substitution
//   out = z (mode 0) or out = u + z (mode 1)
// One thread per row (child, slot) with the children in hyperplane order, so
// the rows of plane s are threads [off[s] W, off[s+1] W).  Each thread keeps
// the rows of its lower and upper couplings G in registers; only y lives in
// LDS.  A plane step is one LDS read per coupling entry, the products, a store
// and a barrier.  Missing neighbours read the thread's own child with weight 0.
// SM holds D^-1 and the couplings as the threads read them: per parent the
// matrices d (0: D^-1; agg 4: 1 + 2 ax below, 2 + 2 ax above; agg 2, where a
// child has one sibling along an axis: 1 + ax), each column b of all the rows
// side by side.
// With few parents the time of a workgroup is a chain: at 64 parents of 64 x 9
// rows the rows' arrival (0.3 MB a CU at 20 to 30 bytes a clock) takes 14k
// clocks of 32k, the 20 plane steps 11.5k (LDS reads), in mode 1 the residual
// 15k more.  With rows read from row-major blocks, one axis at a time, mode 0
// took 16.2 us and mode 1 19.1; now 13.0 and 17.6 (64 parents of 64 x 9); the two
// together 23.2 us before and after with 27 of 64 x 7, 111 and 112 with 512 of 64 x 11.
template <typename T, int LP, bool A2, int MODE>
__global__ __launch_bounds__(A2 ? 512 : 64 * LP) void k_coarse_sweep(
    CoarseGeom g, const T* __restrict__ AdT, const T* __restrict__ Aoff, const T* __restrict__ SM,
    T* __restrict__ r, const T* u, T* out, const Scalars* sc, int check_done, int npar, int nparts) {
    if (check_done && sc->done) return;
    // row width: LP, except in the widest instantiation, which serves every
    // width above kNarrow (entries b >= W are neither read nor written)
    constexpr bool RT = LP == kMaxLc;
    constexpr int MAXP = sweep_parents(A2 ? 2 : 4, RT ? kNarrow + 1 : LP);
    __shared__ T sY[MAXP * (A2 ? 8 : 64) * LP];
    __shared__ T sU[MODE && !A2 ? kHaloBlocks * LP : 1];
    const int W = RT ? g.L : LP;
    constexpr int agg = A2 ? 2 : 4, nc = agg * agg * agg, sh = A2 ? 1 : 2;
    constexpr int nplanes = 3 * (agg - 1) + 1;
    // npar parents per workgroup (several when a parent has few rows, so
    // that the wavefronts are full), each with its own nc * W rows of sY
    const int per = nc * W;
    const int t = threadIdx.x, qp = t / per, tt = t - qp * per;
    const int E = blockIdx.x * npar + qp;
    const bool row_ok = qp < npar && E < g.M;
    const int base = row_ok ? qp * per : 0;
    const int k = row_ok ? tt / W : 0, a = tt % W;
    const int p = A2 ? kCP.pos2[k] : kCP.pos4[k];
    const int q[3] = {p & (agg - 1), (p >> sh) & (agg - 1), p >> (2 * sh)};
    const int plane = q[0] + q[1] + q[2];
    const int c = child_of(g, row_ok ? E : 0, p);
    // neighbour rows in LDS and weights per direction (lower: 2 ax, upper: 2 ax + 1)
    int nb[6];
    T wgt[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const int ax = d >> 1;
        const bool in = (d & 1) ? (q[ax] < agg - 1) : (q[ax] > 0);
        const int step = 1 << (sh * ax);
        const int pn = in ? ((d & 1) ? p + step : p - step) : p;
        nb[d] = base + (A2 ? kCP.rank2[pn] : kCP.rank4[pn]) * W;
        wgt[d] = in ? T(1) : T(0);
    }
    // slots beyond the child's kept count are zero rows of every block: their
    // threads load nothing and carry zeros
    const bool live = row_ok && (g.nkeep == nullptr || a < g.nkeep[c]);
    // right-hand side t = r (- A_l u): all loads of the row first
    const size_t row = (size_t)c * W + a;
    T tv = T(0), own = T(0);
    if (live) {
        tv = r[row];
        // the restriction's partial sums, in order; their sum is kept in r
        if (MODE == 0 && nparts > 1) tv = gather_parts(r + row, nparts, (int64_t)g.m * W);
    }
    if (MODE == 0 && nparts > 1 && live) r[row] = tv;
    if constexpr (MODE && A2) {
        if (live) {
            own = u[row];
            tv -= block_row_apply<T, LP, false, true>(g, AdT, Aoff, u, c, a);
        }
    } else if constexpr (MODE) {
        using Row = ResidRow<T, LP>;
        const auto at = Row::place(g, c, a, k, p);
        Row rr;
        if (live) rr.load(g, at, AdT, Aoff);
        stage_u<T, LP>(g, u, blockIdx.x, sU);
        __syncthreads();
        if (live) {
            tv -= rr.apply(g, at, Aoff, sU);
            own = sU[k * W + a];
        }
    }
    if (row_ok) sY[t] = tv;
    // The rows of D^-1 and of the couplings, loaded while the block
    // synchronises: up to width 9 all at once, wider ones (register budget)
    // load the upper couplings after the forward sweep.  A2 (agg = 2): along
    // each axis a child couples to exactly one sibling, below or above it, so
    // gl[ax] holds that one row, and the sweeps weight it by direction (gu
    // unused).  Couplings to children outside the parent are never loaded.
    constexpr bool kUpperEarly = LP <= 9 && !A2;
    constexpr int ND = A2 ? 4 : 7;
    T gl[3][LP], gu[3][LP], dv[LP];
    const T* sm = SM + (size_t)(row_ok ? E : 0) * ND * W * per + (row_ok ? tt : 0);
    auto load_row = [&](int d, bool in, T* dst) {
#pragma unroll
        for (int b = 0; b < LP; ++b) dst[b] = in && (!RT || b < W) ? sm[((size_t)d * W + b) * per] : T(0);
    };
    load_row(0, live, dv);
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) load_row(A2 ? 1 + ax : 1 + 2 * ax, live && (A2 || wgt[2 * ax] != T(0)), gl[ax]);
    if (kUpperEarly) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) load_row(2 + 2 * ax, live && wgt[2 * ax + 1] != T(0), gu[ax]);
    }
    __syncthreads();
    T w = T(0);
    {
        const T* ty = sY + base + k * W;
#pragma unroll
        for (int b = 0; b < LP; ++b) w += (!RT || b < W) ? dv[b] * ty[b] : T(0);
    }
    __syncthreads();
    // forward: y = w - sum_lower G y
    T y = T(0);
    for (int s = 0; s < nplanes; ++s) {
        if (row_ok && plane == s) {
            T s0 = T(0), s1 = T(0), s2 = T(0);
#pragma unroll
            for (int b = 0; b < LP; ++b) {
                if (RT && b >= W) continue;
                s0 += gl[0][b] * sY[nb[0] + b];
                s1 += gl[1][b] * sY[nb[2] + b];
                s2 += gl[2][b] * sY[nb[4] + b];
            }
            if (A2) {
                s0 *= wgt[0];
                s1 *= wgt[2];
                s2 *= wgt[4];
            }
            y = w - (s0 + s1 + s2);
            sY[t] = y;
        }
        __syncthreads();
    }
    // backward: z = y - sum_upper G z
    if (!kUpperEarly && !A2) {
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) load_row(2 + 2 * ax, live && wgt[2 * ax + 1] != T(0), gu[ax]);
    }
    T z = T(0);
    for (int s = nplanes - 1; s >= 0; --s) {
        if (row_ok && plane == s) {
            T s0 = T(0), s1 = T(0), s2 = T(0);
            if constexpr (A2) {
#pragma unroll
                for (int b = 0; b < LP; ++b) {
                    if (RT && b >= W) continue;
                    s0 += gl[0][b] * sY[nb[1] + b];
                    s1 += gl[1][b] * sY[nb[3] + b];
                    s2 += gl[2][b] * sY[nb[5] + b];
                }
                s0 *= wgt[1];
                s1 *= wgt[3];
                s2 *= wgt[5];
            } else {
#pragma unroll
                for (int b = 0; b < LP; ++b) {
                    if (RT && b >= W) continue;
                    s0 += gu[0][b] * sY[nb[1] + b];
                    s1 += gu[1][b] * sY[nb[3] + b];
                    s2 += gu[2][b] * sY[nb[5] + b];
                }
            }
            z = y - (s0 + s1 + s2);
            sY[t] = z;
        }
        __syncthreads();
    }
    if (row_ok) out[row] = MODE ? own + z : z;
}

// s = r - A_l u on the children of parent E, then r_up[E] = V_E^T s, one row a
// thread, the wavefronts' sums added in wavefront order.  SPLIT (agg 4, few
// parents): a workgroup is one of the W wavefronts of 64 rows that a parent has,
// and writes its part of the sum (part p at r_up + p M Lup; the kernel that reads
// r_up next adds the parts in order): a parent is a small task for 64 W rows of
// latency, and levels of 27 to 64 parents left most of the chip idle (19.4 -> 8.4 us
// for 64 parents of 64 x 9 rows, 12.5 -> 5.7 for 27 of 64 x 7).  The columns of V
// come in together with the rows: 53 -> 39 us for 512 parents of 64 x 11.
template <typename T, int LP, int LU, bool A2, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 64 : ((A2 ? 8 : 64) * LP + 63) / 64 * 64) void k_coarse_resid_restrict(
    CoarseGeom g, const T* __restrict__ AdT, const T* __restrict__ Aoff, const T* __restrict__ r,
    const T* __restrict__ u, const T* __restrict__ V, const int* __restrict__ nkeep_up, int Lup,
    T* __restrict__ rup, const Scalars* sc, int check_done) {
    if (check_done && sc->done) return;
    constexpr bool RT = LP == kMaxLc;
    constexpr int NC = A2 ? 8 : 64;
    __shared__ double sacc[SPLIT ? 1 : (NC * LP + 63) / 64][LU];
    const int W = RT ? g.L : LP, n = NC * W;
    const int E = SPLIT ? blockIdx.x / W : blockIdx.x, part = SPLIT ? blockIdx.x % W : 0;
    const int nk = nkeep_up[E];
    const int t = 64 * part + threadIdx.x, tr = t < n ? t : 0;
    const int p = tr / W, a = tr % W;
    const int c = child_of(g, E, p);
    const bool live = t < n && (g.nkeep == nullptr || a < g.nkeep[c]);   // zero rows beyond the kept slots
    const T* v = V + (size_t)E * Lup * n + tr;
    T vv[LU];
#pragma unroll
    for (int j = 0; j < LU; ++j) vv[j] = live ? v[(size_t)(j < nk ? j : nk - 1) * n] : T(0);
    double sv = 0.0;
    if (live) sv = (double)(r[(size_t)c * W + a] - block_row_apply<T, LP, SPLIT, false>(g, AdT, Aoff, u, c, a));
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double mine = 0.0;
#pragma unroll
    for (int j = 0; j < LU; ++j) {
        // the product rounded by itself: left bare, it is contracted with the first step of the sum
        const double x = wave_sum(fma((double)vv[j], sv, 0.0));
        if (SPLIT) mine = lane == j ? x : mine;
        else if (lane == 0) sacc[w][j] = x;
    }
    if constexpr (!SPLIT) {
        __syncthreads();
        if ((int)threadIdx.x < Lup)
            for (int ww = 0; ww < (int)(blockDim.x >> 6); ++ww) mine += sacc[ww][threadIdx.x];
    }
    if ((int)threadIdx.x < Lup)
        rup[((size_t)part * g.M + E) * Lup + threadIdx.x] = (int)threadIdx.x < nk ? (T)mine : T(0);
}

// u += V_E e_up[E] on the children of E
template <typename T, int LU>
__global__ __launch_bounds__(kCoarseThreads) void k_coarse_prolong(CoarseGeom g, T* __restrict__ u,
                                                                  const T* __restrict__ V,
                                                                  const int* __restrict__ nkeep_up, int Lup,
                                                                  const T* __restrict__ eup, const Scalars* sc,
                                                                  int check_done) {
    if (check_done && sc->done) return;
    const int E = blockIdx.x;
    const int L = g.L, nc = g.agg * g.agg * g.agg, n = nc * L;
    const int nk = nkeep_up[E];
    const T* ee = eup + (size_t)E * Lup;
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        const int p = t / L, a = t % L;
        T acc = T(0);
#pragma unroll
        for (int j = 0; j < LU; ++j) {
            const int jj = j < nk ? j : nk - 1;
            acc += (j < nk ? V[((size_t)E * Lup + jj) * n + t] : T(0)) * ee[jj];
        }
        u[(size_t)child_of(g, E, p) * L + a] += acc;
    }
}

// e = B r at the coarsest level, B the dense inverse of the regularised
// coarsest matrix, over the compact unknowns (cmap: compact index -> padded
// index), r in LDS.  Spaces beyond kCoarsestChunk unknowns use the packed
// triangle (k_coarsest_sym), with r gathered into a compact vector first.
template <typename T>
__global__ void k_gather_compact(int n, const int* __restrict__ cmap, const T* __restrict__ r, int nparts, int64_t pstride,
                                 double* __restrict__ rc, const Scalars* sc, int check_done) {
    if (check_done && sc->done) return;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        rc[i] = (double)gather_parts(r + cmap[i], nparts, pstride);
}

// Each block gathers the compact right-hand side itself from the level vector r
// through cmap, so no separate gather launch; a wavefront takes RW rows, as many
// as leave a block a CU, since what a block stages (n values, with their indices)
// is then a small part of what its rows read.  One row a wavefront, the only form
// before, took 46 us at n = 4096 (2.7 TB/s) and 104 at 5120; eight wavefronts of two
// rows take 31 and 49.
template <typename T, int RW, int NW>
__global__ __launch_bounds__(64 * NW) void k_coarsest(int n, int np, const double* __restrict__ Pinv,
                                                   const int* __restrict__ cmap, const T* __restrict__ r, int nparts,
                                                   int64_t pstride, T* __restrict__ e, const Scalars* sc,
                                                   int check_done) {
    if (check_done && sc->done) return;
    extern __shared__ double srz[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i0 = blockIdx.x * NW * RW + w * RW;
    for (int j = threadIdx.x; j < n; j += blockDim.x) srz[j] = (double)gather_parts(r + cmap[j], nparts, pstride);
    __syncthreads();
    double acc[RW];
    const double* row[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        acc[q] = 0.0;
        row[q] = Pinv + (size_t)min(i0 + q, n - 1) * np;
    }
    // lane l sums the columns l, l + 64, ... in turn
#pragma unroll 8
    for (int j = lane; j < n; j += 64) {
        const double v = srz[j];
#pragma unroll
        for (int q = 0; q < RW; ++q) acc[q] += row[q][j] * v;
    }
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        const double s = wave_sum(acc[q]);
        if (lane == 0 && i0 + q < n) e[cmap[i0 + q]] = (T)s;
    }
}

// Coarsest product for spaces wider than one LDS chunk, reading the
// symmetric inverse once: only its tiles (I, J) with I >= J are stored,
// packed tile after tile (tile (I, J) at index I (I + 1) / 2 + J, each tile
// kSymT x kSymT row-major and contiguous), half the bytes of the full
// matrix.  Tile (I, J) contributes B_IJ r_J to e_I and, below the diagonal,
// B_IJ^T r_I to e_J.  A workgroup streams a chunk of up to kSymChunk tiles of
// one tile row I: lane l of wave w holds columns 2l, 2l + 1 and rows
// w, w + 4, ... of every tile, so each row of a tile is one coalesced 1 KB
// load per wave.  The row contributions accumulate in registers over the
// chunk and are written once per chunk to Q[I][chunk]; the column
// contributions of each off-diagonal tile are combined over the four waves
// and written to P[J][I].  k_coarsest_sym_reduce then sums, for every
// output tile I, its chunks' Q and the P written by the tiles below it, in a
// fixed order (no atomics: results are reproducible).
constexpr int kSymT = 128;
constexpr int kSymChunk = 8;
constexpr int kSymWaves = 8;                  // 512 threads per workgroup
constexpr int kSymRows = kSymT / kSymWaves;   // rows per wave and tile

__global__ void k_pack_lower_tiles(const double* __restrict__ dense, int np, double* __restrict__ packed) {
    const int t = blockIdx.x;
    int I = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((I + 1) * (I + 2) / 2 <= t) ++I;
    while (I * (I + 1) / 2 > t) --I;
    const int J = t - I * (I + 1) / 2;
    double* dst = packed + (size_t)t * kSymT * kSymT;
    for (int k = threadIdx.x; k < kSymT * kSymT; k += blockDim.x) {
        const int i = k / kSymT, j = k % kSymT;
        dst[k] = dense[(size_t)(I * kSymT + i) * np + (size_t)J * kSymT + j];
    }
}

__global__ __launch_bounds__(64 * kSymWaves) void k_coarsest_sym(int nT, const int2* __restrict__ chunks,
                                                                 const double* __restrict__ packed,
                                                                 const double* __restrict__ rc,
                                                                 double* __restrict__ P, double* __restrict__ Q,
                                                                 int maxc, const Scalars* sc, int check_done) {
    if (check_done && sc->done) return;
    __shared__ double sri[kSymT];
    __shared__ double scol[kSymWaves][kSymT];
    const int2 ch = chunks[blockIdx.x];   // (tile row I, first tile J0)
    const int I = ch.x, J0 = ch.y, J1 = min(I + 1, J0 + kSymChunk);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x < kSymT) sri[threadIdx.x] = rc[(size_t)I * kSymT + threadIdx.x];
    __syncthreads();
    double racc[kSymRows];
#pragma unroll
    for (int k = 0; k < kSymRows; ++k) racc[k] = 0.0;
    for (int J = J0; J < J1; ++J) {
        const double* tile = packed + ((size_t)I * (I + 1) / 2 + J) * kSymT * kSymT + (size_t)w * kSymT + 2 * lane;
        const double2 rj = *reinterpret_cast<const double2*>(rc + (size_t)J * kSymT + 2 * lane);
        double c0 = 0.0, c1 = 0.0;
        // all 16 rows of the wave in flight (16 KB per wave), then the sums
        double2 b[kSymRows];
#pragma unroll
        for (int k = 0; k < kSymRows; ++k)
            b[k] = *reinterpret_cast<const double2*>(tile + (size_t)(kSymWaves * k) * kSymT);
#pragma unroll
        for (int k = 0; k < kSymRows; ++k) {
            const double ri = sri[w + kSymWaves * k];
            racc[k] += b[k].x * rj.x + b[k].y * rj.y;
            c0 += b[k].x * ri;
            c1 += b[k].y * ri;
        }
        if (J < I) {
            scol[w][2 * lane] = c0;
            scol[w][2 * lane + 1] = c1;
            __syncthreads();
            if (threadIdx.x < kSymT) {
                const int j = threadIdx.x;
                double v = 0.0;
#pragma unroll
                for (int ww = 0; ww < kSymWaves; ++ww) v += scol[ww][j];
                P[((size_t)J * nT + I) * kSymT + j] = v;
            }
            __syncthreads();
        }
    }
    const int c = J0 / kSymChunk;
#pragma unroll
    for (int k = 0; k < kSymRows; ++k) {
        const double v = wave_sum(racc[k]);
        if (lane == 0) Q[((size_t)I * maxc + c) * kSymT + w + kSymWaves * k] = v;
    }
}

// One workgroup per output tile I: kSymRedGroups groups of kSymT threads
// split the tile's partial vectors (group q takes the chunks c = q mod G and
// the tiles K = I + 1 + q mod G, four loads in flight), then the group sums
// are added in group order, so the result does not depend on timing.
constexpr int kSymRedGroups = 8;

template <typename T>
__global__ __launch_bounds__(kSymT * kSymRedGroups) void k_coarsest_sym_reduce(
    int nT, int n, const double* __restrict__ P, const double* __restrict__ Q, int maxc,
    const int* __restrict__ cmap, T* __restrict__ e, const Scalars* sc, int check_done) {
    if (check_done && sc->done) return;
    __shared__ double part[kSymRedGroups][kSymT];
    constexpr int G = kSymRedGroups;
    const int I = blockIdx.x, i = threadIdx.x % kSymT, q = threadIdx.x / kSymT;
    const int nc = (I + kSymChunk) / kSymChunk;   // chunks of tile row I (I + 1 tiles)
    double v = 0.0;
    for (int c = q; c < nc; c += G) v += Q[((size_t)I * maxc + c) * kSymT + i];
    const double* pr = P + (size_t)I * nT * kSymT + i;
    int K = I + 1 + q;
    for (; K + 3 * G < nT; K += 4 * G) {
        const double a0 = pr[(size_t)K * kSymT], a1 = pr[(size_t)(K + G) * kSymT];
        const double a2 = pr[(size_t)(K + 2 * G) * kSymT], a3 = pr[(size_t)(K + 3 * G) * kSymT];
        v += (a0 + a1) + (a2 + a3);
    }
    for (; K < nT; K += G) v += pr[(size_t)K * kSymT];
    part[q][i] = v;
    __syncthreads();
    if (q != 0) return;
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < G; ++g) t += part[g][i];
    const int row = I * kSymT + i;
    if (row < n) e[cmap[row]] = (T)t;
}

// ---------------------------------------------------------------------------
// set-up kernels

// Level-2 face blocks from the fine faces on the element boundary:
//   D[e][d] = sum_{tau on face d} T_f phi(tau) phi(tau)^T       (d = -x,+x,-y,+y,-z,+z)
//   Aoff[e][ax] = -sum_{tau on face +ax} T_f phi_e(tau) phi_{e+ax}(tau')^T
// (the terms of eq. discrete varia for faces between elements)
// Bound by the basis: the face cells of a column lie in every one of its lines,
// so the whole of it is fetched, and half of it again for the neighbours.  One sum of 64
// products a thread, from LDS, took 1.90 ms at 256^3 with 11 columns; nine 16 x 16
// products of depth 64 on the matrix cores (which add in the same order), all rows
// loaded at once, take 0.52 (0.20 -> 0.065 ms at 128^3).
__global__ __launch_bounds__(256) void k_galerkin2(FineGeom g, const double* __restrict__ kt,
                                                   const double* __restrict__ phi, const int* __restrict__ nkeep,
                                                   int L, double* __restrict__ D, double* __restrict__ Aoff) {
    constexpr int LD = 66;                     // rows of 64 face cells, padded against bank conflicts
    __shared__ double sT[6][64];
    __shared__ double sP[9][kMaxL2 * LD];      // own faces 2 ax (-), 2 ax + 1 (+); 6 + ax: across the + face
    const int e = blockIdx.x;
    const int ex = e % g.mx, ey = (e / g.mx) % g.my, ez = e / (g.mx * g.my);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int fu = lane & 7, fv = lane >> 3;   // in-face coordinates
    auto across = [&](int ax) {                // the element across the + face, or -1
        const bool in = ax == 0 ? ex + 1 < g.mx : (ax == 1 ? ey + 1 < g.my : ez + 1 < g.mz);
        return in ? e + (ax == 0 ? 1 : (ax == 1 ? g.mx : g.mx * g.my)) : -1;
    };
    // face rows: wavefront w takes columns w, w + 4, ..., all loads in flight
    double v[9][kMaxL2 / 4];
#pragma unroll
    for (int d = 0; d < 9; ++d) {
        const int ax = d < 6 ? d >> 1 : d - 6;
        const int en = d < 6 ? e : across(ax);
        const int at = d < 6 && (d & 1) ? 7 : 0;
        const int pos = phi_pos(ax == 0 ? at + 8 * (fu + 8 * fv) : (ax == 1 ? fu + 8 * (at + 8 * fv) : fu + 8 * (fv + 8 * at)));
#pragma unroll
        for (int m = 0; m < kMaxL2 / 4; ++m) {
            const int jj = w + 4 * m;
            v[d][m] = jj < L && en >= 0 ? phi[((size_t)en * L + jj) * 512 + pos] : 0.0;
        }
    }
    // face transmissibilities
    for (int d = w; d < 6; d += 4) {
        const int ax = d >> 1, at = (d & 1) ? 7 : 0, o = (d & 1) ? 1 : -1;
        const int gx = ex * 8 + (ax == 0 ? at : fu), gy = ey * 8 + (ax == 0 ? fu : (ax == 1 ? at : fv));
        const int gz = ez * 8 + (ax == 2 ? at : fv);
        const int hx = gx + (ax == 0 ? o : 0), hy = gy + (ax == 1 ? o : 0), hz = gz + (ax == 2 ? o : 0);
        double T = 0.0;
        if (hx >= 0 && hx < g.nx && hy >= 0 && hy < g.ny && hz >= 0 && hz < g.nz) {
            // kappa~ of this face's direction (three arrays for orthotropic K)
            const size_t off = g.ortho ? (size_t)ax * g.ncell() : 0;
            const double a = kt[off + eidx(g, gx, gy, gz)], b = kt[off + eidx(g, hx, hy, hz)];
            T = 2.0 * a * b / (a + b) * (ax == 0 ? 1.0 : (ax == 1 ? g.cy : g.cz));
        }
        sT[d][lane] = T;
    }
#pragma unroll
    for (int d = 0; d < 9; ++d)
#pragma unroll
        for (int m = 0; m < kMaxL2 / 4; ++m) sP[d][(w + 4 * m) * LD + lane] = v[d][m];
    __syncthreads();
    // block blk = P^T diag(T) Q over the 64 cells of a face, one 16 x 16
    // product of depth 64 on the matrix cores
    const int li = lane & 15, lk = lane >> 4, LL = L * L;
    typedef double dbl4 __attribute__((ext_vector_type(4)));
    for (int blk = w; blk < 9; blk += 4) {
        const int ax = blk - 6, d = blk < 6 ? blk : 2 * ax + 1;
        dbl4 c{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const int f = 4 * kk + lk;
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(sT[d][f] * sP[d][li * LD + f], sP[blk < 6 ? d : blk][li * LD + f], c,
                                                     0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = lk + 4 * r;
            if (a >= L || li >= L) continue;
            if (blk < 6) D[((size_t)e * 6 + blk) * LL + a * L + li] = c[r];
            else Aoff[((size_t)e * 3 + ax) * LL + a * L + li] = -c[r];
        }
    }
}

// Face blocks of level l+1 from those of level l (Galerkin with V_E):
//   D_up[E][d] = sum_{c on face d of E} V_c^T D[c][d] V_c
//   Aoff_up[E][ax] = sum_{c on face +ax of E} V_c^T Aoff[c][ax] V'_{c+ax}
// A workgroup per parent and block (blockIdx.y: the six D, the three Aoff): each is a
// chain of agg^2 children, and a workgroup a parent ran nine of them in turn (268
// -> 39 us for 64 parents of 64 x 9 rows, 0.36 ms for 512 of 64 x 11 before).
__global__ __launch_bounds__(256) void k_galerkin_up(CoarseGeom lo, CoarseGeom up, const double* __restrict__ Dlo,
                                                     const double* __restrict__ Aofflo,
                                                     const double* __restrict__ V,
                                                     const int* __restrict__ nkeep_up, double* __restrict__ Dup,
                                                     double* __restrict__ Aoffup) {
    __shared__ double sB[kMaxL * kMaxL];     // level-l block
    __shared__ double sV[kMaxL * kMaxL];     // V_c   (Lp x Lu)
    __shared__ double sW[kMaxL * kMaxL];     // V'_c' (Lp x Lu)
    __shared__ double sBW[kMaxL * kMaxL];    // B V'  (Lp x Lu)
    const int E = blockIdx.x;
    const int agg = lo.agg, Lp = lo.L, Lu = up.L;
    const int n = agg * agg * agg * Lp;
    const int Ex = E % up.mx, Ey = (E / up.mx) % up.my, Ez = E / (up.mx * up.my);
    const int Ec[3] = {Ex, Ey, Ez};
    const int ext[3] = {up.mx, up.my, up.mz};
    const int estride[3] = {1, up.mx, up.mx * up.my};
    const int blk = blockIdx.y;
    const bool isD = blk < 6;
    const int d = isD ? blk : 2 * (blk - 6) + 1;
    const int ax = d >> 1;
    const bool plus = d & 1;
    const bool has_nb = isD || (Ec[ax] + 1 < ext[ax]);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (has_nb) {
        for (int f = 0; f < agg * agg; ++f) {
            const int u = f % agg, v = f / agg;
            int q[3];
            q[ax] = plus ? agg - 1 : 0;
            q[(ax + 1) % 3] = u;
            q[(ax + 2) % 3] = v;
            const int p = q[0] + agg * (q[1] + agg * q[2]);
            const int c = (Ex * agg + q[0]) + lo.mx * ((Ey * agg + q[1]) + lo.my * (Ez * agg + q[2]));
            // stage B, V_c and (for couplings) V'_{c'}
            for (int t = threadIdx.x; t < Lp * Lp; t += blockDim.x)
                sB[t] = isD ? Dlo[((size_t)c * 6 + d) * Lp * Lp + t] : Aofflo[((size_t)c * 3 + ax) * Lp * Lp + t];
            for (int t = threadIdx.x; t < Lp * Lu; t += blockDim.x) {
                const int b = t / Lu, j = t % Lu;
                sV[t] = V[((size_t)E * Lu + j) * n + p * Lp + b];
                if (isD) {
                    sW[t] = sV[t];
                } else {
                    int qn[3] = {q[0], q[1], q[2]};
                    qn[ax] = 0;
                    const int pn = qn[0] + agg * (qn[1] + agg * qn[2]);
                    const int En = E + estride[ax];
                    sW[t] = V[((size_t)En * Lu + j) * n + pn * Lp + b];
                }
            }
            __syncthreads();
            for (int t = threadIdx.x; t < Lp * Lu; t += blockDim.x) {
                const int a = t / Lu, j = t % Lu;
                double s = 0.0;
                for (int b = 0; b < Lp; ++b) s += sB[a * Lp + b] * sW[b * Lu + j];
                sBW[t] = s;
            }
            __syncthreads();
            for (int t = threadIdx.x, k = 0; t < Lu * Lu; t += blockDim.x, ++k) {
                const int i = t / Lu, j = t % Lu;
                double s = 0.0;
                for (int a = 0; a < Lp; ++a) s += sV[a * Lu + i] * sBW[a * Lu + j];
                acc[k] += s;
            }
            __syncthreads();
        }
    }
    for (int t = threadIdx.x, k = 0; t < Lu * Lu; t += blockDim.x, ++k) {
        if (isD) Dup[((size_t)E * 6 + d) * Lu * Lu + t] = acc[k];
        else Aoffup[((size_t)E * 3 + ax) * Lu * Lu + t] = acc[k];
    }
}

// Ad = Aint + sum_d D[e][d]
__global__ void k_assemble_diag(CoarseGeom g, const double* __restrict__ Aint, const double* __restrict__ D,
                                double* __restrict__ Ad) {
    const int e = blockIdx.x;
    const int LL = g.L * g.L;
    for (int t = threadIdx.x; t < LL; t += blockDim.x) {
        double v = Aint[(size_t)e * LL + t];
        for (int d = 0; d < 6; ++d) v += D[((size_t)e * 6 + d) * LL + t];
        Ad[(size_t)e * LL + t] = v;
    }
}

// Block IC(0) pivots of the level-l smoother, one workgroup per parent: the
// children of one hyperplane (at most 12, 3 with agg 2) are factored in
// parallel, one wavefront each.  Entry t = lane + 64 u of an L x L block is
// lane's u-th register, U of them; LDS passes blocks and pivot rows around
// the wavefront.  The inverse solves C C^T X = I with the Cholesky factor C:
// the factor and the forward substitution eliminate [A | I] row by row (column k
// of I takes the place that column k of A leaves), the backward substitution
// takes a lane a column.  Every entry sees its products in the order of the
// textbook loops (k ascending, divisions by the pivot's root): the order is part
// of the result, see block_row_apply.  Padded slots (index >= nkeep) are rows of
// the identity.
// A chain: per plane one memory round trip, three Schur updates, L pivots of
// one LDS round trip, a root and a division each, L steps back.  433 -> 114 us for 64
// parents of 64 x 9 rows, 2.2 ms -> 262 us for 512 of 64 x 11, 6.0 ms -> 258 us for
// 4,096 of 8 x 9 and then 512 of 8 x 13, against a form with the blocks in LDS.
constexpr int kMaxPlane = 12;   // children per hyperplane of a 4^3 parent
// Widths beyond 13 occur with agg 2 only (three wavefronts, so that all the registers
// of the widest are there).
constexpr int plane_waves(int width) { return width > 13 ? 3 : kMaxPlane; }
template <int LP>
__global__ __launch_bounds__(64 * plane_waves(LP)) void k_blockic_setup(CoarseGeom g, const double* __restrict__ Ad,
                                                                        const double* __restrict__ Aoff,
                                                                        const int* __restrict__ nkeep, double* Dinv,
                                                                        int* bad) {
    constexpr bool RT = LP == kMaxLc;   // the widest serves every width above kNarrow
    constexpr int U = (LP * LP + 63) / 64;
    __shared__ int pos[kMaxChildren], off[12];
    extern __shared__ double work_lds[];   // [children of the widest plane][3][L * L]
    const int E = blockIdx.x;
    const int L = RT ? g.L : LP, agg = g.agg, LL = L * L;
    build_planes(agg, pos, off);
    const int nplanes = 3 * (agg - 1) + 1;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double* sA = work_lds + (size_t)(3 * w) * LL;
    double* sB = sA + LL;
    double* sR = sB + LL;
    int row[U], col[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = lane + 64 * u;
        in[u] = t < LL;
        row[u] = in[u] ? t / L : 0;
        col[u] = in[u] ? t - row[u] * L : 0;
    }
    for (int s = 0; s < nplanes; ++s) {
        const int cnt = off[s + 1] - off[s];
        if (w < cnt) {
            const int p = pos[off[s] + w];
            const int c = child_of(g, E, p);
            const int q[3] = {p % agg, (p / agg) % agg, p / (agg * agg)};
            const int cstep[3] = {1, g.mx, g.mx * g.my};
            const int nk = nkeep[c];
            constexpr bool ONCE = U <= 2;   // all couplings loaded at once, if the registers hold them
            double P[U], O[ONCE ? 3 : 1][U], Di[ONCE ? 3 : 1][U];
            auto load = [&](int ax, double (&o)[U], double (&di)[U]) {
                const size_t cn = q[ax] > 0 ? c - cstep[ax] : c;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool ld = in[u] && q[ax] > 0;
                    o[u] = ld ? Aoff[(cn * 3 + ax) * LL + lane + 64 * u] : 0.0;   // A(cn, c)
                    di[u] = ld ? Dinv[cn * LL + lane + 64 * u] : 0.0;
                }
            };
#pragma unroll
            for (int u = 0; u < U; ++u) P[u] = in[u] ? Ad[(size_t)c * LL + lane + 64 * u] : 0.0;
            if constexpr (ONCE)
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) load(ax, O[ax], Di[ax]);
            // P -= O^T (Dinv_cn O)
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                if (q[ax] == 0) continue;
                if constexpr (!ONCE) load(ax, O[0], Di[0]);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (in[u]) {
                        sA[lane + 64 * u] = Di[ONCE ? ax : 0][u];
                        sB[lane + 64 * u] = O[ONCE ? ax : 0][u];
                    }
                wave_sync();
                double T[U];
#pragma unroll
                for (int u = 0; u < U; ++u) T[u] = 0.0;
                for (int b = 0; b < L; ++b)
#pragma unroll
                    for (int u = 0; u < U; ++u) T[u] += sA[row[u] * L + b] * sB[b * L + col[u]];
                wave_sync();
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (in[u]) sA[lane + 64 * u] = T[u];
                wave_sync();
#pragma unroll
                for (int u = 0; u < U; ++u) T[u] = 0.0;
                for (int b = 0; b < L; ++b)
#pragma unroll
                    for (int u = 0; u < U; ++u) T[u] += sB[b * L + row[u]] * sA[b * L + col[u]];
#pragma unroll
                for (int u = 0; u < U; ++u) P[u] -= T[u];
                wave_sync();
            }
            // symmetrise, padded slots
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (in[u]) sA[lane + 64 * u] = P[u];
            wave_sync();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                P[u] = 0.5 * (P[u] + sA[col[u] * L + row[u]]);
                if (row[u] >= nk || col[u] >= nk) P[u] = row[u] == col[u] ? 1.0 : 0.0;
            }
            // C (to sA) and C^-1
            bool ok = true;
            for (int k = 0; k < L; ++k) {
                // column k of what is left of A from row k on, row k of what has come of I before
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (in[u]) {
                        if (col[u] == k && row[u] >= k) sR[row[u]] = P[u];
                        if (row[u] == k && col[u] < k) sR[col[u]] = P[u];
                    }
                wave_sync();
                double d = sR[k];
                if (!(d > 0.0)) {
                    ok = false;
                    d = 1.0;
                }
                const double root = sqrt(d);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double l = sR[row[u]] / root, f = (col[u] == k ? 1.0 : sR[col[u]]) / root;
                    if (row[u] > k) {
                        if (in[u] && col[u] == k) sA[row[u] * L + k] = l;
                        P[u] = col[u] == k ? -(l * f) : P[u] - l * f;
                    } else if (row[u] == k && col[u] <= k) {
                        P[u] = f;
                    }
                }
                if (lane == 0) sA[k * L + k] = root;
                wave_sync();
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (in[u]) sB[lane + 64 * u] = col[u] <= row[u] ? P[u] : 0.0;
            wave_sync();
            if (lane < L) {
                double x[LP];
#pragma unroll
                for (int i = LP - 1; i >= 0; --i) {
                    if (RT && i >= L) continue;
                    double v = sB[i * L + lane];
#pragma unroll
                    for (int k = 0; k < LP; ++k)
                        if (k > i && (!RT || k < L)) v -= sA[k * L + i] * x[k];
                    x[i] = v / sA[i * L + i];
                    Dinv[(size_t)c * LL + i * L + lane] = x[i];
                }
            }
            wave_sync();
            if (!ok && lane == 0) atomicOr(bad, 2);
        }
        __syncthreads();   // the plane's pivots are read by this workgroup alone
    }
}

// the sweep's matrices: Dinv_c, and Dinv_c A(c, c -+ e_ax) for neighbours
// inside the same parent (zero otherwise), in the layout of k_coarse_sweep
__global__ __launch_bounds__(256) void k_blockic_couple(CoarseGeom g, const double* __restrict__ Ad,
                                                         const double* __restrict__ Aoff,
                                                         const double* __restrict__ Dinv, double* __restrict__ SM,
                                                         double* __restrict__ AdT) {
    const int c = blockIdx.x;
    const int L = g.L, LL = L * L, agg = g.agg, nc = agg * agg * agg;
    const int cx = c % g.mx, cy = (c / g.mx) % g.my, cz = c / (g.mx * g.my);
    const int q[3] = {cx % agg, cy % agg, cz % agg};
    const int stride[3] = {1, g.mx, g.mx * g.my};
    const int E = cx / agg + g.px * (cy / agg + g.py * (cz / agg)), pos = q[0] + agg * (q[1] + agg * q[2]);
    const int k = agg == 4 ? kCP.rank4[pos] : kCP.rank2[pos], nd = agg == 4 ? 7 : 4, rows = nc * L;
    const double* Di = Dinv + (size_t)c * LL;
    for (int t = threadIdx.x; t < LL; t += blockDim.x) AdT[(size_t)c * LL + t % L * L + t / L] = Ad[(size_t)c * LL + t];
    for (int t = threadIdx.x; t < nd * LL; t += blockDim.x) {
        const int d = t / LL, b = (t % LL) / L, a = t % L;
        double v = 0.0;
        if (d == 0) {
            v = Di[a * L + b];
        } else {
            const int ax = agg == 4 ? (d - 1) >> 1 : d - 1;
            const bool upper = agg == 4 ? (d - 1) & 1 : q[ax] == 0;
            if (upper ? (q[ax] < agg - 1) : (q[ax] > 0)) {
                for (int i = 0; i < L; ++i) {
                    // A(c, c - e) = Aoff[c - e][ax]^T ; A(c, c + e) = Aoff[c][ax]
                    const double A = upper ? Aoff[(((size_t)c * 3 + ax) * L + i) * L + b]
                                           : Aoff[(((size_t)(c - stride[ax]) * 3 + ax) * L + b) * L + i];
                    v += Di[a * L + i] * A;
                }
            }
        }
        SM[(((size_t)E * nd + d) * L + b) * rows + (size_t)k * L + a] = v;
    }
}

// a part a wavefront where one workgroup a parent would leave more than half of
// the CUs idle
int coarse_restrict_parts(const CoarseGeom& g) { return g.agg == 4 && g.M <= 128 ? g.L : 1; }

size_t coarse_sweep_doubles(const CoarseGeom& g) { return (size_t)g.m * (g.agg == 4 ? 7 : 4) * g.L * g.L; }

// coarsest dense matrix over the compact unknowns (cinv: padded -> compact
// or -1); the matrix must be zeroed beforehand
__global__ void k_build_coarsest(CoarseGeom g, const double* __restrict__ Ad, const double* __restrict__ Aoff,
                                 const int* __restrict__ cinv, int np, double* __restrict__ dense) {
    const int e = blockIdx.x;
    const int L = g.L, LL = L * L;
    const int cx = e % g.mx, cy = (e / g.mx) % g.my, cz = e / (g.mx * g.my);
    const int cc[3] = {cx, cy, cz};
    const int ext[3] = {g.mx, g.my, g.mz};
    const int stride[3] = {1, g.mx, g.mx * g.my};
    for (int t = threadIdx.x; t < LL; t += blockDim.x) {
        const int a = t / L, b = t % L;
        const int i = cinv[e * L + a];
        if (i < 0) continue;
        const int jd = cinv[e * L + b];
        if (jd >= 0) dense[(size_t)i * np + jd] = Ad[(size_t)e * LL + t];
        for (int ax = 0; ax < 3; ++ax) {
            if (cc[ax] + 1 >= ext[ax]) continue;
            const int en = e + stride[ax];
            const int j = cinv[en * L + b];
            if (j < 0) continue;
            const double v = Aoff[((size_t)e * 3 + ax) * LL + t];
            dense[(size_t)i * np + j] = v;
            dense[(size_t)j * np + i] = v;
        }
    }
}

template <typename S, typename T>
__global__ void k_convert(const S* __restrict__ src, T* __restrict__ dst, int64_t n, const Scalars* sc) {
    if (sc && sc->done) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = (T)src[i];
}

// ---------------------------------------------------------------------------
// launchers

#define SPECMG_LP_DISPATCH_NARROW(LV, ...) \
    switch (LV) { \
        case 4: { constexpr int LP = 4; __VA_ARGS__; } break; \
        case 5: { constexpr int LP = 5; __VA_ARGS__; } break; \
        case 6: { constexpr int LP = 6; __VA_ARGS__; } break; \
        case 7: { constexpr int LP = 7; __VA_ARGS__; } break; \
        case 8: { constexpr int LP = 8; __VA_ARGS__; } break; \
        case 9: { constexpr int LP = 9; __VA_ARGS__; } break; \
    }

#define SPECMG_LP_DISPATCH_SWEEP4(LV, ...) \
    switch (LV) { \
        case 4: { constexpr int LP = 4; __VA_ARGS__; } break; \
        case 5: { constexpr int LP = 5; __VA_ARGS__; } break; \
        case 6: { constexpr int LP = 6; __VA_ARGS__; } break; \
        case 7: { constexpr int LP = 7; __VA_ARGS__; } break; \
        case 8: { constexpr int LP = 8; __VA_ARGS__; } break; \
        case 9: { constexpr int LP = 9; __VA_ARGS__; } break; \
        case 10: { constexpr int LP = 10; __VA_ARGS__; } break; \
        case 11: { constexpr int LP = 11; __VA_ARGS__; } break; \
        case 12: { constexpr int LP = 12; __VA_ARGS__; } break; \
    }

#define SPECMG_LP_DISPATCH_WIDE(LV, ...) \
    switch (LV) { \
        case 10: { constexpr int LP = 10; __VA_ARGS__; } break; \
        case 11: { constexpr int LP = 11; __VA_ARGS__; } break; \
        case 12: { constexpr int LP = 12; __VA_ARGS__; } break; \
        case 13: { constexpr int LP = 13; __VA_ARGS__; } break; \
        default: { constexpr int LP = kMaxLc; __VA_ARGS__; } break; \
    }

#define SPECMG_LP_DISPATCH(LV, ...) \
    switch (LV) { \
        case 4: { constexpr int LP = 4; __VA_ARGS__; } break; \
        case 5: { constexpr int LP = 5; __VA_ARGS__; } break; \
        case 6: { constexpr int LP = 6; __VA_ARGS__; } break; \
        case 7: { constexpr int LP = 7; __VA_ARGS__; } break; \
        case 8: { constexpr int LP = 8; __VA_ARGS__; } break; \
        case 9: { constexpr int LP = 9; __VA_ARGS__; } break; \
        case 10: { constexpr int LP = 10; __VA_ARGS__; } break; \
        case 11: { constexpr int LP = 11; __VA_ARGS__; } break; \
        case 12: { constexpr int LP = 12; __VA_ARGS__; } break; \
        case 13: { constexpr int LP = 13; __VA_ARGS__; } break; \
        default: { constexpr int LP = kMaxLc; __VA_ARGS__; } break; \
    }

// The same for 2x aggregation and widths up to 9: one wavefront per parent.
// Its lanes take the kept rows of the 8 children in turn (row q of the
// parent is slot a of child position p, q = the kept rows of the positions
// before p, plus a), 64 rows per pass, so the dead padded slots take no
// lanes; the restriction sums are wavefront reductions, with no LDS and no
// block barrier.
template <typename T, int LP, int LU>
__global__ __launch_bounds__(256) void k_coarse_resid_restrict_w(
    CoarseGeom g, const T* __restrict__ AdT, const T* __restrict__ Aoff, const T* __restrict__ r,
    const T* __restrict__ u, const T* __restrict__ V, const int* __restrict__ nkeep_up, int Lup,
    T* __restrict__ rup, const Scalars* sc, int check_done) {
    if (check_done && sc->done) return;
    const int lane = threadIdx.x & 63;
    const int E = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (E >= g.M) return;   // whole wavefront; no block barriers below
    const int L = g.L, n = 8 * L;
    int pre[9];
    pre[0] = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) pre[q + 1] = pre[q] + (g.nkeep ? g.nkeep[child_of(g, E, q)] : L);
    const int rows = pre[8];
    const int nk = nkeep_up[E];
    double acc[LU];
#pragma unroll
    for (int j = 0; j < LU; ++j) acc[j] = 0.0;
    for (int q0 = 0; q0 < rows; q0 += 64) {
        const int qr = q0 + lane;
        if (qr < rows) {
            int p = 0;
#pragma unroll
            for (int q = 1; q < 8; ++q) p += qr >= pre[q] ? 1 : 0;
            const int a = qr - pre[p];
            const int c = child_of(g, E, p);
            const double sv = (double)(r[(size_t)c * L + a] - block_row_apply<T, LP, false, false>(g, AdT, Aoff, u, c, a));
            const T* vc = V + (size_t)E * Lup * n + (size_t)p * L + a;
#pragma unroll
            for (int j = 0; j < LU; ++j)
                if (j < nk) acc[j] += (double)vc[(size_t)j * n] * sv;
        }
    }
    double mine = 0.0;
#pragma unroll
    for (int j = 0; j < LU; ++j) {
        const double v = wave_sum(acc[j]);
        if (lane == j) mine = v;
    }
    if (lane < Lup) rup[(size_t)E * Lup + lane] = lane < nk ? (T)mine : T(0);
}

template <typename T>
void launch_coarse_resid_restrict(const CoarseGeom& g0, const T* AdT, const T* Aoff, const T* r, const T* u,
                                  const T* V, const int* nkeep_up, int Lup, T* rup, const Scalars* sc,
                                  int check_done, hipStream_t s) {
    CoarseGeom g = g0;
    const bool split = coarse_restrict_parts(g) > 1;
    if (split) g.nkeep = nullptr;   // as the sweeps
    const int rows = g.agg * g.agg * g.agg * g.L;
    const dim3 nb(g.M), th((rows + 63) / 64 * 64);
    if (g.L < 4 || g.L > kMaxLc || (g.agg == 4 && g.L > kMaxParts))
        throw HipError{hipErrorInvalidValue, "coarse residual width"};
    if (Lup > kMaxLc) throw HipError{hipErrorInvalidValue, "coarse residual upper width"};
    // wider blocks keep about 8 L > 64 rows per parent, two passes of the
    // wavefront: there the workgroup form is faster
    if (g.agg == 2 && g.L <= 9) {
        const int nb4 = (g.M + 3) / 4;
        if (Lup <= kNarrow) {
            SPECMG_LP_DISPATCH_NARROW(g.L, hipLaunchKernelGGL((k_coarse_resid_restrict_w<T, LP, kNarrow>), dim3(nb4),
                                                       dim3(256), 0, s, g, AdT, Aoff, r, u, V, nkeep_up, Lup, rup, sc,
                                                       check_done));
        } else {
            SPECMG_LP_DISPATCH_NARROW(g.L, hipLaunchKernelGGL((k_coarse_resid_restrict_w<T, LP, kMaxLc>), dim3(nb4),
                                                       dim3(256), 0, s, g, AdT, Aoff, r, u, V, nkeep_up, Lup, rup, sc,
                                                       check_done));
        }
        return;
    }
#define SPECMG_RESTRICT(A2, SPLIT, NB, TH)                                                                            \
    if (Lup <= kNarrow)                                                                                               \
        hipLaunchKernelGGL((k_coarse_resid_restrict<T, LP, kNarrow, A2, SPLIT>), NB, TH, 0, s, g, AdT, Aoff, r, u, V,   \
                           nkeep_up, Lup, rup, sc, check_done);                                                       \
    else                                                                                                              \
        hipLaunchKernelGGL((k_coarse_resid_restrict<T, LP, kMaxLc, A2, SPLIT>), NB, TH, 0, s, g, AdT, Aoff, r, u, V,    \
                           nkeep_up, Lup, rup, sc, check_done)
    if (g.agg == 2) {
        SPECMG_LP_DISPATCH_WIDE(g.L, SPECMG_RESTRICT(true, false, nb, th));
    } else if (split) {
        SPECMG_LP_DISPATCH_SWEEP4(g.L, SPECMG_RESTRICT(false, true, dim3(g.M * g.L), dim3(64)));
    } else {
        SPECMG_LP_DISPATCH_SWEEP4(g.L, SPECMG_RESTRICT(false, false, nb, th));
    }
#undef SPECMG_RESTRICT
}

template <typename T>
void launch_coarse_prolong(const CoarseGeom& g, T* u, const T* V, const int* nkeep_up, int Lup, const T* eup,
                           const Scalars* sc, int check_done, hipStream_t s) {
    const int rows = g.agg * g.agg * g.agg * g.L;
    const int th = std::min(kCoarseThreads, (rows + 63) / 64 * 64);
    if (Lup > kMaxLc) throw HipError{hipErrorInvalidValue, "coarse prolongation upper width"};
    if (Lup <= kNarrow)
        hipLaunchKernelGGL((k_coarse_prolong<T, kNarrow>), dim3(g.M), dim3(th), 0, s, g, u, V, nkeep_up, Lup, eup, sc,
                           check_done);
    else
        hipLaunchKernelGGL((k_coarse_prolong<T, kMaxLc>), dim3(g.M), dim3(th), 0, s, g, u, V, nkeep_up, Lup, eup, sc,
                           check_done);
}

static int sweep_parents(const CoarseGeom& g) { return sweep_parents(g.agg, g.L); }
static int sweep_threads(const CoarseGeom& g) {
    const int rows = sweep_parents(g) * g.agg * g.agg * g.agg * g.L;
    return (rows + 63) / 64 * 64;
}
static int sweep_blocks(const CoarseGeom& g) {
    const int np = sweep_parents(g);
    return (g.M + np - 1) / np;
}

template <typename T, int MODE>
static void launch_sweep(const CoarseGeom& g0, const T* AdT, const T* Aoff, const T* SM, T* r, const T* u, T* out,
                         const Scalars* sc, int check_done, int nparts, hipStream_t s) {
    CoarseGeom g = g0;
    if (g.L < 4 || g.L > kMaxLc || sweep_threads(g) > 768) throw HipError{hipErrorInvalidValue, "coarse sweep shape"};
    const dim3 nb(sweep_blocks(g)), th(sweep_threads(g));
    const int npar = sweep_parents(g);
    // launches of at most one workgroup a CU wait for latency, not for bandwidth:
    // they take the padded rows too (zeros) instead of waiting for the kept counts
    // (27 parents of 64 x 7 rows: 9.8 -> 9.1 us; 64 of 64 x 9: no difference)
    if (sweep_blocks(g) <= 256) g.nkeep = nullptr;
    if (g.agg == 2) {
        SPECMG_LP_DISPATCH(g.L, hipLaunchKernelGGL((k_coarse_sweep<T, LP, true, MODE>), nb, th, 0, s, g, AdT, Aoff, SM, r, u,
                                                   out, sc, check_done, npar, nparts));
    } else {
        SPECMG_LP_DISPATCH_SWEEP4(g.L, hipLaunchKernelGGL((k_coarse_sweep<T, LP, false, MODE>), nb, th, 0, s, g, AdT, Aoff,
                                                          SM, r, u, out, sc, check_done, npar, nparts));
    }
}

// u = M_l^{-1} r; r arrives in nparts parts and is left summed
template <typename T>
void launch_coarse_smooth(const CoarseGeom& g, const T* SM, T* r, int nparts, T* u, const Scalars* sc, int check_done,
                          hipStream_t s) {
    launch_sweep<T, 0>(g, nullptr, nullptr, SM, r, nullptr, u, sc, check_done, nparts, s);
}

// e = u + M_l^{-1} (r - A_l u)
template <typename T>
void launch_coarse_resid_smooth(const CoarseGeom& g, const T* AdT, const T* Aoff, const T* SM, const T* r, const T* u, T* e,
                                const Scalars* sc, int check_done, hipStream_t s) {
    launch_sweep<T, 1>(g, AdT, Aoff, SM, const_cast<T*>(r), u, e, sc, check_done, 1, s);
}

int coarsest_sym_tile() { return kSymT; }

size_t coarsest_sym_packed_doubles(int np) {
    const size_t nT = (size_t)np / kSymT;
    return nT * (nT + 1) / 2 * kSymT * kSymT;
}

// host-side chunk table of the symmetric product: (tile row, first tile)
std::vector<int2> coarsest_sym_chunks(int np, int* maxc) {
    const int nT = np / kSymT;
    std::vector<int2> ch;
    *maxc = (nT + kSymChunk - 1) / kSymChunk;
    for (int I = 0; I < nT; ++I)
        for (int J0 = 0; J0 <= I; J0 += kSymChunk) ch.push_back(make_int2(I, J0));
    return ch;
}

void launch_pack_lower_tiles(const double* dense, int np, double* packed, hipStream_t s) {
    const int nT = np / kSymT;
    hipLaunchKernelGGL(k_pack_lower_tiles, dim3(nT * (nT + 1) / 2), dim3(256), 0, s, dense, np, packed);
}

void launch_coarsest_sym(int n, int np, const double* packed, const int2* chunks, int nchunks, int maxc,
                         const int* cmap, const double* r, int nparts, int64_t pstride, double* e, double* rc, double* P, double* Q,
                         const Scalars* sc, int check_done, hipStream_t s) {
    const int nT = np / kSymT;
    hipLaunchKernelGGL((k_gather_compact<double>), dim3(std::min((n + 255) / 256, 1024)), dim3(256), 0, s, n, cmap,
                       r, nparts, pstride, rc, sc, check_done);
    SPECMG_TIMED_LAUNCH(k_coarsest_sym, dim3(nchunks), dim3(64 * kSymWaves), 0, s, nT, chunks, packed, rc, P, Q,
                        maxc, sc, check_done);
    hipLaunchKernelGGL((k_coarsest_sym_reduce<double>), dim3(nT), dim3(kSymT * kSymRedGroups), 0, s, nT, n, P, Q, maxc, cmap, e, sc,
                       check_done);
}

template <typename T>
void launch_coarsest(int n, int np, const double* Pinv, const int* cmap, const T* r, int nparts, int64_t pstride, T* e,
                     const Scalars* sc, int check_done, hipStream_t s) {
    if (n > kCoarsestChunk) throw HipError{hipErrorInvalidValue, "coarsest product size"};
    const size_t lds = (size_t)n * sizeof(double);
    if (n <= 1024) {
        SPECMG_TIMED_LAUNCH((k_coarsest<T, 1, 4>), dim3((n + 3) / 4), dim3(256), lds, s, n, np, Pinv, cmap, r, nparts,
                            pstride, e, sc, check_done);
    } else if (n <= 2048) {
        SPECMG_TIMED_LAUNCH((k_coarsest<T, 1, 8>), dim3((n + 7) / 8), dim3(512), lds, s, n, np, Pinv, cmap, r, nparts,
                            pstride, e, sc, check_done);
    } else {
        SPECMG_TIMED_LAUNCH((k_coarsest<T, 2, 8>), dim3((n + 15) / 16), dim3(512), lds, s, n, np, Pinv, cmap, r, nparts,
                            pstride, e, sc, check_done);
    }
}

void launch_galerkin2(const FineGeom& g, const double* kt, const double* phi, const int* nkeep, int L, double* D,
                      double* Aoff, hipStream_t s) {
    hipLaunchKernelGGL(k_galerkin2, dim3(g.mx * g.my * g.mz), dim3(256), 0, s, g, kt, phi, nkeep, L, D, Aoff);
}

void launch_galerkin_up(const CoarseGeom& lo, const CoarseGeom& up, const double* Dlo, const double* Aofflo,
                        const double* V, const int* nkeep_up, double* Dup, double* Aoffup, hipStream_t s) {
    hipLaunchKernelGGL(k_galerkin_up, dim3(up.m, 9), dim3(256), 0, s, lo, up, Dlo, Aofflo, V, nkeep_up, Dup, Aoffup);
}

void launch_assemble_diag(const CoarseGeom& g, const double* Aint, const double* D, double* Ad, hipStream_t s) {
    hipLaunchKernelGGL(k_assemble_diag, dim3(g.m), dim3(128), 0, s, g, Aint, D, Ad);
}

void launch_blockic_setup(const CoarseGeom& g, const double* Ad, const double* Aoff, const int* nkeep,
                          double* Dinv, double* SM, double* AdT, int* bad, hipStream_t s) {
    // widest hyperplane of the parent's children: 3 (agg 2) or 12 (agg 4)
    const int wmax = g.agg == 2 ? 3 : kMaxPlane;
    const size_t shmem = (size_t)wmax * 3 * g.L * g.L * sizeof(double);
    if (g.L > kMaxL || wmax > plane_waves(g.L) || shmem > 64 * 1024)
        throw HipError{hipErrorInvalidValue, "block-IC set-up shape"};
    const dim3 nb(g.M), th(64 * wmax);
    SPECMG_LP_DISPATCH(g.L, hipLaunchKernelGGL(k_blockic_setup<LP>, nb, th, shmem, s, g, Ad, Aoff, nkeep, Dinv, bad));
    hipLaunchKernelGGL(k_blockic_couple, dim3(g.m), dim3(256), 0, s, g, Ad, Aoff, Dinv, SM, AdT);
}

void launch_build_coarsest(const CoarseGeom& g, const double* Ad, const double* Aoff, const int* cinv, int np,
                           double* dense, hipStream_t s) {
    hipLaunchKernelGGL(k_build_coarsest, dim3(g.m), dim3(128), 0, s, g, Ad, Aoff, cinv, np, dense);
}

template <typename S, typename T>
void launch_convert(const S* src, T* dst, int64_t n, hipStream_t s, const Scalars* sc) {
    int64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    hipLaunchKernelGGL((k_convert<S, T>), dim3((int)b), dim3(256), 0, s, src, dst, n, sc);
}

template void launch_coarse_smooth<double>(const CoarseGeom&, const double*, double*, int, double*, const Scalars*, int, hipStream_t);
template void launch_coarse_resid_restrict<double>(const CoarseGeom&, const double*, const double*, const double*,
                                                   const double*, const double*, const int*, int, double*,
                                                   const Scalars*, int, hipStream_t);
template void launch_coarse_prolong<double>(const CoarseGeom&, double*, const double*, const int*, int,
                                            const double*, const Scalars*, int, hipStream_t);
template void launch_coarse_resid_smooth<double>(const CoarseGeom&, const double*, const double*, const double*, const double*,
                                                 const double*, double*, const Scalars*, int, hipStream_t);
template void launch_coarsest<double>(int, int, const double*, const int*, const double*, int, int64_t, double*,
                                      const Scalars*, int, hipStream_t);
template void launch_convert<double, float>(const double*, float*, int64_t, hipStream_t, const Scalars*);
template void launch_convert<float, double>(const float*, double*, int64_t, hipStream_t, const Scalars*);

}  // namespace specmg
