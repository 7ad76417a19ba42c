// Fine-level kernels: the 7-point TPFA operator (eq. p / eq. discrete varia
// with harmonic-mean faces, fig. kappa edge), the block-Jacobi IC(0)
// smoother on the 8^3 coarse elements (Section 5), restriction/prolongation
// through the level-2 spectral bases (Algorithm 1, steps 2 and 8) and the
// fused CG vector updates.
//
// Tiling: a workgroup owns EX level-2 elements along x, i.e. an (8 EX)x8x8
// cell tile, with one wavefront per element.  Stencil phases stage the tile
// plus a one-cell halo in LDS; the IC(0) sweeps walk the 22 hyperplanes
// i+j+k = s of each element (cells on a hyperplane only depend on the
// previous one for lexicographic IC(0)).
#include <type_traits>

#include "common.hpp"

namespace specmg {

thread_local KernelEvents g_kev;


// ---------------------------------------------------------------------------
// hyperplane table of an 8^3 block: cells sorted by i+j+k
struct PlaneTable {
    unsigned short cell[512];
    unsigned short off[23];
};

constexpr PlaneTable make_planes() {
    PlaneTable t{};
    int p = 0;
    for (int s = 0; s < kPlanes; ++s) {
        t.off[s] = (unsigned short)p;
        for (int k = 0; k < 8; ++k)
            for (int j = 0; j < 8; ++j) {
                int i = s - j - k;
                if (i >= 0 && i < 8) t.cell[p++] = (unsigned short)(i + 8 * (j + 8 * k));
            }
    }
    t.off[kPlanes] = (unsigned short)p;
    return t;
}

__constant__ PlaneTable kPT = make_planes();

constexpr int kMaxCols = 12;   // padded basis width (target <= 8, plus 3)

template <typename T>
__device__ __forceinline__ T harm(T a, T b) {
    // harmonic mean 2ab/(a+b); zero when a neighbour is outside the domain
    // (a + b = 0).  1/(a+b) by Newton's iteration r <- r (2 - s r) from the
    // hardware reciprocal: two steps in float64, one in float32; no branch
    const T s = a + b;
    T r;
    if constexpr (sizeof(T) == 8) {
        r = __builtin_amdgcn_rcp(s);
        r = fma(fma(-s, r, 1.0), r, r);
        r = fma(fma(-s, r, 1.0), r, r);
    } else {
        r = __builtin_amdgcn_rcpf(s);
        r = fmaf(fmaf(-s, r, 1.0f), r, r);
    }
    const T v = (T(2) * a * b) * r;
    return s > T(0) ? v : T(0);
}

// LDS layouts use odd row pitches so that cells of one hyperplane spread
// over the banks: tile arrays x + PX (y + 8 z), haloed arrays
// (x+1) + HX ((y+1) + 10 (z+1)).
template <int EX>
struct TileT {
    static constexpr int TX = 8 * EX;
    static constexpr int NT = 64 * EX;
    static constexpr int LX = TX + 2;          // haloed row length (logical)
    static constexpr int NH = LX * 100;        // haloed cells (logical)
    static constexpr int HX = TX + 3;          // haloed row pitch (odd)
    static constexpr int HXY = HX * 10;
    static constexpr int NHP = HX * 100;       // haloed array size
    static constexpr int NC = TX * 64;         // tile cells
    static constexpr int PX = TX + 1;          // tile row pitch (odd)
    static constexpr int NCP = PX * 64;        // tile array size
};

template <int EX>
__device__ __forceinline__ int tidx(int x, int y, int z) {
    return x + TileT<EX>::PX * (y + 8 * z);
}

// a wavefront's LDS writes are visible to its later LDS reads; keeps the
// compiler from moving LDS accesses across the point
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void tile_origin(const FineGeom& g, int& x0, int& y0, int& z0) {
    int t = blockIdx.x;
    if (g.xcd_remap) {
        const int per = g.ntiles >> 3;
        t = (t & 7) * per + (t >> 3);
    }
    const int tx = t % g.ntx;
    const int r = t / g.ntx;
    x0 = tx * 8 * g.ex;
    y0 = (r % g.nty) * 8;
    z0 = (r / g.nty) * 8;
}

// Element of the wavefront in kernels that run four level-2 elements per
// 256-thread block (block ids remapped so that each XCD walks a contiguous
// range of elements).
__device__ __forceinline__ int block_element4() {
    const int nb = gridDim.x;
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    return b * 4 + (threadIdx.x >> 6);
}

__device__ __forceinline__ size_t gidx(const FineGeom& g, int x, int y, int z) {
    return (size_t)x + (size_t)g.nx * ((size_t)y + (size_t)g.ny * (size_t)z);
}

// Tiles (with a one-cell halo) of global cell arrays into LDS, zero outside
// Omega.  All loads of a thread are issued before any LDS store, so each
// wavefront keeps its whole share of the tile in flight.
template <int EX>
__device__ __forceinline__ bool halo_cell(const FineGeom& g, int h, int x0, int y0, int z0, size_t& gi,
                                          int& ph) {
    using TT = TileT<EX>;
    const int hx = h % TT::LX;
    const int r = h / TT::LX;
    const int x = x0 + hx - 1, y = y0 + (r % 10) - 1, z = z0 + (r / 10) - 1;
    const bool in = h < TT::NH && x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
    gi = in ? eidx(g, x, y, z) : 0;
    ph = hx + TT::HX * r;
    return in;
}

template <int EX>
__device__ __forceinline__ int hidx(int x, int y, int z) {
    return (x + 1) + TileT<EX>::HX * ((y + 1) + 10 * (z + 1));
}

// ---------------------------------------------------------------------------
// Pencil layout of the block IC(0) solves: one wavefront per 8^3 element;
// lane (j, k) = (lane & 7, lane >> 3) owns the x-pencil of cells (m, j, k).
// Slot r of a lane's registers holds cell m = (r - j - k) & 7, so on the
// hyperplane s = m + j + k every lane works on slot s & 7, a static register
// index.  A cell's neighbours in y and z are the same cell of lanes -+1 and
// -+8, kept there one slot lower (j-1, k-1) or higher (j+1, k+1); the
// neighbours in x are the lane's own slots r -+ 1.

__device__ __forceinline__ int pencil_m(int r, int jk) { return (r - jk) & 7; }

// The lane's 8 cells are contiguous in memory (64 bytes for float64): they
// move with 16-byte vector accesses and are rotated into (out of) the slot
// order in registers by a 3-stage barrel shifter on j + k.  Both candidates
// of each select pass through an empty asm statement: left alone, the
// compiler turns "on ? v[a] : v[b]" into v[on ? a : b], an access by a
// run-time index that it expands into 7 compares and 14 selects per slot
// and stage instead of 2 selects.
__device__ __forceinline__ void keep_value(double& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void keep_value(float& v) { asm volatile("" : "+v"(v)); }

template <typename T>
__device__ __forceinline__ void rotate_slots(T (&v)[8], int jk, bool inverse) {
#pragma unroll
    for (int b = 1; b < 8; b <<= 1) {
        const bool on = (jk & b) != 0;
        T t[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            T moved = v[inverse ? ((s + b) & 7) : ((s - b) & 7)], kept = v[s];
            keep_value(moved);
            keep_value(kept);
            t[s] = on ? moved : kept;
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) v[s] = t[s];
    }
}

// Pencil access in element order: the cells x = 2i, 2i + 1 of lane (j, k)'s
// x-pencil are the pair at p + kPair i, p the lane's cell (0, j, k), so the
// wavefront's load of pair i reads one contiguous block (see eidx).  Stored
// word T, values C (conversions on the way).
constexpr int kPair = 128;

template <typename T, typename C>
__device__ __forceinline__ void load8(const T* __restrict__ p, C (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (sizeof(T) == 8) {
            const double2 d = *reinterpret_cast<const double2*>(p + kPair * i);
            v[2 * i] = (C)d.x;
            v[2 * i + 1] = (C)d.y;
        } else {
            const float2 d = *reinterpret_cast<const float2*>(p + kPair * i);
            v[2 * i] = (C)d.x;
            v[2 * i + 1] = (C)d.y;
        }
    }
}
template <typename T, typename C>
__device__ __forceinline__ void store8(T* p, const C (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (sizeof(T) == 8)
            *reinterpret_cast<double2*>(p + kPair * i) = make_double2((double)v[2 * i], (double)v[2 * i + 1]);
        else
            *reinterpret_cast<float2*>(p + kPair * i) = make_float2((float)v[2 * i], (float)v[2 * i + 1]);
    }
}

// v[slot] = p[pencil cell of slot] (slot order of the IC(0) sweep)
template <typename T, typename C>
__device__ __forceinline__ void load_pencil(const T* __restrict__ p, C (&v)[8], int jk) {
    load8(p, v);
    rotate_slots(v, jk, false);
}
// p[pencil cell of slot] = v[slot] (v is consumed)
template <typename T, typename C>
__device__ __forceinline__ void store_pencil(T* p, C (&v)[8], int jk) {
    rotate_slots(v, jk, true);
    store8(p, v);
}

// Lane shifts by one in y.  DP: DPP row shifts inside the 16-lane rows
// (row_shr:1 / row_shl:1), lane l receives lane l - 1 (l + 1) on the vector
// ALU; otherwise bpermute through the LDS crossbar.  The lanes whose partner
// lies outside a DPP row or the wavefront are lanes j = 0 (j = 7) of a pencil
// row, the element's y faces, which the callers mask or replace.  DPP reads
// a source lane that is off in EXEC as out of range: call these on every
// lane, never inside a branch.
template <bool DP, typename T>
__device__ __forceinline__ T lane_prev(T v) {
    if constexpr (DP) return dpp_move<0x111>(v);
    else return __shfl_up(v, 1, 64);
}
template <bool DP, typename T>
__device__ __forceinline__ T lane_next(T v) {
    if constexpr (DP) return dpp_move<0x101>(v);
    else return __shfl_down(v, 1, 64);
}

// value of the same cell in lanes -+1 (y) and -+8 (z); lanes at the edge of
// the wavefront or of a DPP row get other values, which the callers mask
template <bool DP, typename T>
__device__ __forceinline__ T from_ym(const T (&v)[8], int r) { return lane_prev<DP>(v[(r + 7) & 7]); }
template <typename T>
__device__ __forceinline__ T from_zm(const T (&v)[8], int r) { return __shfl_up(v[(r + 7) & 7], 8, 64); }

// Forward and backward IC(0) substitution of the wavefront's element.
// y: in t, out (D+L^T)^{-1} D (D+L)^{-1} t.  ix: inverse pivots; fx, fy, fz:
// transmissibilities of each cell's minus faces (a_ij = -T).  A cell's plus
// face in y (z) is the minus face of the same cell in lane +1 (+8), fetched
// with the neighbour's value; its plus face in x is fx of the next slot.
// Faces that leave the element are dropped here: in y and z by the lane's
// position, in x at the pencil's ends.
template <bool DP, typename T>
__device__ __forceinline__ void ic_pencil(T (&y)[8], const T (&ix)[8], const T (&fx)[8], const T (&fy)[8],
                                          const T (&fz)[8], int j, int k) {
    const int jk = j + k;
    const T wym = j > 0 ? T(1) : T(0), wyp = j < 7 ? T(1) : T(0);
    const T wzm = k > 0 ? T(1) : T(0), wzp = k < 7 ? T(1) : T(0);
    T cur = T(0);
#pragma unroll
    for (int s = 0; s < kPlanes; ++s) {
        const int r = s & 7, rp = (s + 7) & 7;
        const T ny = lane_prev<DP>(cur);
        const T nz = __shfl_up(cur, 8, 64);
        const T xm = s - jk > 0 ? y[rp] : T(0);
        T acc = y[r];
        acc += fx[r] * xm;
        acc += (fy[r] * wym) * ny;
        acc += (fz[r] * wzm) * nz;
        const T v = acc * ix[r];
        const bool act = (unsigned)(s - jk) < 8u;
        y[r] = act ? v : y[r];
        cur = act ? v : cur;
    }
    cur = T(0);
#pragma unroll
    for (int s = kPlanes - 1; s >= 0; --s) {
        const int r = s & 7, rn = (s + 1) & 7;
        const T ny = lane_next<DP>(cur);
        const T nz = __shfl_down(cur, 8, 64);
        const T gy = lane_next<DP>(fy[rn]) * wyp;
        const T gz = __shfl_down(fz[rn], 8, 64) * wzp;
        const T xp = s - jk < 7 ? y[rn] : T(0);
        T acc = fx[rn] * xp;
        acc += gy * ny;
        acc += gz * nz;
        const T v = y[r] + ix[r] * acc;
        const bool act = (unsigned)(s - jk) < 8u;
        y[r] = act ? v : y[r];
        cur = act ? v : cur;
    }
}

// Minus-face transmissibilities of the pencil's cells inside the element
// (the neighbour's copy of kappa~ comes from the lane below).
template <bool DP, typename T>
__device__ __forceinline__ void pencil_faces(const T (&kc)[8], int jk, T (&fx)[8], T (&fy)[8], T (&fz)[8], T cy,
                                             T cz) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        fx[r] = harm(kc[r], kc[(r + 7) & 7]);
        fy[r] = harm(kc[r], from_ym<DP>(kc, r)) * cy;
        fz[r] = harm(kc[r], from_zm(kc, r)) * cz;
    }
    (void)jk;
}

// The same from three kappa~ pencils (orthotropic K): each axis's faces take
// the harmonic mean of its own component.
template <bool DP, typename T>
__device__ __forceinline__ void pencil_faces3(const T (&kx)[8], const T (&ky)[8], const T (&kz)[8], T (&fx)[8],
                                              T (&fy)[8], T (&fz)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        fx[r] = harm(kx[r], kx[(r + 7) & 7]);
        fy[r] = harm(ky[r], from_ym<DP>(ky, r));
        fz[r] = harm(kz[r], from_zm(kz, r));
    }
}

// minus-face transmissibilities of the lane's pencil (rotated slot order)
template <bool O, bool DP, typename T, typename C>
__device__ __forceinline__ void load_faces(const FineGeom& g, const T* __restrict__ kt, size_t row, int jk,
                                           C (&fx)[8], C (&fy)[8], C (&fz)[8]) {
    C kc[8];
    load_pencil(kt + row, kc, jk);
    if constexpr (O) {
        const size_t N = g.ncell();
        C ky[8], kz[8];
        load_pencil(kt + N + row, ky, jk);
        load_pencil(kt + 2 * N + row, kz, jk);
        pencil_faces3<DP>(kc, ky, kz, fx, fy, fz);
    } else {
        pencil_faces<DP>(kc, jk, fx, fy, fz, (C)g.cy, (C)g.cz);
    }
}

// ---------------------------------------------------------------------------
// pre-smoothing: (optionally r -= alpha q with ||r||^2) then u = M^{-1} r
// mode bit0: update r and reduce ||r||^2 (sets the converged flag)
// mode bit1: return at once when the solve is finished
// T: stored word of kappa~, 1/d and u; C: arithmetic (T, or float64 with
// float32 storage); O: three kappa~ arrays (orthotropic K)
// Held to 128 registers (130 otherwise): the 4096 wavefronts of 128^3 are then
// all resident, 26.0 -> 23.9 us; 256^3 139 -> 137 us.
template <int EX, typename T, typename C, bool O>
__global__ __launch_bounds__(64 * EX) __attribute__((amdgpu_waves_per_eu(O ? 1 : 4))) void k_pre_smooth(FineGeom g, const T* __restrict__ kt,
                                                        const T* __restrict__ invd, double* r,
                                                        const double* __restrict__ q, T* __restrict__ u,
                                                        Scalars* sc, RedBuf rb, int mode) {
    if ((mode & 2) && sc->done) return;
    __shared__ double sred[EX];
    int x0, y0, z0;
    tile_origin(g, x0, y0, z0);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 7, k = lane >> 3, jk = j + k;
    const size_t row = eidx(g, x0 + 8 * w, y0 + j, z0 + k);   // cell (0, j, k) of the element
    const double alpha = (mode & 1) ? sc->alpha : 0.0;
    // phases in order, each one's registers released before the next
    // (faces first, then the residual update, then the pivots)
    C fx[8], fy[8], fz[8];
    load_faces<O, false>(g, kt, row, jk, fx, fy, fz);
    __builtin_amdgcn_sched_barrier(0);
    C y[8];
    double rr = 0.0;
    {
        double vr[8], vq[8];
        load_pencil(r + row, vr, jk);
        if (mode & 1) {
            load_pencil(q + row, vq, jk);
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                vr[s] -= alpha * vq[s];
                rr += vr[s] * vr[s];
            }
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) y[s] = (C)vr[s];
        if (mode & 1) store_pencil(r + row, vr, jk);
    }
    __builtin_amdgcn_sched_barrier(0);
    C ix[8];
    load_pencil(invd + row, ix, jk);
    ic_pencil<false>(y, ix, fx, fy, fz, j, k);
    store_pencil(u + row, y, jk);
    if (mode & 1) {
        double v[1] = {block_sum(rr, sred)};
        write_partials<1>(v, rb);
    }
}

// s = r - A u, then r2[e][j] = sum_c phi[e][j][c] s_c for every element.
// The lane's 8 values of one basis column (phi_pos layout): pair i at
// col + 128 i + 2 lane, so each load instruction reads one contiguous block.
template <typename TB, typename C>
__device__ __forceinline__ void load_col(const TB* __restrict__ col, int lane, C (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (sizeof(TB) == 8) {
            const double2 d = reinterpret_cast<const double2*>(col)[i * 64 + lane];
            v[2 * i] = (C)d.x;
            v[2 * i + 1] = (C)d.y;
        } else {
            const float2 d = reinterpret_cast<const float2*>(col)[i * 64 + lane];
            v[2 * i] = (C)d.x;
            v[2 * i + 1] = (C)d.y;
        }
    }
}


// The cells beyond the element's four y and z faces, in the wavefront's LDS
// area ff[8][64].  All 64 lanes load them together, one cell per face and array
// (lane = (x, row) of the face; zero outside the domain; the face's own component
// for orthotropic K).  Beyond the minus faces u goes to ff[0] (y) and ff[2] (z),
// kappa~ to ff[1] and ff[3], for the lanes whose neighbours they are.  Through the
// plus faces (whose lanes get no transmissibility from a neighbour) it is formed
// here, one face cell a lane, with kappa~ of the row inside passed through LDS:
// ff[4] (y) and ff[6] (z), u beyond in ff[5] and ff[7].
template <bool O, typename T, typename C>
__device__ __forceinline__ void stage_faces_yz(const FineGeom& g, const T* __restrict__ kt, const T* __restrict__ u,
                                               int x0, int y0, int z0, int lane, const C (&ky)[8], const C (&kz)[8],
                                               C* ff) {
    const int fx = lane & 7, fr = lane >> 3;
    const size_t N = O ? g.ncell() : 0;
    C vu[4], vk[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {   // -y, -z, +y, +z
        const int o = f < 2 ? -1 : 8;
        const int yy = f % 2 == 0 ? y0 + o : y0 + fr, zz = f % 2 == 0 ? z0 + fr : z0 + o;
        const bool in = yy >= 0 && yy < g.ny && zz >= 0 && zz < g.nz;
        const size_t gi = in ? eidx(g, x0 + fx, yy, zz) : 0;
        vu[f] = in ? (C)u[gi] : C(0);
        vk[f] = in ? (C)kt[(f % 2 == 0 ? N : 2 * N) + gi] : C(0);
    }
    if ((lane & 7) == 7) {
#pragma unroll
        for (int x = 0; x < 8; ++x) ff[4 * 64 + (lane & ~7) + x] = ky[x];
    }
    if (lane >= 56) {
#pragma unroll
        for (int x = 0; x < 8; ++x) ff[6 * 64 + 8 * (lane & 7) + x] = kz[x];
    }
    wave_lds_sync();
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        const C ki = ff[(4 + 2 * f) * 64 + lane];
        ff[2 * f * 64 + lane] = vu[f];
        ff[(2 * f + 1) * 64 + lane] = vk[f];
        ff[(4 + 2 * f) * 64 + lane] = harm(ki, vk[2 + f]) * (C)(f == 0 ? g.cy : g.cz);
        ff[(5 + 2 * f) * 64 + lane] = vu[2 + f];
    }
    wave_lds_sync();
}

// s -= A u on the x-pencil of row (j, k) of an element, natural order
// inside the pencil: uc, kc the row's u and kappa~ (kappa~_x for orthotropic
// K; ky, kz its y and z components), um, km and up, kp u and kappa~ of the
// cells before and after the pencil in x (used when xlo, xhi: inside the
// domain), ff the staged y and z faces (stage_faces_yz).  A lane forms the
// transmissibilities of its minus faces and hands them to its neighbours, whose
// plus faces they are (the same in both directions to the last bit); neighbours
// inside the element are the lanes -+1 and -+8: through the LDS crossbar
// (bpermute), or with DY those in y by DPP row shifts, which take VALU issue slots
// and registers instead (the better trade where the crossbar also carries an IC(0)
// sweep).  Each face is one product and sum on s, in the order -x, +x, -y, +y, -z,
// +z: on media of contrast 1e6 the last bit of the pressure is visible in the face
// fluxes, so the order of the sums is part of the result.  The barriers bound the
// values in flight; one z cell at a time keeps the isotropic post-smoother (DY) at 167
// registers, three wavefronts a SIMD, where four at a time took 171: 34.6 -> 32.9 us
// at 128^3, 195 -> 170 at 256^3, 1.58 -> 1.40 ms at 512^3.
template <bool O, bool DY, typename C>
__device__ __forceinline__ void pencil_apply(const FineGeom& g, int j, int k, const C (&uc)[8],
                                             const C (&kc)[8], const C (&ky)[8], const C (&kz)[8], C um, C km,
                                             C up, C kp, bool xlo, bool xhi, const C* ff, C (&s)[8]) {
    // x faces: inside the pencil, then the two ends
#pragma unroll
    for (int x = 0; x < 7; ++x) {
        const C d = harm(kc[x], kc[x + 1]) * (uc[x] - uc[x + 1]);
        s[x] -= d;
        s[x + 1] += d;
    }
    if (xlo) s[0] -= harm(kc[0], km) * (uc[0] - um);
    if (xhi) s[7] -= harm(kc[7], kp) * (uc[7] - up);
    __builtin_amdgcn_sched_barrier(0);
    // y and z faces.  The shifts run on every lane before the selects: a DPP
    // source lane that is switched off in EXEC reads as out of range.
    const C* fy = ff + 8 * k;
    const C* fz = ff + 128 + 8 * j;
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const C ko = O ? ky[x] : kc[x];
        const C pu = lane_prev<DY>(uc[x]), pk = lane_prev<DY>(ko), qu = lane_next<DY>(uc[x]);
        const C ou = fy[x], ok = fy[64 + x], ht = fy[256 + x], hu = fy[320 + x];
        const C t = harm(ko, j == 0 ? ok : pk) * (C)g.cy;
        const C nt = lane_next<DY>(t);
        s[x] -= t * (uc[x] - (j == 0 ? ou : pu));
        s[x] -= (j == 7 ? ht : nt) * (uc[x] - (j == 7 ? hu : qu));
        if (x % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const C ko = O ? kz[x] : kc[x];
        const C pu = __shfl_up(uc[x], 8, 64), pk = __shfl_up(ko, 8, 64), qu = __shfl_down(uc[x], 8, 64);
        const C ou = fz[x], ok = fz[64 + x], ht = fz[256 + x], hu = fz[320 + x];
        const C t = harm(ko, k == 0 ? ok : pk) * (C)g.cz;
        const C nt = __shfl_down(t, 8, 64);
        s[x] -= t * (uc[x] - (k == 0 ? ou : pu));
        s[x] -= (k == 7 ? ht : nt) * (uc[x] - (k == 7 ? hu : qu));
        if ((DY && !O) || x % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
}

// s -= A u on the x-pencil of row (j, k) of the element whose first cell is
// (x0, y0, z0); row = element-order index of (x0, y0 + j, z0 + k).  The
// row's u and kappa~ (kappa~_x for orthotropic K) are returned in uc, kc.
// Every load (the row, the pencil ends in x, the staged faces) is issued
// before the arithmetic, so a wavefront waits for memory once.
template <bool O, bool DY, typename T, typename C>
__device__ __forceinline__ void pencil_residual(const FineGeom& g, const T* __restrict__ kt, const T* __restrict__ u,
                                                size_t row, int x0, int y0, int z0, int lane, int j, int k,
                                                C* ff, C (&s)[8], C (&uc)[8], C (&kc)[8]) {
    const size_t N = O ? g.ncell() : 0;   // offsets of the y and z arrays
    C ky[8], kz[8];
    load8(u + row, uc);
    load8(kt + row, kc);
    if constexpr (O) {
        load8(kt + N + row, ky);
        load8(kt + 2 * N + row, kz);
    }
    const bool xlo = x0 > 0, xhi = x0 + 8 < g.nx;
    const size_t im = xlo ? eidx(g, x0 - 1, y0 + j, z0 + k) : row;
    const size_t ip = xhi ? eidx(g, x0 + 8, y0 + j, z0 + k) : row;
    const C um = xlo ? (C)u[im] : C(0), km = xlo ? (C)kt[im] : C(0);
    const C up = xhi ? (C)u[ip] : C(0), kp = xhi ? (C)kt[ip] : C(0);
    stage_faces_yz<O>(g, kt, u, x0, y0, z0, lane, O ? ky : kc, O ? kz : kc, ff);
    pencil_apply<O, DY>(g, j, k, uc, kc, ky, kz, um, km, up, kp, xlo, xhi, ff, s);
}

// Sums the block partials of one reduction and applies the CG scalar update
// of the reduction site.  Block b sums partials [b kFinSpan, (b + 1) kFinSpan);
// with several blocks each publishes its sum, and the block that arrives last
// (an agent-scope ticket, reset by that block) adds them in block order.  Every
// sum runs in a fixed order, so the result does not depend on timing.  A chain
// of memory latencies between two full-grid kernels, so everything that is read
// is read at once, the flag and the scalars too (waited for together before
// the flag is looked at), and a single block (up to 2048 partials, 128^3 and
// below) goes straight on to the scalars: 4.3 -> 2.8 us at 32^3, 4.8 -> 3.7 at
// 96^3, 5.3 -> 4.7 at 128^3.
// ONE: called by the last block of another kernel, for at most kFinSpan partials.
template <bool ONE>
__device__ __forceinline__ void finalize_blocks(int site, int nb, Scalars* sc, RedBuf rb, double* out, int check_done) {
    __shared__ double sred[2][kFinThreads / 64];
    __shared__ int last;
    const int nv = (site == RS_RZ || site == RS_GEN2) ? 2 : 1;
    const int b0 = ONE ? 0 : blockIdx.x * kFinSpan, lim = min(kFinSpan, nb - b0);
    double a[2][kFinPer];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int u = 0; u < kFinPer; ++u) {
            const int i = u * kFinThreads + threadIdx.x;
            a[k][u] = k < nv && i < lim ? rb.partial[(size_t)k * kMaxRedBlocks + b0 + i] : 0.0;
        }
    Scalars in{};
    if (sc) in = *sc;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int u = 0; u < kFinPer; ++u) asm volatile("" : "+v"(a[k][u]));
    if (check_done && in.done) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    auto sum2 = [&](double x, double y, double (&t)[2]) {
        x = wave_sum(x);
        y = wave_sum(y);
        __syncthreads();
        if (lane == 0) {
            sred[0][w] = x;
            sred[1][w] = y;
        }
        __syncthreads();
        t[0] = t[1] = 0.0;
#pragma unroll
        for (int i = 0; i < kFinThreads / 64; ++i) {
            t[0] += sred[0][i];
            t[1] += sred[1][i];
        }
    };
    double v[2] = {0.0, 0.0}, t[2];
#pragma unroll
    for (int u = 0; u < kFinPer; ++u) {
        v[0] += a[0][u];
        v[1] += a[1][u];
    }
    sum2(v[0], v[1], t);
    if (!ONE && gridDim.x > 1) {
        if (threadIdx.x == 0) {
            for (int k = 0; k < nv; ++k)
                __hip_atomic_store(rb.partial2 + k * kFinBlocks + blockIdx.x, t[k], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            const unsigned prev = __hip_atomic_fetch_add(rb.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            last = prev == gridDim.x - 1;
        }
        __syncthreads();
        if (!last) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        for (int k = 0; k < nv; ++k)
            v[k] = threadIdx.x < gridDim.x ? atomic_load_relaxed(rb.partial2 + k * kFinBlocks + threadIdx.x) : 0.0;
        sum2(v[0], nv > 1 ? v[1] : 0.0, t);
        if (threadIdx.x == 0) __hip_atomic_store(rb.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x != 0) return;
    if (site == RS_PQ) {
        sc->pq = t[0];
        sc->iter = in.iter + 1;
        if (!(t[0] > 0.0) || !isfinite(t[0])) {
            sc->done = 2;
            sc->alpha = 0.0;
            sc->alpha_x = 0.0;
        } else {
            sc->alpha = in.rz / t[0];
            sc->alpha_x = in.rz / t[0];
        }
    } else if (site == RS_RR) {
        sc->rr = t[0];
        if (t[0] <= in.thresh2) sc->done = 1;
        else if (!isfinite(t[0])) sc->done = 2;
    } else if (site == RS_RZ) {
        const double old = in.rz;
        double beta = 0.0;
        if (old != 0.0) beta = in.flexible ? (-in.alpha * t[1] / old) : (t[0] / old);
        sc->beta = beta;
        sc->rz_new = t[0];
        sc->zq = t[1];
        sc->rz = t[0];
    } else {
        out[0] = t[0];
        if (nv == 2) out[1] = t[1];
    }
}

// T: stored word of kappa~ and u; TB: stored word of the basis; C: the
// arithmetic and the word of the level-2 residual r2.  rr_parts: one block more
// than the elements need sums the pre-smoother's ||r||^2, whose outcome (the
// converged flag) stops the kernels after this one: a launch of its own, 4.7 us
// at 128^3, waited for nothing that this kernel does.
template <typename T, typename TB, typename C, bool O>
__global__ __launch_bounds__(256) void k_resid_restrict(FineGeom g, const T* __restrict__ kt,
                                                       const T* __restrict__ u, const double* __restrict__ r,
                                                       const TB* __restrict__ phi, const int* __restrict__ nkeep,
                                                       int L, C* __restrict__ r2, Scalars* sc, RedBuf rb,
                                                       int rr_parts, int check_done) {
    if (rr_parts && blockIdx.x == gridDim.x - 1) {
        finalize_blocks<true>(RS_RR, rr_parts, sc, rb, nullptr, check_done);
        return;
    }
    if (check_done && sc->done) return;
    __shared__ C sff[4][512];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = g.mx * g.my * g.mz;
    const int nb = gridDim.x - (rr_parts ? 1 : 0);
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int e = b * 4 + (threadIdx.x >> 6);
    if (e >= m) return;   // whole wavefront; no block barriers below
    const int ex = e % g.mx, ey = (e / g.mx) % g.my, ez = e / (g.mx * g.my);
    const int j = lane & 7, k = lane >> 3;
    const int x0 = ex * 8;
    const size_t row = (size_t)e * kSub3 + 2 * lane;   // cell (0, j, k)
    C s[8];
    {
        load8(r + row, s);
        C uc[8], kc[8];
        pencil_residual<O, false>(g, kt, u, row, x0, ey * 8, ez * 8, lane, j, k, sff[w], s, uc, kc);
    }
    // restriction onto the element's kept basis vectors
    const int nkp = nkeep[e];
    const TB* ph = phi + (size_t)e * L * kSub3;
    C acc[kMaxCols];
#pragma unroll
    for (int jj = 0; jj < kMaxCols; ++jj) {
        C a = C(0);
        if (jj < nkp) {
            C pv[8];
            load_col(ph + (size_t)jj * kSub3, lane, pv);
#pragma unroll
            for (int x = 0; x < 8; ++x) a += (C)pv[x] * s[x];
        }
        acc[jj] = a;
        // at most three columns of loads in flight (register budget)
        if (jj % 3 == 2) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int jj = 0; jj < kMaxCols; ++jj) {
        const C v = wave_sum(acc[jj]);
        if (lane == 0 && jj < L) r2[(size_t)e * L + jj] = v;
    }
}

// u += phi e2 on every element (prolongation, Algorithm 1 step 8), one
// wavefront per element: lane = pencil, the basis read column by column
// (load_col); the sum is formed in C, the word of e2
template <typename T, typename TB, typename C>
__global__ __launch_bounds__(256) void k_prolong(FineGeom g, T* u, const TB* __restrict__ phi,
                                                  const int* __restrict__ nkeep, int L,
                                                  const C* __restrict__ e2, const Scalars* sc,
                                                  int check_done) {
    if (check_done && sc->done) return;
    const int lane = threadIdx.x & 63;
    const int e = block_element4();
    if (e >= g.mx * g.my * g.mz) return;   // whole wavefront; no block barriers
    const int nk = nkeep[e];
    const TB* ph = phi + (size_t)e * L * kSub3;
    const C* ee = e2 + (size_t)e * L;
    const size_t row = (size_t)e * kSub3 + 2 * lane;   // cell (0, j, k)
    C uc[8];
    load8(u + row, uc);
#pragma unroll
    for (int jj = 0; jj < kMaxCols; ++jj) {
        if (jj < nk) {
            C pv[8];
            load_col(ph + (size_t)jj * kSub3, lane, pv);
            const C a = ee[jj];
#pragma unroll
            for (int x = 0; x < 8; ++x) uc[x] += pv[x] * a;
        }
        if (jj % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    store8(u + row, uc);
}

// Post-smoothing with its residual (Algorithm 1 step 9): t = r - A u on
// the wavefront's element (pencil_residual), z = u + M^{-1} t, without t
// going through memory.  The row's r and u wait in the wavefront's LDS area
// while the IC(0) sweep holds the registers.  mode bit0: reduce r.z (and
// z.q when flexible) for the CG beta; bit1: return at once when the solve is
// finished.
template <int EX, typename T, typename C, bool O>
__global__ __launch_bounds__(64 * EX) void k_post_fused(FineGeom g, const T* __restrict__ kt,
                                                        const T* __restrict__ invd, const T* __restrict__ u,
                                                        const double* __restrict__ r, const double* __restrict__ q,
                                                        double* __restrict__ z, Scalars* sc, RedBuf rb, int mode) {
    if ((mode & 2) && sc->done) return;
    __shared__ double sred[EX];
    __shared__ C sa[EX][512];        // y and z faces, then the row's u
    __shared__ double srr[EX][512];  // the row's r
    int x0, y0, z0;
    tile_origin(g, x0, y0, z0);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 7, k = lane >> 3, jk = j + k;
    const int ex0 = x0 + 8 * w;
    const size_t row = eidx(g, ex0, y0 + j, z0 + k);
    C s[8], uc[8], kc[8];
    {
        double rv[8];
        load8(r + row, rv);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            s[x] = (C)rv[x];
            srr[w][x * 64 + lane] = rv[x];
        }
    }
    pencil_residual<O, true>(g, kt, u, row, ex0, y0, z0, lane, j, k, sa[w], s, uc, kc);
    wave_lds_sync();
#pragma unroll
    for (int x = 0; x < 8; ++x) sa[w][x * 64 + lane] = uc[x];
    __builtin_amdgcn_sched_barrier(0);
    // faces and pivots of the IC(0) sweep in slot order
    C fx[8], fy[8], fz[8];
    if constexpr (O) {
        load_faces<true, true>(g, kt, row, jk, fx, fy, fz);
    } else {
        rotate_slots(kc, jk, false);
        pencil_faces<true>(kc, jk, fx, fy, fz, (C)g.cy, (C)g.cz);
    }
    C ix[8];
    load_pencil(invd + row, ix, jk);
    rotate_slots(s, jk, false);
    ic_pencil<true>(s, ix, fx, fy, fz, j, k);
    rotate_slots(s, jk, true);
    __builtin_amdgcn_sched_barrier(0);
    double rz = 0.0, zq = 0.0;
    const int flex = (mode & 1) ? sc->flexible : 0;
    double qv[8];
    if (flex) load8(q + row, qv);
    double zv[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        zv[x] = (double)sa[w][x * 64 + lane] + (double)s[x];
        if (mode & 1) {
            rz += srr[w][x * 64 + lane] * zv[x];
            if (flex) zq += zv[x] * qv[x];
        }
    }
    store8(z + row, zv);
    if (mode & 1) {
        double v[2] = {block_sum(rz, sred), block_sum(zq, sred)};
        write_partials<2>(v, rb);
    }
}

// First half of a CG step: p = z + beta p_old (p = z on the first
// iteration) and x += alpha_x p_old (the x update deferred from the
// previous iteration), one double2 per thread.
__global__ __launch_bounds__(256) void k_p_update(const double2* __restrict__ z, const double2* __restrict__ pold,
                                                  double2* __restrict__ pnew, double2* __restrict__ x,
                                                  const Scalars* sc, int first, int64_t n2) {
    if (sc->done) return;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n2) return;
    double2 p = z[i];
    if (!first) {
        const double beta = sc->beta, ax = sc->alpha_x;
        const double2 po = pold[i];
        p.x += beta * po.x;
        p.y += beta * po.y;
        if (ax != 0.0) {
            double2 xv = x[i];
            xv.x += ax * po.x;
            xv.y += ax * po.y;
            x[i] = xv;
        }
    }
    pnew[i] = p;
}

// Second half: q = A p and the block sums of p.q, one level-2 element per
// wavefront (pencil_residual with a zero right-hand side).
template <bool O>
__global__ __launch_bounds__(256) void k_spmv_pcg(FineGeom g, const double* __restrict__ kt,
                                                  const double* __restrict__ p, double* __restrict__ q,
                                                  Scalars* sc, RedBuf rb, int pbuf) {
    if (sc->done) return;
    __shared__ double sff[4][512];
    __shared__ double sred[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = block_element4();
    double pq = 0.0;
    if (e < g.mx * g.my * g.mz) {   // whole wavefront; the block sum below is reached by all
        const int ex = e % g.mx, ey = (e / g.mx) % g.my, ez = e / (g.mx * g.my);
        const int j = lane & 7, k = lane >> 3;
        const size_t row = (size_t)e * kSub3 + 2 * lane;   // cell (0, j, k)
        double s[8], pc[8], kc[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = 0.0;
        pencil_residual<O, false>(g, kt, p, row, ex * 8, ey * 8, ez * 8, lane, j, k, sff[w], s, pc, kc);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s[i] = -s[i];
            pq += pc[i] * s[i];
        }
        store8(q + row, s);
    }
    double v[1] = {block_sum(pq, sred)};
    write_partials<1>(v, rb);
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->pbuf = pbuf;
}

// y = A x (resid = 0) or y = b - A x (resid = 1), element order; O:
// orthotropic K
template <bool O>
__global__ __launch_bounds__(256) void k_apply_A(FineGeom g, const double* __restrict__ kt,
                                                 const double* __restrict__ xv, const double* __restrict__ b,
                                                 double* __restrict__ y, int resid) {
    __shared__ double sff[4][512];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = block_element4();
    if (e >= g.mx * g.my * g.mz) return;   // whole wavefront; no block barriers
    const int ex = e % g.mx, ey = (e / g.mx) % g.my, ez = e / (g.mx * g.my);
    const int j = lane & 7, k = lane >> 3;
    const size_t row = (size_t)e * kSub3 + 2 * lane;   // cell (0, j, k)
    double s[8], uc[8], kc[8];
    if (resid) {
        load8(b + row, s);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = 0.0;
    }
    pencil_residual<O, false>(g, kt, xv, row, ex * 8, ey * 8, ez * 8, lane, j, k, sff[w], s, uc, kc);
    if (!resid) {
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = -s[i];
    }
    store8(y + row, s);
}

// IC(0) pivots of every 8^3 block: d_i = a_ii - sum_{j<i} a_ij^2 / d_j, with
// a_ii summing all six faces (faces leaving the block included).
template <int EX>
__global__ __launch_bounds__(64 * EX) void k_ic_setup(FineGeom g, const double* __restrict__ kt,
                                                      double* __restrict__ invd, float* invd32,
                                                      int* bad) {
    using TT = TileT<EX>;
    __shared__ double sK[3][TT::NHP];
    __shared__ double sDg[TT::NCP];
    int x0, y0, z0;
    tile_origin(g, x0, y0, z0);
    // kappa~ of each face direction (one array, or three for orthotropic K)
    const size_t N = g.ortho ? g.ncell() : 0;
    for (int h = threadIdx.x; h < TT::NH; h += TT::NT) {
        size_t gi;
        int ph;
        const bool in = halo_cell<EX>(g, h, x0, y0, z0, gi, ph);
        for (int d = 0; d < 3; ++d) sK[d][ph] = in ? kt[d * N + gi] : 0.0;
    }
    __syncthreads();
    constexpr int HX = TT::HX, HXY = TT::HXY, TX = TT::TX;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int s = 0; s < kPlanes; ++s) {
        const int o = kPT.off[s];
        const int cnt = kPT.off[s + 1] - o;
        if (lane < cnt) {
            const int c = kPT.cell[o + lane];
            const int i = c & 7, j = (c >> 3) & 7, k = c >> 6;
            const int ti = 8 * w + i + TX * (j + 8 * k);
            const int h = hidx<EX>(8 * w + i, j, k);
            const double kx = sK[0][h], ky = sK[1][h], kz = sK[2][h];
            double diag = harm(kx, sK[0][h - 1]) + harm(kx, sK[0][h + 1]) + harm(ky, sK[1][h - HX]) * g.cy +
                          harm(ky, sK[1][h + HX]) * g.cy + harm(kz, sK[2][h - HXY]) * g.cz +
                          harm(kz, sK[2][h + HXY]) * g.cz;
            if (i > 0) {
                const double t = harm(kx, sK[0][h - 1]);
                diag -= t * t / sDg[ti - 1];
            }
            if (j > 0) {
                const double t = harm(ky, sK[1][h - HX]) * g.cy;
                diag -= t * t / sDg[ti - TX];
            }
            if (k > 0) {
                const double t = harm(kz, sK[2][h - HXY]) * g.cz;
                diag -= t * t / sDg[ti - 8 * TX];
            }
            sDg[ti] = diag;
            if (!(diag > 0.0)) atomicOr(bad, 1);
        }
        __syncthreads();
    }
    for (int c = threadIdx.x; c < TT::NC; c += TT::NT) {
        const int x = c % TX, y = (c / TX) & 7, z = c / (TX * 8);
        const size_t gi = eidx(g, x0 + x, y0 + y, z0 + z);
        const double v = 1.0 / sDg[c];
        invd[gi] = v;
        if (invd32) invd32[gi] = (float)v;
    }
}

// kappa~ = perm * scale, read in natural order and written in element order
__global__ void k_perm_to_kt(FineGeom g, const double* __restrict__ perm, double* __restrict__ kt, float* kt32,
                             double scale, int* bad) {
    const int64_t n = (int64_t)g.ncell();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double p = perm[i];
        if (!(p > 0.0) || !isfinite(p)) atomicOr(bad, 1);
        const double v = p * scale;
        const int x = (int)(i % g.nx), y = (int)((i / g.nx) % g.ny), z = (int)(i / ((int64_t)g.nx * g.ny));
        const size_t ei = eidx(g, x, y, z);
        kt[ei] = v;
        if (kt32) kt32[ei] = (float)v;
    }
}
__global__ void k_perm3_to_kt(FineGeom g, const double* __restrict__ perm, double* __restrict__ kt, double sx,
                              double sy, double sz, int* bad) {
    const int64_t n = (int64_t)g.ncell();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < 3 * n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double p = perm[i];
        if (!(p > 0.0) || !isfinite(p)) atomicOr(bad, 1);
        const int64_t d = i / n, c = i - d * n;
        const int x = (int)(c % g.nx), y = (int)((c / g.nx) % g.ny), z = (int)(c / ((int64_t)g.nx * g.ny));
        kt[(size_t)d * n + eidx(g, x, y, z)] = p * (d == 0 ? sx : (d == 1 ? sy : sz));
    }
}
// one cell array between natural order and element order
__global__ void k_to_elem(FineGeom g, const double* __restrict__ nat, double* __restrict__ el) {
    const int64_t n = (int64_t)g.ncell();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(i % g.nx), y = (int)((i / g.nx) % g.ny), z = (int)(i / ((int64_t)g.nx * g.ny));
        el[eidx(g, x, y, z)] = nat[i];
    }
}
__global__ void k_to_natural(FineGeom g, const double* __restrict__ el, double* __restrict__ nat) {
    const int64_t n = (int64_t)g.ncell();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(i % g.nx), y = (int)((i / g.nx) % g.ny), z = (int)(i / ((int64_t)g.nx * g.ny));
        nat[i] = el[eidx(g, x, y, z)];
    }
}

__global__ __launch_bounds__(256) void k_dot(const double* __restrict__ a, const double* __restrict__ b,
                                              int64_t n, RedBuf rb) {
    __shared__ double sred[4];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        s += a[i] * b[i];
    double v[1] = {block_sum(s, sred)};
    write_partials<1>(v, rb);
}

__global__ __launch_bounds__(256) void k_sum_abs(const double* __restrict__ a, int64_t n, RedBuf rb) {
    __shared__ double sred[4];
    double s = 0.0, t = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        s += a[i];
        t += fabs(a[i]);
    }
    double v[2] = {block_sum(s, sred), block_sum(t, sred)};
    write_partials<2>(v, rb);
}

__global__ __launch_bounds__(kFinThreads) void k_finalize(int site, int nb, Scalars* sc, RedBuf rb, double* out,
                                                          int check_done) {
    finalize_blocks<false>(site, nb, sc, rb, out, check_done);
}

void launch_finalize(int site, int nblocks, Scalars* sc, RedBuf rb, double* out, int check_done,
                     hipStream_t s) {
    const int nfb = nblocks > 0 ? (nblocks + kFinSpan - 1) / kFinSpan : 1;
    hipLaunchKernelGGL(k_finalize, dim3(nfb), dim3(kFinThreads), 0, s, site, nblocks, sc, rb, out, check_done);
}

__global__ void k_axpy_x(double* x, const double* __restrict__ p0, const double* __restrict__ p1,
                         Scalars* sc, int64_t n) {
    const double a = sc->alpha_x;
    const double* p = sc->pbuf ? p1 : p0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] += a * p[i];
}

__global__ void k_clear_alpha_x(Scalars* sc) { sc->alpha_x = 0.0; }

__global__ void k_sub_mean(double* x, int64_t n, const double* sum) {
    const double m = *sum / (double)n;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] -= m;
}

__global__ void k_fill(double* d, double v, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        d[i] = v;
}

__global__ void k_copy(double* d, const double* __restrict__ s, int64_t n, const Scalars* sc) {
    if (sc && sc->done) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        d[i] = s[i];
}

__global__ void k_pcg_init(Scalars* sc, double thresh2, int flexible) {
    sc->rz = 0.0;
    sc->rz_new = 0.0;
    sc->pq = 0.0;
    sc->alpha = 0.0;
    sc->alpha_x = 0.0;
    sc->beta = 0.0;
    sc->rr = 0.0;
    sc->thresh2 = thresh2;
    sc->zq = 0.0;
    sc->sum = 0.0;
    sc->sum2 = 0.0;
    sc->done = 0;
    sc->iter = 0;
    sc->flexible = flexible;
    sc->pbuf = 0;
}

// ---------------------------------------------------------------------------
// launchers

static inline int grid_1d(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    return (int)b;
}

// tiles of 2 elements (mx even) or 1; set-up never builds wider ones
#define SPECMG_EX_DISPATCH(EXV, ...)          \
    switch (EXV) {                            \
        case 2: {                             \
            constexpr int EX = 2;             \
            __VA_ARGS__;                      \
        } break;                              \
        default: {                            \
            constexpr int EX = 1;             \
            __VA_ARGS__;                      \
        } break;                              \
    }

// O = g.ortho as a compile-time flag; orthotropic kernels exist for float64
// coefficients only (set-up rejects the float32 fine level with three
// components)
#define SPECMG_O_DISPATCH(T, ...)                                                          \
    if (g.ortho) {                                                                         \
        if constexpr (std::is_same<T, double>::value) {                                    \
            constexpr bool O = true;                                                       \
            __VA_ARGS__;                                                                   \
        } else {                                                                           \
            throw HipError{hipErrorInvalidValue, "orthotropic K needs float64 coefficients"}; \
        }                                                                                  \
    } else {                                                                               \
        constexpr bool O = false;                                                          \
        __VA_ARGS__;                                                                       \
    }

// the sum of ||r||^2 rides in the residual's launch if one block can form it
bool rr_with_restrict(const FineGeom& g) { return g.ntiles <= kFinSpan; }

template <typename T, typename C>
void launch_pre_smooth(const FineGeom& g, const T* kt, const T* invd, double* r, const double* q, T* u,
                       Scalars* sc, RedBuf rb, int mode, bool rr_rides, hipStream_t s) {
    SPECMG_O_DISPATCH(T, SPECMG_EX_DISPATCH(g.ex, SPECMG_TIMED_LAUNCH((k_pre_smooth<EX, T, C, O>), dim3(g.ntiles),
                                                                      dim3(64 * EX), 0, s, g, kt, invd, r, q, u, sc,
                                                                      rb, mode)));
    if ((mode & 1) && !rr_rides) launch_finalize(RS_RR, g.ntiles, sc, rb, nullptr, (mode & 2) ? 1 : 0, s);
}

template <typename T, typename TB, typename C>
void launch_resid_restrict(const FineGeom& g, const T* kt, const T* u, const double* r, const TB* phi,
                           const int* nkeep, int L, C* r2, Scalars* sc, RedBuf rb, bool rr_rides, int check_done,
                          hipStream_t s) {
    const int m = g.mx * g.my * g.mz;
    const int rr_parts = rr_rides ? g.ntiles : 0;
    SPECMG_O_DISPATCH(T, SPECMG_TIMED_LAUNCH((k_resid_restrict<T, TB, C, O>), dim3((m + 3) / 4 + (rr_parts ? 1 : 0)),
                                             dim3(256), 0, s, g, kt, u, r, phi, nkeep, L, r2, sc, rb, rr_parts,
                                             check_done));
}

template <typename T, typename TB, typename C>
void launch_prolong(const FineGeom& g, T* u, const TB* phi, const int* nkeep, int L, const C* e2,
                    Scalars* sc, int check_done, hipStream_t s) {
    SPECMG_TIMED_LAUNCH((k_prolong<T, TB, C>), dim3((g.mx * g.my * g.mz + 3) / 4), dim3(256), 0, s, g, u, phi, nkeep,
                        L, e2, sc, check_done);
}

template <typename T, typename C>
void launch_post_fused(const FineGeom& g, const T* kt, const T* invd, const T* u, const double* r,
                       const double* q, double* z, Scalars* sc, RedBuf rb, int mode, hipStream_t s) {
    SPECMG_O_DISPATCH(T, SPECMG_EX_DISPATCH(g.ex, SPECMG_TIMED_LAUNCH((k_post_fused<EX, T, C, O>), dim3(g.ntiles),
                                                                      dim3(64 * EX), 0, s, g, kt, invd, u, r, q, z,
                                                                      sc, rb, mode)));
    if (mode & 1) launch_finalize(RS_RZ, g.ntiles, sc, rb, nullptr, (mode & 2) ? 1 : 0, s);
}

void launch_p_update(const FineGeom& g, const double* z, const double* pold, double* pnew, double* x, Scalars* sc,
                     int first, hipStream_t s) {
    const int64_t n2 = (int64_t)g.ncell() / 2;
    SPECMG_TIMED_LAUNCH(k_p_update, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, s,
                        reinterpret_cast<const double2*>(z), reinterpret_cast<const double2*>(pold),
                        reinterpret_cast<double2*>(pnew), reinterpret_cast<double2*>(x), sc, first, n2);
}

void launch_spmv_pcg(const FineGeom& g, const double* kt, const double* p, double* q, Scalars* sc, RedBuf rb,
                     int pbuf, hipStream_t s) {
    const int nblocks = (g.mx * g.my * g.mz + 3) / 4;
    if (nblocks > kMaxRedBlocks) throw HipError{hipErrorInvalidValue, "spmv grid too large for the reduction buffer"};
    if (g.ortho)
        SPECMG_TIMED_LAUNCH(k_spmv_pcg<true>, dim3(nblocks), dim3(256), 0, s, g, kt, p, q, sc, rb, pbuf);
    else
        SPECMG_TIMED_LAUNCH(k_spmv_pcg<false>, dim3(nblocks), dim3(256), 0, s, g, kt, p, q, sc, rb, pbuf);
    launch_finalize(RS_PQ, nblocks, sc, rb, nullptr, 1, s);
}

void launch_apply_A(const FineGeom& g, const double* kt, const double* x, const double* b, double* y,
                    int resid, hipStream_t s) {
    const int m = g.mx * g.my * g.mz;
    if (g.ortho) hipLaunchKernelGGL(k_apply_A<true>, dim3((m + 3) / 4), dim3(256), 0, s, g, kt, x, b, y, resid);
    else hipLaunchKernelGGL(k_apply_A<false>, dim3((m + 3) / 4), dim3(256), 0, s, g, kt, x, b, y, resid);
}

void launch_ic_setup(const FineGeom& g, const double* kt, double* invd, float* invd32, int* bad,
                     hipStream_t s) {
    SPECMG_EX_DISPATCH(g.ex, hipLaunchKernelGGL((k_ic_setup<EX>), dim3(g.ntiles), dim3(64 * EX), 0, s, g,
                                                kt, invd, invd32, bad));
}

void launch_perm3_to_kt(const FineGeom& g, const double* perm, double* kt, double sx, double sy, double sz,
                        int* bad, hipStream_t s) {
    hipLaunchKernelGGL(k_perm3_to_kt, dim3(grid_1d(3 * (int64_t)g.ncell())), dim3(256), 0, s, g, perm, kt, sx, sy,
                       sz, bad);
}

void launch_perm_to_kt(const FineGeom& g, const double* perm, double* kt, float* kt32, double scale, int* bad,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_perm_to_kt, dim3(grid_1d((int64_t)g.ncell())), dim3(256), 0, s, g, perm, kt, kt32, scale,
                       bad);
}

void launch_to_elem(const FineGeom& g, const double* nat, double* el, hipStream_t s) {
    hipLaunchKernelGGL(k_to_elem, dim3(grid_1d((int64_t)g.ncell())), dim3(256), 0, s, g, nat, el);
}

void launch_to_natural(const FineGeom& g, const double* el, double* nat, hipStream_t s) {
    hipLaunchKernelGGL(k_to_natural, dim3(grid_1d((int64_t)g.ncell())), dim3(256), 0, s, g, el, nat);
}

void launch_dot(const double* a, const double* b, int64_t n, double* out, RedBuf rb, int site,
                hipStream_t s) {
    (void)site;
    const int nb = grid_1d(n);
    hipLaunchKernelGGL(k_dot, dim3(nb), dim3(256), 0, s, a, b, n, rb);
    launch_finalize(RS_GEN, nb, nullptr, rb, out, 0, s);
}

void launch_sum_abs(const double* a, int64_t n, double* out_sum, double* out_abs, RedBuf rb,
                    hipStream_t s) {
    const int nb = grid_1d(n);
    hipLaunchKernelGGL(k_sum_abs, dim3(nb), dim3(256), 0, s, a, n, rb);
    // the two totals land in out_sum[0], out_sum[1]; callers pass out_abs = out_sum + 1
    (void)out_abs;
    launch_finalize(RS_GEN2, nb, nullptr, rb, out_sum, 0, s);
}

void launch_axpy_x(double* x, const double* p0, const double* p1, Scalars* sc, int64_t n,
                   hipStream_t s) {
    hipLaunchKernelGGL(k_axpy_x, dim3(grid_1d(n)), dim3(256), 0, s, x, p0, p1, sc, n);
    hipLaunchKernelGGL(k_clear_alpha_x, dim3(1), dim3(1), 0, s, sc);
}

void launch_sub_mean(double* x, int64_t n, const double* sum, hipStream_t s) {
    hipLaunchKernelGGL(k_sub_mean, dim3(grid_1d(n)), dim3(256), 0, s, x, n, sum);
}

void launch_copy(double* dst, const double* src, int64_t n, hipStream_t s, const Scalars* sc) {
    hipLaunchKernelGGL(k_copy, dim3(grid_1d(n)), dim3(256), 0, s, dst, src, n, sc);
}

void launch_fill(double* dst, double v, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_fill, dim3(grid_1d(n)), dim3(256), 0, s, dst, v, n);
}

void launch_pcg_init(Scalars* sc, double thresh2, int flexible, hipStream_t s) {
    hipLaunchKernelGGL(k_pcg_init, dim3(1), dim3(1), 0, s, sc, thresh2, flexible);
}

// (T, C): (double, double) float64; (float, float) the FP32 V-cycle;
// (float, double) float32 storage with float64 arithmetic
#define SPECMG_FINE_INST(T, TB, C)                                                                                 \
    template void launch_pre_smooth<T, C>(const FineGeom&, const T*, const T*, double*, const double*, T*,         \
                                          Scalars*, RedBuf, int, bool, hipStream_t);                               \
    template void launch_resid_restrict<T, TB, C>(const FineGeom&, const T*, const T*, const double*, const TB*,   \
                                                  const int*, int, C*, Scalars*, RedBuf, bool, int, hipStream_t);  \
    template void launch_prolong<T, TB, C>(const FineGeom&, T*, const TB*, const int*, int, const C*, Scalars*,    \
                                           int, hipStream_t);                                                      \
    template void launch_post_fused<T, C>(const FineGeom&, const T*, const T*, const T*, const double*,            \
                                          const double*, double*, Scalars*, RedBuf, int, hipStream_t);
SPECMG_FINE_INST(double, double, double)
SPECMG_FINE_INST(float, float, float)
SPECMG_FINE_INST(float, float, double)
template void launch_resid_restrict<double, float, double>(const FineGeom&, const double*, const double*,
                                                           const double*, const float*, const int*, int, double*,
                                                           Scalars*, RedBuf, bool, int, hipStream_t);
template void launch_prolong<double, float, double>(const FineGeom&, double*, const float*, const int*, int,
                                                    const double*, Scalars*, int, hipStream_t);
#undef SPECMG_FINE_INST

}  // namespace specmg
