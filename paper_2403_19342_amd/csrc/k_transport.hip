// Two-phase flow of Section 6: the total-mobility scaling of the pressure
// permeability (eq. v) and the explicit saturation sub-steps of the improved
// IMPES scheme (eq. ES), plus their C-ABI entry points.
//
// Fluid model: S* = clamp((S - 0.2) / 0.6, 0, 1), k_w = S*^2,
// k_o = (1 - S*)^2, mu_w = 0.3, mu_o = 3.0; lambda = k_w/mu_w + k_o/mu_o
// and f_w = (k_w/mu_w) / lambda.  Wells are rate controlled: q > 0 injects
// water, q < 0 produces the cell's mixture (q_w = f_w(S) q).
//
// One sub-step is two grid-stride passes over the cells:
//   k_sat_rate    r_i = (q_w - sum_d (F_+ - F_-) / h_d) / phi_i with the
//                 face water flux F = f_w(S_upstream) v; each block writes
//                 the largest |r| of its cells to its own slot;
//   k_sat_update  every block reduces those slots to the grid's
//                 largest rate (a max is exact in any order), then
//                 dt = DS_max / max|r| (0 when every rate is zero),
//                 S_i += dt r_i, and block 0 adds dt to the elapsed time.
// f_w of every cell is evaluated once per sub-step, by the pass that writes
// S (k_transport_begin for the initial S), and stored: the rate pass reads
// it for the cell and its upstream neighbours instead of re-evaluating the
// four divisions of the fluid law up to seven times per cell.
// A single atomic max per block onto one word serialises thousands of
// blocks at one L2 address; the slot array keeps the reduction in plain
// loads and stores.  Nothing is copied to the host between sub-steps.
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <string>

#include "common.hpp"
#include "../../include/specmg.h"

namespace specmg {
int fail_message(int code, const char* msg);   // sets the thread's last error, returns code
}

// Kernels live in the named namespace so that profiles show their names.
namespace specmg {

constexpr double kSwc = 0.2;
constexpr double kSpan = 0.6;
constexpr double kMuW = 0.3;
constexpr double kMuO = 3.0;

__device__ __forceinline__ void phase_mobilities(double s, double& lw, double& lo) {
    double sn = (s - kSwc) / kSpan;
    sn = fmin(fmax(sn, 0.0), 1.0);
    lw = sn * sn / kMuW;
    lo = (1.0 - sn) * (1.0 - sn) / kMuO;
}

__device__ __forceinline__ double water_fraction(double s) {
    double lw, lo;
    phase_mobilities(s, lw, lo);
    return lw / (lw + lo);
}

__global__ __launch_bounds__(256) void k_total_mobility(int64_t n, const double* __restrict__ perm,
                                                        const double* __restrict__ s, double* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double lw, lo;
        phase_mobilities(s[i], lw, lo);
        out[i] = perm[i] * (lw + lo);
    }
}

constexpr int kMaxRateBlocks = 2048;   // slots of the per-block maxima in the workspace
constexpr int kRateThreads = 512;
constexpr int kUpdateBlocks = 1280;    // about five workgroups of four wavefronts a CU

__global__ __launch_bounds__(256) void k_transport_begin(int64_t n, const double* __restrict__ s,
                                                         double* __restrict__ fw, double* t) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        fw[i] = water_fraction(s[i]);
    if (blockIdx.x == 0 && threadIdx.x == 0) *t = 0.0;
}

// cell coordinates of a flat index; 32-bit division when the grid allows it
__device__ __forceinline__ void cell_xyz(int64_t i, int nx, int ny, int64_t n, int& x, int& y, int& z) {
    if (n <= 0xffffffffll) {
        const uint32_t u = (uint32_t)i, row = u / (uint32_t)nx;
        x = (int)(u - row * (uint32_t)nx);
        z = (int)(row / (uint32_t)ny);
        y = (int)(row - (uint32_t)z * (uint32_t)ny);
    } else {
        const int64_t row = i / nx;
        x = (int)(i - row * nx);
        z = (int)(row / ny);
        y = (int)(row - (int64_t)z * ny);
    }
}

// Workgroups go to the 8 XCDs in turn; numbered like this, each XCD works on
// one contiguous eighth of the cells, so that the neighbours of a cell, and what
// the previous pass wrote of it, are in its own L2 (grids of a multiple of 8).
// Both passes, in turn / like this: 23.0 / 21.4 us for 0.88 million cells, 25.4 /
// 24.6 for 1.12, 40.4 / 38.6 for 2.1, 71.4 / 70.4 for 4.1, 169 / 176 for 8.4.
__device__ __forceinline__ int64_t block_in_order() {
    const int b = blockIdx.x, nb = gridDim.x;
    return nb & 7 ? b : (b & 7) * (nb >> 3) + (b >> 3);
}

// cell coordinates kRateThreads cells on: the step as (x, y, z), carries added
struct CellStep {
    int x, y, z;
};

// K cells a thread and pass, kRateThreads apart.  Whether a neighbour is
// upstream is known only from the velocities, so its f_w is loaded in any case
// (from the cell itself at the boundary, and in place of the boundary's velocity,
// whose array need not reach that far): all 15 values of all K cells are
// then in flight at once, one wait for memory, where loads behind the tests
// took two and a cell at a time as many again: 20.0 -> 14.8 us for 1.12 million
// cells (54 MB in, 9 MB out), three cells a thread.  Both passes of a sub-step,
// before and after, at 0.26, 0.88, 1.12, 2.1, 4.1 and 8.4 million cells: 11.1,
// 25.6, 31.2, 44.6, 79.4, 200 -> 10.4, 21.4, 24.6, 38.6, 70.4, 176 us.
template <int K>
__global__ __launch_bounds__(kRateThreads) void k_sat_rate(int nx, int ny, int nz, double hx, double hy, double hz,
                                                           CellStep step, const double* __restrict__ phi,
                                                           const double* __restrict__ q, const double* __restrict__ vx,
                                                           const double* __restrict__ vy, const double* __restrict__ vz,
                                                           const double* __restrict__ fw, double* __restrict__ rate,
                                                           double* __restrict__ block_max) {
    __shared__ double red[kRateThreads / 64];
    const int64_t sy = nx, sz = (int64_t)nx * ny, n = sz * nz;
    double m = 0.0;
    for (int64_t i0 = block_in_order() * (K * kRateThreads) + threadIdx.x; i0 < n;
         i0 += (int64_t)gridDim.x * (K * kRateThreads)) {
        int x, y, z;
        cell_xyz(i0, nx, ny, n, x, y, z);
        double f0[K], qi[K], ph[K], vp[K][3], vm[K][3], fp[K][3], fm[K][3];
        bool up[K][3], dn[K][3];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = i0 + (int64_t)k * kRateThreads;
            const bool in = i < n;
            const int64_t c = in ? i : i0;
            up[k][0] = in && x + 1 < nx;
            up[k][1] = in && y + 1 < ny;
            up[k][2] = in && z + 1 < nz;
            dn[k][0] = in && x > 0;
            dn[k][1] = in && y > 0;
            dn[k][2] = in && z > 0;
            f0[k] = fw[c];
            qi[k] = q[c];
            ph[k] = phi[c];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int64_t st = d == 0 ? 1 : (d == 1 ? sy : sz);
                const double* v = d == 0 ? vx : (d == 1 ? vy : vz);
                const int64_t cu = up[k][d] ? c + st : c, cd = dn[k][d] ? c - st : c;
                vp[k][d] = (up[k][d] ? v : fw)[c];   // the boundary's velocities are not read
                vm[k][d] = (dn[k][d] ? v : fw)[cd];
                fp[k][d] = fw[cu];
                fm[k][d] = fw[cd];
            }
            x += step.x;
            if (x >= nx) {
                x -= nx;
                ++y;
            }
            y += step.y;
            if (y >= ny) {
                y -= ny;
                ++z;
            }
            z += step.z;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = i0 + (int64_t)k * kRateThreads;
            // water flux through the + and - faces of one axis, upstream
            // weighted; the boundary faces carry nothing
            auto axis_div = [&](int d, double h) {
                const double p = up[k][d] ? (vp[k][d] >= 0.0 ? f0[k] : fp[k][d]) * vp[k][d] : 0.0;
                const double q_ = dn[k][d] ? (vm[k][d] >= 0.0 ? fm[k][d] : f0[k]) * vm[k][d] : 0.0;
                return (p - q_) / h;
            };
            double div = axis_div(0, hx);
            div += axis_div(1, hy);
            div += axis_div(2, hz);
            const double qw = qi[k] > 0.0 ? qi[k] : f0[k] * qi[k];
            const double r = (qw - div) / ph[k];
            if (i < n) {
                rate[i] = r;
                m = fmax(m, fabs(r));
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kRateThreads / 64; ++w) m = fmax(m, red[w]);
        block_max[blockIdx.x] = m;
    }
}

// The first K cells of a thread are loaded beside the slots of the maxima
// (11.7 -> 10.4 us for 1.12 million cells, 36 MB).
constexpr int kUpdateCells = 4;
__global__ __launch_bounds__(256) void k_sat_update(int64_t n, const double* __restrict__ rate,
                                                    double* __restrict__ s, double* __restrict__ fw,
                                                    const double* __restrict__ block_max, int nmax, double ds_max,
                                                    double* t) {
    constexpr int K = kUpdateCells;
    __shared__ double red[4];
    const int64_t first = block_in_order() * (K * 256) + threadIdx.x, stride = (int64_t)gridDim.x * (K * 256);
    double sv[K], rv[K];
    auto load = [&](int64_t i0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = i0 + 256 * k;
            const int64_t c = i < n ? i : n - 1;
            sv[k] = s[c];
            rv[k] = rate[c];
        }
    };
    load(first);
    double m = 0.0;
#pragma unroll
    for (int u = 0; u < kMaxRateBlocks / 256; ++u) {
        const int k = threadIdx.x + 256 * u;
        if (k < nmax) m = fmax(m, block_max[k]);
    }
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    const double dt = m > 0.0 ? ds_max / m : 0.0;
    for (int64_t i0 = first; i0 < n; i0 += stride) {
        if (i0 != first) load(i0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t i = i0 + 256 * k;
            if (i >= n) break;
            const double si = sv[k] + dt * rv[k];
            s[i] = si;
            fw[i] = water_fraction(si);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *t += dt;
}

static int blocks_for(int64_t n, int cap) {
    const int64_t b = (n + 255) / 256;
    return (int)(b < cap ? (b < 1 ? 1 : b) : cap);
}

static int device_error(hipError_t e, const char* what) {
    return fail_message(SPECMG_EDEVICE, (std::string(what) + ": " + hipGetErrorString(e)).c_str());
}

}  // namespace specmg

using namespace specmg;

extern "C" int specmg_total_mobility(const double* perm_dev, const double* s_dev, double* perm_eff_dev, int64_t n,
                                     void* stream) {
    if (!perm_dev || !s_dev || !perm_eff_dev || n < 0) return fail_message(SPECMG_EINVAL, "bad arguments");
    if (n == 0) return SPECMG_OK;
    hipLaunchKernelGGL(k_total_mobility, dim3(blocks_for(n, 8192)), dim3(256), 0, (hipStream_t)stream, n, perm_dev,
                       s_dev, perm_eff_dev);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPECMG_OK : device_error(e, "k_total_mobility");
}

// Checks and launches shared by specmg_transport and its allocation-free
// variant; work holds 2 n + kMaxRateBlocks doubles (rates, f_w, block maxima).
static int run_transport(const specmg_grid* grid, const double* phi_dev, const double* q_dev, const double* vx_dev,
                         const double* vy_dev, const double* vz_dev, double* s_dev, int32_t substeps, double ds_max,
                         double* work_dev, double* t_dev, hipStream_t s) {
    const int64_t n = (int64_t)grid->nx * grid->ny * grid->nz;
    double* rate = work_dev;
    double* fw = work_dev + n;
    double* block_max = work_dev + 2 * n;
    // cells a thread: what brings the grid down to 1024 workgroups, up to 3 (four
    // take 176 registers); beyond kMaxRateBlocks of them, passes of equal length
    const int64_t per = (int64_t)kRateThreads * 1024;
    const int K = (int)std::min<int64_t>(3, (n + per - 1) / per);
    auto blocks = [&](int64_t cells, int cap) {   // a multiple of 8 from 64 workgroups
        const int64_t chunks = (n + cells - 1) / cells, passes = (chunks + cap - 1) / cap;
        const int64_t b = (chunks + passes - 1) / passes;
        return (int)(b < 64 ? b : (b + 7) / 8 * 8);
    };
    const int nb = blocks((int64_t)K * kRateThreads, kMaxRateBlocks), nu = blocks(256 * kUpdateCells, kUpdateBlocks);
    const int64_t row = kRateThreads / grid->nx;
    const CellStep step{kRateThreads % grid->nx, (int)(row % grid->ny), (int)(row / grid->ny)};
    const auto k_rate = K == 1 ? k_sat_rate<1> : (K == 2 ? k_sat_rate<2> : k_sat_rate<3>);
    hipLaunchKernelGGL(k_transport_begin, dim3(blocks_for(n, 8192)), dim3(256), 0, s, n, s_dev, fw, t_dev);
    for (int m = 0; m < substeps; ++m) {
        hipLaunchKernelGGL(k_rate, dim3(nb), dim3(kRateThreads), 0, s, grid->nx, grid->ny, grid->nz, grid->hx, grid->hy,
                           grid->hz, step, phi_dev, q_dev, vx_dev, vy_dev, vz_dev, fw, rate, block_max);
        hipLaunchKernelGGL(k_sat_update, dim3(nu), dim3(256), 0, s, n, rate, s_dev, fw, block_max, nb, ds_max,
                           t_dev);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPECMG_OK : device_error(e, "saturation sub-steps");
}

static int check_transport_args(const specmg_grid* grid, const double* phi_dev, const double* q_dev,
                                const double* vx_dev, const double* vy_dev, const double* vz_dev, const double* s_dev,
                                int32_t substeps, double ds_max, const double* t_dev) {
    if (!grid || !phi_dev || !q_dev || !vx_dev || !vy_dev || !vz_dev || !s_dev || !t_dev)
        return fail_message(SPECMG_EINVAL, "null argument");
    if (grid->nx < 1 || grid->ny < 1 || grid->nz < 1) return fail_message(SPECMG_EINVAL, "grid sizes must be >= 1");
    if (!(grid->hx > 0) || !(grid->hy > 0) || !(grid->hz > 0))
        return fail_message(SPECMG_EINVAL, "spacings must be positive");
    if (substeps < 0) return fail_message(SPECMG_EINVAL, "substeps must be >= 0");
    if (!(ds_max > 0) || ds_max > 1.0) return fail_message(SPECMG_EINVAL, "ds_max must be in (0, 1]");
    return SPECMG_OK;
}

extern "C" int specmg_transport(const specmg_grid* grid, const double* phi_dev, const double* q_dev,
                                const double* vx_dev, const double* vy_dev, const double* vz_dev, double* s_dev,
                                int32_t substeps, double ds_max, double* work_dev, double* t_dev, void* stream) {
    if (!work_dev) return fail_message(SPECMG_EINVAL, "null argument");
    const int rc = check_transport_args(grid, phi_dev, q_dev, vx_dev, vy_dev, vz_dev, s_dev, substeps, ds_max, t_dev);
    if (rc != SPECMG_OK) return rc;
    return run_transport(grid, phi_dev, q_dev, vx_dev, vy_dev, vz_dev, s_dev, substeps, ds_max, work_dev, t_dev,
                         (hipStream_t)stream);
}

// ---------------------------------------------------------------------------
// Allocation-free variant: the workspace is a file-scope device array,
// `scratch`, sized for SPECMG_TRANSPORT_NOALLOC_MAX_CELLS cells.  Each GPU
// holds its own copy (32 MiB + 16 KiB) from the library's load until the
// process ends.  Its device address is looked up once per device (with that
// device current) by hipGetSymbolAddress; host code never passes the
// array's name itself to a kernel.  Nothing in it needs clearing: every
// sub-step writes the rates and slots before reading them and the first
// kernel writes f_w.  Calls that overlap on one GPU share the array and race.
constexpr int64_t kNoAllocMaxCells = SPECMG_TRANSPORT_NOALLOC_MAX_CELLS;
constexpr int64_t kScratchDoubles = 2 * kNoAllocMaxCells + kMaxRateBlocks;
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// device address of this device's scratch array (looked up on first use)
static int scratch_address(double** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return device_error(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail_message(SPECMG_EINVAL, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return device_error(e != hipSuccess ? e : hipErrorInvalidSymbol, "scratch address");
        g_scratch_ptr[dev] = (double*)ptr;
    }
    *out = g_scratch_ptr[dev];
    return SPECMG_OK;
}

extern "C" int specmg_transport_noalloc(const specmg_grid* grid, const double* phi_dev, const double* q_dev,
                                        const double* vx_dev, const double* vy_dev, const double* vz_dev,
                                        double* s_dev, int32_t substeps, double ds_max, double* t_dev, void* stream) {
    const int rc = check_transport_args(grid, phi_dev, q_dev, vx_dev, vy_dev, vz_dev, s_dev, substeps, ds_max, t_dev);
    if (rc != SPECMG_OK) return rc;
    const int64_t n = (int64_t)grid->nx * grid->ny * grid->nz;
    if (n > kNoAllocMaxCells)
        return fail_message(SPECMG_EINVAL, ("grid of " + std::to_string(n) + " cells exceeds the " +
                                            std::to_string(kNoAllocMaxCells) + " cells of the built-in workspace")
                                               .c_str());
    double* work = nullptr;
    const int ra = scratch_address(&work);
    if (ra != SPECMG_OK) return ra;
    return run_transport(grid, phi_dev, q_dev, vx_dev, vy_dev, vz_dev, s_dev, substeps, ds_max, work, t_dev,
                         (hipStream_t)stream);
}
