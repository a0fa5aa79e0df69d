// kernels_mc.hip -- Monte-Carlo wave-function (quantum-jump) trajectories on gfx950.
//
// arXiv:2504.21440, Sec. 3.3.  One 256-thread workgroup integrates one trajectory at a time with
// the adaptive Dormand-Prince 5(4) scheme and then claims the next trajectory from a device-wide
// queue, so trajectories with many jumps do not hold up the others.  Each thread owns R rows of the
// state; the state and all seven stages stay in registers.  Only the stage input is shared: it is
// written to one of two LDS buffers and the right-hand side A psi (A = -i H_eff, stored in ELL
// column-major order so every load of a row slice is coalesced) gathers from it.
//
// After an accepted step the squared norm of the new state (FP64) is compared with the trajectory's
// threshold r.  Below it, the crossing time is located with the Illinois variant of regula falsi on
// g(theta) = ln |psi(t + theta h)|^2 - ln r, each probe a fresh DP5 step of size theta h from the
// step's start (no interpolant needed); the channel k is the first whose cumulative |C_k psi|^2
// reaches u * sum_k |C_k psi|^2; psi <- C_k psi / |C_k psi|; a new threshold is drawn.  Draws come
// from Philox-4x32-10 keyed by the seed with counter (trajectory, event): event 0 gives the first
// threshold, event m >= 1 the channel uniform and the next threshold of jump m.
//
// Time-dependent problems (TD): A(t) = A_0 + sum_i f_i(t) (-i H_i) + sum_k |g_k(t)|^2 (-1/2 C_k^dag C_k)
// is one ELL whose entries carry their term in the high column bits; before each right-hand side
// the workgroup evaluates the coefficients at the stage time (its own trajectory's t + c_s h) into
// LDS, and a jump weights channel k by |g_k(t*)|^2.
#include <algorithm>

#include "mc_kernel.h"

namespace qt {

// Ensemble mean and standard error (unbiased variance of the real part), one block per (e_op, t).
__global__ __launch_bounds__(256) void k_mc_stats(const double2 *__restrict__ tr, int64_t ntraj, int ne, int nt,
                                                  double2 *mean, double *se)
{
    __shared__ double scr[16];
    const int q = blockIdx.x;  // e_op * nt + time
    const size_t stride = (size_t)ne * nt;
    double sr = 0.0, si = 0.0;
    for (int64_t j = threadIdx.x; j < ntraj; j += blockDim.x) {
        const double2 v = tr[j * stride + q];
        sr += v.x;
        si += v.y;
    }
    sr = block_sum(sr, scr);
    si = block_sum(si, scr);
    const double mr = sr / (double)ntraj, mi = si / (double)ntraj;
    double vv = 0.0;
    for (int64_t j = threadIdx.x; j < ntraj; j += blockDim.x) {
        const double x = tr[j * stride + q].x - mr;
        vv += x * x;
    }
    vv = block_sum(vv, scr);
    if (threadIdx.x == 0) {
        mean[q] = make_double2(mr, mi);
        se[q] = ntraj > 1 ? sqrt(vv / (double)(ntraj - 1) / (double)ntraj) : 0.0;
    }
}

__global__ void k_mc_queue_reset(unsigned long long *q) { *q = 0ull; }

template <typename T, int R, bool TD, int OCC> static const void *mc_fn()
{
    return (const void *)k_mc<T, R, TD, OCC>;
}

// Ensembles of at least this many complex64 trajectories with 2, 4 or 8 rows per thread take the
// variant held to 3 waves per SIMD (2 at 8 rows): more trajectories in flight outweigh the spilled
// registers; a lone trajectory runs 10-20% slower there, so it keeps the other one.  Constant matrices of up
// to 12 entries per row are held in registers instead (kernels_mc_reg.hip).  What is left, trajectories/s of
// 2,047 (unconstrained) and of 2,048: constant, 15 entries per row, d = 512 680,000 and 689,000, d = 1,024
// 258,000 and 362,000, d = 2,048 85,200 and 130,600; driven chains (time-dependent) of L = 9 192,000 and
// 196,000, L = 10 64,000 and 81,700, L = 11 15,300 and 26,000.
constexpr int64_t MC_DENSE_ENSEMBLE = 2048;
static bool mc_occ3(const McParams &p, bool f64)
{
    return !f64 && (p.rows == 2 || p.rows == 4 || p.rows == 8) && p.ntraj >= MC_DENSE_ENSEMBLE;
}

static size_t mc_lds(const McParams &p, bool f64) { return (size_t)2 * p.d * (f64 ? 16 : 8); }

template <typename T, bool TD> static const void *mc_pick(int rows, bool occ3)
{
    switch (rows) {
    case 1: return mc_fn<T, 1, TD, 1>();
    case 2: return occ3 ? mc_fn<T, 2, TD, 3>() : mc_fn<T, 2, TD, 1>();
    case 4: return occ3 ? mc_fn<T, 4, TD, 3>() : mc_fn<T, 4, TD, 1>();
    case 8: return occ3 ? mc_fn<T, 8, TD, 2>() : mc_fn<T, 8, TD, 1>();
    default: return mc_fn<T, 16, TD, 1>();
    }
}

template <typename T, int R, int OCC>
static void mc_launch_t(const McParams *dev_p, bool td, int grid, size_t lds, hipStream_t s)
{
    if (td) hipLaunchKernelGGL((k_mc<T, R, true, OCC>), dim3(grid), dim3(MC_THREADS), lds, s, dev_p);
    else hipLaunchKernelGGL((k_mc<T, R, false, OCC>), dim3(grid), dim3(MC_THREADS), lds, s, dev_p);
}

int mc_grid(const McParams &p, bool f64, bool td, int device)
{
    const bool o3 = mc_occ3(p, f64);
    const void *fn = f64 ? (td ? mc_pick<double, true>(p.rows, o3) : mc_pick<double, false>(p.rows, o3))
                         : (td ? mc_pick<float, true>(p.rows, o3) : mc_pick<float, false>(p.rows, o3));
    size_t lds = mc_lds(p, f64);
    int threads = MC_THREADS;
    if (const void *reg = mc_reg_kernel(p, f64, td, &threads, &lds)) fn = reg;
    if (lds > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) cus = 256;
    const int64_t g = std::min<int64_t>(p.ntraj, (int64_t)per_cu * cus);
    return (int)std::max<int64_t>(1, g);
}

void mc_launch(const McParams &p, const McParams *dev_p, bool f64, bool td, int grid, hipStream_t s)
{
    size_t lds = mc_lds(p, f64);
    int threads = MC_THREADS;
    if (const void *reg = mc_reg_kernel(p, f64, td, &threads, &lds)) {
        void *args[] = {(void *)&dev_p};
        (void)hipLaunchKernel(reg, dim3(grid), dim3(threads), args, lds, s);
        return;
    }
    if (f64) {
        switch (p.rows) {
        case 1: mc_launch_t<double, 1, 1>(dev_p, td, grid, lds, s); break;
        case 2: mc_launch_t<double, 2, 1>(dev_p, td, grid, lds, s); break;
        case 4: mc_launch_t<double, 4, 1>(dev_p, td, grid, lds, s); break;
        case 8: mc_launch_t<double, 8, 1>(dev_p, td, grid, lds, s); break;
        default: mc_launch_t<double, 16, 1>(dev_p, td, grid, lds, s); break;
        }
    } else {
        switch (p.rows) {
        case 1: mc_launch_t<float, 1, 1>(dev_p, td, grid, lds, s); break;
        case 2:
            if (mc_occ3(p, f64)) mc_launch_t<float, 2, 3>(dev_p, td, grid, lds, s);
            else mc_launch_t<float, 2, 1>(dev_p, td, grid, lds, s);
            break;
        case 4:
            if (mc_occ3(p, f64)) mc_launch_t<float, 4, 3>(dev_p, td, grid, lds, s);
            else mc_launch_t<float, 4, 1>(dev_p, td, grid, lds, s);
            break;
        case 8:
            if (mc_occ3(p, f64)) mc_launch_t<float, 8, 2>(dev_p, td, grid, lds, s);
            else mc_launch_t<float, 8, 1>(dev_p, td, grid, lds, s);
            break;
        default: mc_launch_t<float, 16, 1>(dev_p, td, grid, lds, s); break;
        }
    }
}

void mc_launch_stats(const double2 *expect_tr, int64_t ntraj, int ne, int nt, double2 *mean, double *se, hipStream_t s)
{
    if (ne * nt > 0) hipLaunchKernelGGL(k_mc_stats, dim3(ne * nt), dim3(256), 0, s, expect_tr, ntraj, ne, nt, mean, se);
}

void mc_launch_queue_reset(unsigned long long *q, hipStream_t s)
{
    hipLaunchKernelGGL(k_mc_queue_reset, dim3(1), dim3(1), 0, s, q);
}

}  // namespace qt
