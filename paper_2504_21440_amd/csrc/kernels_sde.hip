// kernels_sde.hip -- stochastic Schrodinger and master equations under homodyne detection on gfx950.
//
// arXiv:2504.21440, Sec. 3.5 (Ito form): one workgroup of 256 threads (512 for complex128 states of more
// than 2,048 entries) integrates one trajectory at a time and claims the next from a device-wide
// queue.  Each thread owns R rows of the state vector x (the ket, or vec(rho)); x, the drift and the new
// state stay in registers, the products B_n x of the thread's rows in LDS, and the vector every gather
// reads (x, then each supporting value) in one LDS buffer.  The operators A and B_n are ELL,
// column-major, read through L2.
//
// Step: the tlist interval is cut into equal steps of at most dt.  With a = a(x) and
// b_n = B_n x - cg mu_n x,
//     x' = x + a h + sum_n b_n dW_n + sum_n (b_n(U_n) - b_n) (dW_n^2 - h) / (2 sqrt h),
//     U_n = x + a h + b_n sqrt h,
// the derivative-free order-1.0 strong scheme of Platen (Kloeden & Platen, Sec. 11.1) taken for
// each Wiener process with its own supporting value, then x' is renormalised (unit norm for the
// SSE, unit trace for the SME).  All reductions (mu_n, norms, traces, expectation values) are FP64
// in a fixed order.  dW_n = sqrt(h) z with z from Philox-4x32-10 and the Box-Muller transform,
// counter (trajectory, step, 1 + n/2).
//
// Thread n draws dW_n, before the step's rows are in registers, and mu_n and dW_n pass through LDS: the
// processes are a loop, not unrolled code.  With the draws in every thread amid a step unrolled for eight
// processes, the kernel filled the register file across the sine's and cosine's branch for large angles,
// and the compiler saved registers in that branch's join block ahead of the instruction that restores the
// execution mask.  The angle is never large, so the saves ran for no lane: one was the step counter, and
// the step loop of a complex128 ket of 1,025 entries did not end.
//
// What bounds it: the round trips of the operator reads from L2 and 6 + 3 m barriers a step (m processes).  Two
// measured operators, 400 steps, before and after the processes became a loop: 500 trajectories of n = 1,024
// (master equation, complex64) 7.00 and 6.27 ms, of n = 256 in complex128 3.37 and 2.57 ms; 500 kets of 1,024
// in complex64 6.44 and 5.79 ms; 200 in complex128 5.54 and 5.53 ms.
#include <algorithm>

#include "qt_common.h"
#include "qt_rng.h"
#include "qt_sde.h"

namespace qt {

// LDS doubles behind the state and the images: the partial sums of a step, one per wave (m + 1 of them, or the
// three of an expectation value); then, in the same place, mu and dW of every process and the two partial
// sums of a supporting value.  Then the trajectory number.
__host__ __device__ inline int sde_slots(int m, int nw)
{
    const int a = (m + 1 > 3 ? m + 1 : 3) * nw, b = 2 * m + 2 * nw;
    return a > b ? a : b;
}

template <typename T, int TPB, int R, bool SME>
__global__ __launch_bounds__(TPB) void k_sde(const SdeParams *__restrict__ Pp)
{
    using V = typename vec2<T>::type;
    constexpr int NW = TPB / 64;
    const SdeParams &P = *Pp;
    extern __shared__ __align__(16) char smem[];  // 16-byte LDS accesses: off by 8 bytes they take hundreds of cycles
    const int n = P.n, m = P.m;
    V *xs = (V *)smem;  // the vector the gathers read
    V *bx = xs + n;     // B_k x at the thread's own rows, m blocks of n
    double *scr = (double *)(bx + (size_t)m * n);  // partial sum s of wave w at s * NW + w; later mu, dW of process k at 2 k
    double *sup = scr + 2 * m;                     // partial sums beside mu and dW
    unsigned long long *jsh = (unsigned long long *)(scr + sde_slots(m, NW));
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const V *__restrict__ av = (const V *)P.a_val;
    const V *__restrict__ bv = (const V *)P.b_val;
    auto row = [&](int q) { return tid + q * TPB; };
    auto is_diag = [&](int r) { return r % (P.d + 1) == 0; };
    // (A xs) at own row r
    auto a_row = [&](int r) {
        V acc;
        acc.x = 0;
        acc.y = 0;
        // global-only loads of the operator streams, apart from the LDS gathers of the state
        for (int k = 0; k < P.WA; ++k) cfma(acc, gld(av + (size_t)k * n + r), xs[gld(P.a_col + (size_t)k * n + r)]);
        return acc;
    };
    // (B_j xs) at own row r
    auto b_row = [&](int j, int r) {
        V acc;
        acc.x = 0;
        acc.y = 0;
        const size_t base = (size_t)j * P.WB * n;
        for (int k = 0; k < P.WB; ++k)
            cfma(acc, gld(bv + base + (size_t)k * n + r), xs[gld(P.b_col + base + (size_t)k * n + r)]);
        return acc;
    };
    // this thread's share of mu for the state u (its own rows) and its image Bu:
    // SSE: Re sum conj(u) Bu (the caller divides by |u|^2 and doubles), SME: Re of the diagonal of Bu
    auto mu_part = [&](V u, V bu, int r) {
        if constexpr (SME) return is_diag(r) ? (double)bu.x : 0.0;
        else return (double)u.x * (double)bu.x + (double)u.y * (double)bu.y;
    };
    // this wave's part of a sum; after the next barrier total() is the block's, in a fixed order
    auto post = [&](double *slot, double v) {
        v = wave_sum(v);
        if (lane == 0) slot[w] = v;
    };
    auto total = [&](const double *slot) {
        double t = slot[0];
#pragma unroll
        for (int u = 1; u < NW; ++u) t += slot[u];
        return t;
    };
    auto record = [&](uint64_t j, int idx) {
        // expectation values of the state in xs
        for (int q = 0; q < P.ne; ++q) {
            const int32_t *ep = P.eptr + (size_t)q * (P.d + 1);
            double v[3] = {0.0, 0.0, 0.0};
            if constexpr (SME) {
                // Tr(O rho) = sum_{(i,j) in O} O_ij rho_ji
                for (int p = ep[0] + tid; p < ep[P.d]; p += TPB) {
                    const double2 o = P.eval[p];
                    const double2 r = to_d2(xs[P.evidx[p]]);
                    v[0] += o.x * r.x - o.y * r.y;
                    v[1] += o.x * r.y + o.y * r.x;
                }
            } else {
                for (int i = tid; i < P.d; i += TPB) {
                    double rr = 0.0, ri = 0.0;
                    for (int p = ep[i]; p < ep[i + 1]; ++p) {
                        const double2 o = P.eval[p];
                        const double2 xv = to_d2(xs[P.ecol[p]]);
                        rr += o.x * xv.x - o.y * xv.y;
                        ri += o.x * xv.y + o.y * xv.x;
                    }
                    const double2 c = to_d2(xs[i]);
                    v[0] += c.x * rr + c.y * ri;
                    v[1] += c.x * ri - c.y * rr;
                    v[2] += c.x * c.x + c.y * c.y;
                }
            }
            post(scr, v[0]);
            post(scr + NW, v[1]);
            if constexpr (!SME) post(scr + 2 * NW, v[2]);
            __syncthreads();
            if (tid == 0) {
                const double nn = SME ? 1.0 : total(scr + 2 * NW);
                P.expect_tr[((size_t)j * P.ne + q) * P.nt + idx] = make_double2(total(scr) / nn, total(scr + NW) / nn);
            }
            __syncthreads();
        }
    };

    for (;;) {
        if (tid == 0) *jsh = atomicAdd(P.queue, 1ull);
        __syncthreads();
        const uint64_t j = *jsh;
        __syncthreads();
        if ((int64_t)j >= P.ntraj) break;

        const V *x0 = (const V *)P.x0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = row(q);
            if (r < n) xs[r] = x0[r];
        }
        __syncthreads();
        record(j, 0);
        int status = ST_RUNNING;
        uint32_t step = 0;
        for (int iv = 0; iv + 1 < P.nt && status == ST_RUNNING; ++iv) {
            const double len = P.tlist[iv + 1] - P.tlist[iv];
            const int ns = P.nsub[iv];
            const double h = len / (double)ns, sq = sqrt(h);
            double cur = 0.0;  // thread k < m: the current of process k, summed over the interval
            for (int s = 0; s < ns; ++s, ++step) {
                // xs holds x here (written by the previous step or the start)
                double dw = 0.0;  // thread k < m: the increment of process k
                if (tid < m) {
                    double z0, z1;
                    wiener_normals(P.seed, j, step, (uint32_t)(tid / 2), &z0, &z1);
                    dw = sq * (tid & 1 ? z1 : z0);
                }
                V x[R], a[R], xn[R];
                double n2 = 0.0;  // |x|^2 (SSE)
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int r = row(q);
                    x[q].x = x[q].y = a[q].x = a[q].y = 0;
                    if (r >= n) continue;
                    x[q] = xs[r];
                    a[q] = a_row(r);
                    if constexpr (!SME) n2 += abs2d(x[q]);
                }
#pragma unroll 1
                for (int k = 0; k < m; ++k) {
                    double mk = 0.0;
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int r = row(q);
                        if (r >= n) continue;
                        const V b = b_row(k, r);
                        bx[(size_t)k * n + r] = b;
                        mk += mu_part(x[q], b, r);
                    }
                    post(scr + k * NW, mk);
                }
                if constexpr (!SME) post(scr + m * NW, n2);
                __syncthreads();  // the sums; every gather of x is done
                double mk = 0.0;
                if (tid < m) {
                    mk = total(scr + tid * NW);
                    if constexpr (!SME) mk = 2.0 * mk / total(scr + m * NW);
                    cur += mk * h + dw;
                }
                __syncthreads();
                if (tid < m) {
                    scr[2 * tid] = mk;
                    scr[2 * tid + 1] = dw;
                }
                __syncthreads();
                // drift (SSE: + sum mu/2 B x - mu^2/8 x) and the Euler-Maruyama part of the update
                if constexpr (!SME) {
#pragma unroll 1
                    for (int k = 0; k < m; ++k) {
                        const double mu = scr[2 * k];
#pragma unroll
                        for (int q = 0; q < R; ++q) {
                            const int r = row(q);
                            if (r >= n) continue;
                            caxpy(a[q], (T)(0.5 * mu), bx[(size_t)k * n + r]);
                            caxpy(a[q], (T)(-0.125 * mu * mu), x[q]);
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    xn[q] = x[q];
                    caxpy(xn[q], (T)h, a[q]);
                }
#pragma unroll 1
                for (int k = 0; k < m; ++k) {
                    const double mu = scr[2 * k], dW = scr[2 * k + 1];
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int r = row(q);
                        if (r >= n) continue;
                        V b = bx[(size_t)k * n + r];
                        caxpy(b, (T)(-P.cg * mu), x[q]);
                        caxpy(xn[q], (T)dW, b);
                    }
                }
                // supporting values U_k = x + a h + b_k sqrt(h) and the correction of each process
#pragma unroll 1
                for (int k = 0; k < m; ++k) {
                    const double mu = scr[2 * k], dW = scr[2 * k + 1];
                    __syncthreads();  // every gather of xs is done
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int r = row(q);
                        if (r >= n) continue;
                        V b = bx[(size_t)k * n + r];
                        caxpy(b, (T)(-P.cg * mu), x[q]);
                        V u = x[q];
                        caxpy(u, (T)h, a[q]);
                        caxpy(u, (T)sq, b);
                        xs[r] = u;
                    }
                    __syncthreads();
                    double s0 = 0.0, s1 = 0.0;  // mu part, |U|^2
                    V bu[R];
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int r = row(q);
                        bu[q].x = bu[q].y = 0;
                        if (r >= n) continue;
                        bu[q] = b_row(k, r);
                        s0 += mu_part(xs[r], bu[q], r);
                        if constexpr (!SME) s1 += abs2d(xs[r]);
                    }
                    post(sup, s0);
                    if constexpr (!SME) post(sup + NW, s1);
                    __syncthreads();
                    const double mus = SME ? total(sup) : 2.0 * total(sup) / total(sup + NW);
                    const double wgt = (dW * dW - h) / (2.0 * sq);
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int r = row(q);
                        if (r >= n) continue;
                        V b = bx[(size_t)k * n + r];
                        caxpy(b, (T)(-P.cg * mu), x[q]);
                        caxpy(bu[q], (T)(-P.cg * mus), xs[r]);
                        caxpy(xn[q], (T)wgt, bu[q]);
                        caxpy(xn[q], (T)(-wgt), b);
                    }
                }
                // renormalise: unit norm (SSE) or unit trace (SME)
                double nr = 0.0;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int r = row(q);
                    if (r >= n) continue;
                    if constexpr (SME) nr += is_diag(r) ? (double)xn[q].x : 0.0;
                    else nr += abs2d(xn[q]);
                }
                __syncthreads();  // the last supporting value and its sums have been read
                post(sup, nr);
                __syncthreads();
                const double sc = SME ? total(sup) : sqrt(total(sup));
                if (!isfinite(sc) || sc == 0.0) {
                    status = 6;  // QT_ENONFINITE
                    break;
                }
                const T inv = (T)(1.0 / sc);
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int r = row(q);
                    if (r < n) xs[r] = cscale(xn[q], inv);
                }
                __syncthreads();
            }
            if (status != ST_RUNNING) break;
            if (tid < m) P.meas[((size_t)j * m + tid) * (P.nt - 1) + iv] = cur / len;
            record(j, iv + 1);
        }
        if (tid == 0) P.status[j] = status == ST_RUNNING ? ST_DONE : status;
        __syncthreads();
    }
}

static int device_cus(int device)
{
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) cus = 256;
    return cus;
}

// 256 threads with up to 16 rows each; complex128 states of more than 2,048 entries 512 threads with 8 rows
// (16 rows of them would not fit the registers).
static int sde_threads(const SdeParams &p, bool f64) { return f64 && p.rows > 8 ? 2 * SDE_THREADS : SDE_THREADS; }

size_t sde_lds_bytes(const SdeParams &p, bool f64)
{
    return (size_t)(1 + p.m) * p.n * (f64 ? 16 : 8) + ((size_t)sde_slots(p.m, sde_threads(p, f64) / 64) + 1) * 8;
}

template <typename T, int TPB, int R> static const void *sde_fn(bool sme)
{
    return sme ? (const void *)k_sde<T, TPB, R, true> : (const void *)k_sde<T, TPB, R, false>;
}

template <typename T> static const void *sde_pick(int rows, bool sme)
{
    if (rows > 8) {
        if constexpr (sizeof(T) == 8) return sde_fn<T, 2 * SDE_THREADS, 8>(sme);
        else return sde_fn<T, SDE_THREADS, 16>(sme);
    }
    switch (rows) {
    case 1: return sde_fn<T, SDE_THREADS, 1>(sme);
    case 2: return sde_fn<T, SDE_THREADS, 2>(sme);
    case 4: return sde_fn<T, SDE_THREADS, 4>(sme);
    default: return sde_fn<T, SDE_THREADS, 8>(sme);
    }
}

static const void *sde_kernel(const SdeParams &p, bool f64)
{
    return f64 ? sde_pick<double>(p.rows, p.sme != 0) : sde_pick<float>(p.rows, p.sme != 0);
}

int sde_grid(const SdeParams &p, bool f64, int device)
{
    const void *fn = sde_kernel(p, f64);
    size_t lds = sde_lds_bytes(p, f64);
    int threads = sde_threads(p, f64);
    if (const void *reg = sde_reg_kernel(p, f64, &threads)) fn = reg, lds = 0;
    if (lds > 65536) (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    return (int)std::max<int64_t>(1, std::min<int64_t>(p.ntraj, (int64_t)per_cu * device_cus(device)));
}

void sde_launch(const SdeParams &p, const SdeParams *dev_p, bool f64, int grid, hipStream_t s)
{
    void *args[] = {(void *)&dev_p};
    int threads = sde_threads(p, f64);
    if (const void *reg = sde_reg_kernel(p, f64, &threads)) {
        (void)hipLaunchKernel(reg, dim3(grid), dim3(threads), args, 0, s);
        return;
    }
    (void)hipLaunchKernel(sde_kernel(p, f64), dim3(grid), dim3(threads), args, sde_lds_bytes(p, f64), s);
}

}  // namespace qt
