// mc_kernel.h -- device code of the trajectory kernel, shared by its two translation units: the variants
// that read A from memory (kernels_mc.hip) and those that hold it in registers (kernels_mc_reg.hip).
// What the kernel does is described at the top of kernels_mc.hip.
#pragma once
#include "qt_coef.h"
#include "qt_common.h"
#include "qt_mc.h"
#include "qt_rng.h"

namespace qt {

constexpr int MC_MAXC = 64;  // collapse channels handled by the jump kernel

__device__ __forceinline__ void traj_draw(uint64_t seed, uint64_t traj, uint32_t event, double *a, double *b)
{
    uint32_t c[4] = {(uint32_t)traj, (uint32_t)(traj >> 32), event, 0u};
    philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    *a = u01(c[0], c[1]);
    *b = u01(c[2], c[3]);
}

// Block sums of N doubles of the 256 virtual threads that own rows t, t + 256, t + 512, ... (result in
// every thread), whatever the workgroup size: f(m, c) gives the contributions of the thread's m-th row,
// a virtual thread adds its rows in order, then the wave sums and the waves are added in order.  So a
// trajectory is bitwise the same in every kernel variant.  With more than 256 threads the rows pass
// through `stage` (N * TPB * R doubles of LDS).
template <int N, int TPB, int R, typename F>
__device__ __forceinline__ void row_sums(F f, double (&v)[N], double *scr, double *stage)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = 0.0;
    if constexpr (TPB == MC_THREADS) {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            double c[N];
#pragma unroll
            for (int i = 0; i < N; ++i) c[i] = 0.0;
            f(m, c);
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] += c[i];
        }
    } else {
#pragma unroll
        for (int m = 0; m < R; ++m) {
            double c[N];
#pragma unroll
            for (int i = 0; i < N; ++i) c[i] = 0.0;
            f(m, c);
#pragma unroll
            for (int i = 0; i < N; ++i) stage[i * TPB * R + tid + m * TPB] = c[i];
        }
        __syncthreads();
        if (tid < MC_THREADS) {
#pragma unroll
            for (int q = 0; q < R * TPB / MC_THREADS; ++q)
#pragma unroll
                for (int i = 0; i < N; ++i) v[i] += stage[i * TPB * R + tid + q * MC_THREADS];
        }
    }
    if (tid < MC_THREADS) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = wave_sum(v[i]);
    }
    if constexpr (TPB == MC_THREADS) __syncthreads();
    if (lane == 0 && w < MC_THREADS / 64)
#pragma unroll
        for (int i = 0; i < N; ++i) scr[i * 16 + w] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < MC_THREADS / 64; ++k) s += scr[i * 16 + k];
        v[i] = uni(s);
    }
    __syncthreads();
}

// OCC: the waves per SIMD the register allocation must allow (1: no constraint).  A large ensemble
// gains from more resident trajectories even at the price of spilled registers; a single
// trajectory does not.  W > 0 (constant A of at most W entries per row): every thread holds the entries
// of its rows in registers, as a value and a 16-bit LDS byte offset.
template <typename T, int R, bool TD, int OCC, int TPB = MC_THREADS, int W = 0>
__global__ __launch_bounds__(TPB) __attribute__((amdgpu_waves_per_eu(OCC))) void k_mc(
    const McParams *__restrict__ Pp)
{
    using V = typename vec2<T>::type;
    const McParams &P = *Pp;
    extern __shared__ __align__(16) char smem[];  // 16-byte LDS accesses: off by 8 bytes they take hundreds of cycles
    const int d = P.d;
    V *xs0 = (V *)smem;
    V *xs1 = xs0 + (W > 0 ? TPB * R : d);
    // rows on their way into a block sum (more than 256 threads); three sums at most
    double *stage = (double *)(xs1 + (W > 0 ? TPB * R : d));
    __shared__ double scr[48];
    __shared__ double pk[MC_MAXC];  // channel weights |g_k(t*)|^2 |C_k psi|^2
    __shared__ double pn[MC_MAXC];  // |C_k psi|^2, for the post-jump normalisation
    __shared__ unsigned long long jsh;
    __shared__ double fsh;  // the step-size factor
    __shared__ V cwsh[MC_MAX_TERMS + 1];  // coefficients of the current right-hand side (TD)
    const int tid = threadIdx.x;
    const V *__restrict__ ev = (const V *)P.ell_val;
    const int32_t *__restrict__ ec = P.ell_col;
    const V *__restrict__ cv = (const V *)P.cval;

    constexpr int WR = W > 0 ? W : 2;
    V av[R][WR];
    uint32_t ao[R][WR / 2];
    if constexpr (W > 0) {
        static_assert(W % 2 == 0 && TPB * R * sizeof(V) <= 65536, "packed byte offsets");
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const int r = threadIdx.x + m * TPB;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                V a;
                a.x = a.y = T(0);
                uint32_t o = 0;
                if (r < d && k < P.W) {
                    a = gld(ev + (size_t)k * d + r);
                    o = (uint32_t)gld(ec + (size_t)k * d + r) * (uint32_t)sizeof(V);
                }
                av[m][k] = a;
                if (k & 1) ao[m][k / 2] |= o << 16;
                else ao[m][k / 2] = o;
            }
        }
        // the rows past d are read by nobody's entries but stay finite
        for (int i = threadIdx.x; i < 2 * TPB * R; i += TPB) xs0[i].x = xs0[i].y = T(0);
        __syncthreads();
    }

    const double ql = DP5_Q[min(tid & 63, (int)QN - 1)];
    auto row = [&](int m) { return tid + m * TPB; };
    // out = A(ts) x for own rows.  Every call site is preceded by a barrier after the previous
    // call, so the coefficient row may be rewritten here.
    auto rhs = [&](const V *x, V(&out)[R], double ts) {
        if constexpr (TD) {
            if (tid <= P.nterms) {
                double2 w = make_double2(1.0, 0.0);
                if (tid > 0) w = coef_value(P.coefs[tid - 1], ts);
                cwsh[tid] = from_d2<V>(w);
            }
            __syncthreads();
        }
        // complex64: entry k of all R rows of this thread at once, R independent load-gather-FMA
        // chains per entry rather than one row's W entries after another (measured: the L = 10
        // ensemble 58,700 -> 69,700 trajectories/s); complex128 keeps one row at a time, whose
        // registers the wider values would otherwise spill (22,000 -> 17,800).  Each row is summed
        // in the order k = 0 .. W-1 either way.  Global-only loads of the matrix stream: generic ones
        // would be ordered against, and waited for with, the LDS gathers of the state.
        V acc[R];
#pragma unroll
        for (int m = 0; m < R; ++m) {
            acc[m].x = 0;
            acc[m].y = 0;
        }
        if constexpr (W > 0) {
            const char *xb = (const char *)x;
#pragma unroll
            for (int k = 0; k < W; k += 2) {
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    uint32_t o = ao[m][k / 2];
                    // several rows: unpacked at each use (kept, the offsets would double); one row has
                    // the registers, and needs all its gathers in flight at once
                    if constexpr (R > 1) asm volatile("" : "+v"(o));
                    cfma(acc[m], av[m][k], *(const V *)(xb + (o & 0xffffu)));
                    cfma(acc[m], av[m][k + 1], *(const V *)(xb + (o >> 16)));
                }
                // 2 R gathers in flight: with all W R of them the rows would not fit the registers
                if constexpr (R * sizeof(T) >= 16) __builtin_amdgcn_sched_barrier(0);
            }
        } else if constexpr (sizeof(T) == 8) {
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d)
                    for (int k = 0; k < P.W; ++k) {
                        const size_t at = (size_t)k * d + r;
                        const int32_t c = gld(ec + at);
                        const V a = gld(ev + at);
                        if constexpr (TD)
                            cfma(acc[m], cmul(a, cwsh[c >> MC_TAG_SHIFT]), x[c & ((1 << MC_TAG_SHIFT) - 1)]);
                        else
                            cfma(acc[m], a, x[c]);
                    }
            }
        } else
        for (int k = 0; k < P.W; ++k) {
            int32_t c[R];
            V a[R];
#pragma unroll
            for (int m = 0; m < R; ++m)
                if (row(m) < d) {
                    const size_t at = (size_t)k * d + row(m);
                    c[m] = gld(ec + at);
                    a[m] = gld(ev + at);
                }
#pragma unroll
            for (int m = 0; m < R; ++m)
                if (row(m) < d) {
                    if constexpr (TD)
                        cfma(acc[m], cmul(a[m], cwsh[c[m] >> MC_TAG_SHIFT]), x[c[m] & ((1 << MC_TAG_SHIFT) - 1)]);
                    else
                        cfma(acc[m], a[m], x[c[m]]);
                }
        }
#pragma unroll
        for (int m = 0; m < R; ++m) out[m] = acc[m];
    };
    // weight |g_k(t)|^2 of collapse channel k (1 when constant)
    auto cweight = [&](int k, double tt) {
        if constexpr (TD) {
            const int q = P.cweight[k];
            if (q >= 0) return coef_value(P.coefs[q], tt).x;  // stored with modsq: the squared modulus
        }
        return 1.0;
    };
    // <x|O_q|x> / <x|x> for every e_op, into expect_tr[j][q][idx]
    auto record = [&](const V *x, uint64_t j, int idx) {
        for (int q = 0; q < P.ne; ++q) {
            const int32_t *ep = P.eptr + (size_t)q * (d + 1);
            double v[3];
            row_sums<3, TPB, R>([&](int m, double (&c3)[3]) {
                const int i = row(m);
                if (i >= d) return;
                double rr = 0.0, ri = 0.0;
                for (int p = ep[i]; p < ep[i + 1]; ++p) {
                    const double2 o = P.eval[p];
                    const double2 xv = to_d2(x[P.ecol[p]]);
                    rr += o.x * xv.x - o.y * xv.y;
                    ri += o.x * xv.y + o.y * xv.x;
                }
                const double2 c = to_d2(x[i]);
                c3[0] = c.x * rr + c.y * ri;
                c3[1] = c.x * ri - c.y * rr;
                c3[2] = c.x * c.x + c.y * c.y;
            }, v, scr, stage);
            if (tid == 0) P.expect_tr[((size_t)j * P.ne + q) * P.nt + idx] = make_double2(v[0] / v[2], v[1] / v[2]);
        }
    };

    for (;;) {
        if (tid == 0) jsh = atomicAdd(P.queue, 1ull);
        __syncthreads();
        const uint64_t j = (uint64_t)__double_as_longlong(uni(__longlong_as_double((long long)jsh)));
        __syncthreads();
        if ((int64_t)j >= P.ntraj) break;

        V y[R], k[7][R], yn[R];
        const V *p0 = (const V *)P.psi0;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const int r = row(m);
            if (r < d) {
                y[m] = p0[r];
                xs0[r] = y[m];
            } else {
                y[m].x = 0;
                y[m].y = 0;
            }
        }
        double r_th, unused;
        traj_draw(P.seed, j, 0u, &r_th, &unused);
        uint32_t event = 1;
        int64_t njump = 0, nrhs = 0, nacc = 0, nrej = 0, steps = 0;
        int status = ST_RUNNING;
        double t = P.tlist[0];
        __syncthreads();
        record(xs0, j, 0);
        int idx = 1;

        // DP5 trial step of size hh from (t, y) with k[0] = A y: fills k[1..6], yn (also in xs1)
        // and returns the FP64 error norm; nn receives |yn|^2.
        // keep the scheduler from mixing rows where they fill the registers
        auto fence = [] {
            if constexpr (W > 0 && R * sizeof(T) >= 16) __builtin_amdgcn_sched_barrier(0);
        };
        auto attempt = [&](double hh, double &nn) -> double {
            __syncthreads();
            const double hq = hh * ql;  // hh times every weight, one a lane
            const T tq = (T)hq;
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d) {
                    V x = y[m];
                    caxpy(x, lane_of(tq, Q21), k[0][m]);
                    xs0[r] = x;
                }
                fence();
            }
            __syncthreads();
            rhs(xs0, k[1], t + DP5::c2 * hh);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d) {
                    V x = y[m];
                    caxpy(x, lane_of(tq, Q31), k[0][m]);
                    caxpy(x, lane_of(tq, Q32), k[1][m]);
                    xs1[r] = x;
                }
                fence();
            }
            __syncthreads();
            rhs(xs1, k[2], t + DP5::c3 * hh);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d) {
                    V x = y[m];
                    caxpy(x, lane_of(tq, Q41), k[0][m]);
                    caxpy(x, lane_of(tq, Q42), k[1][m]);
                    caxpy(x, lane_of(tq, Q43), k[2][m]);
                    xs0[r] = x;
                }
                fence();
            }
            __syncthreads();
            rhs(xs0, k[3], t + DP5::c4 * hh);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d) {
                    V x = y[m];
                    caxpy(x, lane_of(tq, Q51), k[0][m]);
                    caxpy(x, lane_of(tq, Q52), k[1][m]);
                    caxpy(x, lane_of(tq, Q53), k[2][m]);
                    caxpy(x, lane_of(tq, Q54), k[3][m]);
                    xs1[r] = x;
                }
                fence();
            }
            __syncthreads();
            rhs(xs1, k[4], t + DP5::c5 * hh);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                if (r < d) {
                    V x = y[m];
                    caxpy(x, lane_of(tq, Q61), k[0][m]);
                    caxpy(x, lane_of(tq, Q62), k[1][m]);
                    caxpy(x, lane_of(tq, Q63), k[2][m]);
                    caxpy(x, lane_of(tq, Q64), k[3][m]);
                    caxpy(x, lane_of(tq, Q65), k[4][m]);
                    xs0[r] = x;
                }
                fence();
            }
            __syncthreads();
            rhs(xs0, k[5], t + hh);
            double2 er[R];
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                V x = y[m];
                caxpy(x, lane_of(tq, QB1), k[0][m]);
                caxpy(x, lane_of(tq, QB3), k[2][m]);
                caxpy(x, lane_of(tq, QB4), k[3][m]);
                caxpy(x, lane_of(tq, QB5), k[4][m]);
                caxpy(x, lane_of(tq, QB6), k[5][m]);
                yn[m] = x;
                if (r < d) xs1[r] = x;
                // the error estimate up to k6: k3 .. k6 need no registers in the last right-hand side
                er[m] = make_double2(0.0, 0.0);
                caxpy(er[m], lane_of(hq, QE1), to_d2(k[0][m]));
                caxpy(er[m], lane_of(hq, QE3), to_d2(k[2][m]));
                caxpy(er[m], lane_of(hq, QE4), to_d2(k[3][m]));
                caxpy(er[m], lane_of(hq, QE5), to_d2(k[4][m]));
                caxpy(er[m], lane_of(hq, QE6), to_d2(k[5][m]));
                fence();
            }
            __syncthreads();
            rhs(xs1, k[6], t + hh);
            nrhs += 6;
            double v[2];
            row_sums<2, TPB, R>([&](int m, double (&c)[2]) {
                if (row(m) >= d) return;
                double2 e = er[m];
                caxpy(e, lane_of(hq, QE7), to_d2(k[6][m]));
                // the larger modulus by the squares: one square root, the same value
                const double n2 = abs2d(yn[m]), sc = P.atol + P.rtol * sqrt(fmax(abs2d(y[m]), n2));
                c[0] = (e.x * e.x + e.y * e.y) / (sc * sc);
                c[1] = n2;
            }, v, scr, stage);
            nn = v[1];
            return uni(sqrt(v[0] / d));
        };

        double h = 0.0;
        if (P.nt > 1) {
            rhs(xs0, k[0], t);
            nrhs += 1;
            if (P.use_h0) {
                h = P.h0;
            } else {
                double v[2];
                row_sums<2, TPB, R>([&](int m, double (&c)[2]) {
                    if (row(m) >= d) return;
                    const double ya = sqrt(abs2d(y[m]));
                    const double sc = P.atol + P.rtol * ya;
                    c[0] = ya * ya / (sc * sc);
                    c[1] = abs2d(k[0][m]) / (sc * sc);
                }, v, scr, stage);
                const double d0 = sqrt(v[0] / d), d1 = sqrt(v[1] / d);
                const double h0 = (d0 < 1e-5 || d1 < 1e-5) ? 1e-6 : 0.01 * d0 / d1;
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    const int r = row(m);
                    if (r < d) {
                        V x = y[m];
                        caxpy(x, (T)h0, k[0][m]);
                        xs1[r] = x;
                    }
                }
                __syncthreads();
                rhs(xs1, k[1], t + h0);
                nrhs += 1;
                double w2[1];
                row_sums<1, TPB, R>([&](int m, double (&c)[1]) {
                    if (row(m) >= d) return;
                    const double2 f1 = to_d2(k[1][m]), f0 = to_d2(k[0][m]);
                    const double sc = P.atol + P.rtol * sqrt(abs2d(y[m]));
                    const double dx = (f1.x - f0.x) / h0, dy = (f1.y - f0.y) / h0;
                    c[0] = (dx * dx + dy * dy) / (sc * sc);
                }, w2, scr, stage);
                const double d2 = sqrt(w2[0] / d);
                const double mx = fmax(d1, d2);
                const double h1 = (mx <= 1e-15) ? fmax(1e-6, h0 * 1e-3) : pow(0.01 / mx, 0.2);
                h = fmin(100.0 * h0, h1);
            }
        }
        double lprev = log(1e-4);  // logarithm of the last accepted error (floored), in the first wave
        int last_rej = 0;
        while (idx < P.nt) {
            if (steps >= P.max_steps) {
                status = 4;  // QT_EMAXSTEPS
                break;
            }
            ++steps;
            int32_t land;
            const double ht = uni(clip_step(t, h, P.tlist[idx], &land));
            land = __builtin_amdgcn_readfirstlane(land);
            double nrm;
            const double err = attempt(ht, nrm);
            if (!isfinite(err)) {
                status = 6;  // QT_ENONFINITE
                break;
            }
            // The step-size factor, 0.9 err^-0.17 err_prev^0.04 or 0.9 err^-0.17 after a rejection, within
            // [0.2, 10], from one logarithm and one exponential in the first wave (the two powers in
            // every wave were a quarter of the kernel's instructions).
            if (tid < 64) {
                const double le = log(err), lx = err > 1.0 ? -0.17 * le : 0.04 * lprev - 0.17 * le;
                const double f = err == 0.0 ? 10.0 : fmax(0.2, 0.9 * exp(lx));
                if (err <= 1.0) lprev = err > 1e-4 ? le : log(1e-4);
                if (tid == 0) fsh = err > 1.0 ? f : fmin(10.0, f);
            }
            __syncthreads();
            const double fac = uni(fsh);
            if (err > 1.0) {
                ++nrej;
                h = uni(ht * fac);
                last_rej = 1;
                if (h < 1e-14 * fmax(1.0, fabs(t))) {
                    status = 5;  // QT_EDTMIN
                    break;
                }
                continue;
            }
            ++nacc;
            double hn = uni(ht * fac);
            if (last_rej && hn > ht) hn = ht;
            last_rej = 0;
            if (nrm >= r_th || P.nc == 0) {  // no collapse channel: nothing to jump into
                t = uni(land ? P.tlist[idx] : t + ht);
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    y[m] = yn[m];
                    k[0][m] = k[6][m];
                }
                h = hn;
                if (land) record(xs1, j, idx++);
                continue;
            }
            // ---- quantum jump inside [t, t + ht]: locate the crossing of |psi|^2 = r ----
            double ny[1];
            row_sums<1, TPB, R>([&](int m, double (&c)[1]) {
                if (row(m) < d) c[0] = abs2d(y[m]);
            }, ny, scr, stage);
            const double lr = log(r_th);
            double a = 0.0, ga = log(ny[0]) - lr, b = 1.0, gb = log(nrm) - lr;
            double th = 1.0, thp = 1.0;
            int side = 0;
            for (int it = 0; it < 64; ++it) {
                th = (a * gb - b * ga) / (gb - ga);
                if (!(th > a && th < b)) th = 0.5 * (a + b);
                double nn;
                (void)attempt(uni(th * ht), nn);
                const double g = log(nn) - lr;
                if (fabs(g) <= 1e-12) break;
                if (fabs(th - thp) * ht <= 1e-10 * fmax(1.0, fabs(t))) break;
                thp = th;
                if (g > 0.0) {
                    a = th;
                    ga = g;
                    if (side == 1) gb *= 0.5;
                    side = 1;
                } else {
                    b = th;
                    gb = g;
                    if (side == -1) ga *= 0.5;
                    side = -1;
                }
            }
            // xs1 (and yn) hold psi at the crossing
            const double tj = uni(t + th * ht);
            double u, rnext;
            traj_draw(P.seed, j, event, &u, &rnext);
            ++event;
            for (int c = 0; c < P.nc; ++c) {
                const int32_t *cp = P.cptr + (size_t)c * (d + 1);
                double v[1];
                row_sums<1, TPB, R>([&](int m, double (&c1)[1]) {
                    const int i = row(m);
                    if (i >= d) return;
                    V acc;
                    acc.x = 0;
                    acc.y = 0;
                    for (int p = cp[i]; p < cp[i + 1]; ++p) cfma(acc, cv[p], xs1[P.ccol[p]]);
                    c1[0] = abs2d(acc);
                }, v, scr, stage);
                if (tid == 0) {
                    pn[c] = v[0];
                    pk[c] = v[0] * cweight(c, tj);
                }
            }
            __syncthreads();
            double tot = 0.0;
            for (int c = 0; c < P.nc; ++c) tot += pk[c];
            const double target = u * tot;
            double cum = 0.0;
            int ch = P.nc - 1;
            for (int c = 0; c < P.nc; ++c) {
                cum += pk[c];
                if (cum >= target) {
                    ch = c;
                    break;
                }
            }
            const double inv = 1.0 / sqrt(pn[ch]);
            const int32_t *cp = P.cptr + (size_t)ch * (d + 1);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const int r = row(m);
                V acc;
                acc.x = 0;
                acc.y = 0;
                if (r < d)
                    for (int p = cp[r]; p < cp[r + 1]; ++p) cfma(acc, cv[p], xs1[P.ccol[p]]);
                y[m] = cscale(acc, (T)inv);
            }
            if (tid == 0 && njump < P.maxj) {
                P.jtimes[(size_t)j * P.maxj + njump] = tj;
                P.jchan[(size_t)j * P.maxj + njump] = ch;
            }
            ++njump;
            r_th = rnext;
            // the root search keeps th strictly inside (0, 1), so a jump always falls before the end
            // of the step, and the save time it was aiming at (if any) is recorded by a later step
            t = tj;
            __syncthreads();  // every thread is done reading xs1 / pk / pn
#pragma unroll
            for (int m = 0; m < R; ++m)
                if (row(m) < d) xs0[row(m)] = y[m];
            __syncthreads();
            rhs(xs0, k[0], t);
            nrhs += 1;
            h = hn;
        }
        if (tid == 0) {
            P.njumps[j] = njump;
            P.status[j] = status == ST_RUNNING ? ST_DONE : status;
            P.nrhs[j] = nrhs;
            P.naccept[j] = nacc;
            P.nreject[j] = nrej;
        }
        __syncthreads();
    }
}

}  // namespace qt
