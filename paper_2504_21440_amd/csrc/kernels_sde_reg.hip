// kernels_sde_reg.hip -- stochastic trajectories with one measured operator, operators in registers.
//
// The scheme, the draws and the outputs are those of kernels_sde.hip (its header has the formulas).  That
// kernel reads A and B from L2 at every product, draws increments (an FP64 logarithm, square root, sine and cosine)
// at every step and passes nine barriers a step with one measured operator.  With one measured
// operator and few entries per row (the Lindbladian of a cavity and a qubit has 5, its measured operator
// 2), here
//   * a thread keeps the entries of its rows in registers, as values and 16-bit LDS byte offsets;
//   * thread t draws the increment of step s0 + t, so one round of draws serves TPB steps;
//   * a block sum is one barrier (each sum has its own slots), and the barrier that publishes mu also
//     frees the gathered vector for the supporting value: 5 barriers a step.
// What remains is the latency of those five gather-sum-barrier rounds; a workgroup is as small as the
// rows allow, so that several trajectories share a CU (states of up to 64 elements take one wave each,
// whose barriers cost nothing).
#include <algorithm>
#include <type_traits>

#include "qt_common.h"
#include "qt_rng.h"
#include "qt_sde.h"

namespace qt {

template <typename T, int TPB, int R, bool SME, int WA, int WB>
__global__ __launch_bounds__(TPB) void k_sde_reg(const SdeParams *__restrict__ Pp)
{
    using V = typename vec2<T>::type;
    constexpr int NW = TPB / 64;
    static_assert(WA % 2 == 0 && WB % 2 == 0 && TPB * R * sizeof(V) <= 65536, "packed byte offsets");
    const SdeParams &P = *Pp;
    __shared__ __align__(16) V xs[TPB * R];  // the vector the gathers read
    __shared__ double scr[6 * NW];
    __shared__ double zs[TPB];               // standard normals of steps s0 .. s0 + TPB - 1
    __shared__ unsigned long long jsh;
    const int n = P.n, d = P.d;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;

    V av[R][WA], bv[R][WB];
    uint32_t ao[R][WA / 2], bo[R][WB / 2];
    uint32_t dmask = 0;  // bit q: row q of this thread is a diagonal element (SME)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int r = tid + q * TPB;
        auto load = [&](const void *val, const int32_t *col, int width, int k, V &a, uint32_t &o) {
            a.x = a.y = T(0);
            o = 0;
            if (r < n && k < width) {
                a = gld((const V *)val + (size_t)k * n + r);
                o = (uint32_t)gld(col + (size_t)k * n + r) * (uint32_t)sizeof(V);
            }
        };
#pragma unroll
        for (int k = 0; k < WA; k += 2) {
            uint32_t o0, o1;
            load(P.a_val, P.a_col, P.WA, k, av[q][k], o0);
            load(P.a_val, P.a_col, P.WA, k + 1, av[q][k + 1], o1);
            ao[q][k / 2] = o0 | o1 << 16;
        }
#pragma unroll
        for (int k = 0; k < WB; k += 2) {
            uint32_t o0, o1;
            load(P.b_val, P.b_col, P.WB, k, bv[q][k], o0);
            load(P.b_val, P.b_col, P.WB, k + 1, bv[q][k + 1], o1);
            bo[q][k / 2] = o0 | o1 << 16;
        }
        if (SME && r < n && r % (d + 1) == 0) dmask |= 1u << q;
    }
    // sum_k val[k] x(col[k]) of one row, in the order of the entries
    auto dot = [&](const auto &val, const auto &off, auto width) {
        V acc;
        acc.x = acc.y = T(0);
#pragma unroll
        for (int k = 0; k < decltype(width)::value; k += 2) {
            cfma(acc, val[k], *(const V *)((const char *)xs + (off[k / 2] & 0xffffu)));
            cfma(acc, val[k + 1], *(const V *)((const char *)xs + (off[k / 2] >> 16)));
        }
        return acc;
    };
    constexpr std::integral_constant<int, WA> CA{};
    constexpr std::integral_constant<int, WB> CB{};
    // this wave's part of sum s; after the next barrier total(s) is the block's
    auto post = [&](int s, double v) {
        v = wave_sum(v);
        if (lane == 0) scr[s * NW + w] = v;
    };
    auto total = [&](int s) {
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < NW; ++u) t += scr[s * NW + u];
        return uni(t);
    };
    // this thread's share of mu for the state u and its image Bu, as in kernels_sde.hip
    auto mu_part = [&](V u, V bu, int q) {
        if constexpr (SME) return (dmask >> q) & 1u ? (double)bu.x : 0.0;
        else return (double)u.x * (double)bu.x + (double)u.y * (double)bu.y;
    };
    auto record = [&](uint64_t j, int idx) {
        for (int e = 0; e < P.ne; ++e) {
            const int32_t *ep = P.eptr + (size_t)e * (d + 1);
            double v[3] = {0.0, 0.0, 0.0};
            if constexpr (SME) {
                for (int p = ep[0] + tid; p < ep[d]; p += TPB) {
                    const double2 o = P.eval[p];
                    const double2 r = to_d2(xs[P.evidx[p]]);
                    v[0] += o.x * r.x - o.y * r.y;
                    v[1] += o.x * r.y + o.y * r.x;
                }
            } else {
                for (int i = tid; i < d; i += TPB) {
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
            post(0, v[0]);
            post(1, v[1]);
            if constexpr (!SME) post(2, v[2]);
            __syncthreads();
            const double nn = SME ? 1.0 : total(2);
            const double2 out = make_double2(total(0) / nn, total(1) / nn);
            if (tid == 0) P.expect_tr[((size_t)j * P.ne + e) * P.nt + idx] = out;
            __syncthreads();
        }
    };

    for (;;) {
        if (tid == 0) jsh = atomicAdd(P.queue, 1ull);
        __syncthreads();
        const uint64_t j = (uint64_t)__double_as_longlong(uni(__longlong_as_double((long long)jsh)));
        __syncthreads();
        if ((int64_t)j >= P.ntraj) break;
        V x[R];
        const V *x0 = (const V *)P.x0;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int r = tid + q * TPB;
            x[q].x = x[q].y = T(0);
            if (r < n) x[q] = x0[r];
            xs[r] = x[q];
        }
        __syncthreads();
        record(j, 0);
        int status = ST_RUNNING;
        uint32_t step = 0, s0 = 0;
        bool drawn = false;
        for (int iv = 0; iv + 1 < P.nt && status == ST_RUNNING; ++iv) {
            const double len = P.tlist[iv + 1] - P.tlist[iv];
            const int ns = P.nsub[iv];
            const double h = uni(len / (double)ns), sq = uni(sqrt(h));
            double cur = 0.0;
            for (int s = 0; s < ns; ++s, ++step) {
                if (!drawn || step - s0 == (uint32_t)TPB) {
                    // the normals of the next TPB steps (the others were last read before a barrier)
                    drawn = true;
                    s0 = step;
                    double z0, z1;
                    wiener_normals(P.seed, j, step + tid, 0u, &z0, &z1);
                    zs[tid] = z0;
                }
                V a[R], b[R];
                double m0 = 0.0, m1 = 0.0;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    a[q] = dot(av[q], ao[q], CA);
                    b[q] = dot(bv[q], bo[q], CB);
                    m0 += mu_part(x[q], b[q], q);
                    if constexpr (!SME) m1 += abs2d(x[q]);
                }
                post(0, m0);
                if constexpr (!SME) post(1, m1);
                __syncthreads();  // mu, the normals; every gather of x is done
                const double mu = uni(SME ? total(0) : 2.0 * total(0) / total(1));
                const double dW = uni(sq * zs[step - s0]);
                cur += mu * h + dW;
                V u[R], xn[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    if constexpr (!SME) {
                        caxpy(a[q], (T)(0.5 * mu), b[q]);
                        caxpy(a[q], (T)(-0.125 * mu * mu), x[q]);
                    }
                    caxpy(b[q], (T)(-P.cg * mu), x[q]);
                    V y = x[q];
                    caxpy(y, (T)h, a[q]);
                    u[q] = y;
                    caxpy(u[q], (T)sq, b[q]);
                    caxpy(y, (T)dW, b[q]);
                    xn[q] = y;
                    xs[tid + q * TPB] = u[q];
                }
                __syncthreads();
                m0 = m1 = 0.0;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    a[q] = dot(bv[q], bo[q], CB);  // B u
                    m0 += mu_part(u[q], a[q], q);
                    if constexpr (!SME) m1 += abs2d(u[q]);
                }
                post(2, m0);
                if constexpr (!SME) post(3, m1);
                __syncthreads();
                const double mus = uni(SME ? total(2) : 2.0 * total(2) / total(3));
                const double wgt = uni((dW * dW - h) / (2.0 * sq));
                double nr = 0.0;
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    caxpy(a[q], (T)(-P.cg * mus), u[q]);
                    caxpy(xn[q], (T)wgt, a[q]);
                    caxpy(xn[q], (T)(-wgt), b[q]);
                    if constexpr (SME) nr += (dmask >> q) & 1u ? (double)xn[q].x : 0.0;
                    else nr += abs2d(xn[q]);
                }
                post(4, nr);
                __syncthreads();
                const double sc = uni(SME ? total(4) : sqrt(total(4)));
                if (!isfinite(sc) || sc == 0.0) {
                    status = 6;  // QT_ENONFINITE
                    break;
                }
                const T inv = (T)(1.0 / sc);
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    x[q] = cscale(xn[q], inv);
                    xs[tid + q * TPB] = x[q];
                }
                __syncthreads();
            }
            if (status != ST_RUNNING) break;
            if (tid == 0) P.meas[(size_t)j * (P.nt - 1) + iv] = cur / len;
            record(j, iv + 1);
        }
        if (tid == 0) P.status[j] = status == ST_RUNNING ? ST_DONE : status;
        __syncthreads();
    }
}

template <typename T, int TPB, int R, bool SME> static const void *sde_reg_fn(int wa, int *threads)
{
    *threads = TPB;
    if (wa <= 6) return (const void *)k_sde_reg<T, TPB, R, SME, 6, 2>;
    return (const void *)k_sde_reg<T, TPB, R, SME, 12, 2>;
}

const void *sde_reg_kernel(const SdeParams &p, bool f64, int *threads)
{
    if (p.m != 1 || p.WB > 2 || p.WA > 12) return nullptr;
    const int n = p.n;
    // The smallest workgroup that holds the state.  500 trajectories of the 40-dimensional homodyne master
    // equation (n = 1,600, complex64, us a step): 7 rows in 256 threads 6.3, 4 in 512 6.5, 2 in 1,024 8.7,
    // from memory 21.5; complex128, 4 rows in 512 threads with spills: 24, from memory 35.
#define QT_SDE(T, TPB, R, SME)                                                  \
    if (f64 == (sizeof(T) == 8) && (p.sme != 0) == SME && n <= TPB * R)        \
        return sde_reg_fn<T, TPB, R, SME>(p.WA, threads);
    QT_SDE(float, 64, 1, false)
    QT_SDE(float, 256, 1, false)
    QT_SDE(float, 256, 4, false)
    QT_SDE(float, 512, 4, false)
    QT_SDE(float, 64, 1, true)
    QT_SDE(float, 256, 1, true)
    QT_SDE(float, 256, 2, true)
    QT_SDE(float, 256, 4, true)
    QT_SDE(float, 256, 7, true)
    QT_SDE(float, 512, 5, true)
    QT_SDE(double, 64, 1, false)
    QT_SDE(double, 256, 1, false)
    QT_SDE(double, 512, 2, false)
    QT_SDE(double, 512, 4, false)
    QT_SDE(double, 64, 1, true)
    QT_SDE(double, 256, 1, true)
    QT_SDE(double, 256, 2, true)
    QT_SDE(double, 512, 2, true)
    QT_SDE(double, 512, 4, true)
#undef QT_SDE
    return nullptr;
}

}  // namespace qt
