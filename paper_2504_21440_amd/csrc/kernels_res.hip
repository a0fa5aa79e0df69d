// kernels_res.hip -- resident solver for small master-equation problems on gfx950.
//
// A small problem's right-hand side (arXiv:2504.21440, Sec. 3.2) is a few thousand complex
// multiply-adds: spread over launches it costs launch latency (3 to 8 us a stage whatever the size),
// and as dense matrix products it is nearly all multiplications by zero (a driven cavity of cutoff 80
// has 6 generator entries per element against 3 x 80 inner steps on the matrix cores).  Here one
// workgroup integrates one problem for the whole launch: the adaptive Dormand-Prince 5(4) loop, step
// control, save-time landing and expectation values included.
//
// The problems taken are constant generators with a Hermitian initial state.  L(rho)^dag = L(rho^dag)
// for every Lindblad form, so rho stays Hermitian and only the elements i <= j are integrated; each
// is written to LDS together with its mirror image, with a real diagonal, so every stage input is
// exactly Hermitian.  A thread owns R elements, with the stages of each and the W generator entries of
// each (value and 16-bit LDS offset) in registers, so a right-hand side is W LDS gathers per element
// and no memory traffic: what bounds it is LDS gathers and multiply-add issue for the large
// classes and the latency of one gather-accumulate-write-barrier round for the small ones.
// LDS holds two matrices, so one barrier separates consecutive stages; their row stride is that of the
// largest dimension of the kernel class, made odd, which keeps the mirror writes (a column of the matrix) on
// distinct banks.
//
// A step is six rounds.  For a constant L, k2 = L (y + a21 h k1) = k1 + a21 h (L k1) with k1 = k7 of
// the step before, so k7 is written to LDS as soon as it is known, and the product L k7 is formed while
// the step control (FP64 logarithm, exponential, square root) runs: the control's latency is hidden
// behind the gathers, and a rejection (rare) forms L k1 again.
//
// Measured (MI355X, lone driven cavities, us a step of six right-hand sides in solves of 20 to 130 steps, start and
// 20 save times included; before: the staged CSR kernels below d = 55 in FP64, the matrix-core kernel for mixed
// precision):
//   d = 20 FP64 3.6 (21.2 before; 2.8 over 783 steps), d = 44 FP64 5.6, d = 60 mixed 8.9, d = 80 mixed 15.2 (120
//   before).
// A sweep of 64 cavities of cutoff 10 to 80 over t = 1 went from 71 to 8.4 ms.  With 16-bit offsets in
// registers instead of the band's constant ones the d = 80 step took 23.4 us (spilled registers).
//
// FP64, as in the other solvers: step control, error norm (an element above the diagonal counts for
// itself and its mirror), trace renormalisation (mixed precision) and expectation values.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "qt_common.h"
#include "qt_host.h"
#include "qt_res.h"

namespace qt {

// One DPP step of a wave sum of doubles: v += v shifted as CTRL says, zero where nothing arrives.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// The sum over the wave, in lane 63 (row shifts within 16 lanes, then row broadcasts: no LDS traffic).
__device__ __forceinline__ double wave_sum63(double v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    return dpp_add<0x143, 0xc>(v);
}

// Largest dimension whose upper triangle a workgroup of `elems` elements holds.
template <typename T> constexpr int res_dmax(int elems)
{
    int d = 1;
    while (d < (sizeof(T) == 8 ? RES_MAX_D_F64 : RES_MAX_D) && (d + 1) * (d + 2) / 2 <= elems) ++d;
    return d;
}
// One LDS matrix: rows of S elements behind S + 1 and before S + 2 elements that stay zero (the
// neighbours a band reads past the matrix; the threads without an element write a zero to the one in
// front of the first row).  S, and so the offset of the second matrix, is a constant of the class, so
// a gather is one LDS read with an immediate offset; byte offsets inside a matrix fit 16 bits.
constexpr int res_stride(int dmax) { return dmax | 1; }
constexpr int res_elems(int dmax) { return (dmax + 2) * res_stride(dmax) + 3; }
// Band classes (W = 0): the sources of element (i, j) are (i-1,j), (i,j-1), (i,j), (i,j+1), (i+1,j) and
// (i+1,j+1), which is a tridiagonal Hamiltonian with lowering operators (a driven cavity).  Their six
// reads need no offsets in registers and no address arithmetic.
constexpr int RES_BAND = 6;

template <typename T, int TPB, int R, int W>
__global__ __launch_bounds__(TPB) void k_res(const ResInst *__restrict__ insts, ResCtl *__restrict__ ctls,
                                             const int32_t *__restrict__ order, int budget, int reset)
{
    using V = typename vec2<T>::type;
    constexpr int NW = TPB / 64;
    constexpr bool BAND = W == 0;
    constexpr int WE = BAND ? RES_BAND : W;      // entries per element
    constexpr int WP = BAND ? 1 : (W + 1) / 2;  // packed offset words per element
    constexpr int XP = 2;            // expectation entries per lane held in registers
    constexpr int DMAX = res_dmax<T>(TPB * R), S = res_stride(DMAX), ES = (int)sizeof(V);
    constexpr int LB = (res_elems(DMAX) * ES + 15) / 16 * 16;
    static_assert(LB <= 65536, "16-bit byte offsets");
    constexpr int FRONT = S + 1;  // elements before (0, 0)
    __shared__ __align__(16) char smem[2 * LB];
    __shared__ double red[3 * NW];
    const int ii = order[blockIdx.x];
    const ResInst &g = insts[ii];
    ResCtl *C = ctls + ii;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int d = g.d, ntri = d * (d + 1) / 2, n = d * d;
    const double nd = (double)n, atol = g.atol, rtol = g.rtol;
    const bool renorm = g.renorm != 0, steady = g.steady_tol2 > 0.0;
    V *yv = (V *)g.vec, *kv = yv + n, *lv = kv + ntri;

    if (!reset && C->status != ST_RUNNING && C->status != RES_ST_INIT) return;

    // This thread's elements: the LDS byte offsets of (i, j), low half, and of its mirror, high half
    // (equal on the diagonal).  Elements past the triangle hold zeros and write the spare slot, so
    // they add nothing to any sum and need no branch.
    uint32_t o12[R];
    V val[R][WE];
    uint32_t off[R][WP];
    // row and column of element e, row-major over i <= j: the largest i with i d - i (i - 1) / 2 <= e
    auto place = [&](int e, int &i, int &j) {
        const float q = 2.0f * d + 1.0f;
        i = (int)((q - sqrtf(fmaxf(0.0f, q * q - 8.0f * e))) * 0.5f);
        i = max(0, min(d - 1, i));
        while (i > 0 && i * d - i * (i - 1) / 2 > e) --i;
        while (i + 1 < d && (i + 1) * d - (i + 1) * i / 2 <= e) ++i;
        j = i + e - (i * d - i * (i - 1) / 2);
    };
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int e = tid + m * TPB;
        const bool ok = e < ntri;
        int i = 0, j = 0, beg = 0, len = 0;
        o12[m] = (uint32_t)((FRONT - 1) * ES) * 0x10001u;
        if (ok) {
            place(e, i, j);
            o12[m] = (uint32_t)((FRONT + i * S + j) * ES) | (uint32_t)((FRONT + j * S + i) * ES) << 16;
            if (g.rowptr) {
                beg = g.rowptr[i * d + j];
                len = g.rowptr[i * d + j + 1] - beg;
            }
        }
#pragma unroll
        for (int p = 0; p < WP; ++p) off[m][p] = 0;
#pragma unroll
        for (int k = 0; k < WE; ++k) val[m][k].x = val[m][k].y = T(0);
#pragma unroll
        for (int k = 0; k < WE; ++k) {
            V a;
            a.x = a.y = T(0);
            int c = i * d + j;
            if (g.rowptr) {
                if (k < len) {
                    a = gld((const V *)g.val + beg + k);
                    c = gld(g.col + beg + k);
                }
            } else if (ok && k < g.W) {
                a = gld((const V *)g.val + (size_t)k * ntri + e);
                c = gld(g.col + (size_t)k * ntri + e);
            }
            const int ci = c / d, cj = c - ci * d;
            if constexpr (BAND) {
                const int di = ci - i, dj = cj - j;
                const int q = di < 0 ? 0 : di == 0 ? 2 + dj : 4 + dj;  // -1: (i-1,j) .. as listed above
#pragma unroll
                for (int u = 0; u < WE; ++u)
                    if (u == q && (a.x != T(0) || a.y != T(0))) val[m][u] = a;
            } else {
                val[m][k] = a;
                off[m][k >> 1] |= (uint32_t)((FRONT + ci * S + cj) * ES) << (16 * (k & 1));
            }
        }
    }
    for (int q = tid; q < 2 * LB / 16; q += TPB) *(double2 *)(smem + 16 * q) = make_double2(0.0, 0.0);
    __syncthreads();
    const V *b0 = (const V *)smem + FRONT;  // element (0, 0) of the first matrix, for the expectation values
    constexpr std::integral_constant<int, 0> M0{};
    constexpr std::integral_constant<int, 1> M1{};
    // this wave's first expectation operator: its first entries per lane
    int xb = 0, xe = 0, xo[XP];
    double2 xv[XP];
#pragma unroll
    for (int u = 0; u < XP; ++u) {
        xo[u] = 0;
        xv[u] = make_double2(0.0, 0.0);
    }
    if (w < g.ne) {
        xb = g.eptr[(size_t)w * (d + 1)];
        xe = g.eptr[(size_t)w * (d + 1) + d];
#pragma unroll
        for (int u = 0; u < XP; ++u) {
            const int p = xb + lane + 64 * u;
            if (p < xe) {
                const int c = g.evidx[p];
                xo[u] = (c / d) * S + c % d;
                xv[u] = gld(g.eval + p);
            }
        }
    }

    // v and its mirror image into matrix B (0 or 1)
    auto put = [&](auto B, int m, V v) {
        char *p = smem + decltype(B)::value * LB;
        V c = v;
        c.y = -v.y;
        *(V *)(p + (o12[m] >> 16)) = c;
        *(V *)(p + (o12[m] & 0xffffu)) = v;
    };
    auto diag = [&](int m) { return (o12[m] >> 16) == (o12[m] & 0xffffu); };
    // Large element counts leave few registers: keep the scheduler from mixing elements, whose
    // gathers in flight it would otherwise spill for.
    auto fence = [] {
        if constexpr (R * sizeof(T) >= 20) __builtin_amdgcn_sched_barrier(0);
    };
    // (L x) of every own element for the x in matrix B, two accumulation chains per component.  With
    // several elements a thread, packed offsets are unpacked at every use (an opaque copy): unpacked
    // once, they would take the registers that the elements need.
    auto apply = [&](auto B, V(&out)[R]) {
        const char *x = smem + decltype(B)::value * LB;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            T pr = 0, nr = 0, pi = 0, qi = 0;
            if constexpr (BAND) {
                // byte offsets from element (i - 1, j - 1)
                constexpr int rel[RES_BAND] = {1, S, S + 1, S + 2, 2 * S + 1, 2 * S + 2};
                const char *p = x + (o12[m] & 0xffffu) - (S + 1) * ES;
#pragma unroll
                for (int k = 0; k < RES_BAND; ++k) {
                    const V z = *(const V *)(p + rel[k] * ES);
                    pr = fma(val[m][k].x, z.x, pr);
                    nr = fma(val[m][k].y, z.y, nr);
                    pi = fma(val[m][k].x, z.y, pi);
                    qi = fma(val[m][k].y, z.x, qi);
                }
            } else {
#pragma unroll
                for (int k = 0; k < W; k += 2) {
                    uint32_t o = off[m][k >> 1];
                    if constexpr (R > 1) asm volatile("" : "+v"(o));
                    const V z = *(const V *)(x + (o & 0xffffu));
                    pr = fma(val[m][k].x, z.x, pr);
                    nr = fma(val[m][k].y, z.y, nr);
                    pi = fma(val[m][k].x, z.y, pi);
                    qi = fma(val[m][k].y, z.x, qi);
                    const V z1 = *(const V *)(x + (o >> 16));
                    pr = fma(val[m][k + 1].x, z1.x, pr);
                    nr = fma(val[m][k + 1].y, z1.y, nr);
                    pi = fma(val[m][k + 1].x, z1.y, pi);
                    qi = fma(val[m][k + 1].y, z1.x, qi);
                }
            }
            out[m].x = pr - nr;
            out[m].y = diag(m) ? T(0) : pi + qi;
            fence();
        }
    };
    auto weight = [&](int m) { return diag(m) ? 1.0 : 2.0; };
    // Publish this wave's part of N sums; after the next barrier total(q) is the block's sum.
    auto post = [&](int q, double v) {
        v = wave_sum63(v);
        if (lane == 63) red[q * NW + w] = v;
    };
    auto total = [&](int q) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < NW; ++u) s += red[q * NW + u];
        return uni(s);
    };
    // expectation values of the state in buf times sc, one wave per operator in turn
    auto record = [&](const V *buf, int idx, double sc) {
        for (int k = w; k < g.ne; k += NW) {
            double sr = 0.0, si = 0.0;
            int b = xb, e = xe;
            if (k == w) {
#pragma unroll
                for (int u = 0; u < XP; ++u) {
                    const double2 r = to_d2(buf[xo[u]]);
                    if (b + lane + 64 * u < e) {
                        sr += xv[u].x * r.x - xv[u].y * r.y;
                        si += xv[u].x * r.y + xv[u].y * r.x;
                    }
                }
                b += 64 * XP;
            } else {
                b = g.eptr[(size_t)k * (d + 1)];
                e = g.eptr[(size_t)k * (d + 1) + d];
            }
            for (int p = b + lane; p < e; p += 64) {
                const int c = g.evidx[p];
                const double2 o = gld(g.eval + p);
                const double2 r = to_d2(buf[(c / d) * S + c % d]);
                sr += o.x * r.x - o.y * r.y;
                si += o.x * r.y + o.y * r.x;
            }
            sr = wave_sum63(sr);
            si = wave_sum63(si);
            if (lane == 63) gst(g.expect + (size_t)k * g.nt + idx, make_double2(sr * sc, si * sc));
        }
    };

    V y[R], k1[R], lk[R];
    const double ql = DP5_Q[min(lane, (int)QN - 1)];
    double t, h, lprev, err_prev, tr0;
    int status, save_idx, last_rejected;
    int64_t n_accept, n_reject, n_steps, n_rhs;
    if (reset || C->status == RES_ST_INIT) {
        // the Hermitian part of the initial state
        const V *r0 = (const V *)g.rho0;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            y[m].x = y[m].y = T(0);
            if (tid + m * TPB < ntri) {
                int i, j;
                place(tid + m * TPB, i, j);
                const V a = gld(r0 + (size_t)i * d + j), b = gld(r0 + (size_t)j * d + i);
                y[m].x = T(0.5) * (a.x + b.x);
                y[m].y = T(0.5) * (a.y - b.y);
            }
            put(M0, m, y[m]);
        }
        __syncthreads();
        t = gld(g.tlist);
        err_prev = 1e-4;
        save_idx = 1;
        last_rejected = 0;
        n_accept = n_reject = n_steps = n_rhs = 0;
        status = ST_RUNNING;
        record(b0, 0, 1.0);
        apply(M0, k1);
        double s0 = 0.0, s1 = 0.0, tr = 0.0;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const double wt = weight(m), y2 = abs2d(y[m]), sc = atol + rtol * sqrt(y2);
            s0 += wt * (y2 / (sc * sc));
            s1 += wt * (abs2d(k1[m]) / (sc * sc));
            if (diag(m)) tr += (double)y[m].x;
        }
        post(0, s0);
        post(1, s1);
        post(2, tr);
        __syncthreads();
        const double d0 = sqrt(total(0) / nd), d1 = sqrt(total(1) / nd);
        tr0 = total(2);
        h = 0.0;
        n_rhs = 1;
        if (g.nt <= 1) {
            status = ST_DONE;
        } else if (g.use_h0) {
            h = g.h0;
        } else {
            const double h0 = (d0 < 1e-5 || d1 < 1e-5) ? 1e-6 : 0.01 * d0 / d1;
#pragma unroll
            for (int m = 0; m < R; ++m) {
                V v = y[m];
                caxpy(v, (T)h0, k1[m]);
                put(M1, m, v);
            }
            __syncthreads();  // every thread has read the sums of the first evaluation, too
            V f1[R];
            apply(M1, f1);
            double s2 = 0.0;
#pragma unroll
            for (int m = 0; m < R; ++m) {
                const double sc = atol + rtol * sqrt(abs2d(y[m]));
                const double dx = ((double)f1[m].x - (double)k1[m].x) / h0, dy = ((double)f1[m].y - (double)k1[m].y) / h0;
                s2 += weight(m) * ((dx * dx + dy * dy) / (sc * sc));
            }
            post(0, s2);
            __syncthreads();
            const double d2 = sqrt(total(0) / nd), mx = fmax(d1, d2);
            const double h1 = (mx <= 1e-15) ? fmax(1e-6, h0 * 1e-3) : pow(0.01 / mx, 0.2);
            h = fmin(100.0 * h0, h1);
            n_rhs = 2;
        }
        __syncthreads();
        // L k1 for the first step
#pragma unroll
        for (int m = 0; m < R; ++m) put(M1, m, k1[m]);
        __syncthreads();
        apply(M1, lk);
    } else {
        t = C->t;
        h = C->h;
        err_prev = C->err_prev;
        tr0 = C->tr0;
        status = C->status;
        save_idx = C->save_idx;
        last_rejected = C->last_rejected;
        n_accept = C->n_accept;
        n_reject = C->n_reject;
        n_steps = C->n_steps;
        n_rhs = C->n_rhs;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            y[m].x = y[m].y = T(0);
            k1[m] = y[m];
            lk[m] = y[m];
            const int e = tid + m * TPB;
            if (e < ntri) {
                int i, j;
                place(e, i, j);
                y[m] = gld(yv + (size_t)i * d + j);
                k1[m] = gld(kv + e);
                lk[m] = gld(lv + e);
            }
        }
    }
    lprev = uni(log(err_prev));
    // the save time a step may land on, and the one after it (requested one landing ahead)
    double tsave = save_idx < g.nt ? gld(g.tlist + save_idx) : 0.0;
    double tnext = save_idx + 1 < g.nt ? gld(g.tlist + save_idx + 1) : 0.0;

    while (status == ST_RUNNING && budget != 0) {
        if (budget > 0) --budget;
        int32_t land;
        const double ht = uni(clip_step(t, h, tsave, &land));
        land = __builtin_amdgcn_readfirstlane(land);
        V k2[R], k3[R], k4[R], k5[R];
        const double hq = ht * ql;  // h times every weight, one a lane
        const T tq = (T)hq;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            k2[m] = k1[m];
            caxpy(k2[m], lane_of(tq, Q21), lk[m]);
            V o = y[m];
            caxpy(o, lane_of(tq, Q31), k1[m]);
            caxpy(o, lane_of(tq, Q32), k2[m]);
            put(M0, m, o);
            fence();
        }
        __syncthreads();
        apply(M0, k3);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            V o = y[m];
            caxpy(o, lane_of(tq, Q41), k1[m]);
            caxpy(o, lane_of(tq, Q42), k2[m]);
            caxpy(o, lane_of(tq, Q43), k3[m]);
            put(M1, m, o);
            fence();
        }
        __syncthreads();
        apply(M1, k4);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            V o = y[m];
            caxpy(o, lane_of(tq, Q51), k1[m]);
            caxpy(o, lane_of(tq, Q52), k2[m]);
            caxpy(o, lane_of(tq, Q53), k3[m]);
            caxpy(o, lane_of(tq, Q54), k4[m]);
            put(M0, m, o);
            fence();
        }
        __syncthreads();
        apply(M0, k5);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            V o = y[m];
            caxpy(o, lane_of(tq, Q61), k1[m]);
            caxpy(o, lane_of(tq, Q62), k2[m]);
            caxpy(o, lane_of(tq, Q63), k3[m]);
            caxpy(o, lane_of(tq, Q64), k4[m]);
            caxpy(o, lane_of(tq, Q65), k5[m]);
            put(M1, m, o);
            fence();
        }
        __syncthreads();
        V yn[R];
        double2 er[R];  // h sum_j (b_j - bhat_j) k_j up to k6, FP64
        double tr = 0.0;
        {
            V k6[R];
            apply(M1, k6);
#pragma unroll
            for (int m = 0; m < R; ++m) {
                V o = y[m];
                caxpy(o, lane_of(tq, QB1), k1[m]);
                caxpy(o, lane_of(tq, QB3), k3[m]);
                caxpy(o, lane_of(tq, QB4), k4[m]);
                caxpy(o, lane_of(tq, QB5), k5[m]);
                caxpy(o, lane_of(tq, QB6), k6[m]);
                yn[m] = o;
                put(M0, m, o);
                if (diag(m)) tr += (double)o.x;
                er[m] = make_double2(0.0, 0.0);
                caxpy(er[m], lane_of(hq, QE1), to_d2(k1[m]));
                caxpy(er[m], lane_of(hq, QE3), to_d2(k3[m]));
                caxpy(er[m], lane_of(hq, QE4), to_d2(k4[m]));
                caxpy(er[m], lane_of(hq, QE5), to_d2(k5[m]));
                caxpy(er[m], lane_of(hq, QE6), to_d2(k6[m]));
                fence();
            }
        }
        __syncthreads();
        V k7[R];
        apply(M0, k7);
        double e2 = 0.0, l2 = 0.0;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            put(M1, m, k7[m]);
            caxpy(er[m], lane_of(hq, QE7), to_d2(k7[m]));
            // max(|y|, |y_new|) by the squares: one square root per element
            const double sc = atol + rtol * sqrt(fmax(abs2d(y[m]), abs2d(yn[m])));
            e2 += weight(m) * ((er[m].x * er[m].x + er[m].y * er[m].y) / (sc * sc));
            if (steady) l2 += weight(m) * abs2d(k7[m]);
            fence();
        }
        post(0, e2);
        if (renorm) post(1, tr);
        if (steady) post(2, l2);
        __syncthreads();
        apply(M1, lk);  // L k7: stage 2 of the next step, while the control below decides
        n_rhs += 6;
        ++n_steps;
        const double err = uni(sqrt(total(0) / nd));
        if (!isfinite(err)) {
            status = 6;  // QT_ENONFINITE
            break;
        }
        const double le = uni(log(err));
        if (err <= 1.0) {
            ++n_accept;
            const double sc = renorm ? tr0 / total(1) : 1.0;
            const bool conv = steady && total(2) * sc * sc <= g.steady_tol2;
            if (conv) {
                for (int k = save_idx; k < g.nt; ++k) record(b0, k, sc);
            } else if (land) {
                record(b0, save_idx, sc);
            }
            t = uni(land ? tsave : t + ht);
            const T ts = (T)sc;
#pragma unroll
            for (int m = 0; m < R; ++m) {
                y[m] = renorm ? cscale(yn[m], ts) : yn[m];
                k1[m] = renorm ? cscale(k7[m], ts) : k7[m];
                if (renorm) lk[m] = cscale(lk[m], ts);
            }
            // h clamp(0.9 err^-0.17 err_prev^0.04, 0.2, 10) from the logarithms
            double hn = ht * (err == 0.0 ? 10.0 : fmin(10.0, fmax(0.2, 0.9 * exp(0.04 * lprev - 0.17 * le))));
            if (last_rejected && hn > ht) hn = ht;
            h = uni(hn);
            err_prev = fmax(err, 1e-4);
            lprev = err > 1e-4 ? le : log(1e-4);
            last_rejected = 0;
            if (conv) {
                save_idx = g.nt;
                status = ST_DONE;
            } else if (land) {
                ++save_idx;
                if (save_idx >= g.nt) status = steady ? 4 : ST_DONE;  // QT_EMAXSTEPS: not converged
                tsave = uni(tnext);
                if (save_idx + 1 < g.nt) tnext = gld(g.tlist + save_idx + 1);
            }
            if (land) __syncthreads();  // the expectation values are read before b0 is written again
        } else {
            ++n_reject;
            h = uni(ht * fmax(0.2, 0.9 * exp(-0.17 * le)));
            last_rejected = 1;
            __syncthreads();
#pragma unroll
            for (int m = 0; m < R; ++m) put(M1, m, k1[m]);
            __syncthreads();
            apply(M1, lk);
        }
        if (status == ST_RUNNING) {
            if (n_steps >= g.max_steps) status = 4;  // QT_EMAXSTEPS
            else if (h < 1e-14 * fmax(1.0, fabs(t))) status = 5;  // QT_EDTMIN
        }
    }
    // the state, whole; while the problem runs on, k1 and L k1 too
#pragma unroll
    for (int m = 0; m < R; ++m)
        if (tid + m * TPB < ntri) {
            int i, j;
            place(tid + m * TPB, i, j);
            V c = y[m];
            c.y = -c.y;
            if (i != j) gst(yv + (size_t)j * d + i, c);
            gst(yv + (size_t)i * d + j, y[m]);
            if (status == ST_RUNNING) {
                gst(kv + tid + m * TPB, k1[m]);
                gst(lv + tid + m * TPB, lk[m]);
            }
        }
    if (tid == 0) {
        C->t = t;
        C->h = h;
        C->err_prev = err_prev;
        C->tr0 = tr0;
        C->status = status;
        C->save_idx = save_idx;
        C->last_rejected = last_rejected;
        C->n_accept = n_accept;
        C->n_reject = n_reject;
        C->n_steps = n_steps;
        C->n_rhs = n_rhs;
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
int res_width(const HCsr &A, const std::vector<HCsr> &cs, bool *band)
{
    const int d = A.d;
    *band = false;
    if (d > RES_MAX_D) return 0;
    bool in = true;  // A tridiagonal, every C_k on the diagonal (alone) or one above it (alone)
    for (int i = 0; i < d; ++i)
        for (int64_t p = A.ptr[i]; p < A.ptr[i + 1]; ++p) in = in && std::abs(A.idx[p] - i) <= 1;
    for (const HCsr &c : cs) {
        int kinds = 0;
        for (int i = 0; i < d; ++i)
            for (int64_t p = c.ptr[i]; p < c.ptr[i + 1]; ++p)
                kinds |= c.idx[p] == i ? 1 : c.idx[p] == i + 1 ? 2 : 4;
        in = in && (kinds == 0 || kinds == 1 || kinds == 2);
    }
    *band = in;
    int w = 0;
    std::vector<int> offd(d, 0);
    for (int i = 0; i < d; ++i)
        for (int64_t p = A.ptr[i]; p < A.ptr[i + 1]; ++p) offd[i] += A.idx[p] != i;
    for (int i = 0; i < d; ++i)
        for (int j = i; j < d; ++j) {
            int64_t k = 1 + offd[i] + offd[j];
            for (const HCsr &c : cs) k += (c.ptr[i + 1] - c.ptr[i]) * (c.ptr[j + 1] - c.ptr[j]);
            if (k > RES_MAX_W) return 0;
            w = std::max(w, (int)k);
        }
    return w;
}

void res_build_ell(const HCsr &A, const std::vector<HCsr> &cs, int W, std::vector<int32_t> &col,
                   std::vector<double2> &val)
{
    const int d = A.d, ntri = d * (d + 1) / 2;
    col.assign((size_t)W * ntri, 0);
    val.assign((size_t)W * ntri, make_double2(0.0, 0.0));
    // the entries of one element, sorted by source: at most W of them, so insertion is the cheap way
    int32_t src[RES_MAX_W + 1];
    cd v[RES_MAX_W + 1];
    int e = 0, k = 0;
    auto add = [&](int32_t c, cd x) {
        int q = k;
        while (q > 0 && src[q - 1] > c) --q;
        if (q > 0 && src[q - 1] == c) {
            v[q - 1] += x;
            return;
        }
        for (int u = k; u > q; --u) src[u] = src[u - 1], v[u] = v[u - 1];
        src[q] = c;
        v[q] = x;
        ++k;
    };
    for (int i = 0; i < d; ++i)
        for (int j = i; j < d; ++j, ++e) {
            k = 0;
            for (int64_t p = A.ptr[i]; p < A.ptr[i + 1]; ++p) add(A.idx[p] * d + j, A.val[p]);
            for (int64_t p = A.ptr[j]; p < A.ptr[j + 1]; ++p) add(i * d + A.idx[p], std::conj(A.val[p]));
            for (const HCsr &c : cs)
                for (int64_t p = c.ptr[i]; p < c.ptr[i + 1]; ++p)
                    for (int64_t q = c.ptr[j]; q < c.ptr[j + 1]; ++q)
                        add(c.idx[p] * d + c.idx[q], c.val[p] * std::conj(c.val[q]));
            for (int u = 0; u < k; ++u) {
                col[(size_t)u * ntri + e] = src[u];
                val[(size_t)u * ntri + e] = make_double2(v[u].real(), v[u].imag());
            }
        }
}

// Kernel classes: threads per workgroup, elements per thread and entries per element (0: the band).
// The smallest class that holds a problem is taken.  The element counts are what 256 registers per lane
// hold at two waves per SIMD: in the band FP32 takes about 30 a piece and FP64 50, at 16 entries 67 and 100.
struct ResClass {
    int tpb, r, w, f64;
};
static const ResClass RES_CLASSES[] = {
    {256, 1, 0, 0}, {512, 1, 0, 0}, {512, 2, 0, 0}, {512, 4, 0, 0}, {512, 7, 0, 0},
    {256, 1, 16, 0}, {512, 1, 16, 0}, {512, 2, 16, 0},
    {256, 1, 0, 1}, {512, 1, 0, 1}, {512, 2, 0, 1}, {512, 3, 0, 1}, {512, 4, 0, 1},
    {256, 1, 16, 1}, {512, 1, 16, 1}, {512, 2, 16, 1},
};
constexpr int RES_NCLASSES = sizeof(RES_CLASSES) / sizeof(RES_CLASSES[0]);
int res_classes() { return RES_NCLASSES; }

int res_class(int d, int W, bool band, int prec)
{
    if (W <= 0 || W > RES_MAX_W || d > RES_MAX_D) return -1;
    for (int k = 0; k < RES_NCLASSES; ++k) {
        const ResClass &c = RES_CLASSES[k];
        const int dmax = c.f64 ? res_dmax<double>(c.tpb * c.r) : res_dmax<float>(c.tpb * c.r);
        if (c.f64 == (prec == QT_F64) && (c.w ? W <= c.w : band) && d <= dmax) return k;
    }
    return -1;
}

template <typename T, int TPB, int R, int W>
static qt_status launch_res(const ResInst *insts, ResCtl *ctls, const int32_t *order, int count, int msl,
                            int reset, hipStream_t s)
{
    hipLaunchKernelGGL((k_res<T, TPB, R, W>), dim3(count), dim3(TPB), 0, s, insts, ctls, order, msl, reset);
    QT_HIP(hipGetLastError());
    return QT_OK;
}

qt_status res_launch(int cls, bool f64, const ResInst *insts, ResCtl *ctls, const int32_t *order,
                     int count, int msl, int reset, hipStream_t s)
{
    if (count <= 0) return QT_OK;
    if (cls < 0 || cls >= RES_NCLASSES || RES_CLASSES[cls].f64 != (f64 ? 1 : 0))
        return set_error(QT_EINVAL, "resident solver: no such class");
    const ResClass &c = RES_CLASSES[cls];
#define QT_RES(T, TPB, R, W) \
    if (f64 == (sizeof(T) == 8) && c.tpb == TPB && c.r == R && c.w == W) \
        return launch_res<T, TPB, R, W>(insts, ctls, order, count, msl, reset, s);
    QT_RES(float, 256, 1, 0)
    QT_RES(float, 512, 1, 0)
    QT_RES(float, 512, 2, 0)
    QT_RES(float, 512, 4, 0)
    QT_RES(float, 512, 7, 0)
    QT_RES(float, 256, 1, 16)
    QT_RES(float, 512, 1, 16)
    QT_RES(float, 512, 2, 16)
    QT_RES(double, 256, 1, 0)
    QT_RES(double, 512, 1, 0)
    QT_RES(double, 512, 2, 0)
    QT_RES(double, 512, 3, 0)
    QT_RES(double, 512, 4, 0)
    QT_RES(double, 256, 1, 16)
    QT_RES(double, 512, 1, 16)
    QT_RES(double, 512, 2, 16)
#undef QT_RES
    return set_error(QT_EINVAL, "resident solver: class not built");
}

}  // namespace qt
