// kernels_op.hip -- the staged solver's right-hand side in operator form on gfx950.
//
// The superoperator of a chain of L spins has 4^L (1 + 2 L + L / 4) entries: 12 or 20 bytes of matrix per
// complex multiply-add, streamed at every stage (317 / 531 MB at L = 10), although it is made of d x d
// operators.  Where A = -i H - 1/2 sum C^dag C has few off-diagonal entries per row and every collapse
// operator at most one entry per row, the kernels here apply
//     L(rho)_ij = (A_ii + conj A_jj) rho_ij + sum_k A_ik rho_kj + sum_l conj(A_jl) rho_il
//               + sum_c C_c(i, k_c(i)) conj(C_c(j, k_c(j))) rho_{k_c(i) k_c(j)}
// from tables of a few hundred KB that stay in the caches, so the only memory traffic left is the state
// vectors.  The state is exactly Hermitian (the caller checks the initial one), so only the tiles on and
// above the diagonal are evaluated, and a workgroup writes its elements and, transposed through LDS, their
// conjugates below: half the sums and half the reads of the epilogue.
//
// What bounds it: one chain of L = 8 (160 workgroups) the latency of a wave, kernel by kernel -- 4.8 us a stage in
// complex64, of which the launch is about 2 -- so there a wave takes one row, the descriptor, the control record
// and the column's entries are requested together, and every source before the first sum; with descriptor
// words read where they are used it took 5.0 us (a solve to t = 10, 126 steps, 4.29 ms against 4.14, in complex128
// 4.05 against 3.66 ms), with two rows 6.1 us.
// L = 10 (complex128) the vector L1: 30 sources and 20 table words per element at 4 lanes a cycle are 12 us,
// beside 130 MB of state vectors from the L2s and the MALL; 28 us a stage (118 us for the matrix kernels, which
// stream 531 MB; 40 us without the Hermitian halving).  Two rows a wave read each column entry for two
// elements; four rows took 40 us (too few waves in flight), one row 33 us.  Sixteen chains of L = 8: 20 us a
// stage against 45 to 60 us.
//
// Precision: as in the assembled matrix, the factor of the element itself (the diagonals of A and the jumps that
// start from the element) is summed in FP64 and rounded once, and so is each product of two C entries.  With
// products of rounded C entries a diagonal channel's decay and jump, which cancel in the matrix, left 2e-7 of
// the rate: after t = 20 with C = sqrt(0.1) n (d = 160) populations were off by 7e-4 of the largest (now 3e-8, as
// with the matrix).  The derivative of a diagonal element is real, so the state stays exactly Hermitian.
// Everything else of a step -- stage combinations, error partials, control, expectation values -- is that of kernels_csr.hip, on
// the same descriptors, with op_blocks(d) partials a problem.
#include <type_traits>

#include "csr_kernels.h"

namespace qt {

// Scalar (uniform) views of a row's record: the constant address space makes the compiler read it with
// scalar loads, which the stores of the epilogue would otherwise rule out.
#define QT_CONST __attribute__((address_space(4)))
typedef float uf2 __attribute__((ext_vector_type(2)));
typedef double ud2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float2 uld(const float2 *p)
{
    const uf2 v = *(const QT_CONST uf2 *)p;
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ double2 uld(const double2 *p)
{
    const ud2 v = *(const QT_CONST ud2 *)p;
    return make_double2(v.x, v.y);
}
__device__ __forceinline__ int32_t uld(const int32_t *p) { return *(const QT_CONST int32_t *)p; }

// The element at a 32-bit byte offset of a vector (one address register, the base in scalar ones; vectors
// hold up to 4 GB: d <= OP_MAX_D).
template <typename V> __device__ __forceinline__ V at(const V *p, uint32_t off)
{
    return gld((const V *)((const char *)p + off));
}
template <typename P> __device__ __forceinline__ P *uniform_ptr(P *p)
{
    const uint64_t b = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return (P *)(((uint64_t)hi << 32) | lo);
}

// Rows and columns of a workgroup and of this wave: four waves' rows, RB each, of a 64 x 64 tile on or above
// the diagonal.  Row b of the triangle of T tiles has T - b of them; rows b and T - 1 - b together have
// T + 1, which makes the tile of a number one division.
template <int RB> struct OpItem {
    static constexpr int ROWS = 4 * RB;
    int ib, jb;  // the workgroup's first row and column
    int i0, j;   // this wave's first row; this lane's column (past the end: the last)
    bool jok;
    int i[RB];   // rows (past the end: the last)
    __device__ __forceinline__ OpItem(int blk, int d)
    {
        const int T = (d + 63) / 64, q = blk / (64 / ROWS), sub = blk % (64 / ROWS);
        int b = q / (T + 1), t = q % (T + 1);
        if (t < T - b) {
            t += b;
        } else {
            t -= T - b;
            b = T - 1 - b;
            t += b;
        }
        ib = b * 64 + sub * ROWS;
        jb = t * 64;
        i0 = ib + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * RB;
        const int jl = jb + (int)(threadIdx.x & 63);
        jok = jl < d;
        j = jok ? jl : d - 1;
#pragma unroll
        for (int r = 0; r < RB; ++r) i[r] = min(i0 + r, d - 1);
    }
    // whether this lane holds an element of the upper triangle in its row r
    __device__ __forceinline__ bool has(int r, int d) const { return jok && i0 + r < d && i0 + r <= j; }
};

// The elements below the diagonal, conj of those above: a workgroup's rows x 64 columns through LDS, so that
// runs of ROWS elements are written.  Uniform over the workgroup.
template <typename V, int RB> struct OpMirror {
    static constexpr int ROWS = 4 * RB;
    V m[ROWS][65];  // 65: the columns of a row and the rows of a column both start in different banks
};
template <typename V, int RB>
__device__ __forceinline__ void op_mirror(const OpMirror<V, RB> &sh, const OpItem<RB> &it, int d, V *out)
{
    constexpr int ROWS = 4 * RB;
#pragma unroll
    for (int n = 0; n < RB; ++n) {
        const int e = n * CSR_THREADS + (int)threadIdx.x, r = e % ROWS, c = e / ROWS;
        const int i = it.ib + r, j = it.jb + c;
        if (j < d && i < j) {  // i < j: also i < d
            V v = sh.m[r][c];
            v.y = -v.y;
            gst((V *)((char *)out + (uint32_t)(j * d + i) * (uint32_t)sizeof(V)), v);
        }
    }
}

// A wave-uniform value in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ double uniform(double v)
{
    return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

// Keeps a uniform value where it is read: the compiler would otherwise move each read of a descriptor to its
// first use, one round trip to memory after the other.
template <typename P> __device__ __forceinline__ void keep(P &p) { asm volatile("" : "+s"(p)); }

// A problem's tables (es: bytes of a state element; SHORT: the channels' column entries in FP32), their descriptor
// read at once.
struct OpTabs {
    int w;
    const double2 *diag;
    const int32_t *lcol;
    const void *aval, *cval, *rows;
    __device__ __forceinline__ OpTabs(const OpForm &O, int d, uint32_t es, bool shorts)
    {
        const char *mem = (const char *)O.mem;
        w = O.w;
        keep(w), keep(mem);
        const OpOffsets o(d, w, es);
        diag = (const double2 *)mem;
        lcol = (const int32_t *)(mem + o.lcol);
        aval = mem + o.aval;
        cval = mem + (shorts ? o.cshort : o.cval);
        rows = mem + o.rows;
    }
};

// M entries of this lane's column, from entry k on.
template <typename V, int M, int K> struct OpCols {
    using CV = typename std::conditional<(K & OP_SHORT) != 0, float2, double2>::type;
    V a[M];         // conj A_jl
    CV c[M];        // C_c's value
    uint32_t l[M];  // their columns
    __device__ __forceinline__ void load(const OpTabs &O, int d, int j, int k)
    {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const uint32_t q = (uint32_t)((k + m) * d + j);
            l[m] = (uint32_t)gld((const int32_t *)((const char *)O.lcol + q * 4u));
            a[m] = at((const V *)O.aval, q * (uint32_t)sizeof(V));
            a[m].y = -a[m].y;
            c[m] = at((const CV *)O.cval, q * (uint32_t)sizeof(CV));
        }
    }
};

// L x at the wave's RB rows in this lane's column; x(o) is the input at byte offset o.  The loops run over
// the entries, a few at a time for all rows: a column's entries are read once for the RB rows, and nothing but
// the sums stays in registers.  pre: the first M0 entries (the first group).  One row (small problems, bound
// by the latency of a wave): every source of a group is requested before its first sum; more: up to four
// entries of RB rows in flight.
template <typename T, int RB, int M0, int K, typename X>
__device__ __forceinline__ void op_sum(const OpTabs &O, int d, const OpItem<RB> &it, double2 dj,
                                       const OpCols<typename vec2<T>::type, M0, K> &pre, X x,
                                       typename vec2<T>::type (&acc)[RB])
{
    using V = typename vec2<T>::type;
    constexpr uint32_t ES = sizeof(V);
    const int w = O.w;
    const uint32_t ds = (uint32_t)d * ES, jo = (uint32_t)it.j * ES;
    const int32_t *rac[RB];
    const V *rav[RB];
    const double2 *rcv[RB];
    V own[RB];
    double2 dd[RB];  // what the element itself is multiplied by
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const char *rec = (const char *)O.rows + (uint32_t)it.i[r] * OpOffsets::rec(w, ES);
        rac[r] = (const int32_t *)rec;              // [w] columns of A, [w] columns of the jumps
        rav[r] = (const V *)(rec + 8 * (size_t)w);  // [w] values of A
        rcv[r] = (const double2 *)(rec + (8 + ES) * (size_t)w);  // [w] of the jumps
        dd[r] = uld(O.diag + it.i[r]);
        dd[r].x += dj.x;
        dd[r].y -= dj.y;
        own[r] = x((uint32_t)it.i[r] * ds + jo);
        acc[r].x = acc[r].y = T(0);
    }
    auto part = [&](auto first, const auto &col, int k) {
        constexpr int M = sizeof(col.l) / 4;
        constexpr bool FIRST = decltype(first)::value;
        V up[RB][M], side[RB][M], jump[RB][M];
        // A rho: the column's other rows
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m) up[r][m] = x((uint32_t)uld(rac[r] + k + m) * ds + jo);
        auto load_side = [&]() {  // rho A^dag: the row's other columns
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int m = 0; m < M; ++m) side[r][m] = x((uint32_t)it.i[r] * ds + (col.l[m] & 0xffffu) * ES);
        };
        // the jumps; an element without one takes itself, times zero, as does one whose jump starts from the element
        // (counted in dd: OP_SELF)
        V v[RB][M];
        auto load_jump = [&]() {
            uint32_t o[RB][M];
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int ki = uld(rac[r] + w + k + m);
                    const uint32_t own_o = (uint32_t)it.i[r] * ds + jo, to = (uint32_t)ki * ds + (col.l[m] >> 16) * ES;
                    const uint32_t none = (uint32_t)(ki >> 31) | (uint32_t)(((int32_t)(col.l[m] >> 16 ^ 0xffffu) - 1) >> 31);
                    o[r][m] = to ^ ((to ^ own_o) & none);  // (bit operations: a select became a branch)
                    jump[r][m] = x(o[r][m]);
                }
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    v[r][m] = from_d2<V>(cmulc(uld(rcv[r] + k + m), to_d2(col.c[m])));
                    if constexpr ((K & OP_SELF) != 0) {
                        const bool own = o[r][m] == (uint32_t)it.i[r] * ds + jo;
                        v[r][m].x = own ? T(0) : v[r][m].x;
                        v[r][m].y = own ? T(0) : v[r][m].y;
                    }
                }
        };
        V va[RB][M];
        if constexpr (RB == 1) {
            load_side();
#pragma unroll
            for (int m = 0; m < M; ++m) va[0][m] = uld(rav[0] + k + m);
            load_jump();
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (FIRST) {
#pragma unroll
            for (int r = 0; r < RB; ++r) cfma(acc[r], from_d2<V>(dd[r]), own[r]);
        }
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m) cfma(acc[r], RB == 1 ? va[r][m] : uld(rav[r] + k + m), up[r][m]);
        if constexpr (RB > 1) load_side();
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m) cfma(acc[r], col.a[m], side[r][m]);
        if constexpr (RB > 1) load_jump();
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int m = 0; m < M; ++m) cfma(acc[r], v[r][m], jump[r][m]);
    };
    if constexpr ((K & OP_SELF) != 0) {  // jumps that start from the element itself
        auto add = [&](int k, uint32_t l, double2 c) {
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const double2 p = cmulc(uld(rcv[r] + k), c);
                const bool own = uld(rac[r] + w + k) == it.i[r] && (int)(l >> 16) == it.j;
                dd[r].x += own ? p.x : 0.0;
                dd[r].y += own ? p.y : 0.0;
            }
        };
#pragma unroll
        for (int m = 0; m < M0; ++m) add(m, pre.l[m], to_d2(pre.c[m]));
#pragma unroll 1
        for (int k = M0; k < w; ++k) {
            const uint32_t q = (uint32_t)(k * d + it.j);
            add(k, (uint32_t)gld((const int32_t *)((const char *)O.lcol + q * 4u)),
                at((const double2 *)O.cval, q * 16u));
        }
    }
    part(std::true_type{}, pre, 0);
    int k = M0;
#pragma unroll 1
    for (; k + 4 <= w; k += 4) {
        OpCols<V, 4, K> col;
        col.load(O, d, it.j, k);
        part(std::false_type{}, col, k);
    }
    if (k < w) {
        OpCols<V, 2, K> col;
        col.load(O, d, it.j, k);
        part(std::false_type{}, col, k);
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)  // rho A^dag is the conjugate of A rho on the diagonal, but their sums round in turn
        if (it.i[r] == it.j) acc[r].y = T(0);
}

// Starting step: which = 0 the first evaluation (k1 = L rho0, y <- rho0), 1 the second.
template <typename T, int RB, int M0, int K>
__device__ __forceinline__ void op_init_body(const CsrInst &I, const CsrCtl *C, int blk, int which)
{
    using V = typename vec2<T>::type;
    __shared__ double scr[16];
    __shared__ OpMirror<V, RB> tr;
    if (C->status != ST_RUNNING || C->phase != (which ? PH_INIT1 : PH_INIT0)) return;
    const int d = I.d;
    const OpItem<RB> it(blk, d);
    const double h0 = C->h0;
    const T th0 = (T)h0;
    const V *__restrict__ x0 = uniform_ptr((const V *)I.rho0);
    V *__restrict__ y = uniform_ptr((V *)I.Y[0]);
    V *__restrict__ k1 = uniform_ptr((V *)I.K[0]);
    double sa = 0.0, sb = 0.0;
    const OpTabs O(I.op, d, sizeof(V), (K & OP_SHORT) != 0);
    if (it.i0 < d) {
        OpCols<V, M0, K> pre;
        pre.load(O, d, it.j, 0);
        const double2 dj = gld(O.diag + it.j);
        V acc[RB];
        if (which)
            op_sum<T, RB, M0, K>(O, d, it, dj, pre, [&](uint32_t o) {
                V v = at((const V *)y, o);
                caxpy(v, th0, at((const V *)k1, o));
                return v;
            }, acc);
        else
            op_sum<T, RB, M0, K>(O, d, it, dj, pre, [&](uint32_t o) { return at(x0, o); }, acc);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            if (!it.has(r, d)) continue;
            const uint32_t row = (uint32_t)(it.i[r] * d + it.j) * (uint32_t)sizeof(V);
            const double wt = it.j > it.i[r] ? 2.0 : 1.0;  // the element below the diagonal counts as well
            if (which) {
                const double2 yr = to_d2(at((const V *)y, row)), f0 = to_d2(at((const V *)k1, row)), f1 = to_d2(acc[r]);
                const double sc = I.atol + I.rtol * sqrt(yr.x * yr.x + yr.y * yr.y);
                const double dx = (f1.x - f0.x) / h0, dy = (f1.y - f0.y) / h0;
                sa += wt * ((dx * dx + dy * dy) / (sc * sc));
            } else {
                const V yv = at(x0, row);
                gst((V *)((char *)k1 + row), acc[r]);
                gst((V *)((char *)y + row), yv);
                tr.m[it.i0 - it.ib + r][threadIdx.x & 63] = acc[r];
                const double sc = I.atol + I.rtol * sqrt(abs2d(yv));
                sa += wt * (abs2d(yv) / (sc * sc));
                sb += wt * (abs2d(acc[r]) / (sc * sc));
            }
        }
    }
    if (!which) {
        __syncthreads();
        op_mirror(tr, it, d, k1);
        // the initial state is copied below the diagonal as well
#pragma unroll
        for (int n = 0; n < RB; ++n) {
            const int e = n * CSR_THREADS + (int)threadIdx.x, i = it.ib + e % (4 * RB), j = it.jb + e / (4 * RB);
            const uint32_t o = (uint32_t)(j * d + i) * (uint32_t)sizeof(V);
            if (j < d && i < j) gst((V *)((char *)y + o), at(x0, o));
        }
    }
    sa = block_sum(sa, scr);
    if (!which) sb = block_sum(sb, scr);
    if (threadIdx.x == 0) {
        I.partials[2 * blk] = sa;
        if (!which) I.partials[2 * blk + 1] = sb;
    }
}

// One Runge-Kutta stage S (2..7), uniform over the launch.
template <typename T, int RB, int M0, int K>
__device__ __forceinline__ void op_stage_body(const CsrInst &I, const CsrCtl *C, int blk, int S)
{
    using V = typename vec2<T>::type;
    __shared__ double scr[16];
    __shared__ OpMirror<V, RB> tk, tx;
    int d = I.d;
    V *Y0 = (V *)I.Y[0], *Y1 = (V *)I.Y[1], *K0 = (V *)I.K[0], *K1 = (V *)I.K[1], *ys0 = (V *)I.ys[0], *ys1 = (V *)I.ys[1];
    V *k2 = (V *)I.ks[0], *k3 = (V *)I.ks[1], *k4 = (V *)I.ks[2], *k5 = (V *)I.ks[3], *k6 = (V *)I.ks[4];
    keep(d), keep(Y0), keep(Y1), keep(K0), keep(K1), keep(ys0), keep(ys1);
    keep(k2), keep(k3), keep(k4), keep(k5), keep(k6);
    const OpTabs O(I.op, d, sizeof(V), (K & OP_SHORT) != 0);
    // the column's first entries do not depend on the control record: in flight beside it
    const OpItem<RB> it(blk, d);
    OpCols<V, M0, K> pre;
    pre.load(O, d, it.j, 0);
    const double2 dj = gld(O.diag + it.j);
    int status = uniform(C->status), phase = uniform(C->phase), p = uniform(C->parity);
    double h = uniform(C->h_try), scale = uniform(C->scale);
    keep(status), keep(phase), keep(p), keep(h), keep(scale);
    if ((status != ST_RUNNING) | (phase != PH_STEP)) return;
    const T s = (T)scale;
    const V *__restrict__ y = p ? Y1 : Y0;
    const V *__restrict__ k1 = p ? K1 : K0;
    const V *__restrict__ ynew = p ? Y0 : Y1;
    const V *__restrict__ xin = S == 2 ? k1 : S == 7 ? ynew : S & 1 ? ys0 : ys1;
    // where the stage's derivative and the next stage's input go
    V *__restrict__ kout = S == 7 ? (p ? K0 : K1) : S == 2 ? k2 : S == 3 ? k3 : S == 4 ? k4 : S == 5 ? k5 : k6;
    V *__restrict__ xout = S == 6 ? (p ? Y0 : Y1) : S & 1 ? ys1 : ys0;
    const V *__restrict__ q0 = S == 7 ? k6 : k2;
    const V *__restrict__ q1 = k3;
    const V *__restrict__ q2 = k4;
    const V *__restrict__ q3 = k5;
    double e2 = 0.0, l2 = 0.0;
    if (it.i0 < d) {
        V acc[RB], yr, k1r, kr[4]{}, ynr{};
        auto operands = [&](int r) {  // of the stage combination
            const uint32_t row = (uint32_t)(it.i[r] * d + it.j) * (uint32_t)sizeof(V);
            yr = at(y, row);
            k1r = at(k1, row);
            // one row: all of them at once, also what this stage does not use (no branch, no wait)
            if (RB == 1 || (S >= 3 && S <= 5) || S == 7) kr[0] = at(q0, row);
            if (RB == 1 || S >= 4) kr[1] = at(q1, row);
            if (RB == 1 || S >= 5) kr[2] = at(q2, row);
            if (RB == 1 || S >= 6) kr[3] = at(q3, row);
            if (RB == 1 || S == 7) ynr = at(ynew, row);
        };
        if constexpr (RB == 1) operands(0);
        op_sum<T, RB, M0, K>(O, d, it, dj, pre, [&](uint32_t o) { return at(xin, o); }, acc);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            if (!it.has(r, d)) continue;
            const uint32_t row = (uint32_t)(it.i[r] * d + it.j) * (uint32_t)sizeof(V);
            if constexpr (RB > 1) operands(r);
            V a = acc[r];
            yr = cscale(yr, s);
            k1r = cscale(k1r, s);
            V o = yr;
            if (S == 2) {
                // k2 = L (y + a21 h k1) = k1 + a21 h (L k1); the trace scale applies to y and k1 alike
                const V lk1 = a;
                a = k1r;
                caxpy(a, (T)(h * DP5::a21) * s, lk1);
                caxpy(o, (T)(h * DP5::a31), k1r);
                caxpy(o, (T)(h * DP5::a32), a);
            } else if (S == 3) {
                caxpy(o, (T)(h * DP5::a41), k1r);
                caxpy(o, (T)(h * DP5::a42), kr[0]);
                caxpy(o, (T)(h * DP5::a43), a);
            } else if (S == 4) {
                caxpy(o, (T)(h * DP5::a51), k1r);
                caxpy(o, (T)(h * DP5::a52), kr[0]);
                caxpy(o, (T)(h * DP5::a53), kr[1]);
                caxpy(o, (T)(h * DP5::a54), a);
            } else if (S == 5) {
                caxpy(o, (T)(h * DP5::a61), k1r);
                caxpy(o, (T)(h * DP5::a62), kr[0]);
                caxpy(o, (T)(h * DP5::a63), kr[1]);
                caxpy(o, (T)(h * DP5::a64), kr[2]);
                caxpy(o, (T)(h * DP5::a65), a);
            } else if (S == 6) {
                caxpy(o, (T)(h * DP5::b1), k1r);
                caxpy(o, (T)(h * DP5::b3), kr[1]);
                caxpy(o, (T)(h * DP5::b4), kr[2]);
                caxpy(o, (T)(h * DP5::b5), kr[3]);
                caxpy(o, (T)(h * DP5::b6), a);
            } else {
                double2 e = make_double2(0.0, 0.0);
                caxpy(e, h * DP5::e1, to_d2(k1r));
                caxpy(e, h * DP5::e3, to_d2(kr[1]));
                caxpy(e, h * DP5::e4, to_d2(kr[2]));
                caxpy(e, h * DP5::e5, to_d2(kr[3]));
                caxpy(e, h * DP5::e6, to_d2(kr[0]));
                caxpy(e, h * DP5::e7, to_d2(a));
                const double sc = I.atol + I.rtol * sqrt(fmax(abs2d(yr), abs2d(ynr)));
                const double wt = it.j > it.i[r] ? 2.0 : 1.0;  // the element below the diagonal counts as well
                e2 += wt * ((e.x * e.x + e.y * e.y) / (sc * sc));
                l2 += wt * abs2d(a);
            }
            gst((V *)((char *)kout + row), a);
            tk.m[it.i0 - it.ib + r][threadIdx.x & 63] = a;
            if (S < 7) {
                gst((V *)((char *)xout + row), o);
                tx.m[it.i0 - it.ib + r][threadIdx.x & 63] = o;
            }
        }
    }
    __syncthreads();
    op_mirror(tk, it, d, kout);
    if (S < 7) op_mirror(tx, it, d, xout);
    if (S == 7) {
        e2 = block_sum(e2, scr);
        const bool steady = I.steady_tol2 > 0.0;
        if (steady) l2 = block_sum(l2, scr);
        if (threadIdx.x == 0) {
            I.partials[2 * blk] = e2;
            if (steady) I.partials[2 * blk + 1] = l2;
        }
    }
}

// The stage or starting step `what` of one workgroup: the row count by the dimension, the entries requested
// at once by the table width (small problems).
template <typename T, bool INIT, bool SMALL, int K>
__device__ __forceinline__ void op_body(const CsrInst &I, const CsrCtl *C, int blk, int what)
{
    if constexpr (SMALL) {
        if (I.op.w >= 8) {
            if constexpr (INIT) op_init_body<T, OP_ROWS_SMALL, 8, K>(I, C, blk, what);
            else op_stage_body<T, OP_ROWS_SMALL, 8, K>(I, C, blk, what);
        } else {
            if constexpr (INIT) op_init_body<T, OP_ROWS_SMALL, 4, K>(I, C, blk, what);
            else op_stage_body<T, OP_ROWS_SMALL, 4, K>(I, C, blk, what);
        }
    } else {
        if constexpr (INIT) op_init_body<T, OP_ROWS, 4, K>(I, C, blk, what);
        else op_stage_body<T, OP_ROWS, 4, K>(I, C, blk, what);
    }
}

// Block index in XCD-contiguous order (as csr_block, with the grid as an argument: one line less to read).
__device__ __forceinline__ int op_block(int n)
{
    const int b = blockIdx.x, q = n >> 3, r = n & 7, x = b & 7;
    return n ? x * q + min(x, r) + (b >> 3) : b;
}

// what: 0 / 1 the starting-step evaluations, 2..7 a stage.  ONE: one problem, descriptor by value (SMALL: of up
// to OP_SMALL_D); otherwise the block table (bi: problem, br: its block).  n: the grid, for the XCD-contiguous
// order (a row's sources are then mostly rows of the same XCD's L2), 0: the launch order.  K: OP_SELF if
// some problem of the launch has a diagonal entry in a channel, OP_SHORT if all have short column entries.  (The
// sums of the others are the same either way; the mask and its registers cost chains of lowering operators 3 to
// 4%, 16-byte column entries 16 chains of L = 8 5%.)
// The complex64 stages are held to 128 registers, four waves a SIMD (130 otherwise).
template <typename T, bool SMALL, bool ONE, bool INIT, int K>
__global__ __launch_bounds__(CSR_THREADS, sizeof(T) == 4 && !INIT ? 4 : 1) void k_op(const CsrInst *__restrict__ insts, const CsrInst one,
                                                    const CsrCtl *__restrict__ ctls, const int32_t *__restrict__ bi,
                                                    const int32_t *__restrict__ br, int n,
                                                    const int32_t *__restrict__ bound, int what)
{
    const int lb = op_block(n);
    if constexpr (ONE) {
        op_body<T, INIT, SMALL, K>(one, ctls, lb, what);
    } else {
        if (bound && lb >= bound[0]) return;
        const int ii = bi[lb], blk = br[lb];
        if (insts[ii].d <= OP_SMALL_D) op_body<T, INIT, true, K>(insts[ii], ctls + ii, blk, what);
        else op_body<T, INIT, false, K>(insts[ii], ctls + ii, blk, what);
    }
}

// Stage 2 with the previous step's control folded in, as k_csr_stage2_ctl.
template <typename T, bool SMALL, int K>
__global__ __launch_bounds__(CSR_THREADS) void k_op_stage2_ctl(const CsrInst one, const CsrCtl *__restrict__ rd,
                                                               CsrCtl *__restrict__ wr, int n)
{
    using V = typename vec2<T>::type;
    __shared__ CsrCtl nsh;
    if (!ctl_fold<V, false>(one, rd, wr, nsh, nullptr)) return;
    op_body<T, false, SMALL, K>(one, &nsh, op_block(n), 2);
}

template <typename T, bool SMALL, bool ONE, int K> static void op_launch_t(const CsrArgs &a, int what)
{
    const dim3 g(a.nblk), t(CSR_THREADS);
    const int n = a.xcd ? a.nblk : 0;
#define QT_ARGS a.insts, a.one, a.ctls, a.bi, a.br, n, a.bound, what
    if (what < 2) hipLaunchKernelGGL((k_op<T, SMALL, ONE, true, K>), g, t, 0, a.s, QT_ARGS);
    else hipLaunchKernelGGL((k_op<T, SMALL, ONE, false, K>), g, t, 0, a.s, QT_ARGS);
#undef QT_ARGS
}

template <typename T, int K> static void op_launch(const CsrArgs &a, int what)
{
    if (!a.use_one) op_launch_t<T, false, false, K>(a, what);
    else if (a.one.d <= OP_SMALL_D) op_launch_t<T, true, true, K>(a, what);
    else op_launch_t<T, false, true, K>(a, what);
}

template <typename T, int K> static void op_ctl(const CsrArgs &a, const CsrCtl *rd, CsrCtl *wr)
{
    const dim3 g(a.nblk), t(CSR_THREADS);
    const int n = a.xcd ? a.nblk : 0;
    if (a.one.d <= OP_SMALL_D) hipLaunchKernelGGL((k_op_stage2_ctl<T, true, K>), g, t, 0, a.s, a.one, rd, wr, n);
    else hipLaunchKernelGGL((k_op_stage2_ctl<T, false, K>), g, t, 0, a.s, a.one, rd, wr, n);
}

// K: the flags of OpForm a kernel serves (op_common); short column entries only without the self-jump mask.
void op_spmv(const CsrLaunch &L, const CsrArgs &a, int first, int last)
{
    const bool self = L.op_flags & OP_SELF, shorts = L.op_flags & OP_SHORT;
    const auto launch = L.f64 ? (self ? op_launch<double, OP_SELF> : op_launch<double, 0>)
                              : (self ? op_launch<float, OP_SELF> : shorts ? op_launch<float, OP_SHORT> : op_launch<float, 0>);
    for (int what = first; what <= last; ++what) launch(a, what);
}

void op_stage2_ctl(const CsrLaunch &L, const CsrArgs &a, const CsrCtl *rd, CsrCtl *wr)
{
    const bool self = L.op_flags & OP_SELF, shorts = L.op_flags & OP_SHORT;
    const auto launch = L.f64 ? (self ? op_ctl<double, OP_SELF> : op_ctl<double, 0>)
                              : (self ? op_ctl<float, OP_SELF> : shorts ? op_ctl<float, OP_SHORT> : op_ctl<float, 0>);
    launch(a, rd, wr);
}

}  // namespace qt
