// qt_op.h -- operator tables of the staged solver's operator-form right-hand side (kernels_op.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qt {

constexpr int OP_MAX_W = 12;  // off-diagonal entries per row of A, and collapse operators
// Below OP_MIN_D the matrix kernels' shorter chain of loads is faster for one problem: a chain of L = 7 (d = 128)
// took 1.97 ms in operator form against 1.62 ms to t = 2 (rtol 1e-5), L = 8 1.97 ms against 2.51 ms.  (From
// 32 on a problem has no more workgroups (op_blocks) than their default shape has, which is what partial sums and
// block tables are sized for.)  Up to OP_MAX_D a state's byte offsets have 32 bits.
//
// Above it the rule looks at batches as much as at lone problems, since a problem's solver may not depend on what it
// runs with.  Matrix kernels and operator form, us a step, banded problems of w off-diagonal entries per row and nc
// channels, complex64 (complex128 is more favourable by 5 to 20%):
//                       one problem                              16 problems
//             w 2, nc 1   w 8, nc 8   w 12, nc 12     w 2, nc 1   w 8, nc 8   w 12, nc 12
//   d = 130   30  30      32  35      35  41          86  69      152  90     170  119
//   d = 160   32  32      38  37      36  39          114 81      193  103    211  117
//   d = 192   33  30      41  37      45  41          146 80      226  107    266  126
//   d = 257   43  48      60  53      67  62          291 144     405  175    483  214
//   d = 320   53  40      87  53      99  62          347 140     596  186    737  231
//   d = 512   97  51      173 63      192 74          939 305     1477 375    1795 459
// So one problem of d up to 160 with wide operators pays up to 15%, and one just above d = 256, where a wave takes
// two rows, up to 10% if its operators are narrow; batches gain 1.2 to 4 times everywhere.
constexpr int OP_MIN_D = 129, OP_MAX_D = 8192;

// L(rho) = A rho + rho A^dag + sum_c C_c rho C_c^dag from d x d tables (device pointers; w = 0: none).
// w is the problem's table width, even and at least 4: entries past a row's own (and channels past the last)
// are the row itself with value 0 (jumps: column -1).  Kernels index a problem's tables with its own w, never with
// another's of the same launch.  Every table exists twice, entry by entry over the columns (what 64 lanes
// read) and row by row (what a wave reads for its rows).
//   diag [d]     A_ii
//   lcol [w][d]  column of A's off-diagonal entry | column of C_c's entry << 16 (0xffff: none)
//   aval [w][d]  A's values, state precision
//   cval [w][d]  C_c's value over a factor f_c of the channel, FP64 (a product of two entries is rounded once, as
//                the assembled matrix rounds it)
//   cshort [w][d]  cval in FP32 (mixed precision; used where that is exact)
//   rows [d]     records: columns of A [w], of the jumps [w] (-1: none), values of A [w] (state precision), of the
//                jumps times conj f_c [w] (FP64)
// f_c is the channel's first entry, where that makes every cval exact in FP32 (a rate's root times entries +-1,
// +-i, as spin operators have), else 1.
// One allocation holds them, so that descriptors (kernel arguments of every CSR launch) stay short.
struct OpForm {
    const void *mem;
    int32_t w;
    int32_t flags;
};
constexpr int32_t OP_SELF = 1;   // some C_c has an entry on its diagonal, so jumps reach the element itself
constexpr int32_t OP_SHORT = 2;  // cshort is exact

// Byte offsets of the tables (diag at 0) for state elements of es bytes, and the bytes of all.
struct OpOffsets {
    uint32_t lcol, aval, cval, cshort, rows, total;
    __host__ __device__ OpOffsets(int d, int w, uint32_t es)
    {
        const uint32_t n = (uint32_t)w * (uint32_t)d;
        lcol = up((uint32_t)d * 16u);
        aval = lcol + up(n * 4u);
        cval = aval + up(n * es);
        cshort = cval + up(n * 16u);
        rows = cshort + (es == 8 ? up(n * 8u) : 0u);
        total = rows + up((uint32_t)d * rec(w, es));
    }
    static __host__ __device__ uint32_t rec(int w, uint32_t es) { return (uint32_t)w * (8u + es + 16u); }  // bytes of a row's record
    static __host__ __device__ uint32_t up(uint32_t b) { return (b + 255u) & ~255u; }
};

// Rows one wave serves: fixed by the dimension, so that a problem's sums do not depend on the plan.  Up to
// d = 256 one problem does not fill the chip and the latency of a wave counts (one chain of L = 8: 4.3 ms to t = 10
// with one row, 5.4 ms with two); above, the vector L1 (L = 10, complex128: 14.2 ms and 12.4 ms).  In between one
// row suits one problem, two a batch (d = 320, w = 8, complex64: one problem 38 and 53 us a step, sixteen 212
// and 186; d = 257: 37 and 53, 204 and 175).
constexpr int OP_ROWS = 2, OP_ROWS_SMALL = 1, OP_SMALL_D = 256;
__host__ __device__ inline int op_rows(int d) { return d > OP_SMALL_D ? OP_ROWS : OP_ROWS_SMALL; }

// Workgroups of a problem: the 64 x 64 tiles of the upper triangle, each cut into groups of four waves' rows.
__host__ __device__ inline int op_blocks(int d)
{
    const int t = (d + 63) / 64;
    return t * (t + 1) / 2 * (16 / op_rows(d));
}

}  // namespace qt
