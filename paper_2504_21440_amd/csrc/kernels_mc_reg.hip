// kernels_mc_reg.hip -- the trajectory kernel with A = -i H_eff in registers.
//
// Reading A from L2 at every right-hand side (132 KB per evaluation at d = 1,024) is what the variants of
// kernels_mc.hip wait for: a chain of W dependent load-gather pairs per stage.  A constant A of few
// entries per row is loaded once per workgroup instead: a thread keeps the entries of its rows as a
// value and a 16-bit LDS byte offset, so a right-hand side is W LDS gathers per row and nothing else.
//
// One row per thread up to d = 1,024, in 256, 512 or 1,024 threads: the 16 waves of a CU are then one, two
// or four trajectories, within 128 registers a lane in complex64 (9 state and stage values, 12 entries;
// complex128 spills some 50 registers at d = 1,024).  d up to 2,048 takes 4 rows in 512 threads, complex64
// only.  The sums run over the same virtual threads in every variant, so a trajectory is bitwise the
// same in all of them.
#include "mc_kernel.h"

namespace qt {

template <typename T, int R, int TPB, int W> static const void *reg_fn(int *threads, size_t *lds)
{
    using V = typename vec2<T>::type;
    *threads = TPB;
    *lds = (size_t)2 * TPB * R * sizeof(V) + (TPB > MC_THREADS ? (size_t)3 * TPB * R * 8 : 0);
    return (const void *)k_mc<T, R, false, 1, TPB, W>;
}

template <typename T, int TPB> static const void *reg_w(int w, int *threads, size_t *lds)
{
    return w <= 4 ? reg_fn<T, 1, TPB, 4>(threads, lds)
                  : w <= 8 ? reg_fn<T, 1, TPB, 8>(threads, lds) : reg_fn<T, 1, TPB, 12>(threads, lds);
}

template <typename T> static const void *reg_rows(int rows, int w, int *threads, size_t *lds)
{
    switch (rows) {
    case 1: return reg_w<T, 256>(w, threads, lds);
    case 2: return reg_w<T, 512>(w, threads, lds);
    case 4: return reg_w<T, 1024>(w, threads, lds);
    case 8: return sizeof(T) == 4 ? reg_fn<float, 4, 512, 12>(threads, lds) : nullptr;
    default: return nullptr;
    }
}

// p.rows: the rows per thread of 256 (1, 2, 4, ...); 12 entries per row hold chains of up to 11 spins.
const void *mc_reg_kernel(const McParams &p, bool f64, bool td, int *threads, size_t *lds)
{
    if (td || p.nterms > 0 || p.W > 12) return nullptr;
    return f64 ? reg_rows<double>(p.rows, p.W, threads, lds) : reg_rows<float>(p.rows, p.W, threads, lds);
}

}  // namespace qt
