// qt_res.h -- descriptors of the resident master-equation solver (kernels_res.hip): one workgroup
// integrates one small problem with its generator in registers and its state in LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "../../include/qtamd.h"

namespace qt {

constexpr int RES_MAX_W = 16;  // generator entries per element held in registers
constexpr int RES_MAX_D = 80;      // two d x (d | 1) matrices in LDS, 16-bit byte offsets
constexpr int RES_MAX_D_F64 = 62;

enum : int32_t { RES_ST_INIT = 200 };

struct ResInst {
    int32_t d, nt, ne, W;
    int32_t use_h0, renorm;
    double atol, rtol, h0;
    int64_t max_steps;
    double steady_tol2;  // steady-state mode (0: off): stop once |L y|_2^2 <= steady_tol2
    // generator: the CSR rows (rowptr / col / val, padding zeros at the end of each row), or, with
    // rowptr null, an ELL of the upper triangle (entry k of element e at k * ntri + e; elements in
    // row-major order over i <= j; col = row-major index of the source element)
    const int32_t *rowptr, *col;
    const void *val;     // state precision
    const void *rho0;    // d x d row-major, state precision
    void *vec;           // 2 d d elements: the state (d x d), then k1 and L k1 (upper triangles)
    const double *tlist;
    const int32_t *eptr; // ne * (d + 1)
    const int32_t *evidx;
    const double2 *eval;
    double2 *expect;
};

struct ResCtl {
    double t, h, err_prev, tr0;
    int32_t status, save_idx, last_rejected, pad;
    int64_t n_accept, n_reject, n_steps, n_rhs;
};

// Upper bound of the generator entries of any element, from the operators A and C_k (row lengths);
// 0 when it is above RES_MAX_W or d is above RES_MAX_D (the problem is not eligible).  band: whether
// the entries lie in the band classes' stencil.
struct HCsr;
struct Liouv;
int res_width(const HCsr &A, const std::vector<HCsr> &cs, bool *band);
// The upper-triangle ELL of the generator of A and C_k at width W, values in FP64.
void res_build_ell(const HCsr &A, const std::vector<HCsr> &cs, int W, std::vector<int32_t> &col,
                   std::vector<double2> &val);
// Kernel class of a problem (problems of one class share launches), -1: none holds it; classes are
// 0 .. res_classes() - 1.
int res_class(int d, int W, bool band, int prec);
int res_classes();
// Launch the solver for `count` problems of one class (order[] lists them).  max_steps_launch < 0: run to completion.  reset: start every problem from rho0.
qt_status res_launch(int cls, bool f64, const ResInst *insts, ResCtl *ctls, const int32_t *order,
                     int count, int max_steps_launch, int reset, hipStream_t s);

// ---- host side of plans and servers (qtamd_me.cpp) ----
bool exactly_hermitian(int32_t d, const double *rho0);
bool res_problem(const Liouv &L, bool dense, const double *rho0);
void res_fill_inst(ResInst *g, const Liouv &L, bool dense, int nt, int ne, const void *rho0, void *vec,
                   const double *tlist, const int32_t *eptr, const int32_t *evidx, const double2 *eval,
                   double2 *expect, const qt_opts &opts, double steady_tol2);
qt_status res_upload_ell(const Liouv &L, void *vec, std::vector<char> &stage, hipStream_t s);
// Where a dense-form problem's ELL lies behind its state vectors (bytes), and its size: values, then columns.
size_t res_ell_offset(int d, int prec);
size_t res_ell_bytes(const Liouv &L);

}  // namespace qt
