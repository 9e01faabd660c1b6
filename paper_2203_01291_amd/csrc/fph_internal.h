// Declarations shared by the library's translation units (not part of the
// C ABI): recording a HIP error for fph_strerror(), the operator under an HMC
// context, and the parameters of an SSH context.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/holstein_hmc.h"

namespace fph {

// Records hipGetErrorString(e) as the message of FPH_E_HIP and returns FPH_E_HIP.
int record_hip_error(hipError_t e);

// Builds what a solve's applies of F F^T to nrhs vectors in precision prec on the
// current field gain from and a single apply does not (pc_dense); call once per solve.
int precond_matrices(fph_handle_t h, int32_t prec, int32_t nrhs, void* stream);

// F F^T of a solver: fph_precond_apply that takes the matrices of
// precond_matrices where there are any and also writes partial sums of in_r . out_r,
// part_dev[r * nparts + k], k < nparts; nparts (at most N) = precond_parts.
int precond_parts(fph_handle_t h, int32_t prec, int32_t nrhs);
int precond_apply_dot(fph_handle_t h, int32_t prec, int32_t nrhs, const void* in_dev, void* out_dev,
                      double* part_dev, void* stream);

// The operator an HMC context runs on (its Holstein handle or SSH context):
// two contexts on the same one must not run side by side.
const void* hmc_operator(fph_hmc_t c);

// Lattice, right-hand-side capacity and coupling of an SSH context (each
// output may be NULL).
int ssh_info(fph_ssh_t c, fph_lattice_t* lat, int32_t* max_rhs, double* g);

// The Holstein handle whose preconditioner an SSH context uses (or NULL),
// and the one under an HMC context on an SSH context (NULL otherwise).
fph_handle_t ssh_precond(fph_ssh_t c);
fph_handle_t hmc_aux(fph_hmc_t c);

}  // namespace fph
