// gsn_corrector_internal.hpp -- hooks between the grid solver and the learned
// corrector (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>

#include "gsn.h"

// One image, queued on s: with u = e^{i theta} psi the state as the caller
// reads it (theta: the grid's FP64 global phase, a device scalar),
// psi_out <- psi + s_out e^{-i theta} net(Re u, Im u, phi).  psi_out may be psi;
// the fused inference (corrector_fused) then goes through its spare image, from
// which it can as well take psi (corrector_spare).
gsn_status corrector_correct(gsn_corrector c, const float2 *psi, const float *phi, float2 *psi_out,
                             const double *theta, hipStream_t s);
bool corrector_fused(gsn_corrector c);
float2 *corrector_spare(gsn_corrector c);
int corrector_height(gsn_corrector c);
int corrector_width(gsn_corrector c);
// device scratch of the corrector for one image: phi (float), two psi copies
float *corrector_phi_buffer(gsn_corrector c);
float2 *corrector_psi_buffer(gsn_corrector c, int which);
