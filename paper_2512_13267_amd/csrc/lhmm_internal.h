// lhmm_internal.h -- helpers shared by the library's translation units (not
// part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include "lhmm.h"

// Record a thread-local error message for lhmm_last_error(); returns code.
int lhmm_fail(int code, const char* fmt, ...);
// Clear the thread-local error message.
void lhmm_clear_error();
// The caller stream a micro engine was created with.
hipStream_t lhmm_micro_caller_stream(const lhmm_micro* m);
// The stream an SPH engine launches on, its particle count and mobile count.
hipStream_t lhmm_sph_caller_stream(const lhmm_sph* s);
void lhmm_sph_counts(const lhmm_sph* s, int* n, int* n_mobile);
// The stream of a surrogate engine and its dimensions.
hipStream_t lhmm_sur_caller_stream(const lhmm_sur* s);
void lhmm_sur_dims(const lhmm_sur* s, int* n_members, int* n_in, int* n_out, int* max_batch);
// Passes of the hybrid macro step, on device memory or (flag, use_dpd) pinned
// host memory; n particles of three-output members.
// Sample t into the ring and the feature rows after it (lhmm_sur_push_history
// and lhmm_sur_features in one launch).
int lhmm_sur_push_features(float* ring, int n, const double* gradL, long long t, float scale, const float* phi,
                           float* X, hipStream_t stream);
// Ensemble mean and gate flags: bit 0 the spread gate (lhmm_sur_gate); with
// max2 >= 0 bits 1 and 2 where |L|^2 exceeds max2 and warm2.
int lhmm_sur_decide(const float* Y, int n_members, int n, float threshold, float floor_, const double* gradL,
                    double max2, double warm2, float* mean, unsigned* flag, hipStream_t stream);
// lhmm_sur_blend of the first n_blend particles, then sum += sigma for all n.
int lhmm_sur_settle(const float* mean, const unsigned* use_dpd, const double* sigma_dpd, int n_blend, int n,
                    float scale, double* sigma, double* sum, hipStream_t stream);

#define LHMM_HIPCHK(expr)                                                                        \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) return lhmm_fail(LHMM_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)
