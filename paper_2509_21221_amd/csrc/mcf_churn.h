// Internal interface of the warm-started churn re-solve: the general form
// (mcf_churn.hip) and the packed one (mcf_churn_packed.hip).  Not part of the
// public C ABI.
#pragma once

#include "mcf_internal.h"

namespace gwtf {

// Warm-started re-solve of churn variants (mcf_churn.hip): one workgroup per
// instance with the instance in LDS, so S*n <= kChurnMaxNodes and
// (S-1)*n*n <= kChurnMaxLinks.
constexpr int kChurnMaxNodes = 512;
constexpr int kChurnMaxLinks = 4096;
struct ChurnParams {
    int32_t B, S, n, start_per_instance;
    const int32_t *cap, *ncost, *acost, *src, *snk, *supply; // caller inputs
    const int32_t *nf0, *af0, *sf0, *tf0;                    // start flow ([B] or [1])
    int64_t *F_out, *cost_out;                               // [B]
    int32_t *status_out;                                     // [B]
    int32_t *nf_out, *af_out, *sf_out, *tf_out;              // result flows, or all NULL
    int64_t *work;                                           // [B][4] or NULL
    int32_t passed_on;                                       // general form: only instances so marked
};
size_t churn_lds_bytes(int S, int n);
hipError_t launch_churn_resolve(const ChurnParams &p, const LaunchInfo &l, hipStream_t stream);

// The packed form: several instances per wave for S <= kChurnPackedStages,
// n <= 16.  Marks what it does not hold with kChurnPassedOn in status_out; the
// general form, launched after it, solves those.
constexpr int kChurnPackedStages = 8;
constexpr int32_t kChurnPassedOn = -1;
hipError_t launch_churn_packed(const ChurnParams &p, const LaunchInfo &l, hipStream_t stream);

} // namespace gwtf
