// A row's log-softmax and its Gumbel-max sample, shared by the loss, sampling and head kernels.
#pragma once

#include "common.h"

namespace cb {

// Log-softmax of one row, kept as (zmax, lse): log pi_j = (z_j - zmax) - lse, recomputed from
// the logits where needed (no per-row array, so nothing spills to scratch). Also the entropy.
struct RowLsm {
    float zmax, lse, H;
    CB_DEV float l(float zj) const { return (zj - zmax) - lse; }
};

CB_DEV RowLsm row_log_softmax(const float* z, int A) {
    RowLsm r;
    r.zmax = z[0];
    for (int j = 1; j < A; ++j) r.zmax = fmaxf(r.zmax, z[j]);
    float se = 0.f;
    for (int j = 0; j < A; ++j) se += expf(z[j] - r.zmax);
    r.lse = logf(se);
    r.H = 0.f;
    for (int j = 0; j < A; ++j) {
        const float l = r.l(z[j]);
        r.H -= expf(l) * l;
    }
    return r;
}

// argmax_j (z_j + g_j), ties to the lowest index, and its log-probability under z.
CB_DEV void row_gumbel_max(const float* z, const float* g, int A, int32_t& act, float& logp) {
    int best = 0;
    float bv = z[0] + g[0];
    for (int j = 1; j < A; ++j) {
        const float v = z[j] + g[j];
        if (v > bv) { bv = v; best = j; }
    }
    const RowLsm rs = row_log_softmax(z, A);
    act = best;
    logp = rs.l(z[best]);
}

}  // namespace cb
