// Host interface of the reduction kernels (reduce.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/cast.h"

namespace cast {

struct PauliSumGroup {
    uint64_t x;
    int first, count;
};
struct PauliSumTerm {
    uint64_t z;
    double cre, cim;  // coefficient times i^{|x&z|}
};

// Doubles of device scratch pauli_inner and expval_sum need.
constexpr size_t kReduceScratch = 16384;

// S(x, z) = sum_y conj(a[y^x]) (-1)^{|z & y|} b[y], FP64, fixed reduction order:
// pauli_inner leaves inner_partials(n) <= kReduceScratch / 8 doubles,
// finish_inner sums `count` consecutive sets of them, the i-th to re, im at
// dev_out - 2 i.  Stream-ordered.
size_t inner_partials(int n);
cast_status pauli_inner(const void *a, const void *b, int n, cast_dtype dt, uint64_t x, uint64_t z, double *partials,
                        hipStream_t s);
cast_status finish_inner(const double *partials, int n, int count, double *dev_out, hipStream_t s);

// dev_out[0] = sum_m coeff_m <psi|P_m|psi> (1 <= n_terms <= 65536; real, since every P_m is Hermitian),
// FP64, fixed reduction order.  `order`: host scratch, n_terms entries.  Stream-ordered; the terms are consumed
// before it returns.
cast_status expval_sum(const void *psi, int n, cast_dtype dt, const cast_pauli_term *terms, size_t n_terms,
                       uint16_t *order, double *scratch, double *dev_out, hipStream_t s);

// out = (sum of Pauli terms) psi; term tables in device memory.  out != psi.
cast_status apply_pauli_sum(const void *psi, void *out, int n, cast_dtype dt, const PauliSumGroup *dgroups,
                            int ngroups, const PauliSumTerm *dterms, hipStream_t s);

}  // namespace cast
