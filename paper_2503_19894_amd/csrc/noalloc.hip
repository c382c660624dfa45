// Allocation-free variant of expval for callers that cannot allocate device
// memory (code under stream capture, tight serving loops, harnesses that
// forbid hipMalloc).
//
// expval needs device scratch for the reduction partials and the result;
// expval takes it from the reuse pool.  Here it
// is one file-scope device array per GPU, whose device address is looked up
// once per device with hipGetSymbolAddress (in host code the array's name is
// not a device address) and passed to the same kernels expval uses.  Every
// call on a GPU uses that GPU's array, so calls that overlap on one GPU (from
// several threads, or queued on different streams) race.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "internal.hpp"
#include "reduce.hpp"

namespace cast {

namespace {

static __device__ __align__(256) double scratch[kReduceScratch + 1];

constexpr int kMaxDevices = 64;
std::mutex g_sym_mu;
double *g_sym_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on the current device (looked up on the first
// call per device, with that device current).
cast_status scratch_ptr(double **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(CAST_EHIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(CAST_EUNSUPPORTED, "device index beyond the scratch table");
    std::lock_guard<std::mutex> g(g_sym_mu);
    if (!g_sym_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(CAST_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_sym_ptr[dev] = (double *)p;
    }
    *out = g_sym_ptr[dev];
    return CAST_OK;
}

}  // namespace

}  // namespace cast

using namespace cast;

extern "C" {

cast_status expval_noalloc(const cast_sv *sv, const cast_pauli_term *terms, size_t n_terms, double *out) {
    if (!sv || !sv->data) return fail(CAST_EINVAL, "state is NULL");
    if (!out) return fail(CAST_EINVAL, "out is NULL");
    if (n_terms && !terms) return fail(CAST_EINVAL, "terms is NULL");
    if (n_terms > (size_t)CAST_EXPVAL_NOALLOC_MAX_TERMS)
        return fail(CAST_EINVAL, "expval_noalloc: more terms than the fixed scratch holds (" +
                                     std::to_string(CAST_EXPVAL_NOALLOC_MAX_TERMS) + ")");
    const uint64_t full = sv->n >= 64 ? ~0ull : ((1ull << sv->n) - 1);
    for (size_t i = 0; i < n_terms; ++i)
        if ((terms[i].xmask | terms[i].zmask) & ~full) return fail(CAST_EINVAL, "Pauli term acts outside the state");
    out[0] = out[1] = 0.0;
    if (!n_terms) return CAST_OK;
    double *base = nullptr;
    if (cast_status rc = scratch_ptr(&base)) return rc;
    // fixed-size host array: nothing is allocated, on the host either
    uint16_t order[CAST_EXPVAL_NOALLOC_MAX_TERMS];
    if (cast_status rc = expval_sum(sv->data, sv->n, sv->dt, terms, n_terms, order, base, base + kReduceScratch,
                                    sv->stream))
        return rc;
    double e = 0.0;
    CAST_HIP_TRY(hipMemcpyAsync(&e, base + kReduceScratch, sizeof e, hipMemcpyDeviceToHost, sv->stream));
    CAST_HIP_TRY(hipStreamSynchronize(sv->stream));
    out[0] = e;
    return CAST_OK;
}

}  // extern "C"
