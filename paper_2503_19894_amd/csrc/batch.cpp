// Host side of batched adjoint gradients (batch.hpp): builds the op programs
// of many parametrised circuits, binds parameters into a pinned matrix
// buffer, and runs the program as per-step launches, per-step launches
// captured in a hipGraph, or one persistent launch captured in a hipGraph.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>

#include "batch.hpp"
#include "internal.hpp"

namespace cast {

struct HostOp {
    uint32_t kind;
    std::vector<int> gates;   // FWD/ADJ: gates in processing order
};

// Coefficients of a rotation operation, rewritten for every run: the angle
// is the sum over its gates (equal rotations that met in a segment).
struct BoundOp {
    uint64_t mat;             // offset in reals
    bool dagger, diag;        // U^dag; diagonal generator (phase form)
    std::vector<int> gates;
};

struct InstPlan {
    int n;
    std::vector<cast_gate> gates;          // copied descriptors
    std::vector<std::vector<cplx>> fixed;  // fixed matrices (sorted-qubit order), per gate
    std::vector<int> sq0, sq1;             // sorted targets per gate
    std::vector<char> diag;                // diagonal for every parameter value
    std::vector<uint64_t> gx, gz;          // generator masks per gate (qubits)
    std::vector<int> gslot;                // result slot per gate (-1: none)
    std::vector<HostOp> ops;
    std::vector<BoundOp> bound;
    bool unitary = true;                   // every fixed gate is
    int tb = 0;                            // tile bits of this instance's segments
    size_t nparams = 0;
    int nslots = 0;
    uint32_t wgs = 1;
};

// A batch's program on the host: the device tables and their sizes.
struct Program {
    int ninst = 0;
    cast_dtype dt = CAST_C128;
    std::vector<InstPlan> inst;
    std::vector<BatchRec> recs;         // step-major
    std::vector<SegOp> ops;
    std::vector<uint32_t> slots;
    std::vector<SegSweep> sweeps;
    std::vector<BatchInst> insts;       // psi, lam and init_src: set by the owner
    std::vector<BatchHGroup> tg;
    std::vector<BatchHTerm> tt;
    std::vector<double> coefs;          // fixed gates' coefficients; rotations are bound per run
    std::vector<uint64_t> step_rec, step_item;
    std::vector<uint64_t> step_items;   // items per step
    std::vector<size_t> step_lds;       // LDS bytes of each step's launch
    uint64_t part_doubles = 0, result_doubles = 0, total_items = 0;
    size_t state_elems = 0;             // psi and lambda of every instance, in order
    int nsteps = 0;
};

}  // namespace cast

struct cast_batch : cast::Program {
    int mode = 0;
    hipStream_t stream = nullptr;
    // device
    void *states = nullptr;
    cast::BatchRec *d_recs = nullptr;
    cast::SegOp *d_ops = nullptr;
    uint32_t *d_slots = nullptr;
    cast::SegSweep *d_sweeps = nullptr;
    size_t lds_bytes = 0;
    uint64_t *d_step_rec = nullptr, *d_step_item = nullptr;
    cast::BatchInst *d_insts = nullptr;
    void *d_mats = nullptr;
    cast::BatchHGroup *d_tg = nullptr;
    cast::BatchHTerm *d_tt = nullptr;
    double *d_partials = nullptr, *d_results = nullptr;
    unsigned long long *d_counters = nullptr;
    // host
    void *h_mats = nullptr;      // pinned, matrices in the state dtype
    double *h_results = nullptr; // pinned
    cast::BatchDev dev;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int persistent_grid = 1024;
    uint32_t persistent_chunk = 16;
    uint32_t spin_limit = 1u << 24;
};

namespace cast {

static void sorted_matrix(int k, const int *qubits, const std::vector<cplx> &m, int *q0, int *q1,
                          std::vector<cplx> *out) {
    PassPlan p;
    make_plan(k, qubits, m.data(), 0.0, 0.0, &p);
    *q0 = p.q[0];
    *q1 = k == 2 ? p.q[1] : -1;
    *out = p.full;
}

// Whether a two-qubit matrix is a I + b P for one Pauli string P that flips
// bits: nonzeros only on the diagonal (all equal) and at (r, r ^ x) for one
// x != 0, with the off-diagonal signs those of a Z mask z (the i^{|x & z|}
// of the Y letters folds into b).  On success, *xm and *zm (local bits).
static bool pauli_pair(const std::vector<cplx> &m, uint32_t *xm, uint32_t *zm) {
    const int D = 4;
    for (uint32_t x = 1; x < (uint32_t)D; ++x) {
        bool ok = true;
        for (int r = 0; r < D && ok; ++r)
            for (int c = 0; c < D && ok; ++c)
                if (c != r && c != (int)(r ^ x) && m[(size_t)r * D + c] != cplx(0, 0)) ok = false;
        for (int r = 1; r < D && ok; ++r)
            if (m[(size_t)r * D + r] != m[0]) ok = false;
        if (!ok) continue;
        for (uint32_t z = 0; z < (uint32_t)D; ++z) {
            const cplx b0 = m[x] * ((__builtin_popcount(z & x) & 1) ? -1.0 : 1.0);
            bool good = true;
            for (int r = 1; r < D && good; ++r) {
                const cplx br = m[(size_t)r * D + (r ^ x)] * ((__builtin_popcount(z & (r ^ x)) & 1) ? -1.0 : 1.0);
                if (std::abs(br - b0) > 1e-15 * (1.0 + std::abs(b0))) good = false;
            }
            if (good) {
                *xm = x;
                *zm = z;
                return true;
            }
        }
    }
    return false;
}

// (cos, sin) of a rotation -> (t, sin) of its three shears, up to a common
// sign: cos >= 0 keeps |t| <= 1.
static void shear_coefs(double *cs) {
    if (cs[0] < 0) cs[0] = -cs[0], cs[1] = -cs[1];
    cs[0] = -cs[1] / (1.0 + cs[0]);
}

// Operation code and coefficients (FP64; dagger: of the adjoint) of a fixed
// gate on sweep bits t0 < t1 (t1 = -1: one qubit), local bit i of its matrix
// index belonging to t_i.
static uint32_t fixed_op(const std::vector<cplx> &mat, int t0, int t1, bool dagger, bool c128,
                         std::vector<double> *out) {
    const int D = t1 < 0 ? 2 : 4, bit = t0, pair = t1 < 0 ? 0 : t0 + t1 - 1;
    auto at = [&](int r, int c) { return dagger ? std::conj(mat[(size_t)c * D + r]) : mat[(size_t)r * D + c]; };
    auto put = [&](cplx z) { out->push_back(z.real()), out->push_back(z.imag()); };
    bool diag = true, real = true, sign = true;
    for (int r = 0; r < D; ++r)
        for (int c = 0; c < D; ++c) {
            const cplx z = mat[(size_t)r * D + c];
            if (r != c && z != cplx(0, 0)) diag = false;
            if (z.imag() != 0.0) real = false;
            if (r == c && z != cplx(1, 0) && z != cplx(-1, 0)) sign = false;
        }
    const cplx one(1, 0);
    // local masks of a one- or two-qubit Pauli string -> sweep bits
    auto spread = [&](uint32_t m) { return ((m & 1u) << t0) | (t1 < 0 ? 0u : ((m >> 1) & 1u) << t1); };
    if (diag && sign) {
        uint32_t neg = 0;
        for (int r = 0; r < D; ++r)
            if (mat[(size_t)r * D + r] == -one) neg |= 1u << r;
        if (D == 4 && neg == 8u) return SO_CZ + pair;
        uint32_t neg8 = 0;
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t loc = ((j >> t0) & 1u) | (t1 < 0 ? 0u : ((j >> t1) & 1u) << 1);
            neg8 |= ((neg >> loc) & 1u) << j;
        }
        return SO_SIGN | neg8 << 8;
    }
    if (diag && D == 2) {
        if (c128 && mat[0] == one) {   // a phase on bit 1: the diagonal rotation's form
            put(at(1, 1));
            return spread(1);
        }
        for (int r = 0; r < D; ++r) put(at(r, r));
        return SO_DIAG1 + bit;
    }
    if (diag) {
        if (mat[0] == one && mat[5] == one && mat[10] == one) {
            put(at(3, 3));
            return SO_CP + pair;
        }
        for (int r = 0; r < D; ++r) put(at(r, r));
        return SO_DIAG2 + pair;
    }
    if (real) {
        for (int r = 0; r < D; ++r)
            for (int c = 0; c < D; ++c) out->push_back(at(r, c).real());
        return (D == 2 ? SO_REAL1 + bit : SO_REAL2 + pair);
    }
    // c I - i s P: the rotation's form (complex128: its shears are orthogonal
    // whatever c and s, so they need a unitary matrix)
    auto rotation = [&](double c, double s) {
        if (c128 && std::fabs(c * c + s * s - 1.0) > 4e-16) return false;
        double cs[2] = {c, s};
        if (c128) shear_coefs(cs);
        out->insert(out->end(), cs, cs + 2);
        return true;
    };
    if (D == 2 && mat[0] == mat[3] && mat[1] == mat[2] && mat[0].imag() == 0.0 && mat[1].real() == 0.0 &&
        rotation(mat[0].real(), -at(0, 1).imag()))
        return 8 * spread(1);
    uint32_t xm, zm;
    if (D == 4 && pauli_pair(mat, &xm, &zm)) {
        const cplx a = at(0, 0), b = at(0, (int)xm) * ((__builtin_popcount(zm & xm) & 1) ? -1.0 : 1.0);
        const int pw = __builtin_popcount(xm & zm);
        // every row agrees with b exactly, so that the pair stands for the matrix
        bool same = true;
        for (int r = 0; r < D; ++r)
            same &= at(r, r ^ (int)xm) == b * ((__builtin_popcount(zm & (r ^ xm)) & 1) ? -1.0 : 1.0);
        const bool two_qubit = (xm | zm) == 3u;
        if (same && two_qubit && a.imag() == 0.0 && (pw & 1 ? b.imag() : b.real()) == 0.0 &&
            rotation(a.real(), pw == 0 ? -b.imag() : pw == 1 ? b.real() : b.imag()))
            return 8 * spread(xm) + spread(zm);
        put(a);
        put(b);
        return (SO_PAULI + spread(xm)) | spread(zm) << 8;
    }
    for (int r = 0; r < D; ++r)
        for (int c = 0; c < D; ++c) put(at(r, c));
    return D == 2 ? SO_GEN1 + bit : SO_GEN2 + pair;
}

// Writes coefficients into a table in the state dtype.
static void put_reals(cast_dtype dt, void *table, uint64_t off, const double *v, size_t n) {
    for (size_t i = 0; i < n; ++i) {
        if (dt == CAST_C128) ((double *)table)[off + i] = v[i];
        else ((float *)table)[off + i] = (float)v[i];
    }
}

// Binds parameters (host FP64, cast once).
static void bind_rotations(const Program &p, const double *const *theta, void *table) {
    for (int i = 0; i < p.ninst; ++i)
        for (const BoundOp &o : p.inst[i].bound) {
            const std::vector<cast_gate> &g = p.inst[i].gates;
            double angle = 0.0;
            for (int l : o.gates) angle += g[l].param_coeff * theta[i][g[l].param_id];
            if (!o.diag || p.dt == CAST_C64) angle *= 0.5;
            double cs[2] = {std::cos(angle), o.dagger ? -std::sin(angle) : std::sin(angle)};
            if (!o.diag && p.dt == CAST_C128) shear_coefs(cs);
            put_reals(p.dt, table, o.mat, cs, 2);
        }
}

// Energy and gradient of one instance from its result slots.
static void read_results(const InstPlan &ip, const double *r, double *energy, double *grad) {
    *energy = r[0];
    for (size_t p = 0; p < ip.nparams; ++p) grad[p] = 0.0;
    for (size_t l = ip.gates.size(); l-- > 0;) {
        const int s = ip.gslot[l];
        if (s < 0) continue;
        // Im i^{|x & z|} S from the part of S the kernel takes
        const double v = __builtin_popcountll(ip.gx[l] & ip.gz[l]) & 2 ? -r[s] : r[s];
        grad[ip.gates[l].param_id] += ip.gates[l].param_coeff * v;
    }
}

static cast_status queue_program(cast_batch *b) {
    hipStream_t s = b->stream;
    const size_t rsz = b->dt == CAST_C128 ? 8 : 4;
    CAST_HIP_TRY(hipMemcpyAsync(b->d_mats, b->h_mats, b->coefs.size() * rsz, hipMemcpyHostToDevice, s));
    if (cast_status rc = batch_init_states(b->dev, b->dt, s)) return rc;
    if (b->mode == 2) {
        if (cast_status rc = batch_zero(b->d_counters, (2 + (size_t)b->ninst) * kCounterStride, s)) return rc;
        if (cast_status rc = batch_launch_persistent(b->dev, b->dt, b->total_items, b->persistent_grid,
                                                     b->d_counters, b->spin_limit, b->persistent_chunk, b->lds_bytes, s))
            return rc;
    } else {
        for (int st = 0; st < b->nsteps; ++st)
            if (cast_status rc = batch_launch_step(b->dev, b->dt, st, b->step_items[st], b->step_lds[st], s)) return rc;
    }
    if (cast_status rc = batch_finish(b->dev, s)) return rc;
    CAST_HIP_TRY(hipMemcpyAsync(b->h_results, b->d_results, b->result_doubles * sizeof(double),
                                hipMemcpyDeviceToHost, s));
    if (b->mode == 2)
        CAST_HIP_TRY(hipMemcpyAsync(b->h_results + b->result_doubles, b->d_counters + kCounterStride, sizeof(unsigned long long),
                                    hipMemcpyDeviceToHost, s));
    return CAST_OK;
}

static void free_batch(cast_batch *b) {
    if (!b) return;
    if (b->stream) (void)hipStreamSynchronize(b->stream);
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    dev_free(b->states);
    dev_free(b->d_recs);
    dev_free(b->d_ops);
    dev_free(b->d_slots);
    dev_free(b->d_sweeps);
    dev_free(b->d_step_rec);
    dev_free(b->d_step_item);
    dev_free(b->d_insts);
    dev_free(b->d_mats);
    dev_free(b->d_tg);
    dev_free(b->d_tt);
    dev_free(b->d_partials);
    dev_free(b->d_results);
    dev_free(b->d_counters);
    if (b->h_mats) (void)hipHostFree(b->h_mats);
    if (b->h_results) (void)hipHostFree(b->h_results);
    if (b->stream) (void)hipStreamDestroy(b->stream);
    delete b;
}

// Tile of a segment: 2^batch_tile_bits amplitudes (the tuning knob, 11 by
// default for both dtypes: psi and lambda together 64 KiB of LDS in
// complex128, 32 KiB in complex64); CAST_BATCH_TILE_BITS overrides.
static int batch_tile_bits(cast_dtype dt) {
    int tb = tuning().batch_tile_bits[dt == CAST_C64 ? CAST_C64 : CAST_C128];
    if (const char *e = std::getenv("CAST_BATCH_TILE_BITS")) tb = std::min(12, std::max(4, atoi(e)));
    return tb;
}

// Low window a segment's tile keeps (the knob batch_min_window, at most
// tb - 2 so that a two-qubit gate on high qubits still fits);
// CAST_BATCH_MIN_WINDOW overrides.
static int batch_min_window(cast_dtype dt, int tb) {
    int w = tuning().batch_min_window[dt == CAST_C64 ? CAST_C64 : CAST_C128];
    if (const char *e = std::getenv("CAST_BATCH_MIN_WINDOW")) w = atoi(e);
    return std::max(0, std::min(w, tb - 2));
}

// Whether segments may take gates out of circuit order (CAST_BATCH_REORDER=0
// keeps the circuit order).
static bool batch_reorder() {
    const char *e = std::getenv("CAST_BATCH_REORDER");
    return !e || atoi(e) != 0;
}

// Cuts a gate list into segments whose qubits fit a tile of 2^tb amplitudes
// (at most kSegMaxGates gates each), returned in application order: the
// circuit's order (reverse: the reverse order) or, with `reorder`, another
// order of the same circuit.  Two gates that share a qubit keep their
// relative order unless both are diagonal (diagonal gates commute); gates on
// disjoint qubits commute.  So any order in which every such pair keeps its
// relative order applies the same operator, and the adjoint sweep evaluates
// each gate's derivative between the states that order gives before and
// after it.  The greedy schedule fills a segment with ready gates (all
// earlier dependent gates applied), preferring those whose qubits the
// segment already holds, then the earliest ready gate that still fits.  On
// a layered ansatz (rotations on every qubit, then an entangling ring) this
// roughly halves the segments of the circuit-order cut, since a layer's
// rotations on the qubits of one tile need not wait for the rest of the
// layer.
// Orders the gates of one segment (given in a valid application order) so
// that consecutive gates share few qubits: the kernel applies each run of
// gates on at most three qubits (a register sweep) with one LDS round trip
// and one barrier, so fewer, longer runs cost less.  List scheduling under
// the same dependence rule as the segments: a run is grown from ready gates,
// first those whose qubits it already holds, then the one adding the fewest
// new qubits (earliest on ties), until no ready gate fits three qubits.  On
// a layered ansatz this interleaves the rotations of neighbouring qubits
// with the entangling gates between them (RY, RZ on q and q + 1, then their
// CZ) instead of running each rotation layer across the whole tile.
static std::vector<int> cluster_sweeps(const std::vector<int> &seg, const std::vector<uint64_t> &gmask,
                                       const std::vector<char> &gdiag) {
    const int n = (int)seg.size();
    std::vector<std::vector<int>> succ(n);
    std::vector<int> indeg(n, 0);
    for (int a = 0; a < n; ++a)
        for (int b = a + 1; b < n; ++b)
            if ((gmask[seg[a]] & gmask[seg[b]]) && !(gdiag[seg[a]] && gdiag[seg[b]])) {
                succ[a].push_back(b);
                ++indeg[b];
            }
    std::vector<int> ready, out;
    for (int a = 0; a < n; ++a)
        if (!indeg[a]) ready.push_back(a);
    while ((int)out.size() < n) {
        uint64_t bits = 0;
        for (;;) {
            int pick = -1, best_new = 4;
            for (size_t r = 0; r < ready.size(); ++r) {
                const uint64_t m = gmask[seg[ready[r]]];
                const int nw = __builtin_popcountll(m & ~bits);
                if (__builtin_popcountll(bits | m) > 3) continue;
                if (nw < best_new) pick = (int)r, best_new = nw;   // ready is ascending: earliest on ties
            }
            if (pick < 0 && bits == 0) pick = 0;   // (a gate on more than three qubits runs alone)
            if (pick < 0) break;
            const int a = ready[pick];
            ready.erase(ready.begin() + pick);
            out.push_back(seg[a]);
            bits |= gmask[seg[a]];
            for (int b : succ[a])
                if (--indeg[b] == 0) ready.insert(std::lower_bound(ready.begin(), ready.end(), b), b);
        }
    }
    return out;
}

static std::vector<std::vector<int>> segment_gates(const std::vector<uint64_t> &gmask, const std::vector<char> &gdiag,
                                                   int tb, bool reverse, bool reorder, int wmin) {
    const int L = (int)gmask.size();
    // a segment's qubits fit a tile of 2^tb amplitudes whose low window
    // [0, W) keeps at least wmin bits: at most tb - wmin of them lie at or
    // above bit wmin, so the tile is read in runs of at least 2^wmin
    // consecutive amplitudes
    const uint64_t hi_mask = wmin >= 64 ? 0 : ~((1ull << wmin) - 1);
    auto fits = [&](uint64_t q) {
        return __builtin_popcountll(q) <= tb && __builtin_popcountll(q & hi_mask) <= tb - wmin;
    };
    auto gate_at = [&](int p) { return reverse ? L - 1 - p : p; };   // base order position -> gate
    std::vector<std::vector<int>> segs;
    if (!reorder) {
        std::vector<int> cur;
        uint64_t qm = 0;
        for (int p = 0; p < L; ++p) {
            const int l = gate_at(p);
            if (!cur.empty() && (!fits(qm | gmask[l]) || cur.size() >= (size_t)kSegMaxGates)) {
                segs.push_back(cur);
                cur.clear();
                qm = 0;
            }
            cur.push_back(l);
            qm |= gmask[l];
        }
        if (!cur.empty()) segs.push_back(cur);
        return segs;
    }
    // dependence graph over base positions: per qubit, the last non-diagonal
    // gate and the diagonal gates since it
    std::vector<std::vector<int>> succ(L);
    std::vector<int> indeg(L, 0);
    std::vector<int> last_nd(64, -1);
    std::vector<std::vector<int>> diag_since(64);
    auto edge = [&](int a, int b) {
        if (a < 0) return;
        succ[a].push_back(b);
        ++indeg[b];
    };
    for (int p = 0; p < L; ++p) {
        const int l = gate_at(p);
        std::vector<int> preds;
        for (int q = 0; q < 64; ++q) {
            if (!((gmask[l] >> q) & 1ull)) continue;
            if (gdiag[l]) {
                preds.push_back(last_nd[q]);
                diag_since[q].push_back(p);
            } else {
                preds.push_back(last_nd[q]);
                for (int d : diag_since[q]) preds.push_back(d);
                diag_since[q].clear();
                last_nd[q] = p;
            }
        }
        std::sort(preds.begin(), preds.end());
        preds.erase(std::unique(preds.begin(), preds.end()), preds.end());
        for (int a : preds) edge(a, p);
    }
    std::vector<int> ready;   // base positions, ascending
    for (int p = 0; p < L; ++p)
        if (!indeg[p]) ready.push_back(p);
    int done = 0;
    while (done < L) {
        std::vector<int> cur;
        uint64_t qm = 0;
        while (cur.size() < (size_t)kSegMaxGates && !ready.empty()) {
            int pick = -1;
            for (size_t r = 0; r < ready.size() && pick < 0; ++r)
                if (!(gmask[gate_at(ready[r])] & ~qm)) pick = (int)r;
            for (size_t r = 0; r < ready.size() && pick < 0; ++r)
                if (fits(qm | gmask[gate_at(ready[r])])) pick = (int)r;
            if (pick < 0) break;
            const int p = ready[pick];
            ready.erase(ready.begin() + pick);
            cur.push_back(gate_at(p));
            qm |= gmask[gate_at(p)];
            ++done;
            for (int b : succ[p])
                if (--indeg[b] == 0) ready.insert(std::lower_bound(ready.begin(), ready.end(), b), b);
        }
        segs.push_back(cluster_sweeps(cur, gmask, gdiag));
    }
    return segs;
}

template <typename T>
static cast_status upload(T **dst, const std::vector<T> &src) {
    if (cast_status rc = dev_alloc((void **)dst, std::max<size_t>(1, src.size()) * sizeof(T))) return rc;
    if (!src.empty()) CAST_HIP_TRY(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
    return CAST_OK;
}

}  // namespace cast

namespace cast {

// Plans a batch (host only).  tile_bits: log2 amplitudes of a segment's tile;
// group_bytes: states of the instances whose programs run side by side (0:
// all of them).  The last two arguments of an instance with init_kind 2 are
// checked here; its state's address is left to the owner.
static cast_status plan_program(int n_inst, const int *n_qubits, cast_dtype dt, const cast_gate *const *circuits,
                                const size_t *n_gates, const size_t *n_params, const cast_pauli_term *const *hams,
                                const size_t *n_terms, const int *init_kind, const cast_sv *const *init_states,
                                int tile_bits, double group_bytes, Program *out) {
    Program *b = out;
    b->ninst = n_inst;
    b->dt = dt;
    b->inst.resize(n_inst);
    std::vector<BatchHGroup> &tg = b->tg;
    std::vector<BatchHTerm> &tt = b->tt;
    std::vector<BatchInst> &hinst = b->insts;
    hinst.resize(n_inst);
    uint64_t part = 0, res = 0;
    for (int i = 0; i < n_inst; ++i) {
        InstPlan &ip = b->inst[i];
        const int n = n_qubits[i];
        if (n < 3 || n > kMaxQubits) return fail(CAST_EINVAL, "instance qubit count must be in [3, 34]");
        if (n_gates[i] && !circuits[i]) return fail(CAST_EINVAL, "circuit is NULL");
        ip.n = n;
        ip.nparams = n_params[i];
        ip.gates.assign(circuits[i], circuits[i] + n_gates[i]);
        const size_t L = ip.gates.size();
        ip.fixed.resize(L);
        ip.diag.assign(L, 0);
        ip.sq0.resize(L);
        ip.sq1.resize(L);
        ip.gx.assign(L, 0);
        ip.gz.assign(L, 0);
        ip.gslot.assign(L, -1);
        int slot = 1;  // slot 0: energy
        for (size_t l = 0; l < L; ++l) {
            const cast_gate &g = ip.gates[l];
            if (g.k < 1 || g.k > 2) return fail(CAST_EUNSUPPORTED, "batched programs take 1- and 2-qubit gates");
            for (int a = 0; a < g.k; ++a) {
                if (g.qubits[a] < 0 || g.qubits[a] >= n) return fail(CAST_EINVAL, "gate qubit out of range");
                for (int c = 0; c < a; ++c)
                    if (g.qubits[a] == g.qubits[c]) return fail(CAST_EINVAL, "duplicate gate qubit");
            }
            const int D = 1 << g.k;
            if (g.param_id >= 0) {
                if ((size_t)g.param_id >= ip.nparams) return fail(CAST_EINVAL, "param_id out of range");
                if (g.generator <= 0 || g.generator >= (1 << (2 * g.k)))
                    return fail(CAST_EINVAL, "parametrised gate needs a Pauli generator");
                ip.gslot[l] = slot++;
                for (int a = 0; a < g.k; ++a) {
                    const int letter = (g.generator >> (2 * a)) & 3;
                    if (letter == 1 || letter == 2) ip.gx[l] |= 1ull << g.qubits[a];
                    if (letter == 2 || letter == 3) ip.gz[l] |= 1ull << g.qubits[a];
                }
                ip.sq0[l] = g.k == 2 ? std::min(g.qubits[0], g.qubits[1]) : g.qubits[0];
                ip.sq1[l] = g.k == 2 ? std::max(g.qubits[0], g.qubits[1]) : -1;
                ip.diag[l] = ip.gx[l] == 0;
                continue;
            }
            if (!g.matrix) return fail(CAST_EINVAL, "fixed gate without a matrix");
            ip.unitary &= unitary_gate(g);
            std::vector<cplx> m((size_t)D * D);
            for (int e = 0; e < D * D; ++e) m[e] = cplx(g.matrix[2 * e], g.matrix[2 * e + 1]);
            sorted_matrix(g.k, g.qubits, m, &ip.sq0[l], &ip.sq1[l], &ip.fixed[l]);
            ip.diag[l] = 1;
            for (int e = 0; e < D * D; ++e)
                if (e / D != e % D && ip.fixed[l][e] != cplx(0, 0)) ip.diag[l] = 0;
        }
        ip.nslots = slot;
        // segments (forward order, then reverse order) whose qubits together
        // fit one tile of 2^tb amplitudes
        ip.tb = std::min(n, tile_bits);
        std::vector<uint64_t> gmask(L, 0);
        for (size_t l = 0; l < L; ++l)
            for (int a = 0; a < ip.gates[l].k; ++a) gmask[l] |= 1ull << ip.gates[l].qubits[a];
        auto segment = [&](bool reverse) {
            return segment_gates(gmask, ip.diag, ip.tb, reverse, batch_reorder(), batch_min_window(dt, ip.tb));
        };
        for (auto &sg : segment(false)) ip.ops.push_back(HostOp{BK_FWD, sg});
        ip.ops.push_back(HostOp{BK_HPSI, {}});
        for (auto &sg : segment(true)) ip.ops.push_back(HostOp{BK_ADJ, sg});
        ip.wgs = 1u << (n - ip.tb);
        // Hamiltonian, grouped by x mask
        if (n_terms[i] && !hams[i]) return fail(CAST_EINVAL, "Hamiltonian is NULL");
        BatchInst &bi = hinst[i];
        bi.n = n;
        bi.nslots = ip.nslots;
        bi.wgs = ip.wgs;
        bi.tg_off = (uint32_t)tg.size();
        bi.tt_off = (uint32_t)tt.size();
        std::map<std::pair<uint64_t, int>, std::vector<size_t>> byx;   // x mask, parity of |x & z|
        std::vector<std::pair<uint64_t, int>> order;
        const uint64_t full = (1ull << n) - 1;
        for (size_t t = 0; t < n_terms[i]; ++t) {
            const cast_pauli_term &pt = hams[i][t];
            if ((pt.xmask | pt.zmask) & ~full) return fail(CAST_EINVAL, "Pauli term acts outside the state");
            const std::pair<uint64_t, int> key(pt.xmask, __builtin_popcountll(pt.xmask & pt.zmask) & 1);
            if (!byx.count(key)) order.push_back(key);
            byx[key].push_back(t);
        }
        uint32_t first = 0;
        for (auto &key : order) {
            tg.push_back(BatchHGroup{key.first, first, (uint32_t)byx[key].size(), (uint32_t)key.second, 0});
            for (size_t t : byx[key]) {
                const cast_pauli_term &pt = hams[i][t];
                // i^{|x & z|}: 1, i, -1, -i
                tt.push_back(BatchHTerm{pt.zmask, __builtin_popcountll(pt.xmask & pt.zmask) & 2 ? -pt.coeff : pt.coeff});
                ++first;
            }
        }
        bi.ngroups = (uint32_t)order.size();
        bi.part_off = part;
        part += (uint64_t)ip.nslots * ip.wgs;
        bi.res_off = res;
        res += (uint64_t)ip.nslots;
        bi.init_kind = init_kind ? init_kind[i] : 0;
        if (bi.init_kind < 0 || bi.init_kind > 2) return fail(CAST_EINVAL, "bad init kind");
        if (bi.init_kind == 2) {
            const cast_sv *src = init_states ? init_states[i] : nullptr;
            if (!src || !src->data || src->n != n || src->dt != dt)
                return fail(CAST_EINVAL, "init state missing or of the wrong size/dtype");
            bi.init_src = src->data;
        }
        b->state_elems += 2ull << n;  // psi and lambda
    }
    b->part_doubles = part;
    b->result_doubles = res;
    // ---- instance groups (consecutive instances whose psi and lambda fit the
    // cache budget run their whole programs before the next group), then
    // steps: step (g, s) holds op s of every instance of group g
    std::vector<std::pair<int, int>> groups;  // [first, last)
    {
        int first = 0;
        double acc = 0;
        const double ab_d = (double)amp_bytes(dt);
        for (int i = 0; i < n_inst; ++i) {
            const double bytes = 2.0 * std::ldexp(1.0, n_qubits[i]) * ab_d;
            if (i > first && group_bytes > 0 && acc + bytes > group_bytes) {
                groups.emplace_back(first, i);
                first = i;
                acc = 0;
            }
            acc += bytes;
        }
        groups.emplace_back(first, n_inst);
        // keep a captured program below 65536 launches: merge groups if needed
        size_t max_ops_all = 0;
        for (auto &ip : b->inst) max_ops_all = std::max(max_ops_all, ip.ops.size());
        const size_t cap = 65536;
        if (groups.size() * max_ops_all > cap) {
            const size_t per = (groups.size() * max_ops_all + cap - 1) / cap;   // groups per merged group
            std::vector<std::pair<int, int>> merged;
            for (size_t gi = 0; gi < groups.size(); gi += per)
                merged.emplace_back(groups[gi].first, groups[std::min(groups.size(), gi + per) - 1].second);
            groups.swap(merged);
        }
    }
    std::vector<BatchRec> &recs = b->recs;
    std::vector<SegOp> &segs = b->ops;
    std::vector<uint32_t> &slots = b->slots;
    std::vector<SegSweep> &sweeps = b->sweeps;
    std::vector<double> &coefs = b->coefs;
    uint64_t item_base = 0;
    for (auto &gr : groups) {
    size_t max_ops = 0;
    for (int i = gr.first; i < gr.second; ++i) max_ops = std::max(max_ops, b->inst[i].ops.size());
    for (size_t s = 0; s < max_ops; ++s) {
        b->step_rec.push_back(recs.size());
        b->step_item.push_back(item_base);
        uint64_t items = 0;
        for (int i = gr.first; i < gr.second; ++i) {
            InstPlan &ip = b->inst[i];
            if (s >= ip.ops.size()) continue;
            const HostOp &op = ip.ops[s];
            BatchRec r;
            memset(&r, 0, sizeof r);
            r.kind = op.kind;
            r.inst = (uint32_t)i;
            r.item0 = (uint32_t)items;
            r.wgs = ip.wgs;
            r.need = (uint64_t)s * ip.wgs;
            r.tb = ip.tb;
            if (op.kind != BK_HPSI) {
                // tile geometry: smallest khi with #{segment qubits >= tb - khi} == khi
                const std::vector<int> &gl = op.gates;
                uint64_t qm = 0;
                for (int l : gl)
                    for (int a = 0; a < ip.gates[l].k; ++a) qm |= 1ull << ip.gates[l].qubits[a];
                int khi = 0;
                for (;; ++khi) {
                    const int lim = ip.tb - khi;
                    const uint64_t above = lim >= 64 ? 0 : (qm & ~((1ull << lim) - 1));
                    if (__builtin_popcountll(above) == khi) break;
                }
                r.W = ip.tb - khi;
                int pos[64];
                int h = 0;
                for (int q = 0; q < r.W; ++q) pos[q] = q, r.bit[q] = 1ull << q;
                for (int q = r.W; q < ip.n; ++q)
                    if ((qm >> q) & 1ull) pos[q] = r.W + h, r.bit[r.W + h] = 1ull << q, ++h;
                // sweeps: consecutive gates on at most three tile bits (padded
                // with the lowest other tile bits to exactly three)
                r.sw0 = (uint32_t)sweeps.size();
                r.ps0 = (uint32_t)slots.size();
                // a rotation equal to an earlier one of the segment, with no
                // gate in between on its qubits, joins it: one inner product
                // (they commute) and one application with the summed angle.
                // complex64 keeps every rotation: each rounds the state, and
                // its results stay those of the gates one by one.  So does an
                // instance with a fixed gate that is not unitary: U^dag does
                // not undo it, so the inner products on its two sides differ.
                std::vector<int> head(gl.size(), -1);     // gate position it joins
                std::vector<std::vector<int>> joined(gl.size());
                {
                    std::vector<int> last(64, -1);        // last position on each qubit
                    for (size_t q = 0; q < gl.size(); ++q) {
                        const int l = gl[q];
                        const int p0 = last[ip.sq0[l]], p1 = ip.sq1[l] < 0 ? p0 : last[ip.sq1[l]];
                        const int lp = p0 >= 0 ? gl[p0] : -1;
                        if (dt == CAST_C128 && ip.unitary && lp >= 0 && p0 == p1 && ip.gates[l].param_id >= 0 && ip.gates[lp].param_id >= 0 &&
                            ip.gx[l] == ip.gx[lp] && ip.gz[l] == ip.gz[lp] && ip.sq0[l] == ip.sq0[lp] &&
                            ip.sq1[l] == ip.sq1[lp]) {
                            head[q] = p0;
                            joined[p0].push_back(l);
                            if (op.kind == BK_ADJ) ip.gslot[l] = ip.gslot[lp];
                            continue;
                        }
                        joined[q].push_back(l);
                        last[ip.sq0[l]] = (int)q;
                        if (ip.sq1[l] >= 0) last[ip.sq1[l]] = (int)q;
                    }
                }
                size_t gi = 0;
                while (gi < gl.size()) {
                    if (head[gi] >= 0) {
                        ++gi;
                        continue;
                    }
                    uint32_t bits = 0;
                    size_t gj = gi;
                    for (; gj < gl.size(); ++gj) {
                        if (head[gj] >= 0) continue;
                        const int l = gl[gj];
                        uint32_t gb = 1u << pos[ip.sq0[l]];
                        if (ip.gates[l].k == 2) gb |= 1u << pos[ip.sq1[l]];
                        if (__builtin_popcount(bits | gb) > 3) break;
                        bits |= gb;
                    }
                    for (int t = 0; __builtin_popcount(bits) < 3 && t < ip.tb; ++t) bits |= 1u << t;
                    SegSweep sw;
                    memset(&sw, 0, sizeof sw);
                    int loc[32];
                    for (int t = 0, c = 0; t < ip.tb; ++t)
                        if ((bits >> t) & 1u) sw.bits |= (uint32_t)t << (8 * c), loc[t] = c++;
                    sw.g0 = (uint32_t)segs.size();
                    sw.p0 = (uint32_t)slots.size() - r.ps0;
                    for (size_t q = gi; q < gj; ++q) {
                        if (head[q] >= 0) continue;
                        const int l = gl[q];
                        const int t0 = loc[pos[ip.sq0[l]]];
                        const int t1 = ip.gates[l].k == 2 ? loc[pos[ip.sq1[l]]] : -1;
                        SegOp o;
                        o.mat = (uint32_t)coefs.size();
                        if (ip.gates[l].param_id >= 0) {
                            auto mask = [&](uint64_t m) {
                                uint32_t v = (uint32_t)((m >> ip.sq0[l]) & 1ull) << t0;
                                if (t1 >= 0) v |= (uint32_t)((m >> ip.sq1[l]) & 1ull) << t1;
                                return v;
                            };
                            o.info = 8 * mask(ip.gx[l]) + mask(ip.gz[l]);
                            ip.bound.push_back(BoundOp{coefs.size(), op.kind == BK_ADJ, ip.diag[l] != 0, joined[q]});
                            coefs.resize(coefs.size() + 2, 0.0);
                            if (op.kind == BK_ADJ) {
                                o.info |= kSegParam;
                                slots.push_back((uint32_t)ip.gslot[l]);
                            }
                        } else {
                            o.info = fixed_op(ip.fixed[l], t0, t1, op.kind == BK_ADJ, dt == CAST_C128, &coefs);
                        }
                        segs.push_back(o);
                    }
                    sw.g1 = (uint32_t)segs.size();
                    sweeps.push_back(sw);
                    gi = gj;
                }
                r.sw1 = (uint32_t)sweeps.size();
                r.np = (uint32_t)slots.size() - r.ps0;
            }
            recs.push_back(r);
            items += ip.wgs;
        }
        if (items > 0x7fffffffull) return fail(CAST_EUNSUPPORTED, "too many work items in one step");
        b->step_items.push_back(items);
        {
            // LDS of this step's launch: the tables, then one tile (forward) or
            // two (adjoint: psi and lambda) of its largest tile
            int tbs = 0, tiles = 0;
            for (size_t q = b->step_rec.back(); q < recs.size(); ++q) {
                if (recs[q].kind == BK_HPSI) continue;
                tbs = std::max(tbs, recs[q].tb);
                tiles = std::max(tiles, recs[q].kind == BK_ADJ ? 2 : 1);
            }
            b->step_lds.push_back(kSegLdsExtra + (size_t)tiles * ((size_t)1 << tbs) * amp_bytes(dt));
        }
        item_base += items;
    }
    }
    // the kernel reads two operations and two coefficients ahead
    segs.resize(segs.size() + 2, SegOp{0, 0});
    coefs.resize(coefs.size() + 2, 0.0);
    if (coefs.size() > 0xffffffffull) return fail(CAST_EUNSUPPORTED, "batch matrix table exceeds 2^32 entries");
    b->nsteps = (int)b->step_items.size();
    b->step_rec.push_back(recs.size());
    b->step_item.push_back(item_base);
    b->total_items = item_base;
    return CAST_OK;
}

cast_status adjoint_segments(const cast_sv *init, const cast_gate *gates, size_t n_gates, const double *theta,
                             size_t n_params, const cast_pauli_term *terms, size_t n_terms, double *energy,
                             double *grad) {
    const int n = init->n, kind = CAST_INIT_STATE;
    const cast_dtype dt = init->dt;
    hipStream_t s = init->stream;
    // one instance has 2^(n - tb) items per step: smaller tiles below 19 qubits
    // keep some 256 workgroups busy; and whatever the knob asks for, psi's and
    // lambda's tiles fit a launch's LDS
    int tb = std::min(batch_tile_bits(dt), std::max(9, n - 8));
    while (kSegLdsExtra + ((2 * amp_bytes(dt)) << tb) > kSegMaxLds) --tb;
    Program p;
    if (cast_status rc = plan_program(1, &n, dt, &gates, &n_gates, &n_params, &terms, &n_terms, &kind, &init, tb, 0.0,
                                      &p))
        return rc;
    const size_t ab = amp_bytes(dt), rsz = ab / 2, N = (size_t)1 << n;
    DevBuf states(s), tables(s), sums(s);
    if (cast_status rc = states.alloc(2 * N * ab)) return rc;
    if (cast_status rc = sums.alloc((p.part_doubles + p.result_doubles) * sizeof(double))) return rc;
    p.insts[0].psi = states.p;
    p.insts[0].lam = (char *)states.p + N * ab;
    p.insts[0].init_src = init->data;
    // all tables in one buffer and one copy
    std::vector<char> h;
    auto put = [&](const void *src, size_t bytes) {
        const size_t off = (h.size() + 255) & ~(size_t)255;
        h.resize(off + std::max<size_t>(bytes, 16));
        if (bytes) std::memcpy(h.data() + off, src, bytes);
        return off;
    };
    auto put_all = [&](const auto &v) { return put(v.data(), v.size() * sizeof(v[0])); };
    const size_t o_recs = put_all(p.recs), o_ops = put_all(p.ops), o_slots = put_all(p.slots),
                 o_sweeps = put_all(p.sweeps), o_srec = put_all(p.step_rec), o_sitem = put_all(p.step_item),
                 o_insts = put_all(p.insts), o_tg = put_all(p.tg), o_tt = put_all(p.tt);
    std::vector<char> mats(p.coefs.size() * rsz);
    put_reals(dt, mats.data(), 0, p.coefs.data(), p.coefs.size());
    bind_rotations(p, &theta, mats.data());
    const size_t o_mats = put_all(mats);
    if (cast_status rc = tables.alloc(h.size())) return rc;
    CAST_HIP_TRY(hipMemcpyAsync(tables.p, h.data(), h.size(), hipMemcpyHostToDevice, s));
    auto at = [&](size_t off) { return (void *)((char *)tables.p + off); };
    BatchDev d;
    d.recs = (const BatchRec *)at(o_recs);
    d.ops = (const SegOp *)at(o_ops);
    d.slots = (const uint32_t *)at(o_slots);
    d.sweeps = (const SegSweep *)at(o_sweeps);
    d.step_rec = (const uint64_t *)at(o_srec);
    d.step_item = (const uint64_t *)at(o_sitem);
    d.insts = (const BatchInst *)at(o_insts);
    d.mats = at(o_mats);
    d.tg = (const BatchHGroup *)at(o_tg);
    d.tt = (const BatchHTerm *)at(o_tt);
    d.partials = sums.as<double>();
    d.results = sums.as<double>() + p.part_doubles;
    d.nsteps = p.nsteps;
    d.ninst = 1;
    if (cast_status rc = batch_init_states(d, dt, s)) return rc;
    for (int st = 0; st < p.nsteps; ++st)
        if (cast_status rc = batch_launch_step(d, dt, st, p.step_items[st], p.step_lds[st], s)) return rc;
    if (cast_status rc = batch_finish(d, s)) return rc;
    std::vector<double> r(p.result_doubles);
    CAST_HIP_TRY(hipMemcpyAsync(r.data(), d.results, r.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    CAST_HIP_TRY(hipStreamSynchronize(s));
    read_results(p.inst[0], r.data(), energy, grad);
    return CAST_OK;
}

}  // namespace cast

using namespace cast;

extern "C" {

cast_status batch_create(int n_inst, const int *n_qubits, cast_dtype dt, const cast_gate *const *circuits,
                         const size_t *n_gates, const size_t *n_params, const cast_pauli_term *const *hams,
                         const size_t *n_terms, const int *init_kind, const cast_sv *const *init_states, int mode,
                         cast_batch **out) {
    if (!out) return fail(CAST_EINVAL, "out is NULL");
    *out = nullptr;
    if (n_inst < 1 || n_inst > 65535) return fail(CAST_EINVAL, "n_inst must be in [1, 65535]");
    if (!n_qubits || !circuits || !n_gates || !n_params || !hams || !n_terms)
        return fail(CAST_EINVAL, "NULL array argument");
    if (dt != CAST_C64 && dt != CAST_C128) return fail(CAST_EINVAL, "bad dtype");
    if (mode < 0 || mode > 2) return fail(CAST_EINVAL, "mode must be 0, 1 or 2");
    cast_batch *b = new cast_batch;
    b->mode = mode;
    auto bail = [&](cast_status rc) {
        free_batch(b);
        return rc;
    };
    // per-step launches: groups of 512 MB of states; the persistent launch keeps
    // every instance in one step-major stream.  The sweeps are bound by latency,
    // so groups need not fit the 256 MB last-level cache, and larger ones make
    // fewer launches with nearly empty last waves: 20 qubits, 64 sets, 39.2 ms
    // with 192 MB, 38.5 with 512, 38.4 with 1024 (complex64 26.1, 25.2, 24.3);
    // 18 qubits 9.7, 9.4, 9.5; instances of 16 to 26 qubits, 0.425 s with 192
    // and 512 MB, 0.431 with 1000.
    double group_bytes = mode == 2 ? 0.0 : 512.0 * (1 << 20);
    if (const char *e = std::getenv("CAST_BATCH_GROUP_MB"))
        if (mode != 2) group_bytes = atof(e) * (1 << 20);
    if (const char *e = std::getenv("CAST_PERSISTENT_GROUP_MB"))
        if (mode == 2) group_bytes = atof(e) * (1 << 20);
    if (cast_status rc = plan_program(n_inst, n_qubits, dt, circuits, n_gates, n_params, hams, n_terms, init_kind,
                                      init_states, batch_tile_bits(dt), group_bytes, b))
        return bail(rc);
    // ---- device and pinned buffers
    const size_t rsz = dt == CAST_C128 ? 8 : 4;
    const size_t ab = amp_bytes(dt);
    if (cast_status rc = dev_alloc(&b->states, b->state_elems * ab)) return bail(rc);
    size_t off = 0;
    for (int i = 0; i < n_inst; ++i) {
        const size_t N = (size_t)1 << b->insts[i].n;
        b->insts[i].psi = (char *)b->states + off * ab;
        b->insts[i].lam = (char *)b->states + (off + N) * ab;
        off += 2 * N;
    }
    if (cast_status rc = upload(&b->d_recs, b->recs)) return bail(rc);
    if (cast_status rc = upload(&b->d_ops, b->ops)) return bail(rc);
    if (cast_status rc = upload(&b->d_slots, b->slots)) return bail(rc);
    if (cast_status rc = upload(&b->d_sweeps, b->sweeps)) return bail(rc);
    {
        int tbm = 0;
        for (auto &ip : b->inst) tbm = std::max(tbm, ip.tb);
        b->lds_bytes = 2 * ((size_t)1 << tbm) * amp_bytes(dt) + kSegLdsExtra;
    }
    if (cast_status rc = upload(&b->d_step_rec, b->step_rec)) return bail(rc);
    if (cast_status rc = upload(&b->d_step_item, b->step_item)) return bail(rc);
    if (cast_status rc = upload(&b->d_insts, b->insts)) return bail(rc);
    if (cast_status rc = upload(&b->d_tg, b->tg)) return bail(rc);
    if (cast_status rc = upload(&b->d_tt, b->tt)) return bail(rc);
    if (cast_status rc = dev_alloc(&b->d_mats, b->coefs.size() * rsz)) return bail(rc);
    if (cast_status rc = dev_alloc((void **)&b->d_partials, std::max<uint64_t>(1, b->part_doubles) * sizeof(double)))
        return bail(rc);
    if (cast_status rc = dev_alloc((void **)&b->d_results, std::max<uint64_t>(1, b->result_doubles) * sizeof(double)))
        return bail(rc);
    if (cast_status rc = dev_alloc((void **)&b->d_counters, (2 + (size_t)n_inst) * kCounterStride * sizeof(unsigned long long)))
        return bail(rc);
    if (hipHostMalloc(&b->h_mats, b->coefs.size() * rsz) != hipSuccess)
        return bail(fail(CAST_ENOMEM, "pinned matrix buffer"));
    if (hipHostMalloc((void **)&b->h_results, (b->result_doubles + 1) * sizeof(double)) != hipSuccess)
        return bail(fail(CAST_ENOMEM, "pinned result buffer"));
    put_reals(dt, b->h_mats, 0, b->coefs.data(), b->coefs.size());
    if (hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking) != hipSuccess)
        return bail(fail(CAST_EHIP, "hipStreamCreate failed"));
    BatchDev &d = b->dev;
    d.recs = b->d_recs;
    d.ops = b->d_ops;
    d.slots = b->d_slots;
    d.sweeps = b->d_sweeps;
    d.step_rec = b->d_step_rec;
    d.step_item = b->d_step_item;
    d.insts = b->d_insts;
    d.mats = b->d_mats;
    d.tg = b->d_tg;
    d.tt = b->d_tt;
    d.partials = b->d_partials;
    d.results = b->d_results;
    d.nsteps = b->nsteps;
    d.ninst = n_inst;
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    b->persistent_grid = cus * 4;
    b->spin_limit = (uint32_t)tuning().persistent_spin_limit[dt == CAST_C64 ? CAST_C64 : CAST_C128];
    // items per claim: 16 (measured best once a step has some 16000 items, see
    // the claim loop) would leave most workgroups without work where steps are
    // small: a 19-qubit instance has 256 items, i.e. 16 busy workgroups of the
    // 512 resident ones.  One claim per resident workgroup and step; and no
    // more workgroups than a step has claims (and a few to step in while others
    // publish), since idle ones poll the counters that the busy ones update.
    // Trotter rings of 10, 13, 16 and 19 qubits, complex64: 23.7 -> 3.4 ms.
    const uint64_t per_step = std::max<uint64_t>(1, b->total_items / (uint64_t)std::max(1, b->nsteps));
    b->persistent_chunk = (uint32_t)std::min<uint64_t>(16, std::max<uint64_t>(1, per_step / (2 * (uint64_t)cus)));
    uint64_t most = 1;
    for (uint64_t m : b->step_items) most = std::max(most, m);
    b->persistent_grid = (int)std::min<uint64_t>(b->persistent_grid, most / b->persistent_chunk + 32);
    if (const char *e = std::getenv("CAST_PERSISTENT_WG_PER_CU")) b->persistent_grid = cus * std::max(1, atoi(e));
    if (const char *e = std::getenv("CAST_PERSISTENT_CHUNK")) b->persistent_chunk = (uint32_t)std::max(1, atoi(e));
    if (mode >= 1) {
        // capture the whole program once; batch_run refreshes the pinned
        // matrices and replays it
        if (hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
            return bail(fail(CAST_EHIP, "hipStreamBeginCapture failed"));
        cast_status rc = queue_program(b);
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(b->stream, &g);
        if (rc) {
            if (g) (void)hipGraphDestroy(g);
            return bail(rc);
        }
        if (e != hipSuccess) return bail(fail(CAST_EHIP, std::string("graph capture: ") + hipGetErrorString(e)));
        b->graph = g;
        e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
        if (e != hipSuccess) return bail(fail(CAST_EHIP, std::string("graph instantiate: ") + hipGetErrorString(e)));
    }
    *out = b;
    return CAST_OK;
}

cast_status batch_run(cast_batch *b, const double *const *theta, double *energies, double *const *grads) {
    if (!b) return fail(CAST_EINVAL, "batch is NULL");
    if (!energies) return fail(CAST_EINVAL, "energies is NULL");
    for (int i = 0; i < b->ninst; ++i) {
        const InstPlan &ip = b->inst[i];
        if (ip.nparams && (!theta || !theta[i] || !grads || !grads[i]))
            return fail(CAST_EINVAL, "theta/grads missing for an instance with parameters");
    }
    bind_rotations(*b, theta, b->h_mats);
    if (b->mode >= 1) {
        CAST_HIP_TRY(hipGraphLaunch(b->exec, b->stream));
    } else {
        if (cast_status rc = queue_program(b)) return rc;
    }
    CAST_HIP_TRY(hipStreamSynchronize(b->stream));
    if (b->mode == 2) {
        unsigned long long err;
        memcpy(&err, b->h_results + b->result_doubles, sizeof err);
        if (err) return fail(CAST_EHIP, "persistent batch: a dependency wait exceeded its bound");
    }
    size_t off = 0;
    for (int i = 0; i < b->ninst; ++i) {
        read_results(b->inst[i], b->h_results + off, &energies[i], b->inst[i].nparams ? grads[i] : nullptr);
        off += (size_t)b->inst[i].nslots;
    }
    return CAST_OK;
}

void batch_destroy(cast_batch *b) { free_batch(b); }

cast_status adjoint_grad_batch(int n_inst, const int *n_qubits, cast_dtype dt, const cast_gate *const *circuits,
                               const size_t *n_gates, const double *const *theta, const size_t *n_params,
                               const cast_pauli_term *const *hams, const size_t *n_terms, const int *init_kind,
                               const cast_sv *const *init_states, int mode, double *energies, double *const *grads) {
    cast_batch *b = nullptr;
    if (cast_status rc = batch_create(n_inst, n_qubits, dt, circuits, n_gates, n_params, hams, n_terms, init_kind,
                                      init_states, mode, &b))
        return rc;
    cast_status rc = batch_run(b, theta, energies, grads);
    batch_destroy(b);
    return rc;
}

cast_status batch_info(const cast_batch *b, int *n_steps, uint64_t *total_items, double *state_bytes) {
    if (!b) return fail(CAST_EINVAL, "batch is NULL");
    if (n_steps) *n_steps = b->nsteps;
    if (total_items) *total_items = b->total_items;
    if (state_bytes) {
        double s = 0;
        for (auto &ip : b->inst) s += 2.0 * std::ldexp(1.0, ip.n) * (double)amp_bytes(b->dt);
        *state_bytes = s;
    }
    return CAST_OK;
}

cast_status batch_segments(int n, const cast_gate *gates, size_t n_gates, cast_dtype dt, int reverse,
                           size_t *n_segments, int *order, int *segment_of) {
    if (!n_segments) return fail(CAST_EINVAL, "n_segments is NULL");
    if (n_gates && !gates) return fail(CAST_EINVAL, "gates is NULL");
    if (dt != CAST_C64 && dt != CAST_C128) return fail(CAST_EINVAL, "bad dtype");
    if (n < 3 || n > kMaxQubits) return fail(CAST_EINVAL, "qubit count must be in [3, 34]");
    std::vector<uint64_t> gmask(n_gates, 0);
    std::vector<char> gdiag(n_gates, 0);
    for (size_t l = 0; l < n_gates; ++l) {
        const cast_gate &g = gates[l];
        if (g.k < 1 || g.k > 2) return fail(CAST_EUNSUPPORTED, "batched programs take 1- and 2-qubit gates");
        for (int a = 0; a < g.k; ++a) {
            if (g.qubits[a] < 0 || g.qubits[a] >= n) return fail(CAST_EINVAL, "gate qubit out of range");
            gmask[l] |= 1ull << g.qubits[a];
        }
        bool diag = true;
        if (g.param_id >= 0) {
            for (int a = 0; a < g.k; ++a) {
                const int letter = (g.generator >> (2 * a)) & 3;
                if (letter == 1 || letter == 2) diag = false;
            }
        } else {
            if (!g.matrix) return fail(CAST_EINVAL, "fixed gate without a matrix");
            const int D = 1 << g.k;
            for (int r = 0; r < D; ++r)
                for (int c = 0; c < D; ++c)
                    if (r != c && (g.matrix[2 * (r * D + c)] != 0.0 || g.matrix[2 * (r * D + c) + 1] != 0.0)) diag = false;
        }
        gdiag[l] = diag;
    }
    const std::vector<std::vector<int>> segs =
        segment_gates(gmask, gdiag, std::min(n, batch_tile_bits(dt)), reverse != 0, batch_reorder(),
                      batch_min_window(dt, std::min(n, batch_tile_bits(dt))));
    *n_segments = segs.size();
    size_t i = 0;
    for (size_t sgi = 0; sgi < segs.size(); ++sgi)
        for (int l : segs[sgi]) {
            if (order) order[i] = l;
            if (segment_of) segment_of[i] = (int)sgi;
            ++i;
        }
    return CAST_OK;
}

cast_status batch_traffic(const cast_batch *b, double *alg_bytes, uint64_t *state_passes) {
    if (!b) return fail(CAST_EINVAL, "batch is NULL");
    double bytes = 0;
    uint64_t passes = 0;
    for (auto &ip : b->inst) {
        const double S = std::ldexp(1.0, ip.n) * (double)amp_bytes(b->dt);
        bytes += S;                           // initial state written
        for (auto &op : ip.ops) {
            if (op.kind == BK_ADJ) {          // psi and lambda read and written
                bytes += 4 * S;
                passes += 2;
            } else {                          // FWD: psi read and written; HPSI: psi read, lambda written
                bytes += 2 * S;
                passes += 1;
            }
        }
    }
    if (alg_bytes) *alg_bytes = bytes;
    if (state_passes) *state_passes = passes;
    return CAST_OK;
}

}  // extern "C"
