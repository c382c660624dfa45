// Batched adjoint-gradient programs: many parametrised circuits (same or
// different qubit counts) evaluated together on one GPU.
//
// Each instance's program is a list of ops, op s of every instance forming
// global step s:
//   FWD  a segment of consecutive gates applied to psi
//   HPSI lambda <- H psi, partial sums of <psi|lambda>  (energy)
//   ADJ  a segment of gates in reverse order: for each, partial sums of
//        <lambda|G|psi>, then psi <- U^dag psi, lambda <- U^dag lambda
// A segment holds consecutive gates whose qubits together fit one LDS tile
// (the low window [0, W) plus the segment's qubits at or above W): a work
// item loads one tile of psi (and lambda), applies every gate of the segment
// in LDS in order, and writes the tile back, so one HBM pass serves many
// gates.  Every op of an instance has `wgs` items (tiles); partial sums of
// item w land in a fixed slot, and a final kernel adds them in a fixed order.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/cast.h"

namespace cast {

enum BatchKind : uint32_t { BK_FWD = 0, BK_HPSI = 1, BK_ADJ = 2 };

constexpr int kSegMaxGates = 64;   // gates per segment (bounds the LDS reduction area)
// LDS of a segment item beyond its two tiles: the inner products' per-wave sums
constexpr size_t kSegLdsExtra = (size_t)kSegMaxGates * 4 * sizeof(double);
constexpr size_t kSegMaxLds = 128u << 10;   // of a launch

// Operations of a register sweep, in sweep coordinates (a thread holds eight
// amplitudes x[j], bit i of j <-> the sweep's tile bit i).  Codes below 64
// are Pauli rotations, code = 8 X + Z with the string's x / z masks over the
// sweep bits: exp(-i a P / 2), two reals.  complex64: cos and +-sin of a / 2.
// complex128 leaves out a global phase, which energies and gradients do not
// see: for X = 0 (diagonal) the phase e^{+-i a} on the amplitudes with odd Z
// parity, (cos, +-sin) of a; for X != 0 the rotation by a / 2 up to a sign
// that makes cos >= 0, as three shears, t = -sin / (1 + cos) and sin.  The
// others are fixed gates; `pair` counts the sweep-bit pairs (0,1), (0,2),
// (1,2).
enum SegCode : uint32_t {
    SO_CZ = 64,      // + pair: x[11] = -x[11]; no coefficients
    SO_CP = 67,      // + pair: x[11] *= p; 2 reals
    SO_DIAG1 = 70,   // + bit: 4 reals
    SO_DIAG2 = 73,   // + pair: 8 reals
    SO_REAL1 = 76,   // + bit: 4 reals
    SO_GEN1 = 79,    // + bit: 8 reals
    SO_REAL2 = 82,   // + pair: 16 reals
    SO_GEN2 = 85,    // + pair: 32 reals
    SO_SIGN = 88,    // x[j] = -x[j] where bit j of info bits 8-15 is set; no coefficients
    SO_PAULI = 88,   // + X (1..7): y_j = a x_j + b (-1)^{popc(z & (j ^ X))} x_{j ^ X}, z = info bits 8-10;
                     // 4 reals
};
struct SegOp {
    uint32_t info;          // bits 0-6 SegCode; bit 7: take the inner product first; bits 8-15 see SegCode
    uint32_t mat;           // offset (reals) of its coefficients
};
constexpr uint32_t kSegParam = 128;

struct SegSweep {           // consecutive gates of a segment on at most three tile bits
    uint32_t bits;          // the sweep's tile bits, ascending, 8 bits each
    uint32_t g0, g1;        // its operations [g0, g1) of the SegOp table
    uint32_t p0;            // index of its first inner product within the segment
};

// Read at wave-uniform addresses: 32- and 64-bit fields only (the scalar unit
// loads no smaller ones).
struct BatchRec {           // op `s` of one instance
    uint32_t kind;
    uint32_t inst;
    uint32_t item0;         // first item of this record within its step
    uint32_t wgs;           // items (workgroups) of this record
    uint32_t sw0, sw1;      // FWD/ADJ: sweeps [sw0, sw1) of the SegSweep table
    uint32_t ps0, np;       // ADJ: result slots [ps0, ps0 + np) of the slot table, one per inner product
    int tb, W;              // tile: 2^tb amplitudes, window [0, W)
    uint64_t bit[16];       // amplitude-index bit of tile bit i (0 past tb)
    uint64_t need;          // persistent mode: items of this instance that must be done first
};

// H's terms by x mask and parity of |x & z|: coefficients are real (even) or
// imaginary (odd), c the nonzero part including i^{|x&z|}.
struct BatchHGroup {
    uint64_t x;
    uint32_t first, count;
    uint32_t odd, pad;
};
struct BatchHTerm {
    uint64_t z;
    double c;
};

struct BatchInst {
    void *psi;
    void *lam;
    int n;
    int nslots;
    uint32_t wgs;
    uint32_t ngroups;       // Pauli-term groups of H
    uint64_t part_off;      // doubles: partial sums, nslots x wgs
    uint64_t res_off;       // doubles: results, nslots
    uint32_t tg_off;        // first BatchHGroup of H
    uint32_t tt_off;        // first BatchHTerm of H (groups' `first` are relative to it)
    int init_kind;          // 0 |0...0>, 1 |+...+>, 2 copy of init_src
    int pad;
    const void *init_src;
};

struct BatchDev {           // device pointers of one program
    const BatchRec *recs;   // all records, step-major
    const SegOp *ops;
    const uint32_t *slots;
    const SegSweep *sweeps;
    const uint64_t *step_rec;    // nsteps + 1: first record of each step
    const uint64_t *step_item;   // nsteps + 1: first global item of each step (persistent mode)
    const BatchInst *insts;
    const void *mats;
    const BatchHGroup *tg;
    const BatchHTerm *tt;
    double *partials;
    double *results;
    int nsteps;
    int ninst;
};

// 64-bit counters of the persistent launch, each on a cache line of its own:
// next item, error flag, then per instance the items completed.
constexpr size_t kCounterStride = 16;

// Queues step s (one launch over all its records).
cast_status batch_launch_step(const BatchDev &d, cast_dtype dt, int s, uint64_t nitems, size_t lds,
                              hipStream_t st);
// Queues the whole program as one persistent launch: workgroups pull items
// in global order from a counter; an item waits until its instance has
// finished the previous op.  Waits are bounded by spin_limit polls; on
// overrun *err becomes nonzero and every workgroup exits.
cast_status batch_launch_persistent(const BatchDev &d, cast_dtype dt, uint64_t total_items, int grid,
                                    unsigned long long *counters, uint32_t spin_limit, uint32_t chunk, size_t lds,
                                    hipStream_t st);
// Zeroes `n` 64-bit counters with a kernel (graph-capture safe).
cast_status batch_zero(unsigned long long *p, size_t n, hipStream_t st);
// Sets every instance's psi to its initial state (BatchInst::init_kind).
cast_status batch_init_states(const BatchDev &d, cast_dtype dt, hipStream_t st);
// Adds each instance's partial sums into results (fixed order).
cast_status batch_finish(const BatchDev &d, hipStream_t st);

}  // namespace cast
