// Cache-blocked execution of a fused gate list: several fused gates per HBM
// pass.
//
// Consecutive fused gates are grouped into segments.  A segment has a tile
// qubit set T = [0, w) + H (w >= 4 low "window" qubits and up to tb - w higher
// qubits H, |T| = tb); every non-diagonal gate of the segment mixes only
// amplitudes that differ on T (its block span, the qubits touched by its first
// d virtual basis vectors, lies in T).  A tile is the 2^tb amplitudes that
// agree off T: 2^|H| contiguous runs of 2^w amplitudes.  One workgroup loads a
// tile into LDS, applies the segment's gates in order (block gates by coset of
// their span, diagonal gates elementwise, with the targets outside T read off
// the tile's base index), and writes it back, so a segment costs one read and
// one write of the state however many gates it holds.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/cast.h"

namespace cast {

constexpr int kBlkMaxHigh = 10;    // tile qubits above the window
constexpr int kBlkMaxD = 3;        // largest block dimension applied inside a tile
constexpr int kBlkMinWindow = 4;   // smallest window: runs of >= 16 amplitudes

// One operation inside a tile: a fused gate's blocks, or a run of consecutive
// diagonal gates as phase tables (neighbouring gates multiplied together on
// the host while their union has at most kRunMaxQ qubits).  Read at
// wave-uniform indices: 32- and 64-bit fields only.
struct BlkGate {
    int kind;                // 0 phase table, 1 blocks of 2^d x 2^d
    int k, d;
    int q[8];                // sorted targets
    int tpos[8];             // tile bit of each target, -1 when the target is outside the tile
    // blocks
    uint32_t colv[6];        // virtual coordinates of local index bit s (the columns of L^-1)
    uint32_t span[kBlkMaxD]; // tile offset of virtual basis vector i < d
    uint32_t amask;          // bit b: block b is not the identity (its matrices lie in block order)
    uint32_t nlane, nuni;    // coset bits given by the lane, and by the wave and iteration
    uint64_t lanepos;        // tile bit of lane bit i (8 bits each)
    uint32_t ent;            // entries of the 2^nuni uniform coset parts in the entry table;
                             // phase tables: of the iterations' uniform local indices
    int run;                 // phase tables: tables of the run from here (0 inside a run)
    int tshift;              // first table of a run: log2 of the tables' stride (entries)
    uint32_t area;           // first table of a run: its LDS bytes
    uint64_t mat;            // offset (reals) of the matrices in the fused list's buffer, or of the
                             // run's tables in the plan's table buffer
};
struct BlkEnt {              // uniform part of a coset: virtual coordinates, LDS element; of a phase
    uint32_t u, a;           // table's iteration: local index (u)
};

// LDS of a segment pass: the tile, then the phase tables: all the segment's
// when they fit kBlkAreaBytes (staged once per workgroup), else two areas,
// the run being applied and the next one, staged meanwhile.  Tile and areas
// stay within 80 KiB, so two workgroups share a compute unit's 160 KiB.
constexpr uint32_t kBlkAreaBytes = 16u << 10;
constexpr uint32_t kBlkRunMax = 8;

struct BlkSeg {              // kernel arguments of one segment pass
    uint64_t ntiles;         // 2^(n - tb)
    uint64_t hlowmask[kBlkMaxHigh];  // per high tile qubit (ascending): global index bits below it
    int tb, w, nh;
    int qh[kBlkMaxHigh];     // high tile qubits, ascending
    uint32_t g0, g1;         // operations [g0, g1) of the gate table
    int resident;            // every run's tables stay in LDS
    uint32_t lds_tabs;       // bytes of phase tables in LDS
};

struct BlkPtrs {             // device tables of a plan
    const void *mats, *tabs;
    const BlkGate *gates;
    const BlkEnt *ent;
};

// Workgroup size of a plan with tiles of 2^tb amplitudes (the knob, at most
// one thread per amplitude).
int blocked_threads(cast_dtype dt, int tb);
cast_status launch_blocked(void *psi, cast_dtype dt, const BlkPtrs &p, const BlkSeg &s, int nt, hipStream_t stream);

}  // namespace cast
