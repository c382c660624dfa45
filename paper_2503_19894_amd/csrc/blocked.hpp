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
constexpr int kBlkMaxD = 3;        // largest block dimension of apply_circuit_blocked's segments
constexpr int kGroupMaxD = 5;      // and of apply_circuit's tile groups (matrix cores from 4)
constexpr int kBlkMinWindow = 4;   // smallest window: runs of >= 16 amplitudes

// One operation inside a tile.  Read at wave-uniform indices: 32- and 64-bit
// fields only.
//   kind 0  a phase table over at most kBlkTabBits tile bits.  A stretch of
//           consecutive diagonal gates becomes a run of such tables: the gates'
//           targets outside the tile are fixed per tile, and gates are put
//           together while their targets inside it fit one table, whatever
//           their number; kind 2 multiplies the gates' phases into the tables,
//           per tile, so that an amplitude meets one lookup and one multiply
//           per table instead of per gate.
//   kind 1  a fused gate's blocks of 2^d x 2^d.
//   kind 2  builds the phase tables up to the next kind 2 (one or more runs,
//           as many as the table area holds).
// A record is read whole, in one go, by scalar loads: what the kernel needs of
// a gate is worked out here rather than derived, load by load, for every tile
// (a 27-qubit QFT, complex64, six passes: 5.35 -> 4.66 ms; a 12-qubit random
// circuit in one launch: 41 -> 34 us).
struct alignas(128) BlkGate {
    int kind;
    int d;
    int run;                 // phase table: tables applied together from here (0 inside a run)
    uint32_t nuni, nlane;    // blocks: coset bits given by the wave and iteration, and by the lane
    uint32_t amask;          // blocks: bit b: block b is not the identity (its matrices lie in block order)
    // first entry in LDS: phase table, in the table area, a multiple of its
    // 2^k entries; blocks of d >= 4, in the matrices
    uint32_t lds;
    uint32_t ent, nent;      // its first entry in the entry table; kind 2: its work units there
    uint32_t span[kGroupMaxD];  // blocks: LDS element of virtual basis vector i < d
    uint64_t mat;            // blocks: offset (reals) of the matrices in the fused list's buffer
    union {
        struct {
            uint32_t lane[6];    // blocks: LDS element of lane bit i < nlane
            uint32_t par[6];     // blocks: bit b of the virtual coordinates that the tile fixes is the
                                 // parity of the tile number's bits par[b]
        };
        struct {
            int k;               // phase table: its tile bits
            int pos[8];          // and their places
            uint32_t m0, m1;     // its gates [m0, m1) of the member table
        };
    };
};
static_assert(sizeof(BlkGate) == 128, "two scalar loads of 16 words");
// Entries of an operation: blocks, the 2^nuni <= 64 uniform coset parts; phase
// table, the uniform local index of each iteration over the tile, a run's
// tables side by side.  The work units of kind 2 follow those of every
// operation.  Every wave reads one entry before it knows whether it has work,
// so the table ends in kBlkEntsPad unused ones.  (64 entries for each operation
// whatever it uses made the upload of a fresh list's tables the largest part of
// its first application.)
constexpr uint32_t kBlkEntsPad = 16;
struct BlkEnt {
    uint32_t u, a;           // blocks: virtual coordinates, LDS element; phase table: local index;
                             // kind 2: phase table (gate index), 64-entry slice
};
struct BlkMember {           // a diagonal gate of a phase table
    int k;
    int q[8];                // targets
    int src[8];              // bit of the table's index each comes from, -1: outside the tile
    uint64_t tab;            // offset (reals) of its 2^k phases
};

// LDS of a segment pass: the tile, then the table area; 80 KiB together, so
// two workgroups share a compute unit's 160 KiB.  Tables of 2^7 entries: three
// of them take a QFT run's targets with all other bits of a tile.
constexpr uint32_t kBlkTileBytes = 64u << 10;   // the largest
constexpr uint32_t kBlkAreaBytes = 16u << 10;
constexpr int kBlkTabBits = 7;
// With dense blocks: one workgroup of kGroupThreads and the matrices besides.
constexpr uint32_t kBlkMaxLds = 160u << 10;
constexpr uint32_t kBlkMatBytes = kBlkMaxLds - kBlkTileBytes - kBlkAreaBytes;
constexpr int kGroupThreads = 1024;
constexpr uint32_t kBlkRunMax = 8;

struct BlkSeg {              // kernel arguments of one segment pass
    uint64_t ntiles;         // 2^(n - tb)
    uint64_t hlowmask[kBlkMaxHigh];  // per high tile qubit (ascending): global index bits below it
    int tb, w, nh;
    int qh[kBlkMaxHigh];     // high tile qubits, ascending
    uint32_t g0, g1;         // operations [g0, g1) of the gate table
    uint32_t lds_tabs;       // bytes of the table area
    uint32_t lds_mats;       // bytes of matrices (blocks of d >= 4; 0: none)
    int nt;                  // workgroup size
};

struct BlkPtrs {             // device tables of a plan
    const void *mats, *tabs;
    const BlkGate *gates;
    const BlkEnt *ent;
    const BlkMember *members;
};

// Workgroup size of a plan with tiles of 2^tb amplitudes (the knob, at most
// one thread per amplitude).
int blocked_threads(cast_dtype dt, int tb);
cast_status launch_blocked(void *psi, cast_dtype dt, const BlkPtrs &p, const BlkSeg &s, hipStream_t stream);

}  // namespace cast
