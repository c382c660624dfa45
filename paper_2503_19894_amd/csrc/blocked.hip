// Segment kernel of the cache-blocked executor: one workgroup per tile (see
// blocked.hpp).  The tile is staged through LDS with the same XOR swizzle as
// the single-gate tile kernel (16-byte chunk c at chunk c ^ hash(c / 16)), so
// coalesced load/store phases and power-of-two-strided group reads are both
// free of bank conflicts.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "blocked.hpp"
#include "internal.hpp"
#include "mfma.hpp"

namespace cast {
namespace {

template <typename R> struct Cx;
template <> struct Cx<double> { using T = double2; };
template <> struct Cx<float> { using T = float2; };
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t swz(uint32_t c) { return c ^ (((c >> 4) ^ (c >> 8)) & 15u); }

template <int S>   // S = log2(amplitudes per 16-byte chunk)
__device__ __forceinline__ uint32_t at(uint32_t y) {
    return (swz(y >> S) << S) | (y & ((1u << S) - 1));
}

// Inserts a zero bit at each position (1 << pos) - 1 = lowmask[i], ascending.
__device__ __forceinline__ uint64_t deposit_bits(uint64_t g, const uint64_t *lowmask, int k) {
    for (int i = 0; i < k; ++i) g = ((g & ~lowmask[i]) << 1) | (g & lowmask[i]);
    return g;
}

// Global index bits of tile position y (without the tile's base): window
// bits keep their place, tile bit w + i is high qubit i.  Like the coset
// enumeration, the L^-1 map and the LDS swizzle, this map is linear over
// GF(2), so the value at y = lane + uniform splits into a per-lane part
// computed once and a wave-uniform part computed on the scalar unit.
__device__ __forceinline__ uint64_t expand(uint32_t y, const BlkSeg &s) {
    uint64_t x = y & ((1u << s.w) - 1);
    const uint32_t hi = y >> s.w;
    for (int i = 0; i < s.nh; ++i)
        if ((hi >> i) & 1u) x |= 1ull << s.qh[i];
    return x;
}

// The plan's tables are read through the constant address space: nothing in
// the kernel writes them, so uniform reads go to the scalar unit.
template <typename T> using CPtr = const __attribute__((address_space(4))) T *;
template <typename T> __device__ __forceinline__ CPtr<T> cptr(const T *p) { return (CPtr<T>)p; }

// Reads a whole record by the widest scalar loads, with one wait.
template <typename T> __device__ __forceinline__ T load_const(CPtr<T> p) {
    typedef uint32_t W __attribute__((ext_vector_type(sizeof(T) >= 64 ? 16 : sizeof(T) / 4)));
    constexpr int C = sizeof(T) / sizeof(W);
    static_assert(C * sizeof(W) == sizeof(T), "whole loads");
    union { W w[C]; T t; } x;
#pragma unroll
    for (int i = 0; i < C; ++i) x.w[i] = reinterpret_cast<CPtr<W>>(p)[i];
    return x.t;
}

template <typename V> __device__ __forceinline__ V cmul(const V &a, const V &b) {
    V r;
    r.x = a.x * b.x - a.y * b.y;
    r.y = a.x * b.y + a.y * b.x;
    return r;
}

// Builds phase tables for the tile at tbase (kind 2): a wave takes 64 entries
// of one table and multiplies its gates' phases, their indices being a part
// fixed by the tile and the entry's bits.
template <typename R, int NT>
__device__ __forceinline__ void build_tables(typename Cx<R>::T *area, CPtr<BlkGate> gates, const BlkGate &g,
                                             CPtr<BlkEnt> ent, CPtr<BlkMember> members, const R *tabs,
                                             uint64_t tbase) {
    using V = typename Cx<R>::T;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint32_t i = wave; i < g.nent; i += NT / 64) {
        const BlkEnt unit = load_const(ent + g.ent + i);
        CPtr<BlkGate> t = gates + unit.u;
        const uint32_t e = unit.a * 64 + lane;
        V p;
        p.x = 1;
        p.y = 0;
        const uint32_t m1 = t->m1;
#pragma unroll 4
        for (uint32_t m = t->m0; m < m1; ++m) {
            CPtr<BlkMember> b = members + m;
            uint32_t j = 0;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (s >= b->k) break;
                const int src = b->src[s];
                j |= (src < 0 ? (uint32_t)((tbase >> b->q[s]) & 1u) : (e >> src) & 1u) << s;
            }
            p = cmul(p, reinterpret_cast<const V *>(tabs + b->tab)[j]);
        }
        if (e < (1u << t->k)) area[t->lds + e] = p;
    }
}

// A run of M phase tables: amplitude y is read once, multiplied by each
// table's phase in order (identity phases are exactly 1), and written once.
// Times 1 an infinite amplitude would turn into NaN, which the single passes
// leave alone, so a result that is NaN is formed again: the amplitude itself
// where the product of its phases is 1, else that product's multiple.  (One
// comparison and a branch of the whole wave: a 27-qubit QFT, complex64, 4.58 ->
// 4.66 ms; 30 qubits, complex128, 62.6 -> 63.1.  With a branch per lane 4.72 and
// 63.7, with a test of every product against 1 4.96 and 66.5.)
// Instantiated per run length so the phase loop is straight code.  A table's
// index is a lane part and a wave-uniform part per iteration.
template <typename R, int S, int NT, int M>
__device__ __forceinline__ void diag_run_m(typename Cx<R>::T *tile, const typename Cx<R>::T *area, CPtr<BlkGate> g,
                                           CPtr<BlkEnt> ent, uint32_t tile_amps) {
    using V = typename Cx<R>::T;
    uint32_t jl[M];
#pragma unroll
    for (int t = 0; t < M; ++t) {
        const BlkGate r = load_const(g + t);
        uint32_t j = r.lds;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < r.k) j |= ((threadIdx.x >> r.pos[i]) & 1u) << i;
        jl[t] = j;
    }
    const uint32_t al = at<S>(threadIdx.x);
    const uint32_t iters = tile_amps > NT ? tile_amps / NT : 1;
    if (threadIdx.x >= tile_amps) return;
    for (uint32_t i = 0; i < iters; ++i) {
        const uint32_t a = al ^ at<S>(i * NT);
        V x = tile[a];
#pragma unroll
        for (int t = 0; t < M; ++t) x = cmul(x, area[jl[t] ^ ent[i * M + t].u]);
        const bool nan = __builtin_isunordered(x.x, x.y);
        if (__builtin_expect(__ballot(nan) != 0, 0)) {
            const V x0 = tile[a];
            V p = area[jl[0] ^ ent[i * M].u];
#pragma unroll
            for (int t = 1; t < M; ++t) p = cmul(p, area[jl[t] ^ ent[i * M + t].u]);
            if (nan) x = p.x == 1 && p.y == 0 ? x0 : cmul(x0, p);
        }
        tile[a] = x;
    }
}

template <typename R, int S, int NT>
__device__ __forceinline__ void diag_run(typename Cx<R>::T *tile, const typename Cx<R>::T *area, CPtr<BlkGate> g,
                                         CPtr<BlkEnt> ent, int run, uint32_t tile_amps) {
    switch (run) {
        case 1: diag_run_m<R, S, NT, 1>(tile, area, g, ent, tile_amps); break;
        case 2: diag_run_m<R, S, NT, 2>(tile, area, g, ent, tile_amps); break;
        case 3: diag_run_m<R, S, NT, 3>(tile, area, g, ent, tile_amps); break;
        case 4: diag_run_m<R, S, NT, 4>(tile, area, g, ent, tile_amps); break;
        case 5: diag_run_m<R, S, NT, 5>(tile, area, g, ent, tile_amps); break;
        case 6: diag_run_m<R, S, NT, 6>(tile, area, g, ent, tile_amps); break;
        case 7: diag_run_m<R, S, NT, 7>(tile, area, g, ent, tile_amps); break;
        default: diag_run_m<R, S, NT, 8>(tile, area, g, ent, tile_amps); break;
    }
}

// The virtual coordinates that the tile's number fixes.
__device__ __forceinline__ uint32_t tile_coords(const BlkGate &g, uint32_t tnum) {
    uint32_t u = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b) u |= ((uint32_t)__popc(tnum & g.par[b]) & 1u) << b;
    return u;
}

// Block gate with 2^D x 2^D blocks: one work item per coset of the span.  The
// virtual coordinates u = L^-1 j of a coset's first position give its block
// (u >> D) and its place in it (u mod 2^D).  The lane's bits of a coset lie on
// tile bits that are no targets, so u is wave-uniform: a wave skips identity
// blocks, and the block's matrix is read with scalar loads.  (With the
// matrices in LDS and a block per lane, a 4 x 4 block cost 16 LDS reads for
// its matrix beside 8 for its amplitudes: 28 qubits, complex128, 0.24 ms more
// per gate and pass.)
template <int D, typename R, int S, int NT>
__device__ __forceinline__ void block_in_tile(typename Cx<R>::T *tile, const BlkGate &g, CPtr<BlkEnt> ent,
                                              CPtr<R> mats, uint32_t tnum) {
    using V = typename Cx<R>::T;
    constexpr int N = 1 << D;
    uint32_t soff[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t o = 0;
#pragma unroll
        for (int i = 0; i < D; ++i)
            if ((c >> i) & 1) o ^= g.span[i];
        soff[c] = o;
    }
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    BlkEnt nxt = load_const(ent + wave);   // wave < kBlkEntsPad
    const uint32_t uuni = tile_coords(g, tnum);
    const uint32_t nl = g.nlane, nq = 1u << g.nuni, amask = g.amask;
    uint32_t al = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i)
        if ((lane >> i) & 1u) al ^= g.lane[i];   // 0 from nlane
    CPtr<R> m0 = mats + g.mat;
    for (uint32_t q = wave; q < nq; q += NT / 64) {
        const BlkEnt e = nxt;
        nxt = load_const(ent + (q + NT / 64 < nq ? q + NT / 64 : q));
        const uint32_t u = uuni ^ e.u, blk = u >> D;
        if (!((amask >> blk) & 1u)) continue;
        uint32_t a0 = e.a;
#pragma unroll
        for (int b = 0; b < D; ++b)
            if ((u >> b) & 1u) a0 ^= soff[1 << b];
        a0 ^= al;
        CPtr<R> m = m0 + (uint32_t)__popc(amask & ((1u << blk) - 1)) * (2 * N * N);
        if (lane >> nl) continue;   // tiles with fewer than 64 cosets of free bits
        V v[N];
#pragma unroll
        for (int c = 0; c < N; ++c) v[c] = tile[a0 ^ soff[c]];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            R ar = 0, ai = 0;
#pragma unroll
            for (int c = 0; c < N; ++c) {
                const R mx = m[2 * (r * N + c)], my = m[2 * (r * N + c) + 1];
                ar = fma(mx, v[c].x, ar);
                ar = fma(-my, v[c].y, ar);
                ai = fma(mx, v[c].y, ai);
                ai = fma(my, v[c].x, ai);
            }
            V o;
            o.x = ar;
            o.y = ai;
            tile[a0 ^ soff[r]] = o;
        }
    }
}

// Dense blocks (d = 4, 5) on the matrix cores: a unit is sixteen cosets of one
// block, one per column, and the wave forms all 2^D output rows as 16 x 16
// tiles (four real products per complex one, as in the single-gate kernels).
// Inputs and matrix (transposed, in LDS for the whole launch) are read one
// k-step ahead.  The outputs are written after the last input is read, so the
// update is in place.
// Rows of a staged matrix's column c are permuted by i ^ matrix_swz(c), so
// that neither the transposing writes (a lane per column) nor the reads (four
// columns, sixteen rows each) meet in a bank.
__device__ __forceinline__ uint32_t matrix_swz(uint32_t c) { return (c & 15u) ^ ((c & 1u) << 4); }

template <int D, typename R, int S, int NT>
__device__ __forceinline__ void mfma_in_tile(typename Cx<R>::T *tile, const BlkGate &g, CPtr<BlkEnt> ent,
                                             const typename Cx<R>::T *mt, uint32_t tnum) {
    using V = typename Cx<R>::T;
    using M = Mfma<R>;
    constexpr int N = 1 << D, T = N / 16, K = N / 4;
    uint32_t sp[D];
#pragma unroll
    for (int i = 0; i < D; ++i) sp[i] = g.span[i];
    auto off = [&](int c) {   // bits 2.. of a row or column: wave-uniform
        uint32_t o = 0;
#pragma unroll
        for (int i = 0; i < D; ++i)
            if ((c >> i) & 1) o ^= sp[i];
        return o;
    };
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t j = lane & 15, kk = lane >> 4;
    BlkEnt nxt = load_const(ent + wave);   // wave < kBlkEntsPad
    const uint32_t uuni = tile_coords(g, tnum);
    const uint32_t nq = 1u << g.nuni, amask = g.amask;
    uint32_t al = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if ((j >> i) & 1u) al ^= g.lane[i];
    // k-row 4 s + kk of the inputs; result rows M::row(lane, v) + 16 t
    uint32_t ain = al, aout = al;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if ((kk >> i) & 1u) {
            ain ^= sp[i];
            aout ^= sizeof(R) == 8 ? sp[i] : sp[2 + i];
        }
    const uint32_t jk = kk * N + ((j ^ matrix_swz(kk)) & (N - 1));   // column kk, row j
    for (uint32_t q = wave; q < nq; q += NT / 64) {
        const BlkEnt e = nxt;
        nxt = load_const(ent + (q + NT / 64 < nq ? q + NT / 64 : q));
        const uint32_t u = uuni ^ e.u, blk = u >> D;
        if (!((amask >> blk) & 1u)) continue;
        const uint32_t a0 = e.a ^ off((int)(u & (N - 1)));
        const V *m0 = mt + g.lds + (uint32_t)__popc(amask & ((1u << blk) - 1)) * (N * N);
        // column 4 s + kk, row 16 t + j
        auto entry = [&](int s, int t) { return m0[(jk ^ (uint32_t)(((4 * s) & 15) ^ (16 * t))) + 4 * s * N]; };
        typename M::acc cr[T], ci[T];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) cr[t][v] = ci[t][v] = 0;
        V x = tile[a0 ^ ain], a[T];
#pragma unroll
        for (int t = 0; t < T; ++t) a[t] = entry(0, t);
#pragma unroll
        for (int s = 0; s < K; ++s) {
            V xn = x, an[T];
            if (s + 1 < K) {
                xn = tile[a0 ^ ain ^ off(4 * (s + 1))];
#pragma unroll
                for (int t = 0; t < T; ++t) an[t] = entry(s + 1, t);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                cr[t] = M::mma(a[t].x, x.x, cr[t]);
                ci[t] = M::mma(a[t].x, x.y, ci[t]);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                cr[t] = M::mma(-a[t].y, x.y, cr[t]);
                ci[t] = M::mma(a[t].y, x.x, ci[t]);
            }
            x = xn;
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (s + 1 < K) a[t] = an[t];
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                V y;
                y.x = cr[t][v];
                y.y = ci[t][v];
                tile[a0 ^ aout ^ off(16 * t + (sizeof(R) == 8 ? 4 * v : v))] = y;
            }
    }
}

// MF: the segment has dense blocks for the matrix cores.  The workgroup then
// holds the tile and every such block's matrix in LDS: two of 512 threads on a
// compute unit where both fit (23 qubits, complex64, two 4-qubit gates: 44 us
// against 53 with one of 1024), else one of 1024.  (Two workgroups that read
// the matrices from global memory ran in step, both loading, then both
// multiplying.)  In a 21-qubit random circuit, complex128, the matrix cores are
// busy for 0.43 of the cycles of the launches with one workgroup, 0.15 of the
// shorter ones with two.
// NB: 16-byte chunks per lane of the tile, 0: any number (tiles of small
// states).  Fixed, so that the wait for a tile's loads need not also wait for
// the stores of the tile before, issued after them.
template <typename R, int NT, bool MF, int NB>
__global__ void __launch_bounds__(NT, 4) k_blocked(R *__restrict__ psi_r, const R *__restrict__ mats_g,
                                                const R *__restrict__ tabs, const BlkGate *__restrict__ gates_g,
                                                const BlkEnt *__restrict__ ent_g,
                                                const BlkMember *__restrict__ members_g, BlkSeg s) {
    using V = typename Cx<R>::T;
    constexpr int S = sizeof(V) == 16 ? 0 : 1;
    constexpr int B = NB ? NB : (int)(kBlkTileBytes / 16) / NT;
    extern __shared__ u4 lds16[];
    V *tile = reinterpret_cast<V *>(lds16);
    const uint32_t tile_amps = 1u << s.tb;
    V *area = tile + tile_amps;
    CPtr<BlkGate> gates = cptr(gates_g);
    CPtr<BlkEnt> ent = cptr(ent_g);
    CPtr<BlkMember> members = cptr(members_g);
    CPtr<R> mats = cptr(mats_g);
    V *mt = area + s.lds_tabs / sizeof(V);
    if (MF) {
        // dense blocks transposed: entry (i, c) at c * 2^d + (i ^ matrix_swz(c))
        for (uint32_t gi = s.g0; gi < s.g1; ++gi) {
            const BlkGate g = load_const(gates + gi);
            if (g.kind != 1 || g.d < 4) continue;
            const V *src = reinterpret_cast<const V *>(mats_g + g.mat);
            const int d = g.d;
            const uint32_t n2 = (1u << d) - 1, count = (uint32_t)__popc(g.amask) << (2 * d);
            for (uint32_t e = threadIdx.x; e < count; e += NT) {
                const uint32_t c = e & n2, i = (e >> d) & n2;
                mt[g.lds + ((e >> (2 * d)) << (2 * d)) + (c << d) + (i ^ (matrix_swz(c) & n2))] = src[e];
            }
        }
    }
    u4 *p16 = reinterpret_cast<u4 *>(psi_r);
    const uint32_t chunks = tile_amps >> S;
    const uint64_t glane = expand(threadIdx.x << S, s) >> S;
    const uint32_t slane = swz(threadIdx.x);
    // One chunk per lane and slot (nb slots; a tile of fewer than NT chunks
    // leaves lanes idle).  The next tile's loads are issued before this tile's
    // gates and wait in registers, so a workgroup always has a tile in flight.
    const int nb = NB ? NB : chunks > NT ? (int)(chunks / NT) : 1;
    const bool mine = NB || threadIdx.x < chunks;
    auto base_of = [&](uint64_t t) { return p16 + (deposit_bits(t << s.w, s.hlowmask, s.nh) >> S) + glane; };
    uint64_t uoff[B];   // uniform
#pragma unroll
    for (int u = 0; u < B; ++u) uoff[u] = expand((uint32_t)(u * NT) << S, s) >> S;
    u4 nxt[B];
    auto load_ahead = [&](uint64_t t) {
        const u4 *src = base_of(t);
        if (!mine) return;
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (u < nb) nxt[u] = __builtin_nontemporal_load(src + uoff[u]);
    };
    load_ahead(blockIdx.x);   // gridDim.x <= ntiles
    for (uint64_t t = blockIdx.x; t < s.ntiles; t += gridDim.x) {
        const uint64_t tbase = deposit_bits(t << s.w, s.hlowmask, s.nh);
        u4 *base16 = p16 + (tbase >> S) + glane;
        // ---- load (chunk c = c0 + lane)
        if (mine) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (u < nb) lds16[slane ^ swz(u * NT)] = nxt[u];
        }
        // ---- the segment's operations (a run of tables counts as one), in
        // order.  The first tables are built before the next tile's loads are
        // issued: loads return in order, so a phase read after them would wait
        // for them.
        uint32_t gi = s.g0;
        BlkGate g = load_const(gates + gi);
        if (g.kind == 2) {
            build_tables<R, NT>(area, gates, g, ent, members, tabs, tbase);
            g = load_const(gates + ++gi);   // a table of it
        }
        if (t + gridDim.x < s.ntiles) load_ahead(t + gridDim.x);
        __syncthreads();
        while (gi < s.g1) {
            CPtr<BlkEnt> e = ent + g.ent;
            if (g.kind == 0) {
                diag_run<R, S, NT>(tile, area, gates + gi, e, g.run, tile_amps);
                gi += (uint32_t)g.run;
            } else {
                if (g.kind == 2) {
                    build_tables<R, NT>(area, gates, g, ent, members, tabs, tbase);
                } else {
                    const uint32_t tnum = (uint32_t)t;
                    switch (g.d) {
                        case 1: block_in_tile<1, R, S, NT>(tile, g, e, mats, tnum); break;
                        case 2: block_in_tile<2, R, S, NT>(tile, g, e, mats, tnum); break;
                        case 4: if (MF) mfma_in_tile<4, R, S, NT>(tile, g, e, mt, tnum); break;
                        case 5: if (MF) mfma_in_tile<5, R, S, NT>(tile, g, e, mt, tnum); break;
                        default: block_in_tile<3, R, S, NT>(tile, g, e, mats, tnum); break;
                    }
                }
                ++gi;
            }
            if (gi < s.g1) g = load_const(gates + gi);
            __syncthreads();
        }
        // ---- store
        if (NB) {
            u4 out[B];
#pragma unroll
            for (int u = 0; u < B; ++u) out[u] = lds16[slane ^ swz(u * NT)];
#pragma unroll
            for (int u = 0; u < B; ++u) __builtin_nontemporal_store(out[u], base16 + uoff[u]);
        } else if (mine) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (u < nb) __builtin_nontemporal_store(lds16[slane ^ swz(u * NT)], base16 + uoff[u]);
        }
        __syncthreads();   // the next tile overwrites LDS
    }
}

template <typename R, int NT, bool MF, int NB>
hipError_t launch_nb(R *psi, const BlkPtrs &p, const BlkSeg &s, uint32_t grid, size_t lds, hipStream_t stream) {
    static const hipError_t attr = hipFuncSetAttribute((const void *)k_blocked<R, NT, MF, NB>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kBlkMaxLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((k_blocked<R, NT, MF, NB>), dim3(grid), dim3(NT), lds, stream, psi, (const R *)p.mats,
                       (const R *)p.tabs, p.gates, p.ent, p.members, s);
    return hipGetLastError();
}

// Whole and half tiles have kernels of their own at the workgroup sizes in use
// (half: complex64 below the largest tile, and two workgroups with matrices).
template <typename R, int NT, bool MF>
hipError_t launch_nt(R *psi, const BlkPtrs &p, const BlkSeg &s, uint32_t grid, size_t lds, hipStream_t stream) {
    constexpr int B = (int)(kBlkTileBytes / 16) / NT;
    const size_t tile = (2 * sizeof(R)) << s.tb;
    if constexpr (MF || NT == 512) {
        if (tile == kBlkTileBytes) return launch_nb<R, NT, MF, B>(psi, p, s, grid, lds, stream);
        if (tile == kBlkTileBytes / 2) return launch_nb<R, NT, MF, B / 2>(psi, p, s, grid, lds, stream);
    }
    if constexpr (MF && NT == 512) return hipErrorInvalidValue;   // at least half a tile
    else return launch_nb<R, NT, MF, 0>(psi, p, s, grid, lds, stream);
}

template <typename R>
hipError_t launch_r(R *psi, const BlkPtrs &p, const BlkSeg &s, uint32_t grid, size_t lds,
                    hipStream_t stream) {
    if (s.lds_mats)
        return s.nt == 512 ? launch_nt<R, 512, true>(psi, p, s, grid, lds, stream)
                           : launch_nt<R, kGroupThreads, true>(psi, p, s, grid, lds, stream);
    switch (s.nt) {
        case 256: return launch_nt<R, 256, false>(psi, p, s, grid, lds, stream);
        case 512: return launch_nt<R, 512, false>(psi, p, s, grid, lds, stream);
        default: return launch_nt<R, 1024, false>(psi, p, s, grid, lds, stream);
    }
}

}  // namespace

int blocked_threads(cast_dtype dt, int tb) {
    int nt = tuning().blocked_threads[dt];   // (an environment variable's may be any number)
    if (nt != 256 && nt != 512) nt = 1024;
    while (nt > 256 && ((size_t)1 << tb) < (size_t)nt) nt >>= 1;   // at least one amplitude per thread
    return nt;
}

cast_status launch_blocked(void *psi, cast_dtype dt, const BlkPtrs &p, const BlkSeg &s, hipStream_t stream) {
    const size_t tile = ((size_t)1 << s.tb) * amp_bytes(dt), lds = tile + s.lds_tabs + s.lds_mats;
    if (tile > kBlkTileBytes || lds > kBlkMaxLds) return fail(CAST_EUNSUPPORTED, "tile and gate tables exceed a compute unit's LDS");
    // two workgroups per compute unit (one with matrices in LDS; their LDS
    // allows no more), each looping over tiles with the next one's loads in
    // flight
    uint64_t grid = s.ntiles;
    const uint64_t cap = std::min<uint64_t>(tuning().max_grid[dt], s.nt == kGroupThreads && s.lds_mats ? 256 : 512);
    if (grid > cap) grid = cap;
    const hipError_t e = dt == CAST_C128 ? launch_r<double>((double *)psi, p, s, (uint32_t)grid, lds, stream)
                                         : launch_r<float>((float *)psi, p, s, (uint32_t)grid, lds, stream);
    if (e != hipSuccess) return fail(CAST_EHIP, std::string("blocked pass launch: ") + hipGetErrorString(e));
    return CAST_OK;
}

}  // namespace cast
