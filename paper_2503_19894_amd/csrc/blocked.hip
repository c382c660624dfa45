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

// Builds phase tables for the tile at tbase (kind 2): a wave takes 64 entries
// of one table and multiplies its gates' phases, their indices being a part
// fixed by the tile and the entry's bits.
template <typename R, int NT>
__device__ __forceinline__ void build_tables(typename Cx<R>::T *area, CPtr<BlkGate> gates, CPtr<BlkGate> g,
                                             CPtr<BlkEnt> ent, CPtr<BlkMember> members, const R *tabs,
                                             uint64_t tbase) {
    using V = typename Cx<R>::T;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (uint32_t i = wave; i < g->nent; i += NT / 64) {
        CPtr<BlkGate> t = gates + ent[g->ent + i].u;
        const uint32_t e = ent[g->ent + i].a * 64 + lane;
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
            const V z = reinterpret_cast<const V *>(tabs + b->tab)[j];
            const R re = p.x * z.x - p.y * z.y;
            p.y = p.x * z.y + p.y * z.x;
            p.x = re;
        }
        if (e < (1u << t->k)) area[t->lds + e] = p;
    }
}

// A run of M phase tables: amplitude y is read once, multiplied by each
// table's phase in order (identity phases are exactly 1), and written once.
// Instantiated per run length so the phase loop is straight code.  A table's
// index is a lane part and a wave-uniform part per iteration.
template <typename R, int S, int NT, int M>
__device__ __forceinline__ void diag_run_m(typename Cx<R>::T *tile, const typename Cx<R>::T *area, CPtr<BlkGate> g,
                                           CPtr<BlkEnt> ent, uint32_t tile_amps) {
    using V = typename Cx<R>::T;
    uint32_t jl[M], e0[M];
#pragma unroll
    for (int t = 0; t < M; ++t) {
        uint32_t j = g[t].lds;
        for (int i = 0; i < g[t].k; ++i) j |= ((threadIdx.x >> g[t].tpos[i]) & 1u) << i;
        jl[t] = j;
        e0[t] = g[t].ent;
    }
    const uint32_t al = at<S>(threadIdx.x);
    const uint32_t iters = tile_amps > NT ? tile_amps / NT : 1;
    if (threadIdx.x >= tile_amps) return;
    for (uint32_t i = 0; i < iters; ++i) {
        const uint32_t a = al ^ at<S>(i * NT);
        V x = tile[a];
#pragma unroll
        for (int t = 0; t < M; ++t) {
            const V ph = area[jl[t] ^ ent[e0[t] + i].u];
            const R re = x.x * ph.x - x.y * ph.y;
            const R im = x.x * ph.y + x.y * ph.x;
            x.x = re;
            x.y = im;
        }
        tile[a] = x;
    }
}

template <typename R, int S, int NT>
__device__ __forceinline__ void diag_run(typename Cx<R>::T *tile, const typename Cx<R>::T *area, CPtr<BlkGate> g,
                                         CPtr<BlkEnt> ent, uint32_t tile_amps) {
    switch (g->run) {
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

// Block gate with 2^D x 2^D blocks: one work item per coset of the span.  The
// virtual coordinates u = L^-1 j of a coset's first position give its block
// (u >> D) and its place in it (u mod 2^D).  The lane's bits of a coset lie on
// tile bits that are no targets, so u is wave-uniform: a wave skips identity
// blocks, and the block's matrix is read with scalar loads.  (With the
// matrices in LDS and a block per lane, a 4 x 4 block cost 16 LDS reads for
// its matrix beside 8 for its amplitudes: 28 qubits, complex128, 0.24 ms more
// per gate and pass.)
template <int D, typename R, int S, int NT>
__device__ __forceinline__ void block_in_tile(typename Cx<R>::T *tile, CPtr<BlkGate> g, CPtr<BlkEnt> ent,
                                              CPtr<R> mats, uint64_t tbase) {
    using V = typename Cx<R>::T;
    constexpr int N = 1 << D;
    uint32_t soff[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
        uint32_t o = 0;
#pragma unroll
        for (int i = 0; i < D; ++i)
            if ((c >> i) & 1) o ^= at<S>(g->span[i]);
        soff[c] = o;
    }
    uint32_t uuni = 0;   // targets outside the tile
    for (int q = 0; q < g->k; ++q)
        if (g->tpos[q] < 0 && ((tbase >> g->q[q]) & 1u)) uuni ^= g->colv[q];
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nl = g->nlane, nq = 1u << g->nuni, amask = g->amask;
    const uint64_t lanepos = g->lanepos;
    uint32_t al = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const uint32_t bit = at<S>(1u << ((lanepos >> (8 * i)) & 255u));
        if (i < (int)nl && ((lane >> i) & 1u)) al ^= bit;
    }
    CPtr<R> m0 = mats + g->mat;
    CPtr<BlkEnt> e0 = ent + g->ent;
    for (uint32_t q = wave; q < nq; q += NT / 64) {
        const uint32_t u = uuni ^ e0[q].u, blk = u >> D;
        if (!((amask >> blk) & 1u)) continue;
        uint32_t a0 = e0[q].a;
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
template <int D, typename R, int S, int NT>
__device__ __forceinline__ void mfma_in_tile(typename Cx<R>::T *tile, CPtr<BlkGate> g, CPtr<BlkEnt> ent,
                                             const typename Cx<R>::T *mt, uint64_t tbase) {
    using V = typename Cx<R>::T;
    using M = Mfma<R>;
    constexpr int N = 1 << D, T = N / 16, K = N / 4;
    uint32_t sp[D];
#pragma unroll
    for (int i = 0; i < D; ++i) sp[i] = at<S>(g->span[i]);
    auto off = [&](int c) {   // bits 2.. of a row or column: wave-uniform
        uint32_t o = 0;
#pragma unroll
        for (int i = 0; i < D; ++i)
            if ((c >> i) & 1) o ^= sp[i];
        return o;
    };
    uint32_t uuni = 0;
    for (int q = 0; q < g->k; ++q)
        if (g->tpos[q] < 0 && ((tbase >> g->q[q]) & 1u)) uuni ^= g->colv[q];
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t j = lane & 15, kk = lane >> 4;
    const uint32_t nq = 1u << g->nuni, amask = g->amask;
    const uint64_t lanepos = g->lanepos;
    uint32_t al = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if ((j >> i) & 1u) al ^= at<S>(1u << ((lanepos >> (8 * i)) & 255u));
    // k-row 4 s + kk of the inputs; result rows M::row(lane, v) + 16 t
    uint32_t ain = al, aout = al;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if ((kk >> i) & 1u) {
            ain ^= sp[i];
            aout ^= sizeof(R) == 8 ? sp[i] : sp[2 + i];
        }
    const V *m0 = mt + g->lds + kk * N + j;   // column kk, row j
    CPtr<BlkEnt> e0 = ent + g->ent;
    for (uint32_t q = wave; q < nq; q += NT / 64) {
        const uint32_t u = uuni ^ e0[q].u, blk = u >> D;
        if (!((amask >> blk) & 1u)) continue;
        const uint32_t a0 = e0[q].a ^ off((int)(u & (N - 1)));
        const V *m = m0 + (uint32_t)__popc(amask & ((1u << blk) - 1)) * (N * N);
        typename M::acc cr[T], ci[T];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) cr[t][v] = ci[t][v] = 0;
        V x = tile[a0 ^ ain], a[T];
#pragma unroll
        for (int t = 0; t < T; ++t) a[t] = m[16 * t];
#pragma unroll
        for (int s = 0; s < K; ++s) {
            V xn = x, an[T];
            if (s + 1 < K) {
                xn = tile[a0 ^ ain ^ off(4 * (s + 1))];
#pragma unroll
                for (int t = 0; t < T; ++t) an[t] = m[4 * (s + 1) * N + 16 * t];
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

// MF: the segment has dense blocks for the matrix cores.  One workgroup of
// 1024 threads per compute unit then holds the tile and every such block's
// matrix in LDS.  (Two workgroups that read the matrices from global memory
// ran in step, both loading, then both multiplying: 24 passes of 4- and
// 5-qubit gates on 26 qubits, complex64, 5.2 ms.)
template <typename R, int NT, bool MF>
__global__ void __launch_bounds__(NT, 4) k_blocked(R *__restrict__ psi_r, const R *__restrict__ mats_g,
                                                const R *__restrict__ tabs, const BlkGate *__restrict__ gates_g,
                                                const BlkEnt *__restrict__ ent_g,
                                                const BlkMember *__restrict__ members_g, BlkSeg s) {
    using V = typename Cx<R>::T;
    constexpr int S = sizeof(V) == 16 ? 0 : 1;
    constexpr int B = 4096 / NT;               // chunks per lane of a 64 KiB tile
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
        // dense blocks transposed: entry (i, c) at c * 2^d + i
        for (uint32_t gi = s.g0; gi < s.g1; ++gi) {
            CPtr<BlkGate> g = gates + gi;
            if (g->kind != 1 || g->d < 4) continue;
            const V *src = reinterpret_cast<const V *>(mats_g + g->mat);
            const int d = g->d;
            const uint32_t n2 = (1u << d) - 1, count = (uint32_t)__popc(g->amask) << (2 * d);
            for (uint32_t e = threadIdx.x; e < count; e += NT)
                mt[g->lds + ((e >> (2 * d)) << (2 * d)) + ((e & n2) << d) + ((e >> d) & n2)] = src[e];
        }
    }
    u4 *p16 = reinterpret_cast<u4 *>(psi_r);
    const uint32_t chunks = tile_amps >> S;
    const uint64_t glane = expand(threadIdx.x << S, s) >> S;
    const uint32_t slane = swz(threadIdx.x);
    // One chunk per lane and slot when the tile is B * NT chunks (the default
    // sizes): the next tile's loads are then issued before this tile's gates
    // and wait in registers, so a workgroup always has a tile in flight.
    const bool ahead = chunks == B * NT;
    auto base_of = [&](uint64_t t) { return p16 + (deposit_bits(t << s.w, s.hlowmask, s.nh) >> S) + glane; };
    uint64_t uoff[B];   // uniform
#pragma unroll
    for (int u = 0; u < B; ++u) uoff[u] = expand((uint32_t)(u * NT) << S, s) >> S;
    u4 nxt[B];
    if (ahead) {
        const u4 *src = base_of(blockIdx.x);   // gridDim.x <= ntiles
#pragma unroll
        for (int u = 0; u < B; ++u) nxt[u] = __builtin_nontemporal_load(src + uoff[u]);
    }
    for (uint64_t t = blockIdx.x; t < s.ntiles; t += gridDim.x) {
        const uint64_t tbase = deposit_bits(t << s.w, s.hlowmask, s.nh);
        u4 *base16 = p16 + (tbase >> S) + glane;
        // ---- load (chunk c = c0 + lane)
        if (ahead) {
#pragma unroll
            for (int u = 0; u < B; ++u) lds16[slane ^ swz(u * NT)] = nxt[u];
        } else {
            for (uint32_t c = threadIdx.x; c < chunks; c += NT)
                lds16[swz(c)] = __builtin_nontemporal_load(base16 + (expand((c - threadIdx.x) << S, s) >> S));
        }
        // ---- the segment's operations (a run of tables counts as one), in
        // order.  The first tables are built before the next tile's loads are
        // issued: loads return in order, so a phase read after them would wait
        // for them.
        uint32_t gi = s.g0;
        if (gates[gi].kind == 2) {
            build_tables<R, NT>(area, gates, gates + gi, ent, members, tabs, tbase);
            ++gi;
        }
        if (ahead && t + gridDim.x < s.ntiles) {
            const u4 *src = base_of(t + gridDim.x);
#pragma unroll
            for (int u = 0; u < B; ++u) nxt[u] = __builtin_nontemporal_load(src + uoff[u]);
        }
        __syncthreads();
        while (gi < s.g1) {
            CPtr<BlkGate> g = gates + gi;
            if (g->kind == 0) {
                diag_run<R, S, NT>(tile, area, g, ent, tile_amps);
                gi += (uint32_t)g->run;
            } else {
                if (g->kind == 2) {
                    build_tables<R, NT>(area, gates, g, ent, members, tabs, tbase);
                } else {
                    switch (g->d) {
                        case 1: block_in_tile<1, R, S, NT>(tile, g, ent, mats, tbase); break;
                        case 2: block_in_tile<2, R, S, NT>(tile, g, ent, mats, tbase); break;
                        case 4: if (MF) mfma_in_tile<4, R, S, NT>(tile, g, ent, mt, tbase); break;
                        case 5: if (MF) mfma_in_tile<5, R, S, NT>(tile, g, ent, mt, tbase); break;
                        default: block_in_tile<3, R, S, NT>(tile, g, ent, mats, tbase); break;
                    }
                }
                ++gi;
            }
            __syncthreads();
        }
        // ---- store
        if (ahead) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                __builtin_nontemporal_store(lds16[slane ^ swz(u * NT)], base16 + uoff[u]);
        } else {
            for (uint32_t c = threadIdx.x; c < chunks; c += NT)
                __builtin_nontemporal_store(lds16[swz(c)], base16 + (expand((c - threadIdx.x) << S, s) >> S));
        }
        __syncthreads();   // the next tile overwrites LDS
    }
}

template <typename R, int NT, bool MF>
hipError_t launch_nt(R *psi, const BlkPtrs &p, const BlkSeg &s, uint32_t grid, size_t lds, hipStream_t stream) {
    static const hipError_t attr = hipFuncSetAttribute((const void *)k_blocked<R, NT, MF>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kBlkMaxLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((k_blocked<R, NT, MF>), dim3(grid), dim3(NT), lds, stream, psi, (const R *)p.mats,
                       (const R *)p.tabs, p.gates, p.ent, p.members, s);
    return hipGetLastError();
}

template <typename R>
hipError_t launch_r(R *psi, const BlkPtrs &p, const BlkSeg &s, uint32_t grid, size_t lds,
                    hipStream_t stream) {
    if (s.lds_mats) return launch_nt<R, kGroupThreads, true>(psi, p, s, grid, lds, stream);
    switch (s.nt) {
        case 256: return launch_nt<R, 256, false>(psi, p, s, grid, lds, stream);
        case 512: return launch_nt<R, 512, false>(psi, p, s, grid, lds, stream);
        default: return launch_nt<R, 1024, false>(psi, p, s, grid, lds, stream);
    }
}

}  // namespace

int blocked_threads(cast_dtype dt, int tb) {
    int nt = tuning().blocked_threads[dt];
    while (nt > 256 && ((size_t)1 << tb) < (size_t)nt) nt >>= 1;   // at least one amplitude per thread
    return nt;
}

cast_status launch_blocked(void *psi, cast_dtype dt, const BlkPtrs &p, const BlkSeg &s, hipStream_t stream) {
    const size_t lds = ((size_t)1 << s.tb) * amp_bytes(dt) + s.lds_tabs + s.lds_mats;
    if (lds > kBlkMaxLds) return fail(CAST_EUNSUPPORTED, "tile and gate tables exceed a compute unit's LDS");
    // two workgroups per compute unit (one with matrices in LDS; their LDS
    // allows no more), each looping over tiles with the next one's loads in
    // flight
    uint64_t grid = s.ntiles;
    const uint64_t cap = std::min<uint64_t>(tuning().max_grid[dt], s.lds_mats ? 256 : 512);
    if (grid > cap) grid = cap;
    const hipError_t e = dt == CAST_C128 ? launch_r<double>((double *)psi, p, s, (uint32_t)grid, lds, stream)
                                         : launch_r<float>((float *)psi, p, s, (uint32_t)grid, lds, stream);
    if (e != hipSuccess) return fail(CAST_EHIP, std::string("blocked pass launch: ") + hipGetErrorString(e));
    return CAST_OK;
}

}  // namespace cast
