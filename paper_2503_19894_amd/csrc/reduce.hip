// Pauli-string reductions and Pauli-sum application for gfx950.
//
// A Pauli string is P = i^{|x&z|} X^x Z^z (bit q of x/z gives qubit q's
// letter), so (P psi)[y ^ x] = i^{|x&z|} (-1)^{|z&y|} psi[y] and
//   <a|P|b> = i^{|x&z|} * S(x, z),  S(x, z) = sum_y conj(a[y^x]) (-1)^{|z&y|} b[y].
// k_pauli_inner computes S of one string between two states, k_expval the
// weighted sum of many strings on one state, k_expval_flip that of strings with
// one x mask; all accumulate products in FP64
// (complex64 inputs are promoted per product).  Reduction order is fixed
// (grid-stride partials, wave shuffles, LDS tree, then one finishing block),
// so results are bitwise reproducible for a given n.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"
#include "reduce.hpp"

namespace cast {

template <typename R> struct AmpR;
template <> struct AmpR<double> { using T = double2; };
template <> struct AmpR<float> { using T = float2; };

constexpr int kRedThreads = 256;
constexpr int kRedMaxBlocks = 1024;
static_assert((size_t)kRedMaxBlocks * 2 <= kReduceScratch, "partials of pauli_inner");

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <typename R>
__global__ void __launch_bounds__(kRedThreads) k_pauli_inner(const R *__restrict__ a_r, const R *__restrict__ b_r,
                                                            uint64_t N, uint64_t x, uint64_t z,
                                                            double *__restrict__ partial) {
    using V = typename AmpR<R>::T;
    const V *a = reinterpret_cast<const V *>(a_r);
    const V *b = reinterpret_cast<const V *>(b_r);
    double re = 0.0, im = 0.0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t y = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; y < N; y += stride) {
        const V av = a[y ^ x];
        const V bv = b[y];
        const double ar = av.x, ai = av.y, br = bv.x, bi = bv.y;
        const double pr = ar * br + ai * bi;
        const double pi = ar * bi - ai * br;
        const bool neg = __popcll(z & y) & 1;
        re += neg ? -pr : pr;
        im += neg ? -pi : pi;
    }
    __shared__ double red[kRedThreads / 64][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    re = wave_sum(re);
    im = wave_sum(im);
    if (lane == 0) {
        red[wave][0] = re;
        red[wave][1] = im;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = 0.0;
        for (int w = 0; w < kRedThreads / 64; ++w) s += red[w][threadIdx.x];
        partial[(size_t)blockIdx.x * 2 + threadIdx.x] = s;
    }
}

// Block i: out[v] = sum over rows of partial[row][v], v < nvals, fixed order, of
// the i-th set of partials; its results lie i sets before the first's.
__global__ void __launch_bounds__(kRedThreads) k_finish(const double *__restrict__ partial, int rows, int nvals,
                                                       double *__restrict__ out) {
    __shared__ double red[kRedThreads];
    partial += (size_t)blockIdx.x * rows * nvals;
    out -= (size_t)blockIdx.x * nvals;
    for (int v = 0; v < nvals; ++v) {
        double s = 0.0;
        for (int b = threadIdx.x; b < rows; b += blockDim.x) s += partial[(size_t)b * nvals + v];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int w = blockDim.x / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) out[v] = red[0];
        __syncthreads();
    }
}

static int red_blocks(int n) {
    const uint64_t N = 1ull << n;
    uint64_t b = (N + kRedThreads * 4 - 1) / (kRedThreads * 4);
    if (b > kRedMaxBlocks) b = kRedMaxBlocks;
    if (b < 1) b = 1;
    return (int)b;
}

size_t inner_partials(int n) { return 2 * (size_t)red_blocks(n); }

static cast_status reduce_error() {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CAST_EHIP, std::string("reduction launch: ") + hipGetErrorString(e));
    return CAST_OK;
}

cast_status pauli_inner(const void *a, const void *b, int n, cast_dtype dt, uint64_t x, uint64_t z, double *partials,
                        hipStream_t s) {
    const int blocks = red_blocks(n);
    const uint64_t N = 1ull << n;
    if (dt == CAST_C128)
        hipLaunchKernelGGL(k_pauli_inner<double>, dim3(blocks), dim3(kRedThreads), 0, s, (const double *)a,
                           (const double *)b, N, x, z, partials);
    else
        hipLaunchKernelGGL(k_pauli_inner<float>, dim3(blocks), dim3(kRedThreads), 0, s, (const float *)a,
                           (const float *)b, N, x, z, partials);
    return reduce_error();
}

cast_status finish_inner(const double *partials, int n, int count, double *dev_out, hipStream_t s) {
    hipLaunchKernelGGL(k_finish, dim3(count), dim3(kRedThreads), 0, s, partials, red_blocks(n), 2, dev_out);
    return reduce_error();
}

// ------------------------------------------------------------------ expval
// Sum of Pauli-term expectation values in as few passes over the state as
// possible.  Every term is a real weighted sum over the amplitudes,
//   coeff <psi|P|psi> = sum_y c (-1)^{|z&y|} f(y),
//   f(y) = Re or Im (conj(psi[y^x]) psi[y])   (|x&z| even / odd),
// so all terms whose x masks stay inside one LDS tile share one read of the
// state: a workgroup loads a tile (the low window and up to T - w high
// qubits), keeps its amplitudes in registers and in LDS, forms f once per x
// mask from the LDS partner, and adds every term's signed c f to one FP64
// accumulator per lane.
//   Bound: HBM for a few terms per tile, else the sign and add per (term,
//   amplitude); terms that share an x mask also share one Walsh-Hadamard
//   transform of f over the lane's amplitudes.
//   Split: tiles of 2^12 amplitudes in 512 lanes, two workgroups per CU, so
//   that one loads while the other sums; smaller tiles below 20 qubits, so
//   that the chip has some 256 of them.
//   Measured (ring of ZZ and X terms): 26 qubits, complex128, 7.22 -> 0.95 ms
//   (three reads of the state instead of 30 two-operand passes, 3.4 TB/s);
//   15 qubits, complex64, 0.18 -> 0.04 ms (2 launches instead of 36).
constexpr int kExpPasses = 4, kExpGroups = 32, kExpTerms = 80;
constexpr int kExpGrid = 512;   // workgroups per pass
enum { kExpDiag = 0, kExpTile = 1, kExpGlobal = 2 };

// Argument tables, read at wave-uniform indices: 32- and 64-bit fields only,
// since the scalar unit loads no smaller ones (a byte field costs a vector
// load and its wait per use).
struct ExpTerm {
    double c;
    uint64_t z;
    uint32_t zl;            // z at the tile bits of the lane index
    uint32_t zj;            // z at those above; bits 16-23: bit j is the parity of zj & j
};
struct ExpGroup {
    uint64_t x;             // flipped qubits (kExpGlobal)
    uint32_t xt;            // flipped tile bits
    int mode, odd;          // odd: Im
    int hb;                 // lane amplitude bit that picks one of each pair (y, y ^ x); -1: all
    int t0, t1;
};
struct ExpPass {
    int w, khi;
    int g0, g1;
    uint64_t bit[12];       // amplitude-index bit of tile bit i
};
struct ExpArgs {
    ExpPass pass[kExpPasses];
    ExpGroup grp[kExpGroups];
    ExpTerm term[kExpTerms];
    uint64_t ntiles;
    uint32_t valid;         // amplitudes of a tile that exist (2^n below one tile)
};

__device__ __forceinline__ double flip_sign(double v, uint32_t odd) {
    return __hiloint2double(__double2hiint(v) ^ (int)(odd << 31), __double2loint(v));
}

// sum_j (-1)^{|zj & j|} f_j for every zj at once (Walsh-Hadamard transform)
template <int J>
__device__ __forceinline__ void walsh(double *f) {
#pragma unroll
    for (int b = 1; b < J; b <<= 1)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (j & b) continue;
            const double u = f[j], v = f[j | b];
            f[j] = u + v;
            f[j | b] = u - v;
        }
}

__device__ __forceinline__ double signed_coeff(double c, uint64_t z, uint32_t zl, uint64_t base, uint32_t t) {
    return flip_sign(c, (uint32_t)(__popcll(z & base) + __popc(zl & t)));
}

// One group's contribution for this lane's J amplitudes `own`, with the
// partners at LDS position (t + NT j) ^ xt (MODE kExpTile) or in the state.
// HB: lane amplitude bit that picks one of each pair (y, y ^ x); -1: all of
// them.  A group of several terms transforms f once and reads each term's sum
// off it (its terms come ordered by zj, so every register index is known at
// compile time); a group of one adds the signed values.
template <int NT, int J, int HB, int MODE, typename V>
__device__ __forceinline__ double group_sum(const ExpArgs &a, const ExpGroup &G, const V (&own)[J], const V *tile,
                                            const V *psi, const uint64_t (&yj)[3], uint64_t yt, bool ok,
                                            uint64_t base, uint32_t t) {
    constexpr auto skip = [](int j) { return HB >= 0 && ((j >> (HB < 0 ? 0 : HB)) & 1); };
    V o[J];
    if (MODE == kExpGlobal) {
        // opaque, so that the J addresses are not kept in registers across groups
        uint64_t yx = yt ^ G.x;
        asm volatile("" : "+v"(yx));
#pragma unroll
        for (int j = 0; j < J; ++j) {
            uint64_t y = yx;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if ((j >> i) & 1) y ^= yj[i];
            o[j].x = o[j].y = 0;
            if (ok) o[j] = psi[y];
        }
    }
    double f[J];
    if (MODE == kExpTile) {
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (!skip(j)) o[j] = tile[(t + NT * j) ^ G.xt];
    }
    if (G.odd) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const V &q = MODE == kExpDiag ? own[j] : o[j];
            f[j] = skip(j) ? 0.0 : (double)q.x * (double)own[j].y - (double)q.y * (double)own[j].x;
        }
    } else {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const V &q = MODE == kExpDiag ? own[j] : o[j];
            f[j] = skip(j) ? 0.0 : (double)q.x * (double)own[j].x + (double)q.y * (double)own[j].y;
        }
    }
    if (G.t1 - G.t0 == 1) {
        const ExpTerm &M = a.term[G.t0];
        const uint32_t sj = M.zj >> 16;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (skip(j)) continue;
            const double v = flip_sign(f[j], sj >> j);
            if (__builtin_popcount(j) & 1) s1 += v;
            else s0 += v;
        }
        return signed_coeff(M.c, M.z, M.zl, base, t) * (s0 + s1);
    }
    walsh<J>(f);
    double e = 0.0;
    int m = G.t0;
    const int t1 = G.t1;
#pragma unroll
    for (int j = 0; j < J; ++j)
        for (; m < t1 && (a.term[m].zj & 0xffffu) == (uint32_t)j; ++m)
            e = fma(signed_coeff(a.term[m].c, a.term[m].z, a.term[m].zl, base, t), f[j], e);
    return e;
}

// J amplitudes per lane: tile position of amplitude j is threadIdx.x + NT j.
// Four waves per SIMD at NT = 512 (two workgroups per CU).
template <typename R, int NT, int J>
__global__ void __launch_bounds__(NT, 4) k_expval(const R *__restrict__ psi_r, ExpArgs a,
                                                   double *__restrict__ partial) {
    using V = typename AmpR<R>::T;
    extern __shared__ uint4 exp_lds[];
    V *tile = reinterpret_cast<V *>(exp_lds);
    const V *psi = reinterpret_cast<const V *>(psi_r);
    const ExpPass &P = a.pass[blockIdx.y];
    constexpr int LB = NT == 512 ? 9 : 8;   // tile bits of the lane index
    const uint32_t t = threadIdx.x;
    const int w = P.w, khi = P.khi;
    auto base_of = [&](uint64_t tl) {
        uint64_t y = tl << w;
        for (int i = 0; i < khi; ++i) {
            const uint64_t lm = P.bit[w + i] - 1;
            y = ((y & ~lm) << 1) | (y & lm);
        }
        return y;
    };
    // tile position -> amplitude index: an OR of lane, j and tile parts
    uint64_t yl = 0;
#pragma unroll
    for (int i = 0; i < LB; ++i)
        if ((t >> i) & 1u) yl |= P.bit[i];
    const uint64_t yj[3] = {P.bit[LB], P.bit[LB + 1], P.bit[LB + 2]};
    const bool ok = t < a.valid;
    double e = 0.0;
    for (uint64_t tl = blockIdx.x; tl < a.ntiles; tl += gridDim.x) {
        const uint64_t base = base_of(tl);
        uint64_t yt = base | yl;
        asm volatile("" : "+v"(yt));   // opaque: the J addresses are formed here, not kept in registers
        V own[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            uint64_t y = yt;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if ((j >> i) & 1) y |= yj[i];
            own[j].x = own[j].y = 0;
            if (ok) own[j] = psi[y];
        }
#pragma unroll
        for (int j = 0; j < J; ++j) tile[t + NT * j] = own[j];
        __syncthreads();
        for (int g = P.g0; g < P.g1; ++g) {
            const ExpGroup &G = a.grp[g];
            if (G.mode == kExpDiag) {
                e += group_sum<NT, J, -1, kExpDiag>(a, G, own, tile, psi, yj, yt, ok, base, t);
            } else if (G.mode == kExpGlobal) {
                e += group_sum<NT, J, -1, kExpGlobal>(a, G, own, tile, psi, yj, yt, ok, base, t);
            } else {
                switch (G.hb) {
                    case 0: e += group_sum<NT, J, 0, kExpTile>(a, G, own, tile, psi, yj, yt, ok, base, t); break;
                    case 1: e += group_sum<NT, J, 1, kExpTile>(a, G, own, tile, psi, yj, yt, ok, base, t); break;
                    case 2: e += group_sum<NT, J, 2, kExpTile>(a, G, own, tile, psi, yj, yt, ok, base, t); break;
                    default: e += group_sum<NT, J, -1, kExpTile>(a, G, own, tile, psi, yj, yt, ok, base, t); break;
                }
            }
        }
        __syncthreads();
    }
    e = wave_sum(e);
    double *red = reinterpret_cast<double *>(exp_lds);
    if ((t & 63) == 0) red[t >> 6] = e;
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
        for (int i = 0; i < NT / 64; ++i) s += red[i];
        partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
}

template <typename R, int NT, int J>
static hipError_t launch_expval_j(const void *psi, const ExpArgs &a, dim3 grid, double *partial, hipStream_t s) {
    using V = typename AmpR<R>::T;
    hipLaunchKernelGGL((k_expval<R, NT, J>), grid, dim3(NT), NT * J * sizeof(V), s, (const R *)psi, a, partial);
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_expval(int T, const void *psi, const ExpArgs &a, dim3 grid, double *partial, hipStream_t s) {
    switch (T) {
        case 8: return launch_expval_j<R, 256, 1>(psi, a, grid, partial, s);
        case 9: return launch_expval_j<R, 256, 2>(psi, a, grid, partial, s);
        case 10: return launch_expval_j<R, 256, 4>(psi, a, grid, partial, s);
        case 11: return launch_expval_j<R, 256, 8>(psi, a, grid, partial, s);
        default: return launch_expval_j<R, 512, 8>(psi, a, grid, partial, s);
    }
}

namespace {

// Launches being filled: passes with their tile qubits, groups in x order.
struct ExpPlan {
    const void *psi;
    int n, T, wmin;
    cast_dtype dt;
    double *scratch;
    hipStream_t s;
    ExpArgs a;
    int npass = 0, ng = 0, nt = 0;
    uint64_t need[kExpPasses];   // qubits the pass's x masks flip
    uint8_t pass_of[kExpGroups];
    size_t used = 0;             // partial sums queued so far

    // window w = T - #{q in need: q >= w} of a tile holding `q`, or -1
    int window(uint64_t q) const {
        for (int w = T;;) {
            const int w2 = T - __builtin_popcountll(q >> w);
            if (w2 < wmin) return -1;
            if (w2 == w) return w;
            w = w2;
        }
    }

    cast_status fold(double *out) {
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, s, scratch, (int)used, 1, out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(CAST_EHIP, std::string("expval launch: ") + hipGetErrorString(e));
        return CAST_OK;
    }

    cast_status flush() {
        if (!npass) return CAST_OK;
        // groups in pass order, then each pass's geometry and tile-space masks
        const int LB = T == 12 ? 9 : 8;   // tile bits of the kernel's lane index
        ExpArgs b;
        b.ntiles = 1ull << (n > T ? n - T : 0);
        b.valid = n < T ? 1u << n : 1u << T;
        int g2 = 0, t2 = 0;
        for (int p = 0; p < npass; ++p) {
            ExpPass &P = b.pass[p];
            const int w = window(need[p]);
            P.w = w;
            P.khi = 0;
            int qhi[12];
            for (int q = w; q < n; ++q)
                if ((need[p] >> q) & 1u) qhi[P.khi++] = q;
            for (int i = 0; i < 12; ++i) P.bit[i] = i < w ? 1ull << i : i - w < P.khi ? 1ull << qhi[i - w] : 0;
            auto to_tile = [&](uint64_t m) {
                uint32_t o = (uint32_t)(m & ((1ull << w) - 1));
                for (int i = 0; i < P.khi; ++i) o |= (uint32_t)((m >> qhi[i]) & 1u) << (w + i);
                return o;
            };
            P.g0 = g2;
            for (int g = 0; g < ng; ++g) {
                if (pass_of[g] != p) continue;
                ExpGroup G = a.grp[g];
                G.hb = -1;
                if (G.mode == kExpTile) {
                    G.xt = to_tile(G.x);
                    if (G.xt >> LB) G.hb = 31 - __builtin_clz(G.xt >> LB);
                }
                const int u0 = t2;
                for (int m = G.t0; m < G.t1; ++m) {
                    ExpTerm M = a.term[m];
                    const uint32_t zt = to_tile(M.z);
                    M.zl = zt & ((1u << LB) - 1);
                    M.zj = zt >> LB;
                    for (uint32_t j = 0; j < 8; ++j) M.zj |= (uint32_t)(__builtin_popcount((zt >> LB) & j) & 1) << (16 + j);
                    // bits inside the tile are zl and zj; z keeps the others
                    uint64_t in = (1ull << w) - 1;
                    for (int i = 0; i < P.khi; ++i) in |= 1ull << qhi[i];
                    M.z &= ~in;
                    if (G.hb >= 0) M.c *= 2.0;   // both of a pair give the same value
                    b.term[t2++] = M;
                }
                std::sort(b.term + u0, b.term + t2, [](const ExpTerm &l, const ExpTerm &r) {
                    return (l.zj & 0xffffu) < (r.zj & 0xffffu);
                });
                G.t0 = u0;
                G.t1 = t2;
                b.grp[g2++] = G;
            }
            P.g1 = g2;
        }
        const uint32_t gx = (uint32_t)std::min<uint64_t>(b.ntiles, kExpGrid);
        // a full partial buffer is folded into its first entry
        if (used + (size_t)gx * npass > kReduceScratch) {
            if (cast_status rc = fold(scratch)) return rc;
            used = 1;
        }
        const hipError_t e = dt == CAST_C128
            ? launch_expval<double>(T, psi, b, dim3(gx, npass), scratch + used, s)
            : launch_expval<float>(T, psi, b, dim3(gx, npass), scratch + used, s);
        if (e != hipSuccess) return fail(CAST_EHIP, std::string("expval launch: ") + hipGetErrorString(e));
        used += (size_t)gx * npass;
        npass = ng = nt = 0;
        return CAST_OK;
    }

    // Pass that takes the x mask (opened if needed), -1: the launch is full.
    int place(uint64_t x) {
        if (window(x) < 0 || x == 0) {   // partner outside any tile, or none: any pass
            if (npass == 0) need[npass++] = 0;
            return npass - 1;
        }
        for (int p = 0; p < npass; ++p)
            if (window(need[p] | x) >= 0) {
                need[p] |= x;
                return p;
            }
        if (npass == kExpPasses) return -1;
        need[npass] = x;
        return npass++;
    }
};

}  // namespace

// Strings that share one x mask: the state is streamed once.  Both of a pair
// (y, y ^ x) give the same value, so a lane takes the one with bit hb clear, the
// highest of x, and reads both; if x lies within a wave's amplitudes (below bit
// 6) every lane takes its own, whose partner is in the same lines.
//   Bound: HBM, one read of the state.
//   For a single string, and for strings whose partner lies in no tile: there
//   k_expval reads the state twice, the second time once for each parity of
//   |x & z|, and its 3 KiB of arguments cost a small state 1 us.
//   Split: J items per lane in flight on 2048 workgroups; full sweeps in
//   complex128, 16 bytes per lane each, are as fast with one on 1024 (27 qubits,
//   409 us; four: 435 where the partner is read too), in complex64 they are not
//   (429; four: 240).
//   Measured: one string that flips all of 27 qubits, complex64, 204 us (k_expval
//   453, each amplitude with its partner 383); two with different parities 210
//   (610).
constexpr int kFlipTerms = 16, kFlipBlocks = 2048;
struct FlipArgs {
    double c[kFlipTerms];
    uint64_t z[kFlipTerms];
    uint32_t odd;           // bit m: Im
    int count, hb;          // hb: -1: every amplitude
};

template <typename R, int J>
__global__ void __launch_bounds__(kRedThreads) k_expval_flip(const R *__restrict__ psi_r, uint64_t items, uint64_t x,
                                                            FlipArgs a, double *__restrict__ partial) {
    using V = typename AmpR<R>::T;
    const V *psi = reinterpret_cast<const V *>(psi_r);
    const uint64_t stride = (uint64_t)gridDim.x * kRedThreads;
    const uint64_t low = a.hb < 0 ? ~0ull : (1ull << a.hb) - 1;
    const double c0 = a.c[0];
    const uint64_t z0 = a.z[0];
    double e = 0.0;
    for (uint64_t i0 = (uint64_t)blockIdx.x * kRedThreads + threadIdx.x; i0 < items; i0 += J * stride) {
        V u[J], w[J];
        uint64_t y[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint64_t i = i0 + j * stride;
            y[j] = ((i & ~low) << 1) | (i & low);
            u[j].x = u[j].y = w[j].x = w[j].y = 0;
            if (i < items) {
                u[j] = psi[y[j]];
                w[j] = x == 0 ? u[j] : psi[y[j] ^ x];
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const double ur = u[j].x, ui = u[j].y, wr = w[j].x, wi = w[j].y;
            const double re = wr * ur + wi * ui, im = wr * ui - wi * ur;
            e = fma(flip_sign(c0, (uint32_t)__popcll(z0 & y[j])), a.odd & 1u ? im : re, e);
            for (int m = 1; m < a.count; ++m)
                e = fma(flip_sign(a.c[m], (uint32_t)__popcll(a.z[m] & y[j])), (a.odd >> m) & 1u ? im : re, e);
        }
    }
    __shared__ double red[kRedThreads / 64];
    e = wave_sum(e);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < kRedThreads / 64; ++i) t += red[i];
        partial[blockIdx.x] = t;
    }
}

// i^{|x&z|} S with S = Re, or i Im for an odd power
static double real_coeff(const cast_pauli_term &t) {
    const int pw = __builtin_popcountll(t.xmask & t.zmask) & 3;
    return pw == 1 || pw == 2 ? -t.coeff : t.coeff;
}

static cast_status expval_flip(const void *psi, int n, cast_dtype dt, const cast_pauli_term *terms, size_t n_terms,
                               double *scratch, double *dev_out, hipStream_t s) {
    const uint64_t x = terms[0].xmask;
    const bool pairs = x >> 6, four = pairs || dt == CAST_C64;
    const uint64_t items = 1ull << (pairs ? n - 1 : n);
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(four ? kFlipBlocks : kFlipBlocks / 2,
                                                         (items + 4 * kRedThreads - 1) / (4 * kRedThreads));
    size_t used = 0;
    auto fold = [&](double *out) {
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, s, scratch, (int)used, 1, out);
        return reduce_error();
    };
    for (size_t t = 0; t < n_terms; t += kFlipTerms) {
        if (used + blocks > kReduceScratch) {   // into its first entry
            if (cast_status rc = fold(scratch)) return rc;
            used = 1;
        }
        FlipArgs a{};
        a.count = (int)std::min<size_t>(kFlipTerms, n_terms - t);
        a.hb = pairs ? 63 - __builtin_clzll(x) : -1;
        for (int m = 0; m < a.count; ++m) {
            const cast_pauli_term &p = terms[t + m];
            a.c[m] = pairs ? 2.0 * real_coeff(p) : real_coeff(p);
            a.z[m] = p.zmask;
            a.odd |= (uint32_t)(__builtin_popcountll(p.xmask & p.zmask) & 1) << m;
        }
        auto launch = [&](auto kernel, auto *state) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kRedThreads), 0, s, state, items, x, a, scratch + used);
        };
        if (dt == CAST_C128) launch(four ? k_expval_flip<double, 4> : k_expval_flip<double, 1>, (const double *)psi);
        else launch(four ? k_expval_flip<float, 4> : k_expval_flip<float, 1>, (const float *)psi);
        if (cast_status rc = reduce_error()) return rc;
        used += blocks;
    }
    return fold(dev_out);
}

cast_status expval_sum(const void *psi, int n, cast_dtype dt, const cast_pauli_term *terms, size_t n_terms,
                       uint16_t *order, double *scratch, double *dev_out, hipStream_t s) {
    ExpPlan pl;
    pl.psi = psi;
    pl.n = n;
    pl.dt = dt;
    pl.T = std::min(12, std::max(8, n - 8));
    // low window: runs of 128 bytes; small states sit in the L2 cache, where
    // shorter runs cost nothing and leave more tile bits for the masks
    pl.wmin = std::min(dt == CAST_C64 && pl.T == 12 ? 4 : 3, n);
    pl.scratch = scratch;
    pl.s = s;
    if (std::all_of(terms, terms + n_terms, [&](const cast_pauli_term &t) { return t.xmask == terms[0].xmask; }) &&
        (n_terms == 1 || pl.window(terms[0].xmask) < 0))
        return expval_flip(psi, n, dt, terms, n_terms, scratch, dev_out, s);
    for (size_t i = 0; i < n_terms; ++i) order[i] = (uint16_t)i;
    auto odd_of = [&](size_t i) { return __builtin_popcountll(terms[i].xmask & terms[i].zmask) & 1; };
    // by x mask, the diagonal terms last (they fit every pass), then by parity
    std::sort(order, order + n_terms, [&](uint16_t i, uint16_t j) {
        const uint64_t xi = terms[i].xmask - 1, xj = terms[j].xmask - 1;
        if (xi != xj) return xi < xj;
        const int oi = odd_of(i), oj = odd_of(j);
        return oi != oj ? oi < oj : i < j;
    });
    for (size_t k = 0; k < n_terms;) {
        const uint64_t x = terms[order[k]].xmask;
        const int odd = odd_of(order[k]);
        if (pl.ng == kExpGroups || pl.nt == kExpTerms)
            if (cast_status rc = pl.flush()) return rc;
        int p = pl.place(x);
        if (p < 0) {
            if (cast_status rc = pl.flush()) return rc;
            p = pl.place(x);
        }
        ExpGroup &G = pl.a.grp[pl.ng];
        pl.pass_of[pl.ng++] = (uint8_t)p;
        G.x = x;
        G.xt = 0;
        G.mode = x == 0 ? kExpDiag : pl.window(x) < 0 ? kExpGlobal : kExpTile;
        G.odd = odd;
        G.t0 = pl.nt;
        for (; k < n_terms && pl.nt < kExpTerms && terms[order[k]].xmask == x && odd_of(order[k]) == odd; ++k) {
            const cast_pauli_term &t = terms[order[k]];
            pl.a.term[pl.nt++] = ExpTerm{real_coeff(t), t.zmask, 0, 0};
        }
        G.t1 = pl.nt;
    }
    if (cast_status rc = pl.flush()) return rc;
    return pl.fold(dev_out);
}

// out[y] = sum_groups sum_{m in group} c_m (-1)^{|z_m & (y^x_g)|} psi[y ^ x_g]
// where c_m already includes i^{|x&z|}.  Term table layout (device):
//   groups: {x, first term, term count}, terms: {z, c_re, c_im}.
template <typename R>
__global__ void __launch_bounds__(256) k_apply_pauli_sum(const R *__restrict__ psi_r, R *__restrict__ out_r,
                                                        uint64_t N, const PauliSumGroup *__restrict__ groups,
                                                        int ngroups, const PauliSumTerm *__restrict__ terms) {
    using V = typename AmpR<R>::T;
    const V *psi = reinterpret_cast<const V *>(psi_r);
    V *out = reinterpret_cast<V *>(out_r);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t y = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; y < N; y += stride) {
        double accr = 0.0, acci = 0.0;
        for (int g = 0; g < ngroups; ++g) {
            const uint64_t x = groups[g].x;
            const uint64_t src = y ^ x;
            const V v = psi[src];
            double sr = 0.0, si = 0.0;
            const int t0 = groups[g].first, t1 = t0 + groups[g].count;
            for (int t = t0; t < t1; ++t) {
                const bool neg = __popcll(terms[t].z & src) & 1;
                sr += neg ? -terms[t].cre : terms[t].cre;
                si += neg ? -terms[t].cim : terms[t].cim;
            }
            const double vr = v.x, vi = v.y;
            accr += sr * vr - si * vi;
            acci += sr * vi + si * vr;
        }
        V o;
        o.x = (R)accr;
        o.y = (R)acci;
        out[y] = o;
    }
}

cast_status apply_pauli_sum(const void *psi, void *out, int n, cast_dtype dt, const PauliSumGroup *dgroups,
                            int ngroups, const PauliSumTerm *dterms, hipStream_t s) {
    const uint64_t N = 1ull << n;
    uint64_t grid = (N + 255) / 256;
    if (grid > 8192) grid = 8192;
    if (dt == CAST_C128)
        hipLaunchKernelGGL(k_apply_pauli_sum<double>, dim3(grid), dim3(256), 0, s, (const double *)psi,
                           (double *)out, N, dgroups, ngroups, dterms);
    else
        hipLaunchKernelGGL(k_apply_pauli_sum<float>, dim3(grid), dim3(256), 0, s, (const float *)psi, (float *)out,
                           N, dgroups, ngroups, dterms);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CAST_EHIP, std::string("pauli-sum launch: ") + hipGetErrorString(e));
    return CAST_OK;
}

}  // namespace cast
