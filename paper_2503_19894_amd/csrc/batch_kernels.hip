// Kernels of the batched adjoint-gradient programs (batch.hpp).
//
// One work item = one workgroup's share (1 / wgs) of one op of one instance.
// The same item routine serves both launch modes: one launch per global step
// (all instances' op s side by side), or one persistent launch in which
// workgroups pull items in global order and wait, per instance, for the
// previous op to finish.
#include <hip/hip_runtime.h>

#include "batch.hpp"
#include "internal.hpp"

namespace cast {

extern __shared__ uint4 batch_lds[];

template <typename R> struct BAmp;
template <> struct BAmp<double> { using T = double2; };
template <> struct BAmp<float> { using T = float2; };

__device__ __forceinline__ uint32_t ins0_32(uint32_t g, int q) {
    const uint32_t lm = (1u << q) - 1;
    return ((g & ~lm) << 1) | (g & lm);
}

// The read-only tables (gate matrices, gate and sweep records) are read
// through the constant address space.  Nothing in a kernel writes them, so
// their loads may use the scalar cache and land in SGPRs.  Through generic
// pointers the compiler must assume that the kernel's own stores to the
// states may alias them, and in a loop over work items (the persistent
// launch) every such load after the first item's stores became a vector load
// into VGPRs: 223 VGPRs instead of 119 for complex128.
template <typename T> using CPtr = const __attribute__((address_space(4))) T *;
template <typename T> __device__ __forceinline__ CPtr<T> cptr(const T *p) { return (CPtr<T>)p; }

__device__ __forceinline__ double block_sum(double v, double *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    return s;
}

// ------------------------------------------------------------------ operations
// On a thread's eight register amplitudes x[j], j over the sweep's three tile
// bits.  Masks and bit positions are template parameters, so every register
// index and sign is known at compile time.
constexpr int par(int v) { return __builtin_popcount(v) & 1; }

// c a + b (NEG: b - c a) with c wave-uniform, in the three-address form: left
// to itself the compiler takes v_fmac, whose result sits in b's register, and
// copies it to a's place after every operation, since all cases of seg_op
// have to leave x[] in the same registers (34 copies per operation).
template <bool NEG>
__device__ __forceinline__ double fma3(double c, double a, double b) {
    double d;
    if (NEG) asm("v_fma_f64 %0, -%1, %2, %3" : "=v"(d) : "s"(c), "v"(a), "v"(b));
    else asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "s"(c), "v"(a), "v"(b));
    return d;
}
template <bool NEG>
__device__ __forceinline__ float fma3(float c, float a, float b) {
    float d;
    if (NEG) asm("v_fma_f32 %0, -%1, %2, %3" : "=v"(d) : "s"(c), "v"(a), "v"(b));
    else asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "s"(c), "v"(a), "v"(b));
    return d;
}

// (p, q) <- (c p - s q, s p + c q) (NEG: the inverse) as three shears,
// t = -s / (1 + c), 0 <= c: in place and three fused operations instead of
// four.
template <bool NEG>
__device__ __forceinline__ void shear(double &p, double &q, double t, double s) {
    p = fma(NEG ? -t : t, q, p);
    q = fma(NEG ? -s : s, p, q);
    p = fma(NEG ? -t : t, q, p);
}

// Pauli rotation (SegCode below 64) with coefficients c, s.  complex128: see
// SegCode.  complex64: the products of an output are rounded in a fixed order
// (contraction off, fused operations written out), so that results do not
// depend on how the compiler contracts them.
template <int X, int Z>
__device__ __forceinline__ void rot(double2 *x, double c, double s) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (X == 0) {
            if (!par(Z & j)) continue;
            const double u = s * x[j].y, v = s * x[j].x;
            x[j].x = fma3<false>(c, x[j].x, -u);
            x[j].y = fma3<false>(c, x[j].y, v);
            continue;
        }
        // x_j <- c x_j - i s P[j][j ^ X] x_{j ^ X},
        // -i P[j][j ^ X] = -i i^{|X & Z|} (-1)^{Z . (j ^ X)}
        constexpr bool flip = __builtin_popcount(X & Z) == 2;
        const int k = j ^ X;
        if (k < j) continue;   // each pair once
        if (par(X & Z)) {
            if (par(Z & j)) shear<true>(x[j].x, x[k].x, c, s), shear<true>(x[j].y, x[k].y, c, s);
            else shear<false>(x[j].x, x[k].x, c, s), shear<false>(x[j].y, x[k].y, c, s);
        } else if (par(Z & k) != (int)flip) {
            shear<false>(x[j].x, x[k].y, c, s), shear<true>(x[j].y, x[k].x, c, s);
        } else {
            shear<true>(x[j].x, x[k].y, c, s), shear<false>(x[j].y, x[k].x, c, s);
        }
    }
}

template <int X, int Z>
__device__ __forceinline__ void rot(float2 *x, float c, float s) {
#pragma clang fp contract(off)
    constexpr bool flip = __builtin_popcount(X & Z) == 2;
    constexpr bool two = __builtin_popcount(X | Z) == 2;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (X == 0) {
            const float u = s * x[j].y, v = s * x[j].x;
            x[j].x = fma3<false>(c, x[j].x, par(Z & j) ? -u : u);
            x[j].y = fma3<false>(c, x[j].y, par(Z & j) ? v : -v);
            continue;
        }
        const int k = j ^ X;
        if (k < j) continue;   // each pair once
        const float2 a = x[j], b = x[k];
        // signs of s in x_j (from x_k) and x_k (from x_j)
        constexpr bool real = par(X & Z);
        const bool nj = par(Z & k) != (int)flip, nk = par(Z & j) != (int)flip;
        if (real && !two) {          // Y
            const float ux = s * b.x, uy = s * b.y, vx = c * b.x, vy = c * b.y;
            x[j].x = fma3<false>(c, a.x, nj ? -ux : ux);
            x[j].y = fma3<false>(c, a.y, nj ? -uy : uy);
            x[k].x = nk ? fma3<true>(s, a.x, vx) : fma3<false>(s, a.x, vx);
            x[k].y = nk ? fma3<true>(s, a.y, vy) : fma3<false>(s, a.y, vy);
        } else if (real) {           // XY, YZ, ...
            const float ux = c * a.x, uy = c * a.y, vx = s * a.x, vy = s * a.y;
            x[j].x = nj ? fma3<true>(s, b.x, ux) : fma3<false>(s, b.x, ux);
            x[j].y = nj ? fma3<true>(s, b.y, uy) : fma3<false>(s, b.y, uy);
            x[k].x = fma3<false>(c, b.x, nk ? -vx : vx);
            x[k].y = fma3<false>(c, b.y, nk ? -vy : vy);
        } else if (!two) {           // X
            const float ux = c * a.x, uy = c * a.y, vx = s * a.x, vy = s * a.y;
            x[j].x = fma3<false>(s, b.y, ux);
            x[j].y = fma3<true>(s, b.x, uy);
            x[k].x = fma3<false>(c, b.x, vy);
            x[k].y = fma3<false>(c, b.y, -vx);
        } else {                     // XX, YY, XZ, ...
            const float sj = nj ? -s : s, sk = nk ? -s : s;
            x[j].x = c * a.x + sj * b.y;
            x[j].y = c * a.y - sj * b.x;
            x[k].x = c * b.x + sk * a.y;
            x[k].y = c * b.y - sk * a.x;
        }
    }
}

// sum_j conj(l[j ^ X]) (-1)^{Z . j} x[j]: its imaginary part, or for odd
// |X & Z| its real part, the one d E / d theta needs.  FP64 products.
template <int X, int Z, typename V>
__device__ __forceinline__ double inner(const V *l, const V *x) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const V a = l[j ^ X];
        const double u = par(X & Z) ? (double)x[j].x : (double)x[j].y;
        const double v = par(X & Z) ? (double)x[j].y : -(double)x[j].x;
        const double ar = par(Z & j) ? -(double)a.x : (double)a.x, ai = par(Z & j) ? -(double)a.y : (double)a.y;
        s0 = fma(ar, u, s0);
        s1 = fma(ai, v, s1);
    }
    return s0 + s1;
}

template <int B, typename V, typename R>
__device__ __forceinline__ void gen1(V *x, CPtr<R> m) {
    const R r00 = m[0], i00 = m[1], r01 = m[2], i01 = m[3], r10 = m[4], i10 = m[5], r11 = m[6], i11 = m[7];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j & (1 << B)) continue;
        const V a = x[j], b = x[j | (1 << B)];
        V y0, y1;
        y0.x = fma(-i01, b.y, fma(r01, b.x, fma(-i00, a.y, r00 * a.x)));
        y0.y = fma(i01, b.x, fma(r01, b.y, fma(i00, a.x, r00 * a.y)));
        y1.x = fma(-i11, b.y, fma(r11, b.x, fma(-i10, a.y, r10 * a.x)));
        y1.y = fma(i11, b.x, fma(r11, b.y, fma(i10, a.x, r10 * a.y)));
        x[j] = y0;
        x[j | (1 << B)] = y1;
    }
}

template <int B, typename V, typename R>
__device__ __forceinline__ void real1(V *x, CPtr<R> m) {
    const R m00 = m[0], m01 = m[1], m10 = m[2], m11 = m[3];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j & (1 << B)) continue;
        const V a = x[j], b = x[j | (1 << B)];
        x[j].x = fma(m00, a.x, m01 * b.x);
        x[j].y = fma(m00, a.y, m01 * b.y);
        x[j | (1 << B)].x = fma(m10, a.x, m11 * b.x);
        x[j | (1 << B)].y = fma(m10, a.y, m11 * b.y);
    }
}

// Local index of j on sweep bits (B0, B1).
template <int B0, int B1>
__device__ __forceinline__ constexpr int loc2(int j) { return ((j >> B0) & 1) | ((j >> B1) & 1) << 1; }

// Two-qubit dense gates, a row of coefficients at a time (all of them would
// take 64 scalar registers in complex128).
template <int B0, int B1, typename V, typename R>
__device__ __forceinline__ void gen2(V *x, CPtr<R> m) {
    V y[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (loc2<B0, B1>(j)) continue;
            V a;
            a.x = a.y = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const R mr = m[2 * (r * 4 + c)], mi = m[2 * (r * 4 + c) + 1];
                const V in = x[j | (c & 1) << B0 | (c >> 1) << B1];
                a.x = fma(-mi, in.y, fma(mr, in.x, a.x));
                a.y = fma(mi, in.x, fma(mr, in.y, a.y));
            }
            y[j | (r & 1) << B0 | (r >> 1) << B1] = a;
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = y[j];
}

template <int B0, int B1, typename V, typename R>
__device__ __forceinline__ void real2(V *x, CPtr<R> m) {
    V y[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (loc2<B0, B1>(j)) continue;
            R yr = 0, yi = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const V in = x[j | (c & 1) << B0 | (c >> 1) << B1];
                yr = fma(m[r * 4 + c], in.x, yr);
                yi = fma(m[r * 4 + c], in.y, yi);
            }
            y[j | (r & 1) << B0 | (r >> 1) << B1].x = yr;
            y[j | (r & 1) << B0 | (r >> 1) << B1].y = yi;
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = y[j];
}

// Diagonal on sweep bits (B0, B1; B1 = B0 for one qubit): x[j] *= m[j's bits].
template <int B0, int B1, typename V, typename R>
__device__ __forceinline__ void diag(V *x, CPtr<R> m) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int e = B0 == B1 ? (j >> B0) & 1 : loc2<B0, B1>(j);
        const R dr = m[2 * e], di = m[2 * e + 1];
        const V a = x[j];
        x[j].x = dr * a.x - di * a.y;
        x[j].y = dr * a.y + di * a.x;
    }
}

// x[11] *= (c, s) / x[11] = -x[11]
template <int B0, int B1, typename V, typename R>
__device__ __forceinline__ void cphase(V *x, R c, R s) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (loc2<B0, B1>(j) != 3) continue;
        const V a = x[j];
        x[j].x = c * a.x - s * a.y;
        x[j].y = c * a.y + s * a.x;
    }
}
template <int B0, int B1, typename V>
__device__ __forceinline__ void cz(V *x) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (loc2<B0, B1>(j) == 3) x[j].x = -x[j].x, x[j].y = -x[j].y;
}

template <typename V>
__device__ __forceinline__ void sign8(V *x, uint32_t neg) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if ((neg >> j) & 1u) x[j].x = -x[j].x, x[j].y = -x[j].y;
}

// y_j = a x_j + b (-1)^{popc(z & (j ^ X))} x_{j ^ X}
template <int X, typename V, typename R>
__device__ __forceinline__ void pauli_pair(V *x, CPtr<R> m, uint32_t z) {
    const R ar = m[0], ai = m[1], br = m[2], bi = m[3];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = j ^ X;
        if (k < j) continue;   // each pair once
        const V xj = x[j], xk = x[k];
        V pj, pk;              // b x_k, b x_j
        pj.x = br * xk.x - bi * xk.y;
        pj.y = br * xk.y + bi * xk.x;
        pk.x = br * xj.x - bi * xj.y;
        pk.y = br * xj.y + bi * xj.x;
        if (__popc(z & (uint32_t)k) & 1) pj.x = -pj.x, pj.y = -pj.y;
        if (__popc(z & (uint32_t)j) & 1) pk.x = -pk.x, pk.y = -pk.y;
        x[j].x = ar * xj.x - ai * xj.y + pj.x;
        x[j].y = ar * xj.y + ai * xj.x + pj.y;
        x[k].x = ar * xk.x - ai * xk.y + pk.x;
        x[k].y = ar * xk.y + ai * xk.x + pk.y;
    }
}

// One operation on x and, with `two`, on l; c, s its first two coefficients
// (read ahead), m all of them.  With the parameter flag, first the inner
// product, whose value is returned.  One dispatch per operation: every case
// is straight code for its masks.
#define CAST_ROT(X, Z)                                                 \
    case 8 * (X) + (Z):                                                \
        if (info & kSegParam) v = inner<X, Z>(l, x);                   \
        rot<X, Z>(x, c, s);                                            \
        if (two) rot<X, Z>(l, c, s);                                   \
        break;
#define CAST_ROT1(B) CAST_ROT(0, B) CAST_ROT(B, 0) CAST_ROT(B, B)
#define CAST_ROT2(P, Q)                                                \
    CAST_ROT(0, P | Q) CAST_ROT(P, Q) CAST_ROT(Q, P) CAST_ROT(P, P | Q) CAST_ROT(Q, P | Q) \
    CAST_ROT(P | Q, 0) CAST_ROT(P | Q, P) CAST_ROT(P | Q, Q) CAST_ROT(P | Q, P | Q)
#define CAST_FIXED(CODE, CALL)                                         \
    case (CODE): {                                                     \
        { V *y = x; CALL; }                                            \
        if (two) { V *y = l; CALL; }                                   \
        break;                                                         \
    }
template <typename V, typename R>
__device__ __forceinline__ double seg_op(uint32_t info, V *x, V *l, bool two, R c, R s, CPtr<R> m) {
    double v = 0.0;
    switch (info & 127u) {
        CAST_ROT1(1) CAST_ROT1(2) CAST_ROT1(4)
        CAST_ROT2(1, 2) CAST_ROT2(1, 4) CAST_ROT2(2, 4)
        CAST_FIXED(SO_CZ, (cz<0, 1>(y)))
        CAST_FIXED(SO_CZ + 1, (cz<0, 2>(y)))
        CAST_FIXED(SO_CZ + 2, (cz<1, 2>(y)))
        CAST_FIXED(SO_CP, (cphase<0, 1>(y, c, s)))
        CAST_FIXED(SO_CP + 1, (cphase<0, 2>(y, c, s)))
        CAST_FIXED(SO_CP + 2, (cphase<1, 2>(y, c, s)))
        CAST_FIXED(SO_DIAG1, (diag<0, 0, V, R>(y, m)))
        CAST_FIXED(SO_DIAG1 + 1, (diag<1, 1, V, R>(y, m)))
        CAST_FIXED(SO_DIAG1 + 2, (diag<2, 2, V, R>(y, m)))
        CAST_FIXED(SO_DIAG2, (diag<0, 1, V, R>(y, m)))
        CAST_FIXED(SO_DIAG2 + 1, (diag<0, 2, V, R>(y, m)))
        CAST_FIXED(SO_DIAG2 + 2, (diag<1, 2, V, R>(y, m)))
        CAST_FIXED(SO_REAL1, (real1<0, V, R>(y, m)))
        CAST_FIXED(SO_REAL1 + 1, (real1<1, V, R>(y, m)))
        CAST_FIXED(SO_REAL1 + 2, (real1<2, V, R>(y, m)))
        CAST_FIXED(SO_GEN1, (gen1<0, V, R>(y, m)))
        CAST_FIXED(SO_GEN1 + 1, (gen1<1, V, R>(y, m)))
        CAST_FIXED(SO_GEN1 + 2, (gen1<2, V, R>(y, m)))
        CAST_FIXED(SO_REAL2, (real2<0, 1, V, R>(y, m)))
        CAST_FIXED(SO_REAL2 + 1, (real2<0, 2, V, R>(y, m)))
        CAST_FIXED(SO_REAL2 + 2, (real2<1, 2, V, R>(y, m)))
        CAST_FIXED(SO_GEN2, (gen2<0, 1, V, R>(y, m)))
        CAST_FIXED(SO_GEN2 + 1, (gen2<0, 2, V, R>(y, m)))
        CAST_FIXED(SO_GEN2 + 2, (gen2<1, 2, V, R>(y, m)))
        CAST_FIXED(SO_SIGN, (sign8(y, info >> 8)))
        CAST_FIXED(SO_PAULI + 1, (pauli_pair<1, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 2, (pauli_pair<2, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 3, (pauli_pair<3, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 4, (pauli_pair<4, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 5, (pauli_pair<5, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 6, (pauli_pair<6, V, R>(y, m, info >> 8)))
        CAST_FIXED(SO_PAULI + 7, (pauli_pair<7, V, R>(y, m, info >> 8)))
        default: break;
    }
    return v;
}
#undef CAST_ROT
#undef CAST_ROT1
#undef CAST_ROT2
#undef CAST_FIXED

// ------------------------------------------------------------------ inner-product sums
// The matrix core sums the inner products over lanes.  With A[m][k] = 1 for
// m = p mod 16 and 0 elsewhere, D = A B + D adds B's four rows (the lanes'
// values, lane l at row l / 16, column l % 16) into row p mod 16 of D: one
// v_mfma_f64_16x16x4 per product instead of six cross-lane adds of two moves
// each, and sixteen products share one accumulator.  flush() adds the
// accumulator's sixteen columns and leaves the sums with the workgroup's.
typedef double acc_v4 __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ double dpp_ror(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_total(double v) {
    v += dpp_ror<0x128>(v);   // rotate within rows of 16 lanes
    v += dpp_ror<0x124>(v);
    v += dpp_ror<0x122>(v);
    v += dpp_ror<0x121>(v);
    return v;
}
// D value v of lane l is row l / 16 + 4 v, column l % 16.
__device__ __forceinline__ void flush_sums(acc_v4 &acc, double *gsum, uint32_t p0, int lane, int wave) {
    const double r0 = row_total(acc[0]), r1 = row_total(acc[1]), r2 = row_total(acc[2]), r3 = row_total(acc[3]);
    const int v = lane & 15;
    if (v < 4) {
        const double r = v == 0 ? r0 : v == 1 ? r1 : v == 2 ? r2 : r3;
        gsum[(p0 + (uint32_t)(lane >> 4) + 4u * (uint32_t)v) * 4 + wave] += r;   // each wave its own entries
    }
    acc[0] = acc[1] = acc[2] = acc[3] = 0.0;
}

__device__ __forceinline__ BatchInst load_inst(CPtr<BatchInst> p) {
    BatchInst b;
    b.psi = p->psi;
    b.lam = p->lam;
    b.n = p->n;
    b.nslots = p->nslots;
    b.wgs = p->wgs;
    b.ngroups = p->ngroups;
    b.part_off = p->part_off;
    b.res_off = p->res_off;
    b.tg_off = p->tg_off;
    b.tt_off = p->tt_off;
    b.init_kind = p->init_kind;
    b.pad = 0;
    b.init_src = p->init_src;
    return b;
}

// LDS position of tile amplitude e: 16-byte chunk c is stored at chunk
// c ^ hash(c / 16), which keeps the coalesced load/store phases conflict-free
// and spreads the sweeps' power-of-two-strided group reads over the banks.
__device__ __forceinline__ uint32_t bswz(uint32_t c) { return c ^ (((c >> 4) ^ (c >> 8)) & 15u); }
template <int S>
__device__ __forceinline__ uint32_t bat(uint32_t e) { return (bswz(e >> S) << S) | (e & ((1u << S) - 1)); }

// FWD / ADJ segment on tile w of an instance.  LDS layout: per-wave sums of
// the segment's inner products (at most kSegMaxGates), then the psi tile and
// (ADJ only) the lambda tile, 2^tb amplitudes each, swizzled as above.  A
// forward step's launch carries one tile's LDS, so more of its workgroups
// share a compute unit.  `pair` (FWD in the persistent launch, whose
// workgroups hold two tiles of LDS anyway): tiles w and w + 1 of psi go
// through the segment together in the two tile slots, the second one taking
// the lambda tile's place.
template <typename R>
__device__ __forceinline__ void seg_item(const BatchDev &d, CPtr<BatchRec> rec, const BatchInst &in, uint32_t w,
                         typename BAmp<R>::T *lds, bool pair) {
    using V = typename BAmp<R>::T;
    typedef unsigned int nu4 __attribute__((ext_vector_type(4)));
    constexpr int S = sizeof(V) == 16 ? 0 : 1;      // log2(amplitudes per 16-byte chunk)
    const bool adj = rec->kind == BK_ADJ;
    const bool two = adj || pair;                    // a second tile in the lambda slot
    const int tb = rec->tb, W = rec->W;
    const uint32_t T = 1u << tb, tid = threadIdx.x;
    double *gsum = reinterpret_cast<double *>(lds);               // [kSegMaxGates][4 waves]
    V *tp = reinterpret_cast<V *>(reinterpret_cast<char *>(lds) + kSegLdsExtra), *tl = tp + T;
    V *psi = reinterpret_cast<V *>(in.psi);
    V *lam = reinterpret_cast<V *>(in.lam);
    // amplitude index of a tile position: an OR of tile, lane and chunk parts
    uint64_t tbase = (uint64_t)w << W, tbase2 = (uint64_t)(w + 1) << W;
    for (int i = W; i < tb; ++i) {
        const uint64_t lm = rec->bit[i] - 1;
        tbase = ((tbase & ~lm) << 1) | (tbase & lm);
        tbase2 = ((tbase2 & ~lm) << 1) | (tbase2 & lm);
    }
    // the second tile: lambda's tile w, or psi's tile w + 1 (its amplitude
    // index differs from tile w's by the XOR of the two tile bases, which
    // lie above the tile's low window)
    V *sec = pair ? psi : lam;
    const uint64_t dsec = pair ? (tbase ^ tbase2) : 0;
    if (adj) gsum[tid] = 0.0;                        // kSegMaxGates * 4 = 256 entries
    // 16-byte chunks of the tile (a run holds at least one chunk when W >= S)
    const bool chunked = W >= S;
    const uint32_t nchunk = chunked ? (T >> S) : T;
    const int s0 = chunked ? S : 0;
    uint64_t xl = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((tid >> i) & 1u) xl |= rec->bit[s0 + i];
    const uint64_t b8 = rec->bit[s0 + 8], b9 = rec->bit[s0 + 9], b10 = rec->bit[s0 + 10], b11 = rec->bit[s0 + 11];
    auto chunk_part = [&](uint32_t u) {   // u < 16
        return ((u & 1) ? b8 : 0) | ((u & 2) ? b9 : 0) | ((u & 4) ? b10 : 0) | ((u & 8) ? b11 : 0);
    };
    const uint64_t x0 = tbase | xl;
    const uint32_t zl = bswz(tid);
    if (chunked) {
        // eight chunks of each state in flight per lane (a whole 2^11-amplitude
        // complex128 or 2^12-amplitude complex64 tile per 256 lanes): the item
        // waits on its loads once instead of twice
        constexpr int DEPTH = 8;
        nu4 *t16p = reinterpret_cast<nu4 *>(tp), *t16l = reinterpret_cast<nu4 *>(tl);
        const nu4 *p16 = reinterpret_cast<const nu4 *>(psi), *l16 = reinterpret_cast<const nu4 *>(sec);
        for (uint32_t u0 = 0; u0 * 256 < nchunk; u0 += DEPTH) {
            nu4 bp[DEPTH], bl[DEPTH];
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if ((u0 + u) * 256 + tid < nchunk) {
                    const uint64_t x = x0 | chunk_part(u0 + u);
                    bp[u] = p16[x >> S];
                    if (two) bl[u] = l16[(x ^ dsec) >> S];
                }
            }
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if ((u0 + u) * 256 + tid < nchunk) {
                    const uint32_t z = zl ^ bswz((u0 + u) * 256);
                    t16p[z] = bp[u];
                    if (two) t16l[z] = bl[u];
                }
            }
        }
    } else {
        for (uint32_t u = 0; u * 256 + tid < nchunk; ++u) {
            const uint64_t x = x0 | chunk_part(u);
            const uint32_t e = bat<S>(u * 256 + tid);
            tp[e] = psi[x];
            if (two) tl[e] = sec[x ^ dsec];
        }
    }
    __syncthreads();
    CPtr<R> mats = cptr(reinterpret_cast<const R *>(d.mats));
    CPtr<SegOp> ops = cptr(d.ops);
    const int lane = tid & 63, wave = tid >> 6;
    acc_v4 acc = {0.0, 0.0, 0.0, 0.0};
    uint32_t p = 0;
    // sweeps: each thread loads 8-amplitude groups over the sweep's three
    // tile bits once, applies the sweep's operations in registers in order
    // (taking each inner product right before its gate), and writes the group back
    const uint32_t groups = 1u << (tb - 3);
    char *tpb = reinterpret_cast<char *>(tp), *tlb = reinterpret_cast<char *>(tl);
    const uint32_t sw1 = rec->sw1;
    for (uint32_t sw = rec->sw0; sw < sw1; ++sw) {
        CPtr<SegSweep> sp = cptr(d.sweeps) + sw;
        const uint32_t bits = sp->bits, g0 = sp->g0, g1 = sp->g1, p0 = sp->p0;
        const int q0 = bits & 255, q1 = (bits >> 8) & 255, q2 = bits >> 16;
        // bat<S> is linear over GF(2) (shifts, masks and XORs) and a group's
        // base and the sweep offsets have disjoint bits, so the LDS slot of
        // base | off[j] is bat(base) ^ bat(off[j]): the eight swizzled
        // offsets are wave-uniform and each access costs one XOR
        // (byte offsets: the XOR of two multiples of sizeof(V) is one)
        const uint32_t o0 = bat<S>(1u << q0) * (uint32_t)sizeof(V), o1 = bat<S>(1u << q1) * (uint32_t)sizeof(V),
                       o2 = bat<S>(1u << q2) * (uint32_t)sizeof(V);
        uint32_t so[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) so[j] = ((j & 1) ? o0 : 0u) ^ ((j & 2) ? o1 : 0u) ^ ((j & 4) ? o2 : 0u);
        for (uint32_t gb = 0; gb < groups; gb += 256) {
            const uint32_t g = gb + tid;
            const bool act = g < groups;
            // lanes past the last group compute on zeros: the operations stay in
            // uniform control flow (within a divergent branch the compiler would
            // linearise the dispatch and copy x and l at each of its joins)
            uint32_t bb = 0;
            V x[8], l[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j].x = x[j].y = l[j].x = l[j].y = 0;
            if (act) {
                bb = bat<S>(ins0_32(ins0_32(ins0_32(g, q0), q1), q2)) * (uint32_t)sizeof(V);
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const V *>(tpb + (bb ^ so[j]));
                if (two) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) l[j] = *reinterpret_cast<const V *>(tlb + (bb ^ so[j]));
                }
            }
            p = p0;
            // read ahead: the record two operations on and the first
            // coefficients of the next one are requested while this one is
            // applied, so an operation's scalar loads never wait on each other
            // (the tables are padded by two entries)
            uint32_t info = ops[g0].info, mat = ops[g0].mat, info1 = ops[g0 + 1].info, mat1 = ops[g0 + 1].mat;
            R c1 = mats[mat], s1 = mats[mat + 1];
            for (uint32_t gi = g0; gi < g1; ++gi) {
                const uint32_t op = info;
                const R c = c1, s = s1;
                CPtr<R> m = mats + mat;
                info = info1;
                mat = mat1;
                c1 = mats[mat];
                s1 = mats[mat + 1];
                info1 = ops[gi + 2].info;
                mat1 = ops[gi + 2].mat;
                const double v = seg_op<V, R>(op, x, l, two, c, s, m);
                if (op & kSegParam) {
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((uint32_t)(lane & 15) == (p & 15u) ? 1.0 : 0.0, v, acc,
                                                               0, 0, 0);
                    ++p;
                    if ((p & 15u) == 0) flush_sums(acc, gsum, p - 16, lane, wave);
                }
            }
            // more groups follow: they start again at p0
            if (adj && groups > 256 && (p & 15u)) flush_sums(acc, gsum, p & ~15u, lane, wave);
            if (act) {
#pragma unroll
                for (int j = 0; j < 8; ++j) *reinterpret_cast<V *>(tpb + (bb ^ so[j])) = x[j];
                if (two) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) *reinterpret_cast<V *>(tlb + (bb ^ so[j])) = l[j];
                }
            }
        }
        __syncthreads();
    }
    if (adj && rec->np) {
        if (groups <= 256 && (p & 15u)) flush_sums(acc, gsum, p & ~15u, lane, wave);
        __syncthreads();
        // one partial per inner product: its four waves in a fixed order
        if (tid < rec->np) {
            const double sum = ((gsum[tid * 4] + gsum[tid * 4 + 1]) + gsum[tid * 4 + 2]) + gsum[tid * 4 + 3];
            d.partials[in.part_off + (uint64_t)d.slots[rec->ps0 + tid] * in.wgs + w] = sum;
        }
    }
    if (chunked) {
        const nu4 *t16p = reinterpret_cast<const nu4 *>(tp), *t16l = reinterpret_cast<const nu4 *>(tl);
        nu4 *p16 = reinterpret_cast<nu4 *>(psi), *l16 = reinterpret_cast<nu4 *>(sec);
        for (uint32_t u = 0; u * 256 + tid < nchunk; ++u) {
            const uint64_t x = x0 | chunk_part(u);
            const uint32_t z = zl ^ bswz(u * 256);
            p16[x >> S] = t16p[z];
            if (two) l16[(x ^ dsec) >> S] = t16l[z];
        }
    } else {
        for (uint32_t u = 0; u * 256 + tid < nchunk; ++u) {
            const uint64_t x = x0 | chunk_part(u);
            const uint32_t e = bat<S>(u * 256 + tid);
            psi[x] = tp[e];
            if (two) sec[x ^ dsec] = tl[e];
        }
    }
    __syncthreads();   // the LDS sums and tiles are reused by the next item
}

// lambda[y] = (H psi)[y] for the 2^tb amplitudes from y0, and the partial sum
// of Re <psi|lambda>.  A lane's amplitudes are y0 + tid + 256 j: a term's sign
// is a per-lane parity, formed once, and a wave-uniform one per j.
template <typename R>
__device__ __forceinline__ double hpsi_range(const BatchDev &d, const BatchInst &in, uint64_t y0, uint32_t count) {
    using V = typename BAmp<R>::T;
    constexpr int J = 4;
    const V *psi = reinterpret_cast<const V *>(in.psi);
    V *lam = reinterpret_cast<V *>(in.lam);
    CPtr<BatchHGroup> groups = cptr(d.tg) + in.tg_off;
    CPtr<BatchHTerm> terms = cptr(d.tt) + in.tt_off;
    double e = 0.0;
    for (uint32_t c0 = 0; c0 < count; c0 += 256 * J) {
        const uint64_t yb = y0 + c0;            // uniform
        const uint64_t yt = yb + threadIdx.x;
        const uint32_t left = count - c0;
        double lr[J], li[J];
#pragma unroll
        for (int j = 0; j < J; ++j) lr[j] = li[j] = 0.0;
        for (uint32_t g = 0; g < in.ngroups; ++g) {
            const uint64_t x = groups[g].x;
            const uint32_t first = groups[g].first, count_g = groups[g].count, odd = groups[g].odd;
            V v[J];
            double c[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                v[j].x = v[j].y = 0;
                if (256u * j + threadIdx.x < left) v[j] = psi[(yt + 256 * j) ^ x];
                c[j] = 0.0;
            }
            for (uint32_t t = first; t < first + count_g; ++t) {
                const uint64_t z = terms[t].z;
                const double ct = terms[t].c;
                const uint32_t neg = (uint32_t)__popcll(z & (yt ^ x)) & 1u;
                const double cs = __hiloint2double(__double2hiint(ct) ^ (int)(neg << 31), __double2loint(ct));
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const uint32_t nj = (uint32_t)__popc((uint32_t)z & (256u * j)) & 1u;   // uniform; bits 8-9 of yt are yb's
                    c[j] += __hiloint2double(__double2hiint(cs) ^ (int)(nj << 31), __double2loint(cs));
                }
            }
            if (odd) {
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    lr[j] = fma(-c[j], (double)v[j].y, lr[j]);
                    li[j] = fma(c[j], (double)v[j].x, li[j]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    lr[j] = fma(c[j], (double)v[j].x, lr[j]);
                    li[j] = fma(c[j], (double)v[j].y, li[j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (256u * j + threadIdx.x >= left) continue;
            V o;
            o.x = (R)lr[j];
            o.y = (R)li[j];
            lam[yt + 256 * j] = o;
            // <psi|lambda> with lambda as stored (rounded to the state dtype)
            const V p = psi[yt + 256 * j];
            e = fma((double)p.y, (double)o.y, fma((double)p.x, (double)o.x, e));
        }
    }
    return e;
}

// One work item: item w of record rec (pair: items w and w + 1 of a FWD record).
template <typename R>
__device__ __forceinline__ void run_item(const BatchDev &d, CPtr<BatchRec> rec, uint32_t w, double *red, bool pair = false) {
    using V = typename BAmp<R>::T;
    const BatchInst in = load_inst(cptr(d.insts) + rec->inst);
    if (rec->kind != BK_HPSI) {
        seg_item<R>(d, rec, in, w, reinterpret_cast<V *>(batch_lds), pair);
        return;
    }
    const uint32_t per = 1u << rec->tb;
    const double sum = block_sum(hpsi_range<R>(d, in, (uint64_t)w << rec->tb, per), red);
    if (threadIdx.x == 0) d.partials[in.part_off + w] = sum;   // slot 0
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Largest r in [lo, hi) with recs[r].item0 <= x.
__device__ __forceinline__ uint64_t find_rec(CPtr<BatchRec> recs, uint64_t lo, uint64_t hi, uint64_t x) {
    while (hi - lo > 1) {
        const uint64_t mid = (lo + hi) / 2;
        if (recs[mid].item0 <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <typename R>
__global__ void __launch_bounds__(256, 3) k_batch_step(BatchDev d, int s) {
    __shared__ double red[4];
    const uint64_t r = find_rec(cptr(d.recs), cptr(d.step_rec)[s], cptr(d.step_rec)[s + 1], blockIdx.x);
    CPtr<BatchRec> rec = cptr(d.recs) + r;   // by pointer: its bit[] is indexed at run time
    run_item<R>(d, rec, blockIdx.x - rec->item0, red);
}

// counters (stride kCounterStride): 0 next item; 1 error flag; 2 + i items of
// instance i completed.  A workgroup claims `chunk` consecutive items per
// counter atomic and publishes its completions per run of items of one
// instance; before any wait it publishes what it holds, so it never waits on
// its own unpublished work.  Items are claimed in global order and every
// dependency is on an earlier item, so the earliest unfinished item can
// always proceed.
template <typename R>
__global__ void __launch_bounds__(256) k_batch_persistent(BatchDev d, uint64_t total, unsigned long long *counters,
                                                          uint32_t spin_limit, uint32_t chunk) {
    __shared__ double red[4];
    __shared__ unsigned long long base_sh;
    __shared__ int stop_sh;
    uint32_t pend_inst = 0;     // thread 0 only: completed, unpublished items
    unsigned long long pend = 0;
    unsigned long long *const err = counters + kCounterStride;
    for (;;) {
        if (threadIdx.x == 0) {
            base_sh = atomicAdd(&counters[0], (unsigned long long)chunk);
            stop_sh = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        }
        __syncthreads();
        // values read from LDS are not known to be uniform; read through
        // readfirstlane they are, so everything derived stays scalar
        const uint64_t base = uniform64(base_sh);
        if (base >= total || __builtin_amdgcn_readfirstlane(stop_sh)) break;
        const uint64_t end = base + chunk < total ? base + chunk : total;
        for (uint64_t item = base; item < end; ++item) {
            uint64_t lo = 0, hi = (uint64_t)d.nsteps;
            while (hi - lo > 1) {
                const uint64_t mid = (lo + hi) / 2;
                if (cptr(d.step_item)[mid] <= item) lo = mid;
                else hi = mid;
            }
            const int s = (int)lo;
            const uint64_t x = item - cptr(d.step_item)[s];
            const uint64_t r = find_rec(cptr(d.recs), cptr(d.step_rec)[s], cptr(d.step_rec)[s + 1], x);
            CPtr<BatchRec> rec = cptr(d.recs) + r;   // by pointer: its bit[] is indexed at run time
            if (threadIdx.x == 0) {
                unsigned long long *done = &counters[(2 + rec->inst) * kCounterStride];
                if (pend && pend_inst != rec->inst) {
                    __hip_atomic_fetch_add(&counters[(2 + pend_inst) * kCounterStride], pend, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                    pend = 0;
                }
                // poll with relaxed loads (an acquire per poll would invalidate the
                // caches under every other workgroup), then acquire once.  A
                // spin limit of 0 fails every item that has a dependency at all,
                // so the error path can be forced from the host.
                const bool force = spin_limit == 0 && rec->need != 0;
                if (force || __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + pend < rec->need) {
                    if (pend) {
                        __hip_atomic_fetch_add(done, pend, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                        pend = 0;
                    }
                    uint32_t spins = 0;
                    while (force || __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < rec->need) {
                        if (++spins > spin_limit ||
                            __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                            atomicExch(err, 1ull);
                            stop_sh = 1;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(2);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(stop_sh)) break;
            // two forward items of one record claimed together run as a pair
            // (same gates, both tile slots of this workgroup's LDS)
            const uint32_t w = (uint32_t)(x - rec->item0);
            const bool pair = rec->kind == BK_FWD && item + 1 < end && w + 1 < rec->wgs;
            run_item<R>(d, rec, w, red, pair);
            // the barrier makes every wave's stores visible to the workgroup;
            // thread 0's agent-scope release later publishes them device-wide
            __syncthreads();
            if (threadIdx.x == 0) {
                pend_inst = rec->inst;
                pend += pair ? 2 : 1;
            }
            if (pair) ++item;
        }
        if (threadIdx.x == 0 && pend) {
            __hip_atomic_fetch_add(&counters[(2 + pend_inst) * kCounterStride], pend, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            pend = 0;
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(stop_sh)) break;
    }
}

__global__ void k_batch_zero(unsigned long long *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

template <typename R>
__global__ void __launch_bounds__(256) k_batch_init(BatchDev d) {
    using V = typename BAmp<R>::T;
    const BatchInst in = d.insts[blockIdx.y];
    V *psi = reinterpret_cast<V *>(in.psi);
    const V *src = reinterpret_cast<const V *>(in.init_src);
    const uint64_t N = 1ull << in.n;
    const R amp = (R)exp2(-0.5 * in.n);
    for (uint64_t y = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; y < N; y += (uint64_t)gridDim.x * blockDim.x) {
        V v;
        if (in.init_kind == 2) {
            v = src[y];
        } else if (in.init_kind == 1) {
            v.x = amp;
            v.y = 0;
        } else {
            v.x = y == 0 ? (R)1 : (R)0;
            v.y = 0;
        }
        psi[y] = v;
    }
}

// One wave per result slot: its partial sums over the work items, in a fixed
// order.
__global__ void __launch_bounds__(256) k_batch_finish(BatchDev d) {
    const BatchInst in = d.insts[blockIdx.x];
    const int lane = threadIdx.x & 63;
    for (int slot = (int)(blockIdx.y * 4 + (threadIdx.x >> 6)); slot < in.nslots; slot += (int)gridDim.y * 4) {
        double s = 0.0;
        for (uint32_t w = lane; w < in.wgs; w += 64) s += d.partials[in.part_off + (uint64_t)slot * in.wgs + w];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) d.results[in.res_off + slot] = s;
    }
}

static cast_status launched(const char *what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(CAST_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return CAST_OK;
}

// Raises the kernels' dynamic-LDS limit once (segment items use more than 64 KiB).
template <typename R>
static hipError_t allow_lds() {
    static hipError_t done = [] {
        hipError_t e = hipFuncSetAttribute((const void *)k_batch_step<R>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kSegMaxLds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)k_batch_persistent<R>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kSegMaxLds);
        return e;
    }();
    return done;
}

cast_status batch_launch_step(const BatchDev &d, cast_dtype dt, int s, uint64_t nitems, size_t lds,
                              hipStream_t st) {
    if (lds > kSegMaxLds) return fail(CAST_EUNSUPPORTED, "segment tiles exceed 128 KiB of LDS");
    const hipError_t ae = dt == CAST_C128 ? allow_lds<double>() : allow_lds<float>();
    if (ae != hipSuccess) return fail(CAST_EHIP, std::string("LDS attribute: ") + hipGetErrorString(ae));
    if (dt == CAST_C128) hipLaunchKernelGGL(k_batch_step<double>, dim3((uint32_t)nitems), dim3(256), lds, st, d, s);
    else hipLaunchKernelGGL(k_batch_step<float>, dim3((uint32_t)nitems), dim3(256), lds, st, d, s);
    return launched("batched step launch");
}

cast_status batch_launch_persistent(const BatchDev &d, cast_dtype dt, uint64_t total_items, int grid,
                                    unsigned long long *counters, uint32_t spin_limit, uint32_t chunk, size_t lds,
                                    hipStream_t st) {
    if (lds > kSegMaxLds) return fail(CAST_EUNSUPPORTED, "segment tiles exceed 128 KiB of LDS");
    const hipError_t ae = dt == CAST_C128 ? allow_lds<double>() : allow_lds<float>();
    if (ae != hipSuccess) return fail(CAST_EHIP, std::string("LDS attribute: ") + hipGetErrorString(ae));
    if (dt == CAST_C128)
        hipLaunchKernelGGL(k_batch_persistent<double>, dim3(grid), dim3(256), lds, st, d, total_items, counters,
                           spin_limit, chunk);
    else
        hipLaunchKernelGGL(k_batch_persistent<float>, dim3(grid), dim3(256), lds, st, d, total_items, counters,
                           spin_limit, chunk);
    return launched("persistent batch launch");
}

cast_status batch_zero(unsigned long long *p, size_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_zero, dim3(1), dim3(256), 0, st, p, n);
    return launched("counter reset");
}

cast_status batch_init_states(const BatchDev &d, cast_dtype dt, hipStream_t st) {
    if (dt == CAST_C128) hipLaunchKernelGGL(k_batch_init<double>, dim3(1024, d.ninst), dim3(256), 0, st, d);
    else hipLaunchKernelGGL(k_batch_init<float>, dim3(1024, d.ninst), dim3(256), 0, st, d);
    return launched("batch init");
}

cast_status batch_finish(const BatchDev &d, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_finish, dim3(d.ninst, 16), dim3(256), 0, st, d);
    return launched("batch finish");
}

}  // namespace cast
