// Two-electron part of the nuclear gradient, one object per angular class:
// device algebra shared by the class kernels (grad_class.hip) and the
// one-electron kernels (grad.hip).
//
// The Coulomb integrals of a primitive quartet are sums over Hermite
// Gaussians, sum_h E^{ab}_h sum_k E^{cd}_k (-1)^{|k|} R_{h+k}(P - Q), with E
// a product of 1-D coefficients per direction.  The centres A, B enter
// through the product centre P and through A - B in E, so with the density
// weights Gamma of the quartet
//   d/dA = (a/p) F_P + g_AB,  d/dB = (b/p) F_P - g_AB,  and likewise
//   d/dC = -(c/q) F_P + g_CD, d/dD = -(d/q) F_P - g_CD,
//   F_P  = sum Gamma E_h E_k (-1)^{|k|} R_{h+k+1},   g = sum Gamma dE/d(A-B) ...,
// nine numbers for the twelve centre derivatives, with Hermite indices that
// never exceed L + 1.  For one direction, with X_PA the distance to the
// first centre and a its exponent,
//   E^{i+1,j}_t = E^{ij}_{t-1}/(2p) + X_PA E^{ij}_t + (t+1) E^{ij}_{t+1}   (j: X_PB),
//   dE^{ij}_t/d(A-B) = 2a (X_PA E^{ij}_t + (t+1) E^{ij}_{t+1}) - i E^{i-1,j}_t
// (the Gaussian product factor is kept out of E; the second line holds with
// it in).
#pragma once

#include "class_ops.hpp"
#include "eri_kernels.hpp"

namespace mess {

// Primitive pair: exponents, p, the product factor times both coefficients,
// and P - A (zero on one centre).
struct GPrim {
    double a, b, p, K;
    double PAx, PAy, PAz, pad;
};

struct GradLists {
    const PairInfo *pairs;     // sorted pairs of the basis
    const GPrim *prims;        // of pair i: prims[off[i] .. off[i] + cnt[i])
    const int *off, *cnt;
    const int *sh_atom;        // atom of every shell
    const double *tab, *tabt;  // Boys tables of the basis
    const double *D;
    int N, nat;
    double *copies;            // kGradCopies gradients, summed at the end
};
constexpr int kGradCopies = 32;   // spreads the atomics of the blocks over cache lines
constexpr int kGradLdsAtoms = 512;  // gradients of up to this many atoms are summed in LDS first

// One class's quartets into the gradient copies.
template <int CB, int CK>
struct GradOps {
    static int run(const GradLists &G, const ClassLaunch &L);
};

// 1-D Hermite coefficients (and their A - B derivatives) for all i <= I,
// j <= J, t <= i + j of one direction, every index known at compile time.
template <int I, int J>
struct Herm1 {
    static constexpr int NT = I + J + 1;
    double e[(I + 1) * (J + 1) * NT], d[(I + 1) * (J + 1) * NT];
    static constexpr int at(int i, int j, int t) { return (i * (J + 1) + j) * NT + t; }
    __device__ __forceinline__ void build(double a, double o2p, double PA, double PB) {
        static_for<0, I + 1>([&](auto II) {
            static_for<0, J + 1>([&](auto JJ) {
                constexpr int i = decltype(II)::value, j = decltype(JJ)::value;
                static_for<0, i + j + 1>([&](auto TT) {
                    constexpr int t = decltype(TT)::value;
                    if constexpr (i + j == 0) {
                        e[0] = 1.0;
                    } else {
                        constexpr int i1 = i > 0 ? i - 1 : i, j1 = i > 0 ? j : j - 1, top = i + j - 1;
                        const double X = i > 0 ? PA : PB;
                        double v = 0.0;
                        if constexpr (t <= top) v = X * e[at(i1, j1, t)];
                        if constexpr (t >= 1) v += o2p * e[at(i1, j1, t - 1)];
                        if constexpr (t + 1 <= top) v += (t + 1) * e[at(i1, j1, t + 1)];
                        e[at(i, j, t)] = v;
                    }
                });
                static_for<0, i + j + 1>([&](auto TT) {
                    constexpr int t = decltype(TT)::value;
                    double v = PA * e[at(i, j, t)];
                    if constexpr (t < i + j) v += (t + 1) * e[at(i, j, t + 1)];
                    v *= 2.0 * a;
                    if constexpr (i > 0 && t <= i - 1 + j) v -= i * e[at(i - 1, j, t)];
                    d[at(i, j, t)] = v;
                });
            });
        });
    }
};

// Component c (0-based) of a shell of angular momentum l.
constexpr Cart comp_of(int l, int c) { return cart_of(cart_off(l) + c); }
constexpr double comp_sc(Cart c) { return cart_is_mixed_d(c) ? kSqrt3 : 1.0; }

// R_c of every Hermite index |c| <= N (in registers): R^n_0 = (-2 alpha)^n
// F_n, R^n_{c+1_i} = X_i R^{n+1}_c + c_i R^{n+1}_{c-1_i}.
template <int N>
__device__ __forceinline__ void hermite_r(double alpha, const double (&X)[3], const double (&F)[N + 1],
                                          double (&R)[cart_off(N + 1)]) {
    double V[N + 1][cart_off(N + 1)];
    double m2a = 1.0;
    static_for<0, N + 1>([&](auto M) {
        V[decltype(M)::value][0] = m2a * F[decltype(M)::value];
        m2a *= -2.0 * alpha;
    });
    static_for<1, cart_off(N + 1)>([&](auto CI) {
        constexpr int c = decltype(CI)::value;
        constexpr Cart k = cart_of(c);
        // lower along the direction with the smallest non-zero exponent
        constexpr int i = [] {
            const Cart q = cart_of(c);
            int best = -1;
            for (int d = 0; d < 3; ++d)
                if (q.get(d) > 0 && (best < 0 || q.get(d) < q.get(best))) best = d;
            return best;
        }();
        constexpr int c1 = k.minus(i).idx();
        static_for<0, N - k.l() + 1>([&](auto M) {
            constexpr int m = decltype(M)::value;
            double v = X[i] * V[m + 1][c1];
            if constexpr (k.get(i) >= 2) v += (k.get(i) - 1) * V[m + 1][k.minus(i, 2).idx()];
            V[m][c] = v;
        });
    });
    static_for<0, cart_off(N + 1)>([&](auto C) { R[decltype(C)::value] = V[0][decltype(C)::value]; });
}

// Adds the nine centre derivatives of a wave's quartet (per-lane partial
// sums g: A, B, C, x y z each; D by translation) to acc (3 per atom; LDS or
// global): a reduce-scatter over the lanes leaves one value a lane group.
__device__ __forceinline__ void grad_add(const double (&g)[9], int lane, const int (&atom)[4], double *acc, bool lds) {
    double v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = k < 9 ? g[k] : 0.0;
    // lane bits 5..2 choose the value
    auto step = [&](auto CC, auto OO) {
        constexpr int C = decltype(CC)::value, O = decltype(OO)::value;
        const bool up = (lane & O) != 0;
        static_for<0, C / 2>([&](auto I) {
            constexpr int k = decltype(I)::value;
            const double send = up ? v[k] : v[k + C / 2], keep = up ? v[k + C / 2] : v[k];
            v[k] = keep + __shfl_xor(send, O, 64);
        });
    };
    using std::integral_constant;
    step(integral_constant<int, 16>{}, integral_constant<int, 32>{});
    step(integral_constant<int, 8>{}, integral_constant<int, 16>{});
    step(integral_constant<int, 4>{}, integral_constant<int, 8>{});
    step(integral_constant<int, 2>{}, integral_constant<int, 4>{});
    double s = v[0];
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 1, 64);
    const int k = ((lane >> 5) & 1) * 8 + ((lane >> 4) & 1) * 4 + ((lane >> 3) & 1) * 2 + ((lane >> 2) & 1);
    if ((lane & 3) || k >= 9) return;
    const int at = k < 3 ? atom[0] : (k < 6 ? atom[1] : atom[2]);
    double *pa = acc + 3 * at + k % 3, *pd = acc + 3 * atom[3] + k % 3;
    if (lds) {
        __hip_atomic_fetch_add(pa, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add(pd, -s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
        unsafeAtomicAdd(pa, s);
        unsafeAtomicAdd(pd, -s);
    }
}

}  // namespace mess
