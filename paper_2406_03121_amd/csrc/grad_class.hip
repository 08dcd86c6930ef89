// Two-electron gradient of one angular class (compiled once per class with
// -DMESS_GCB=<bra pair class> -DMESS_GCK=<ket pair class>).  Two forms:
//   k_grad_lane   a wave per shell quartet, a lane per primitive quartet,
//                 the Hermite algebra unrolled in registers;
//   k_grad_coop   a block per shell quartet (and share of its ket
//                 primitives), a wave per primitive quartet with its lanes
//                 over (ab, k), tables in LDS.
// The lane form serves a class until its unrolled steps outgrow the
// registers by more than the cooperative form costs on 3 waters (45
// functions).  Kernel times there, lane / cooperative, ms: (pp|pp) 0.49 /
// 0.14, (ds|ds) 0.16 / 0.78, (dp|ps) 0.31 / 0.74, (dd|ss) 0.71 / 1.42, but
// (dp|pp) 2.17 / 0.29, (dp|ds) 1.34 / 0.93, (dd|ps) 1.75 / 0.96 (3 to 4 KB of
// spill a lane).  The line moves with the list: on 1 water (dp|ps) 0.18 /
// 0.10 and (dd|ss) 0.22 / 0.07; on 7 waters (dp|ds) 4.9 / 10.0 and (dd|ps)
// 4.2 / 9.3, where a rule on the list's length would choose the lane form.
#include <algorithm>

#include "grad.hpp"

#ifndef MESS_GCB
#error "compile with -DMESS_GCB, -DMESS_GCK"
#endif

namespace mess {

// Density weight of element (m, n, l, s) of a quartet with the half of the
// energy expression and the quartet's permutation count in mult.
__device__ __forceinline__ double grad_weight(const double *__restrict__ D, int N, int m, int n, int l, int s, double mult) {
    const double *Dm = D + (int64_t)m * N, *Dn = D + (int64_t)n * N;
    return mult * (Dm[n] * D[(int64_t)l * N + s] - 0.25 * (Dm[l] * Dn[s] + Dm[s] * Dn[l]));
}

__device__ __forceinline__ double quartet_mult(const PairInfo &bra, const PairInfo &ket, bool same) {
    return 0.5 * (bra.sa == bra.sb ? 1.0 : 2.0) * (ket.sa == ket.sb ? 1.0 : 2.0) * (same ? 1.0 : 2.0);
}

constexpr double k2Pi52 = 34.986836655249725693;  // 2 pi^(5/2)

// Bounded by FP64 arithmetic where it does not spill (vector work on 54 to 72 %
// of the waves' cycles in (ds|ps), (pp|ps), (dp|ss)), by its scratch accesses
// where it does (waits on 54 to 66 % in (pp|pp), (ds|pp), (dd|ss)): about
// nnz(ab) (NK + 6) + NK nnz(ab) FMAs per bra component after the L + 1 order
// R table (126 steps for (ds|ds)), with the density contracted first, so no
// integral is formed.  The primitive
// quartets of one shell quartet (the list leaves out those whose product
// factor is below e^-70) fill the lanes; sums over lanes once per quartet.
template <class Dm>
__global__ void __launch_bounds__(256) k_grad_lane(GradLists G, int bra_off, int ket_off, int nrow, int same_class,
                                                   const int64_t *__restrict__ rowstart, const int2 *__restrict__ rowmap,
                                                   int64_t total) {
    constexpr int LA = Dm::LA, LB = Dm::LB, LC = Dm::LC, LD = Dm::LD, LAB = Dm::LAB, LCD = Dm::LCD, N1 = Dm::L + 1;
    constexpr int NH = cart_off(LAB + 2), NK = cart_off(LCD + 1);
    __shared__ double gam[4][Dm::NOUT];
    extern __shared__ double gacc[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool lds = G.nat <= kGradLdsAtoms;
    double *copy = G.copies + (int64_t)(blockIdx.x % kGradCopies) * 3 * G.nat;
    if (lds)
        for (int i = threadIdx.x; i < 3 * G.nat; i += 256) gacc[i] = 0.0;
    __syncthreads();
    double *gm = gam[wave];
    for (int64_t qt = blockIdx.x * (int64_t)4 + wave; qt < total; qt += (int64_t)gridDim.x * 4) {
        const int2 ij = quartet_pairs(rowstart, rowmap, nrow, qt);
        const int ib = bra_off + ij.x, ik = ket_off + ij.y;
        const PairInfo bra = G.pairs[ib], ket = G.pairs[ik];
        const double mult = quartet_mult(bra, ket, same_class && ij.x == ij.y);
        for (int x = lane; x < Dm::NOUT; x += 64) {
            const int a = x / (Dm::NB * Dm::NCD), b = (x / Dm::NCD) % Dm::NB, c = (x / Dm::ND) % Dm::NC, d = x % Dm::ND;
            double sc = 1.0;
            if (LA == 2 && (a == 1 || a == 2 || a == 4)) sc *= kSqrt3;
            if (LB == 2 && (b == 1 || b == 2 || b == 4)) sc *= kSqrt3;
            if (LC == 2 && (c == 1 || c == 2 || c == 4)) sc *= kSqrt3;
            if (LD == 2 && (d == 1 || d == 2 || d == 4)) sc *= kSqrt3;
            gm[x] = sc * grad_weight(G.D, G.N, bra.bfa + a, bra.bfb + b, ket.bfa + c, ket.bfb + d, mult);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const double AC[3] = {bra.Ax - ket.Ax, bra.Ay - ket.Ay, bra.Az - ket.Az};
        const double AB[3] = {bra.ABx, bra.ABy, bra.ABz}, CD[3] = {ket.ABx, ket.ABy, ket.ABz};
        const int nb = G.cnt[ib], nk = G.cnt[ik];
        const GPrim *pb = G.prims + G.off[ib], *pk = G.prims + G.off[ik];
        double g[9] = {};
        for (int x = lane; x < nb * nk; x += 64) {
            const GPrim P = pb[x / nk], Q = pk[x % nk];
            const double spq = rsqrt_nr(P.p + Q.p), alpha = P.p * Q.p * spq * spq;
            const double X[3] = {AC[0] + (P.PAx - Q.PAx), AC[1] + (P.PAy - Q.PAy), AC[2] + (P.PAz - Q.PAz)};
            double F[N1 + 1], R[cart_off(N1 + 1)];
            boys_f64t<N1>(alpha * (X[0] * X[0] + X[1] * X[1] + X[2] * X[2]), G.tabt, F);
            hermite_r<N1>(alpha, X, F, R);
            const double rp = 1.0 / P.p, rq = 1.0 / Q.p;
            const double pref = k2Pi52 * rp * rq * spq * P.K * Q.K;
            Herm1<LA, LB> Eb[3];
            Herm1<LC, LD> Ek[3];
            const double PA[3] = {P.PAx, P.PAy, P.PAz}, QC[3] = {Q.PAx, Q.PAy, Q.PAz};
            static_for<0, 3>([&](auto Di) {
                constexpr int d = decltype(Di)::value;
                Eb[d].build(P.a, 0.5 * rp, PA[d], PA[d] + AB[d]);
                Ek[d].build(Q.a, 0.5 * rq, QC[d], QC[d] + CD[d]);
            });
            double FP[3] = {}, gab[3] = {}, gcd[3] = {};
            static_for<0, Dm::NAB>([&](auto ABi) {
                constexpr int ab = decltype(ABi)::value;
                constexpr Cart ca = comp_of(LA, ab / Dm::NB), cb = comp_of(LB, ab % Dm::NB);
                constexpr int hx = ca.x + cb.x, hy = ca.y + cb.y, hz = ca.z + cb.z;
                using HB = Herm1<LA, LB>;
                using HK = Herm1<LC, LD>;
                // density-weighted ket coefficients (and their C - D derivatives)
                double T[NK], Td[3][NK];
                static_for<0, NK>([&](auto K) {
                    constexpr int k = decltype(K)::value;
                    T[k] = Td[0][k] = Td[1][k] = Td[2][k] = 0.0;
                });
                static_for<0, Dm::NCD>([&](auto CDi) {
                    constexpr int cd = decltype(CDi)::value;
                    constexpr Cart cc = comp_of(LC, cd / Dm::ND), cdd = comp_of(LD, cd % Dm::ND);
                    const double w = gm[ab * Dm::NCD + cd];
                    static_for<0, NK>([&](auto K) {
                        constexpr int k = decltype(K)::value;
                        constexpr Cart kk = cart_of(k);
                        if constexpr (kk.x <= cc.x + cdd.x && kk.y <= cc.y + cdd.y && kk.z <= cc.z + cdd.z) {
                            constexpr int ix = HK::at(cc.x, cdd.x, kk.x), iy = HK::at(cc.y, cdd.y, kk.y),
                                          iz = HK::at(cc.z, cdd.z, kk.z);
                            const double s = (kk.l() & 1) ? -w : w;
                            const double ex = Ek[0].e[ix], ey = Ek[1].e[iy], ez = Ek[2].e[iz];
                            T[k] += s * (ex * ey * ez);
                            Td[0][k] += s * (Ek[0].d[ix] * ey * ez);
                            Td[1][k] += s * (ex * Ek[1].d[iy] * ez);
                            Td[2][k] += s * (ex * ey * Ek[2].d[iz]);
                        }
                    });
                });
                // potentials of the ket's Hermite density at the bra's indices
                double W[NH];
                static_for<0, NH>([&](auto H) {
                    constexpr int h = decltype(H)::value;
                    constexpr Cart c = cart_of(h);
                    constexpr bool need = (c.x <= hx && c.y <= hy && c.z <= hz) || (c.x == hx + 1 && c.y <= hy && c.z <= hz) ||
                                          (c.x <= hx && c.y == hy + 1 && c.z <= hz) || (c.x <= hx && c.y <= hy && c.z == hz + 1);
                    if constexpr (need) {
                        double s = 0.0;
                        static_for<0, NK>([&](auto K) {
                            constexpr int k = decltype(K)::value;
                            constexpr Cart kk = cart_of(k);
                            s += T[k] * R[cart_idx(c.x + kk.x, c.y + kk.y, c.z + kk.z)];
                        });
                        W[h] = s;
                    }
                });
                static_for<0, cart_off(LAB + 1)>([&](auto H) {
                    constexpr int h = decltype(H)::value;
                    constexpr Cart c = cart_of(h);
                    if constexpr (c.x <= hx && c.y <= hy && c.z <= hz) {
                        constexpr int ix = HB::at(ca.x, cb.x, c.x), iy = HB::at(ca.y, cb.y, c.y), iz = HB::at(ca.z, cb.z, c.z);
                        const double ex = Eb[0].e[ix], ey = Eb[1].e[iy], ez = Eb[2].e[iz];
                        const double e = ex * ey * ez;
                        FP[0] += e * W[cart_idx(c.x + 1, c.y, c.z)];
                        FP[1] += e * W[cart_idx(c.x, c.y + 1, c.z)];
                        FP[2] += e * W[cart_idx(c.x, c.y, c.z + 1)];
                        gab[0] += Eb[0].d[ix] * ey * ez * W[h];
                        gab[1] += ex * Eb[1].d[iy] * ez * W[h];
                        gab[2] += ex * ey * Eb[2].d[iz] * W[h];
                        static_for<0, NK>([&](auto K) {
                            constexpr int k = decltype(K)::value;
                            constexpr Cart kk = cart_of(k);
                            const double v = e * R[cart_idx(c.x + kk.x, c.y + kk.y, c.z + kk.z)];
                            gcd[0] += Td[0][k] * v;
                            gcd[1] += Td[1][k] * v;
                            gcd[2] += Td[2][k] * v;
                        });
                    }
                });
            });
            const double fa = P.a * rp * pref, fb = P.b * rp * pref, fc = Q.a * rq * pref;
            static_for<0, 3>([&](auto Di) {
                constexpr int d = decltype(Di)::value;
                g[d] += fa * FP[d] + pref * gab[d];
                g[3 + d] += fb * FP[d] - pref * gab[d];
                g[6 + d] += pref * gcd[d] - fc * FP[d];
            });
        }
        const int atom[4] = {G.sh_atom[bra.sa], G.sh_atom[bra.sb], G.sh_atom[ket.sa], G.sh_atom[ket.sb]};
        grad_add(g, lane, atom, lds ? gacc : copy, lds);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (lds)
        for (int i = threadIdx.x; i < 3 * G.nat; i += 256)
            if (gacc[i] != 0.0) unsafeAtomicAdd(copy + i, gacc[i]);
}

// A_{t,i} = t! / (i! (t - 2i)! 2^i): R_{tuv} = sum_{ijk} A_{ti} X^{t-2i}
// A_{uj} Y^{u-2j} A_{vk} Z^{v-2k} R^{t+u+v-i-j-k}_{000}, the expansion of the
// recursion, so the entries of one table are independent of one another.
constexpr int kHermMax = 10, kHermHalf = 5;
struct HermCoef {
    double c[kHermMax][kHermHalf];
};
constexpr HermCoef make_herm_coef() {
    HermCoef r{};
    for (int t = 0; t < kHermMax; ++t) {
        double v = 1.0;
        for (int i = 0; 2 * i <= t; ++i) {
            r.c[t][i] = v;
            v *= (double)((t - 2 * i) * (t - 2 * i - 1)) / (2.0 * (i + 1));
        }
    }
    return r;
}
__constant__ HermCoef kHermCoef = make_herm_coef();

// R tables are kept by (t, u, v) with v fastest and only t + u + v <= N:
// entry (t, u, v) at row[t (N + 1) + u] + v.
template <int N>
struct RLayout {
    int row[(N + 1) * (N + 1)];
    unsigned char t[cart_off(N + 1)], u[cart_off(N + 1)], v[cart_off(N + 1)];
};
template <int N>
constexpr RLayout<N> make_r_layout() {
    RLayout<N> r{};
    int n = 0;
    for (int t = 0; t <= N; ++t)
        for (int u = 0; u <= N - t; ++u) {
            r.row[t * (N + 1) + u] = n;
            for (int v = 0; v <= N - t - u; ++v) {
                r.t[n] = (unsigned char)t;
                r.u[n] = (unsigned char)u;
                r.v[n] = (unsigned char)v;
                ++n;
            }
        }
    return r;
}
template <int N>
__constant__ RLayout<N> kRLayout = make_r_layout<N>();

// Powers of the components and of the Hermite indices of one class.
template <class Dm>
struct CoopMap {
    static constexpr int NK = cart_off(Dm::LCD + 1), NAB = Dm::NAB, NCD = Dm::NCD;
    unsigned char ab[NAB][6];  // a_x a_y a_z b_x b_y b_z
    unsigned char cd[NCD][6];
    unsigned char k[NK][3];
};
template <class Dm>
constexpr CoopMap<Dm> make_coop_map() {
    CoopMap<Dm> r{};
    for (int i = 0; i < Dm::NAB; ++i) {
        const Cart a = comp_of(Dm::LA, i / Dm::NB), b = comp_of(Dm::LB, i % Dm::NB);
        for (int d = 0; d < 3; ++d) {
            r.ab[i][d] = (unsigned char)a.get(d);
            r.ab[i][3 + d] = (unsigned char)b.get(d);
        }
    }
    for (int i = 0; i < Dm::NCD; ++i) {
        const Cart c = comp_of(Dm::LC, i / Dm::ND), e = comp_of(Dm::LD, i % Dm::ND);
        for (int d = 0; d < 3; ++d) {
            r.cd[i][d] = (unsigned char)c.get(d);
            r.cd[i][3 + d] = (unsigned char)e.get(d);
        }
    }
    for (int i = 0; i < CoopMap<Dm>::NK; ++i)
        for (int d = 0; d < 3; ++d) r.k[i][d] = (unsigned char)cart_of(i).get(d);
    return r;
}
template <class Dm>
__constant__ CoopMap<Dm> kCoopMap = make_coop_map<Dm>();

// bra primitives whose 1-D tables are in LDS at a time (within 64 KB)
template <class Dm>
inline constexpr int kGradChunk = Dm::NAB * Dm::NCD > 1000 ? 4 : 8;

// Bounded by latency: a lane's (ab, k) entry reads three coefficients and
// four R values from LDS for every Hermite index of ab (up to 12), each chain
// behind an index of its own; waves wait on 49 to 56 % of their cycles, issue
// vector work on 22 to 24 % and to the LDS on 6 %.  The ket's density
// T[ab][k] is formed once per ket primitive and shared by the block's waves,
// which take its bra primitives in turn; V[ab][k] (the bra's potential at
// the ket's indices) is summed over them in LDS, and gives the C - D part
// once per ket primitive.
template <class Dm>
__global__ void __launch_bounds__(256) k_grad_coop(GradLists G, int bra_off, int ket_off, int nrow, int same_class,
                                                   const int64_t *__restrict__ rowstart, const int2 *__restrict__ rowmap,
                                                   int64_t total, int ksplit) {
    constexpr int LA = Dm::LA, LB = Dm::LB, LC = Dm::LC, LD = Dm::LD, N1 = Dm::L + 1;
    constexpr int NK = cart_off(Dm::LCD + 1), NAB = Dm::NAB, NCD = Dm::NCD, CH = kGradChunk<Dm>;
    constexpr int NR = cart_off(N1 + 1), NA1 = N1 + 1;
    using HB = Herm1<LA, LB>;
    using HK = Herm1<LC, LD>;
    constexpr int SB = (LA + 1) * (LB + 1) * HB::NT, SK = (LC + 1) * (LD + 1) * HK::NT;
    static_assert(N1 < kHermMax, "Hermite order");
    __shared__ double gam[NAB * NCD], vv[NAB * NK], tt[NAB * NK];
    double *ecd = vv;  // the ket's coefficients, until tt is formed from them
    __shared__ double eb[CH][3][2][SB], ek[3][2][SK];
    __shared__ int2 desc[NAB * NK];
    __shared__ double Rw[4][NR], Aw[4][3][NA1][kHermHalf], Gw[4][NA1];
    __shared__ int rrow[(N1 + 1) * (N1 + 1)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < (N1 + 1) * (N1 + 1); i += 256) rrow[i] = kRLayout<N1>.row[i];
    // every entry (ab, k): offsets of the 1-D tables, Hermite extents of ab
    // and powers of k, packed
    for (int x = tid; x < NAB * NK; x += 256) {
        const unsigned char *c = kCoopMap<Dm>.ab[x / NK], *k = kCoopMap<Dm>.k[x % NK];
        desc[x] = make_int2(HB::at(c[0], c[3], 0) | HB::at(c[1], c[4], 0) << 8 | HB::at(c[2], c[5], 0) << 16,
                            (c[0] + c[3]) | (c[1] + c[4]) << 4 | (c[2] + c[5]) << 8 | k[0] << 12 | k[1] << 16 | k[2] << 20);
    }
    double *copy = G.copies + (int64_t)(blockIdx.x % kGradCopies) * 3 * G.nat;
    auto wsync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int64_t item = blockIdx.x; item < total * ksplit; item += gridDim.x) {
        const int2 ij = quartet_pairs(rowstart, rowmap, nrow, item / ksplit);
        const int ib = bra_off + ij.x, ik = ket_off + ij.y;
        const PairInfo bra = G.pairs[ib], ket = G.pairs[ik];
        const double mult = quartet_mult(bra, ket, same_class && ij.x == ij.y);
        const int nb = G.cnt[ib], nk = G.cnt[ik];
        const GPrim *pb = G.prims + G.off[ib], *pk = G.prims + G.off[ik];
        __syncthreads();  // LDS of the item before
        for (int x = tid; x < Dm::NOUT; x += 256) {
            const int a = x / (Dm::NB * NCD), b = (x / NCD) % Dm::NB, c = (x / Dm::ND) % Dm::NC, d = x % Dm::ND;
            double sc = 1.0;
            if (LA == 2 && (a == 1 || a == 2 || a == 4)) sc *= kSqrt3;
            if (LB == 2 && (b == 1 || b == 2 || b == 4)) sc *= kSqrt3;
            if (LC == 2 && (c == 1 || c == 2 || c == 4)) sc *= kSqrt3;
            if (LD == 2 && (d == 1 || d == 2 || d == 4)) sc *= kSqrt3;
            gam[x] = sc * grad_weight(G.D, G.N, bra.bfa + a, bra.bfb + b, ket.bfa + c, ket.bfb + d, mult);
        }
        const double AC[3] = {bra.Ax - ket.Ax, bra.Ay - ket.Ay, bra.Az - ket.Az};
        const double AB[3] = {bra.ABx, bra.ABy, bra.ABz}, CD[3] = {ket.ABx, ket.ABy, ket.ABz};
        double g[9] = {};
        const int k0 = (int)(item % ksplit);
        for (int kq = k0; kq < nk; kq += ksplit) {
            const GPrim Q = pk[kq];
            const double rq = 1.0 / Q.p;
            const double QC[3] = {Q.PAx, Q.PAy, Q.PAz};
            __syncthreads();  // readers of ek, ecd, tt of the primitive before
            if (tid < 3) {
                HK h;
                const double qc = tid == 0 ? QC[0] : (tid == 1 ? QC[1] : QC[2]);
                const double cd = tid == 0 ? CD[0] : (tid == 1 ? CD[1] : CD[2]);
                h.build(Q.a, 0.5 * rq, qc, qc + cd);
                static_for<0, LC + 1>([&](auto I) { static_for<0, LD + 1>([&](auto J) {
                    static_for<0, decltype(I)::value + decltype(J)::value + 1>([&](auto T) {
                        constexpr int x = HK::at(decltype(I)::value, decltype(J)::value, decltype(T)::value);
                        ek[tid][0][x] = h.e[x];
                        ek[tid][1][x] = h.d[x];
                    });
                }); });
            }
            __syncthreads();
            for (int x = tid; x < NCD * NK; x += 256) {
                const int cd = x / NK, k = x % NK;
                const unsigned char *c = kCoopMap<Dm>.cd[cd], *h = kCoopMap<Dm>.k[k];
                double v = (h[0] + h[1] + h[2]) & 1 ? -1.0 : 1.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) v *= h[d] <= c[d] + c[3 + d] ? ek[d][0][HK::at(c[d], c[3 + d], h[d])] : 0.0;
                ecd[x] = v;
            }
            __syncthreads();
            for (int x = tid; x < NAB * NK; x += 256) {
                const int ab = x / NK, k = x % NK;
                double v = 0.0;
                for (int cd = 0; cd < NCD; ++cd) v += gam[ab * NCD + cd] * ecd[cd * NK + k];
                tt[x] = v;
            }
            __syncthreads();
            for (int x = tid; x < NAB * NK; x += 256) vv[x] = 0.0;
            for (int c0 = 0; c0 < nb; c0 += CH) {
                __syncthreads();  // tt, vv written; eb read by the chunk before
                if (tid < 3 * CH && c0 + tid / 3 < nb) {
                    const GPrim P = pb[c0 + tid / 3];
                    const int d = tid % 3;
                    HB h;
                    const double pa = d == 0 ? P.PAx : (d == 1 ? P.PAy : P.PAz);
                    const double abd = d == 0 ? AB[0] : (d == 1 ? AB[1] : AB[2]);
                    h.build(P.a, 0.5 / P.p, pa, pa + abd);
                    static_for<0, LA + 1>([&](auto I) { static_for<0, LB + 1>([&](auto J) {
                        static_for<0, decltype(I)::value + decltype(J)::value + 1>([&](auto T) {
                            constexpr int x = HB::at(decltype(I)::value, decltype(J)::value, decltype(T)::value);
                            eb[tid / 3][d][0][x] = h.e[x];
                            eb[tid / 3][d][1][x] = h.d[x];
                        });
                    }); });
                }
                __syncthreads();
                for (int ci = wave; ci < CH && c0 + ci < nb; ci += 4) {
                    const GPrim P = pb[c0 + ci];
                    const double spq = rsqrt_nr(P.p + Q.p), alpha = P.p * Q.p * spq * spq, rp = 1.0 / P.p;
                    const double X[3] = {AC[0] + (P.PAx - Q.PAx), AC[1] + (P.PAy - Q.PAy), AC[2] + (P.PAz - Q.PAz)};
                    const double Tb = alpha * (X[0] * X[0] + X[1] * X[1] + X[2] * X[2]);
                    const double pref = k2Pi52 * rp * rq * spq * P.K * Q.K;
                    wsync();  // readers of this wave's tables of the primitive before
                    if (lane <= N1) {
                        // F_lane(T): Taylor sum about T_k = k/16, or the large-T form
                        double f, m2a = 1.0;
                        if (Tb < kBoysTmax) {
                            const int kk = __double2int_rn(Tb * kBoysInvStep);
                            const double md = (double)kk * (1.0 / kBoysInvStep) - Tb;
                            const double *row = G.tab + kk * kBoysN + lane;
                            const int nt = min(8, kBoysN - lane);
                            f = row[nt - 1];
                            for (int i = nt - 2; i >= 0; --i) f = row[i] + md * f / (i + 1);
                        } else {
                            const double sT = rsqrt_nr(Tb), rT = sT * sT;
                            f = 0.88622692545275801365 * sT;
                            for (int n = 0; n < lane; ++n) f *= (n + 0.5) * rT;
                        }
                        for (int n = 0; n < lane; ++n) m2a *= -2.0 * alpha;
                        Gw[wave][lane] = m2a * f;
                    }
                    if (lane < 3 * NA1) {
                        const int d = lane / NA1, t = lane % NA1;
                        const double x = d == 0 ? X[0] : (d == 1 ? X[1] : X[2]), x2 = x * x;
                        double pw = t & 1 ? x : 1.0;
                        for (int i = t / 2; i >= 0; --i) {
                            Aw[wave][d][t][i] = kHermCoef.c[t][i] * pw;
                            pw *= x2;
                        }
                    }
                    wsync();
                    for (int r = lane; r < NR; r += 64) {
                        const int t = kRLayout<N1>.t[r], u = kRLayout<N1>.u[r], v = kRLayout<N1>.v[r];
                        double s = 0.0;
                        for (int i = 0; 2 * i <= t; ++i)
                            for (int j = 0; 2 * j <= u; ++j) {
                                const double aij = Aw[wave][0][t][i] * Aw[wave][1][u][j];
                                for (int k = 0; 2 * k <= v; ++k)
                                    s += aij * Aw[wave][2][v][k] * Gw[wave][t + u + v - i - j - k];
                            }
                        Rw[wave][r] = s;
                    }
                    wsync();
                    const double *R = Rw[wave];
                    double FP[3] = {}, gab[3] = {};
                    for (int x = lane; x < NAB * NK; x += 64) {
                        const int2 ds = desc[x];
                        const double *Ex = eb[ci][0][0] + (ds.x & 255), *Dx = Ex + SB;
                        const double *Ey = eb[ci][1][0] + (ds.x >> 8 & 255), *Dy = Ey + SB;
                        const double *Ez = eb[ci][2][0] + (ds.x >> 16), *Dz = Ez + SB;
                        const int nx = ds.y & 15, ny = ds.y >> 4 & 15, nz = ds.y >> 8 & 15;
                        const int kx = ds.y >> 12 & 15, ky = ds.y >> 16 & 15, kz = ds.y >> 20;
                        double v = 0.0, vx = 0.0, vy = 0.0, vz = 0.0, wx = 0.0, wy = 0.0, wz = 0.0;
                        for (int t = 0; t <= nx; ++t)
                            for (int u = 0; u <= ny; ++u) {
                                const double exy = Ex[t] * Ey[u], dxy = Dx[t] * Ey[u], xdy = Ex[t] * Dy[u];
                                const int *rr = rrow + (t + kx) * (N1 + 1) + u + ky;
                                const double *r0 = R + rr[0] + kz, *rx = R + rr[N1 + 1] + kz, *ry = R + rr[1] + kz;
                                double s = 0.0;
                                for (int z = 0; z <= nz; ++z) {
                                    const double ez = Ez[z], r = r0[z], ezr = ez * r;
                                    s += ezr;
                                    vx += exy * ez * rx[z];
                                    vy += exy * ez * ry[z];
                                    vz += exy * ez * r0[z + 1];
                                    wz += exy * Dz[z] * r;
                                }
                                v += exy * s;
                                wx += dxy * s;
                                wy += xdy * s;
                            }
                        const double tk = tt[x];
                        __hip_atomic_fetch_add(&vv[x], pref * v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        FP[0] += tk * vx;
                        FP[1] += tk * vy;
                        FP[2] += tk * vz;
                        gab[0] += tk * wx;
                        gab[1] += tk * wy;
                        gab[2] += tk * wz;
                    }
                    const double fa = P.a * rp * pref, fb = P.b * rp * pref, fc = Q.a * rq * pref;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        g[d] += fa * FP[d] + pref * gab[d];
                        g[3 + d] += fb * FP[d] - pref * gab[d];
                        g[6 + d] -= fc * FP[d];
                    }
                }
            }
            // C - D part
            __syncthreads();
            for (int x = tid; x < NAB * NK; x += 256) {
                const int ab = x / NK, k = x % NK;
                const unsigned char *h = kCoopMap<Dm>.k[k];
                double sx = 0.0, sy = 0.0, sz = 0.0;
                for (int cd = 0; cd < NCD; ++cd) {
                    const unsigned char *c = kCoopMap<Dm>.cd[cd];
                    if (h[0] > c[0] + c[3] || h[1] > c[1] + c[4] || h[2] > c[2] + c[5]) continue;
                    const int ix = HK::at(c[0], c[3], h[0]), iy = HK::at(c[1], c[4], h[1]), iz = HK::at(c[2], c[5], h[2]);
                    const double w = gam[ab * NCD + cd];
                    sx += w * ek[0][1][ix] * ek[1][0][iy] * ek[2][0][iz];
                    sy += w * ek[0][0][ix] * ek[1][1][iy] * ek[2][0][iz];
                    sz += w * ek[0][0][ix] * ek[1][0][iy] * ek[2][1][iz];
                }
                const double v = (h[0] + h[1] + h[2]) & 1 ? -vv[x] : vv[x];
                g[6] += sx * v;
                g[7] += sy * v;
                g[8] += sz * v;
            }
        }
        const int atom[4] = {G.sh_atom[bra.sa], G.sh_atom[bra.sb], G.sh_atom[ket.sa], G.sh_atom[ket.sb]};
        grad_add(g, lane, atom, copy, false);
    }
}

template <>
int GradOps<MESS_GCB, MESS_GCK>::run(const GradLists &G, const ClassLaunch &L) {
    using Dm = ClassOf<MESS_GCB, MESS_GCK>;
    if (L.total <= 0) return MESS_OK;
    if constexpr (MESS_GCB < 4 || (MESS_GCB == 4 && MESS_GCK <= 1) || MESS_GCK == 0) {
        // four quartets a block; up to 8 blocks a CU, then blocks loop
        const int64_t g = std::min<int64_t>((L.total + 3) / 4, 2048);
        const size_t lds = G.nat <= kGradLdsAtoms ? sizeof(double) * 3 * G.nat : 0;
        hipLaunchKernelGGL((k_grad_lane<Dm>), dim3((unsigned)g), dim3(256), lds, L.stream, G, L.bra_off, L.ket_off, L.nbra,
                           L.same_class, L.rowstart, L.rowmap, L.total);
    } else {
        // ket primitives split over blocks until about 4096 of them: a block's
        // primitives are a serial chain ((dd|dd) of 3 waters 2.6 -> 1.6 ms
        // from 8 to 16 shares)
        const int ks = (int)std::max<int64_t>(1, std::min<int64_t>(16, 4096 / L.total));
        const int64_t g = std::min<int64_t>(L.total * ks, 1 << 20);
        hipLaunchKernelGGL((k_grad_coop<Dm>), dim3((unsigned)g), dim3(256), 0, L.stream, G, L.bra_off, L.ket_off, L.nbra,
                           L.same_class, L.rowstart, L.rowmap, L.total, ks);
    }
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

}  // namespace mess
