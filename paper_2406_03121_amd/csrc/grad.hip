// Analytic nuclear gradient of the closed-shell Hartree-Fock energy (the
// atomic forces the paper obtains by differentiating its energy, sections 1
// and 4):
//
//   dE/dR_X = sum_{mu nu} D_{mu nu} dH_{mu nu}/dR_X
//           + 1/2 sum_{mu nu la si} P_{mu nu la si} d(mu nu|la si)/dR_X
//           - sum_{mu nu} W_{mu nu} dS_{mu nu}/dR_X + dE_nuc/dR_X,
//
// D the converged density, F its Fock matrix, W = D F D / 2 (energy-weighted
// density; the orthonormality constraint's term), and the symmetrised
// two-particle density P = D_{mu nu} D_{la si} - (D_{mu la} D_{nu si} +
// D_{mu si} D_{nu la}) / 4.  Only basis functions on atom X (and, for the
// nuclear attraction, the operator 1/|r - R_X|) depend on R_X; D and F need
// no response because the SCF energy is stationary.
//
// Integral derivatives by Hermite Gaussians (grad.hpp states the algebra):
// a shell pair's centres enter through the product centre and through A - B,
// and the density is contracted first, so no derivative integral is formed:
//   overlap (pi/p)^{3/2} K_AB prod_k E^{i_k j_k}_0, kinetic from d^2/dx^2 of
//   the ket factor, differentiated as 2a E^{i+1,j} - i E^{i-1,j} on each
//   centre in turn,
//   nuclear attraction -Z_C (2 pi / p) K_AB sum_tuv E_t E_u E_v R_tuv(p, P - C)
//   with d/dC = -(d/dA + d/dB) for each nucleus C,
//   and the two-electron part class by class in grad_class.hip.
//
// One-electron part: a wave per unordered shell pair, its lanes over the
// primitive pairs (overlap, kinetic) and over nucleus x primitive pair
// (attraction).  Two-electron part: the basis's work lists (unique quartets
// that pass the Schwarz test) with a primitive-pair list of its own, which
// keeps every pair whose Gaussian product factor is above e^-70: with
// exponents to 5000 and their derivative factors what is left out stays
// below 1e-18 of an integral derivative.  Kernels add into kGradCopies
// copies of the gradient (a block's atomics would otherwise meet on the few
// cache lines of 3 n_atoms values), summed at the end.  At 45 functions (3
// waters, s to d) the call takes 6.0 ms (9.6 with its classes one after
// another), 1540 before with every Hermite array of a lane's primitive
// quartet in scratch memory and every centre's derivative formed from the
// integrals' expansion.
#include <algorithm>
#include <cmath>
#include <vector>

#include "grad.hpp"
#include "linalg.hpp"

namespace mess {

int zero_async(double *p, int64_t n, hipStream_t s);
int get_work_lists(mess_basis *B, double tau, hipStream_t s, WorkLists **out);
int fill_class_launch(const mess_basis *B, const ClassList &cl, hipStream_t s, ClassLaunch &L);

constexpr double kGradPairExp = 70.0;  // pairs with alpha beta / p |AB|^2 above this are left out

// Primitive pairs of every sorted shell pair, a wave each: the kept ones
// compacted in order.
__global__ void __launch_bounds__(256) k_grad_prims(int npair, const PairInfo *__restrict__ pairs,
                                                    const int *__restrict__ sh_prim0, const int *__restrict__ sh_np,
                                                    const double *__restrict__ alpha, const double *__restrict__ ct,
                                                    const int *__restrict__ off, int *__restrict__ cnt,
                                                    GPrim *__restrict__ prims) {
    const int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= npair) return;
    const PairInfo pr = pairs[i];
    const int na = sh_np[pr.sa], nb = sh_np[pr.sb], a0 = sh_prim0[pr.sa], b0 = sh_prim0[pr.sb];
    const double r2 = pr.ABx * pr.ABx + pr.ABy * pr.ABy + pr.ABz * pr.ABz;
    int n = 0;
    for (int x0 = 0; x0 < na * nb; x0 += 64) {
        const int x = x0 + lane;
        GPrim g{};
        bool keep = false;
        if (x < na * nb) {
            const int u = a0 + x / nb, v = b0 + x % nb;
            g.a = alpha[u];
            g.b = alpha[v];
            g.p = g.a + g.b;
            const double mu = g.a * g.b / g.p * r2, f = -g.b / g.p;
            keep = mu <= kGradPairExp;
            g.K = ct[u] * ct[v] * exp(-mu);
            g.PAx = f * pr.ABx;
            g.PAy = f * pr.ABy;
            g.PAz = f * pr.ABz;
        }
        const unsigned long long m = __ballot(keep);
        if (keep) prims[off[i] + n + __popcll(m & ((1ull << lane) - 1))] = g;
        n += __popcll(m);
    }
    if (lane == 0) cnt[i] = n;
}

// ------------------------------------------------------------ one-electron

// Energy gradient of D (T + V) - W S over the pairs [off, off + n) of one
// pair class, a wave each; the work is small (one launch of a few us beside
// the two-electron part), so a pair's nuclei and primitive pairs share the
// lanes and the sums leave by one atomic per value.
template <int LA, int LB>
__global__ void __launch_bounds__(64) k_grad_1e(GradLists G, int off, const double *__restrict__ xyz,
                                                const double *__restrict__ Zc, const double *__restrict__ W) {
    constexpr int NA = ncart(LA), NB = ncart(LB), LAB = LA + LB;
    __shared__ double dm[NA * NB], fn[64 * 3];
    const int lane = threadIdx.x;
    const PairInfo pr = G.pairs[off + blockIdx.x];
    const GPrim *pp = G.prims + G.off[off + blockIdx.x];
    const int np = G.cnt[off + blockIdx.x], N = G.N;
    double *copy = G.copies + (int64_t)(blockIdx.x % kGradCopies) * 3 * G.nat;
    // block (a, b) and, for two different shells, block (b, a) too
    const double both = pr.sa == pr.sb ? 0.5 : 1.0;
    for (int x = lane; x < NA * NB; x += 64) {
        const int a = x / NB, b = x % NB;
        double sc = both;
        if (LA == 2 && (a == 1 || a == 2 || a == 4)) sc *= kSqrt3;
        if (LB == 2 && (b == 1 || b == 2 || b == 4)) sc *= kSqrt3;
        const int64_t mn = (int64_t)(pr.bfa + a) * N + pr.bfb + b, nm = (int64_t)(pr.bfb + b) * N + pr.bfa + a;
        dm[x] = sc * (G.D[mn] + G.D[nm]);
    }
    __syncthreads();
    const double AB[3] = {pr.ABx, pr.ABy, pr.ABz};
    double gA[3] = {}, gB[3] = {};
    // overlap and kinetic energy: each centre's derivative on its own, for the
    // ordered pairs (a, b) and (b, a)
    auto ordered = [&](auto L1c, auto L2c, bool swapped, double(&g)[3]) {
        constexpr int L1 = decltype(L1c)::value, L2 = decltype(L2c)::value, N1 = ncart(L1), N2 = ncart(L2);
        const int at1 = 3 * G.sh_atom[swapped ? pr.sb : pr.sa], at2 = 3 * G.sh_atom[swapped ? pr.sa : pr.sb];
        const int f1 = swapped ? pr.bfb : pr.bfa, f2 = swapped ? pr.bfa : pr.bfb;
        for (int x = lane; x < np; x += 64) {
            const GPrim P = pp[x];
            const double a = swapped ? P.b : P.a, b = swapped ? P.a : P.b, p = P.p;
            using H = Herm1<L1 + 1, L2 + 2>;
            H E[3];
            static_for<0, 3>([&](auto Di) {
                constexpr int d = decltype(Di)::value;
                // distances from the product centre's coordinates, rounded
                // as one fused step (a tight pair's kinetic derivative
                // multiplies their last bit by alpha^2)
                const double c1 = xyz[at1 + d], c2 = xyz[at2 + d], c = fma(b, c2, a * c1) / p;
                E[d].build(a, 0.5 / p, c - c1, c - c2);
            });
            const double sq = sqrt(M_PI / p);
            static_for<0, N1 * N2>([&](auto Ci) {
                constexpr int i1 = decltype(Ci)::value / N2, i2 = decltype(Ci)::value % N2;
                constexpr Cart ca = comp_of(L1, i1), cb = comp_of(L2, i2);
                double S[3], T[3], dS[3], dT[3];
                static_for<0, 3>([&](auto Di) {
                    constexpr int d = decltype(Di)::value, i = ca.get(d), j = cb.get(d);
                    auto s1 = [&](auto I, auto J) { return E[d].e[H::at(decltype(I)::value, decltype(J)::value, 0)] * sq; };
                    auto t1 = [&](auto I) {
                        double v = 0.0;
                        if constexpr (j >= 2) v = j * (j - 1) * s1(I, std::integral_constant<int, j - 2>{});
                        return -0.5 * (v - 2.0 * b * (2 * j + 1) * s1(I, std::integral_constant<int, j>{}) +
                                       4.0 * b * b * s1(I, std::integral_constant<int, j + 2>{}));
                    };
                    using Ii = std::integral_constant<int, i>;
                    using Iu = std::integral_constant<int, i + 1>;
                    using Jj = std::integral_constant<int, j>;
                    S[d] = s1(Ii{}, Jj{});
                    T[d] = t1(Ii{});
                    dS[d] = 2.0 * a * s1(Iu{}, Jj{});
                    dT[d] = 2.0 * a * t1(Iu{});
                    if constexpr (i > 0) {
                        using Id = std::integral_constant<int, i - 1>;
                        dS[d] -= i * s1(Id{}, Jj{});
                        dT[d] -= i * t1(Id{});
                    }
                });
                const int64_t mn = (int64_t)(f1 + i1) * N + f2 + i2;
                const double w = 2.0 * comp_sc(ca) * comp_sc(cb) * P.K, wd = w * G.D[mn], ww = w * W[mn];
                static_for<0, 3>([&](auto Di) {
                    constexpr int k = decltype(Di)::value, k1 = (k + 1) % 3, k2 = (k + 2) % 3;
                    const double t = dT[k] * S[k1] * S[k2] + dS[k] * (T[k1] * S[k2] + S[k1] * T[k2]);
                    g[k] += wd * t - ww * (dS[k] * S[k1] * S[k2]);
                });
            });
        }
    };
    using std::integral_constant;
    ordered(integral_constant<int, LA>{}, integral_constant<int, LB>{}, false, gA);
    if (pr.sa != pr.sb) ordered(integral_constant<int, LB>{}, integral_constant<int, LA>{}, true, gB);
    // nuclear attraction: lane = nucleus of a chunk x share of the primitive pairs
    for (int c0 = 0; c0 < G.nat; c0 += 64) {
        const int nc = min(G.nat - c0, 64), share = 64 / nc;
        const int c = lane % nc, first = lane / nc;
        double f[3] = {};
        if (first < share) {
            const double A0 = pr.Ax - xyz[3 * (c0 + c)], A1 = pr.Ay - xyz[3 * (c0 + c) + 1], A2 = pr.Az - xyz[3 * (c0 + c) + 2];
            const double z = -2.0 * M_PI * Zc[c0 + c];
            for (int x = first; x < np; x += share) {
                const GPrim P = pp[x];
                const double PA[3] = {P.PAx, P.PAy, P.PAz}, X[3] = {A0 + PA[0], A1 + PA[1], A2 + PA[2]};
                const double rp = 1.0 / P.p, pref = z * rp * P.K;
                double F[LAB + 2], R[cart_off(LAB + 2)];
                boys_f64t<LAB + 1>(P.p * (X[0] * X[0] + X[1] * X[1] + X[2] * X[2]), G.tabt, F);
                hermite_r<LAB + 1>(P.p, X, F, R);
                using H = Herm1<LA, LB>;
                H E[3];
                static_for<0, 3>([&](auto Di) {
                    constexpr int d = decltype(Di)::value;
                    E[d].build(P.a, 0.5 * rp, PA[d], PA[d] + AB[d]);
                });
                double FP[3] = {}, g[3] = {};
                static_for<0, NA * NB>([&](auto ABi) {
                    constexpr int ab = decltype(ABi)::value;
                    constexpr Cart ca = comp_of(LA, ab / NB), cb = comp_of(LB, ab % NB);
                    static_for<0, cart_off(LAB + 1)>([&](auto Hi) {
                        constexpr Cart h = cart_of(decltype(Hi)::value);
                        if constexpr (h.x <= ca.x + cb.x && h.y <= ca.y + cb.y && h.z <= ca.z + cb.z) {
                            constexpr int ix = H::at(ca.x, cb.x, h.x), iy = H::at(ca.y, cb.y, h.y), iz = H::at(ca.z, cb.z, h.z);
                            const double w = dm[ab], ex = E[0].e[ix], ey = E[1].e[iy], ez = E[2].e[iz];
                            const double e = w * (ex * ey * ez), r = w * R[h.idx()];
                            FP[0] += e * R[h.plus(0).idx()];
                            FP[1] += e * R[h.plus(1).idx()];
                            FP[2] += e * R[h.plus(2).idx()];
                            g[0] += E[0].d[ix] * ey * ez * r;
                            g[1] += ex * E[1].d[iy] * ez * r;
                            g[2] += ex * ey * E[2].d[iz] * r;
                        }
                    });
                });
                static_for<0, 3>([&](auto Di) {
                    constexpr int d = decltype(Di)::value;
                    gA[d] += pref * (P.a * rp * FP[d] + g[d]);
                    gB[d] += pref * (P.b * rp * FP[d] - g[d]);
                    f[d] -= pref * FP[d];
                });
            }
        }
        for (int i = lane; i < 3 * nc; i += 64) fn[i] = 0.0;
        __syncthreads();
        if (first < share)
            for (int d = 0; d < 3; ++d)
                __hip_atomic_fetch_add(&fn[3 * c + d], f[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
        for (int i = lane; i < 3 * nc; i += 64) unsafeAtomicAdd(copy + 3 * c0 + i, fn[i]);
        __syncthreads();
    }
    for (int k = 0; k < 3; ++k)
        for (int o = 32; o > 0; o >>= 1) {
            gA[k] += __shfl_xor(gA[k], o, 64);
            gB[k] += __shfl_xor(gB[k], o, 64);
        }
    if (lane < 3) {
        unsafeAtomicAdd(copy + 3 * G.sh_atom[pr.sa] + lane, lane == 0 ? gA[0] : (lane == 1 ? gA[1] : gA[2]));
        unsafeAtomicAdd(copy + 3 * G.sh_atom[pr.sb] + lane, lane == 0 ? gB[0] : (lane == 1 ? gB[1] : gB[2]));
    }
}

// The gradient: the copies' sum plus dE_nuc/dR_A = -sum_B Z_A Z_B (R_A - R_B)
// / |R_A - R_B|^3, a thread per atom and direction.
__global__ void k_grad_finish(int nat, const double *__restrict__ xyz, const double *__restrict__ Zc,
                              const double *__restrict__ copies, double *__restrict__ grad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, a = i / 3, k = i % 3;
    if (a >= nat) return;
    double g = 0.0;
    for (int c = 0; c < kGradCopies; ++c) g += copies[(int64_t)c * 3 * nat + i];
    for (int b = 0; b < nat; ++b) {
        if (b == a) continue;
        const double d[3] = {xyz[3 * a] - xyz[3 * b], xyz[3 * a + 1] - xyz[3 * b + 1], xyz[3 * a + 2] - xyz[3 * b + 2]};
        const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        g -= Zc[a] * Zc[b] / (r2 * sqrt(r2)) * d[k];
    }
    grad[i] = g;
}

void free_grad(mess_basis *B) {
    hipFree(B->grad_ws);
    B->grad_ws = nullptr;
    B->grad_ws_bytes = 0;
}

}  // namespace mess

using namespace mess;

extern "C" int mess_hf_gradient(const mess_basis *basis, const double *D, const double *F, double schwarz_tol,
                                double *grad, mess_stream stream) {
    if (!basis || !D || !F || !grad) {
        set_error("mess_hf_gradient: NULL argument");
        return MESS_E_ARG;
    }
    auto *B = const_cast<mess_basis *>(basis);
    if (B->n_mol != 1) {
        set_error("mess_hf_gradient: a batch of %d molecules; the gradient is built for one molecule", B->n_mol);
        return MESS_E_UNSUPPORTED;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int N = B->nbf, nat = B->nat, nsh = B->nsh, npair = B->npair;
    WorkLists *W = nullptr;
    MESS_TRY(get_work_lists(B, schwarz_tol > 0.0 ? schwarz_tol : 0.0, s, &W));
    const size_t np = B->alpha.size();
    // host tables in one block: exponents, coefficients, then shell and pair indices
    std::vector<int> hi(3 * (size_t)nsh + npair);
    int64_t nprim = 0;
    for (int i = 0; i < nsh; ++i) {
        hi[i] = B->sh_prim0[i];
        hi[nsh + i] = B->sh_np[i];
        hi[2 * nsh + i] = B->sh_atom[i];
    }
    for (int i = 0; i < npair; ++i) {
        hi[3 * (size_t)nsh + i] = (int)nprim;
        nprim += (int64_t)B->sh_np[B->pairs_host[i].sa] * B->sh_np[B->pairs_host[i].sb];
    }
    if (nprim > INT32_MAX) {
        set_error("mess_hf_gradient: %lld primitive pairs", (long long)nprim);
        return MESS_E_SIZE;
    }
    const size_t tab_bytes = (sizeof(double) * 2 * np + sizeof(int) * hi.size() + 63) / 64 * 64;
    std::vector<char> tab(tab_bytes);
    std::copy(B->alpha.begin(), B->alpha.end(), reinterpret_cast<double *>(tab.data()));
    std::copy(B->ctilde.begin(), B->ctilde.end(), reinterpret_cast<double *>(tab.data()) + np);
    std::copy(hi.begin(), hi.end(), reinterpret_cast<int *>(tab.data() + sizeof(double) * 2 * np));
    // one workspace, kept in the basis
    const size_t bytes = tab_bytes + sizeof(GPrim) * nprim +
                         sizeof(double) * (2 * (size_t)N * N + 3 * (size_t)nat * (kGradCopies + 1)) + sizeof(int) * npair;
    if (bytes > B->grad_ws_bytes) {
        MESS_HIP(hipStreamSynchronize(s));
        free_grad(B);
        if (hipMalloc(&B->grad_ws, bytes) != hipSuccess) {
            B->grad_ws = nullptr;
            set_error("mess_hf_gradient: device allocation of %zu bytes failed", bytes);
            return MESS_E_NOMEM;
        }
        B->grad_ws_bytes = bytes;
    }
    char *ws = static_cast<char *>(B->grad_ws);
    auto *d_alpha = reinterpret_cast<double *>(ws);
    auto *d_prim0 = reinterpret_cast<int *>(ws + sizeof(double) * 2 * np);
    auto *prims = reinterpret_cast<GPrim *>(ws + tab_bytes);
    auto *d_T = reinterpret_cast<double *>(prims + nprim), *d_W = d_T + (size_t)N * N;
    double *copies = d_W + (size_t)N * N, *d_g = copies + 3 * (size_t)nat * kGradCopies;
    int *cnt = reinterpret_cast<int *>(d_g + 3 * nat), *off = d_prim0 + 3 * nsh;
    // however this returns, the stream is waited for first: the copy reads tab
    struct Wait {
        hipStream_t s;
        bool due = true;
        ~Wait() { if (due) (void)hipStreamSynchronize(s); }
    } wait{s};
    MESS_HIP(hipMemcpyAsync(ws, tab.data(), tab_bytes, hipMemcpyHostToDevice, s));
    MESS_TRY(zero_async(copies, 3 * (int64_t)nat * kGradCopies, s));
    hipLaunchKernelGGL(k_grad_prims, dim3((unsigned)((npair + 3) / 4)), dim3(256), 0, s, npair, B->d_pairs, d_prim0,
                       d_prim0 + nsh, d_alpha, d_alpha + np, off, cnt, prims);
    // W = D F D / 2
    MESS_TRY(gemm(s, false, false, N, N, N, 1.0, D, N, F, N, 0.0, d_T, N));
    MESS_TRY(gemm(s, false, false, N, N, N, 0.5, d_T, N, D, N, 0.0, d_W, N));
    const GradLists G{B->d_pairs, prims, off, cnt, d_prim0 + 2 * nsh, B->d_boys, B->d_boys_t, D, N, nat, copies};
    auto one = [&](auto kernel, int cls) {
        const int n = B->pair_class_off[cls + 1] - B->pair_class_off[cls];
        if (n > 0)
            hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(64), 0, s, G, B->pair_class_off[cls], B->d_xyz, B->d_Zd, d_W);
    };
    one(k_grad_1e<0, 0>, 0);
    one(k_grad_1e<1, 0>, 1);
    one(k_grad_1e<1, 1>, 2);
    one(k_grad_1e<2, 0>, 3);
    one(k_grad_1e<2, 1>, 4);
    one(k_grad_1e<2, 2>, 5);
    MESS_LAUNCH_CHECK();
    std::vector<const ClassList *> act;
    std::vector<double> cost;
    for (const ClassList &cl : W->classes) {
        if (cl.total == 0) continue;
        double fp = 0.0, fq = 0.0;
        class_flops(cl.cb, cl.ck, &fp, &fq);
        act.push_back(&cl);
        cost.push_back(fp * (double)cl.prim_quartets + fq * (double)cl.total);
    }
    MESS_TRY(run_forked(s, cost, [&](int i, hipStream_t st) {
        const ClassList &cl = *act[i];
        ClassLaunch L;
        MESS_TRY(fill_class_launch(B, cl, st, L));
        return dispatch_class(cl.cb, cl.ck, [&](auto CB, auto CK) {
            return GradOps<decltype(CB)::value, decltype(CK)::value>::run(G, L);
        });
    }));
    hipLaunchKernelGGL(k_grad_finish, dim3((unsigned)((3 * nat + 63) / 64)), dim3(64), 0, s, nat, B->d_xyz, B->d_Zd,
                       copies, d_g);
    MESS_LAUNCH_CHECK();
    MESS_HIP(hipMemcpyAsync(grad, d_g, sizeof(double) * 3 * nat, hipMemcpyDeviceToHost, s));
    wait.due = false;
    MESS_HIP(hipStreamSynchronize(s));
    return MESS_OK;
}
