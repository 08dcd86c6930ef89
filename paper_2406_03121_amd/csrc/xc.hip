// LDA exchange on an atom-centred molecular grid (paper section 5 names the
// local density approximation as the exchange-correlation choice of its
// batched example; functional and grid are this library's readings):
//
//   Dirac-Slater exchange  e_x(rho) = -C_x rho^(4/3),  C_x = (3/4)(3/pi)^(1/3),
//   v_x = de_x/drho = -(3/pi)^(1/3) rho^(1/3)  (points with rho <= 0 add nothing);
//   rho_g = sum_{mu nu} Phi_{g mu} D_{mu nu} Phi_{g nu},
//   E_x = sum_g w_g e_x(rho_g),  V_x = Phi^T diag(w v_x) Phi.
//
// Grid per atom: 75 second-kind Gauss-Chebyshev radial nodes
// x_i = cos(i pi / 76) mapped by r = (1 + x)/(1 - x) bohr, times a product
// angular rule of 17 Gauss-Legendre nodes in cos(theta) and 34 equally
// spaced azimuths; Becke fuzzy-cell weights (three smoothing iterations, no
// size adjustment).  Points are ordered atom, radial node, theta, azimuth.
//
// Device layout: the grid as [G][4] (x, y, z, w) and the basis values
// transposed, PhiT[mu][g] with G (the point count rounded up to 64)
// contiguous, so that the basis-value kernel writes coalesced rows and both
// contractions stream G-contiguous tiles.  Both are built once per basis.
// Per density, both contractions on the FP64 matrix cores: one kernel forms
// U = D PhiT for a tile of points held in LDS and reduces rho_g = sum_nu
// PhiT[nu][g] U[nu][g] in the same pass (with D + D^T above the diagonal
// blocks and nothing below: N^2 flops per point), then the weights f_g = w_g
// v_x(rho_g); a second kernel forms V_x = PhiT diag(f) PhiT^T on 64 x 64
// tiles of the upper block triangle over chunks of points (N^2 flops per
// point), whose partial sums are added in a fixed order.
//
// PBE exchange-correlation (the generalised-gradient functional the paper
// selects for its DFT examples, section 5), closed shell, on the same grid:
//   f(rho, sigma) = rho eps_x^unif F_x(s) + rho (eps_c^PW92(r_s) + H(r_s, t)),
//   sigma = |grad rho|^2, grad rho = 2 sum_{mu nu} D_{mu nu} phi_mu grad phi_nu,
//   E_xc = sum_g w_g f_g,
//   V_xc[mu][nu] = sum_g w_g [f_rho phi_mu phi_nu
//                             + 2 f_sigma grad rho . (phi_mu grad phi_nu + grad phi_mu phi_nu)],
// with the partial derivatives f_rho, f_sigma written out analytically
// (pbe_point); points with rho < 1e-10 add nothing.  The basis gradients
// dPhiT[k][mu][g] (k = x, y, z) are built on the first PBE call.  Per
// density: U = D PhiT per 64-point tile reduced against PhiT and the three
// dPhiT (rho and grad rho in one pass, 2 N^2 + 6 N flops per point), the
// functional per point, and V_xc = PhiT Z^T + Z PhiT^T with
// Z[nu][g] = w (f_rho/2 phi_nu + 2 f_sigma grad rho . grad phi_nu) formed
// while the tiles are staged (all tile pairs, 2 N^2 flops per point; at a
// hundred functions both passes are bound by the 32 bytes per function and
// point that they read).
#include <algorithm>
#include <cmath>
#include <vector>

#include "eri_hgp.hpp"
#include "mess_internal.hpp"

namespace mess {

constexpr int kNRad = 75, kNTheta = 17, kNPhi = 34, kNAng = kNTheta * kNPhi;
constexpr int kPtsPerAtom = kNRad * kNAng;
constexpr int kXT = 64;      // points are padded to a multiple of this; edge of a V_x tile

struct XcShell {
    double x, y, z;
    int l, prim0, nprim, bf0;
};

struct XcGrid {
    int64_t npts = 0, G = 0;
    int nbf = 0;
    double *dphiT = nullptr;  // [3][nbf][G] basis gradients (PBE only)
    double *grad = nullptr;   // [3][G] grad rho (PBE)
    double *hv = nullptr;     // [3][G] 2 w f_sigma grad rho (PBE)
    double *xyzw = nullptr;   // [G][4]
    double *phiT = nullptr;   // [nbf][G]
    double *f = nullptr;      // [G] w_g v_x(rho_g)
    double *rho = nullptr;    // [G]
    double *epart = nullptr;  // [G / 16] partial sums of w_g e_x
    double *Dp = nullptr;     // D in fragment order
    double *vpart[2] = {};    // partial sums of V_x tiles, LDA and PBE
    int4 *groups = nullptr;   // V_x tile groups (VGroup), LDA then PBE
    double *ex = nullptr;     // [1] E_x of the last build
    double *Vacc = nullptr;   // [nbf][nbf] accumulation of the upper block triangle
};

void free_xc(mess_basis *B) {
    XcGrid *X = static_cast<XcGrid *>(B->xc);
    if (!X) return;
    for (double *p : {X->xyzw, X->phiT, X->f, X->rho, X->epart, X->ex, X->Vacc, X->dphiT, X->grad, X->hv, X->Dp,
                      X->vpart[0], X->vpart[1]})
        hipFree(p);
    hipFree(X->groups);
    delete X;
    B->xc = nullptr;
}

// ------------------------------------------------------------ quadrature

// Gauss-Legendre nodes (ascending) and weights on [-1, 1]: Newton's method on
// P_n from the three-term recurrence, started at cos(pi (i - 1/4)/(n + 1/2)).
static void gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w) {
    x.assign(n, 0.0);
    w.assign(n, 0.0);
    for (int i = 1; i <= n; ++i) {
        double z = std::cos(M_PI * (i - 0.25) / (n + 0.5)), dp = 0.0;
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (z * p1 - p0) / (z * z - 1.0);
            const double dz = p1 / dp;
            z -= dz;
            if (std::fabs(dz) < 1e-16) break;
        }
        {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (z * p1 - p0) / (z * z - 1.0);
        }
        x[n - i] = z;  // z decreases with i
        w[n - i] = 2.0 / ((1.0 - z * z) * dp * dp);
    }
}

// Becke cell function s(mu) = (1 - f(f(f(mu))))/2, f(x) = (3x - x^3)/2.
__device__ __forceinline__ double becke_s(double mu) {
    double f = mu;
#pragma unroll
    for (int k = 0; k < 3; ++k) f = 1.5 * f - 0.5 * f * f * f;
    return 0.5 * (1.0 - f);
}

// One thread per point: position and weight (radial x angular x Becke).
__global__ void k_grid(int nat, const double *__restrict__ xyz, const double *__restrict__ rad,
                       const double *__restrict__ ang, int64_t npts, int64_t G, double *__restrict__ xyzw) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= G) return;
    if (g >= npts) {
        xyzw[4 * g] = xyzw[4 * g + 1] = xyzw[4 * g + 2] = xyzw[4 * g + 3] = 0.0;
        return;
    }
    const int a = (int)(g / kPtsPerAtom);
    const int rest = (int)(g % kPtsPerAtom);
    const int ir = rest / kNAng, ia = rest % kNAng;
    const double r = rad[2 * ir], wr = rad[2 * ir + 1];
    const double px = xyz[3 * a] + r * ang[4 * ia], py = xyz[3 * a + 1] + r * ang[4 * ia + 1],
                 pz = xyz[3 * a + 2] + r * ang[4 * ia + 2];
    double Pown = 0.0, Psum = 0.0;
    for (int c = 0; c < nat; ++c) {
        const double dcx = px - xyz[3 * c], dcy = py - xyz[3 * c + 1], dcz = pz - xyz[3 * c + 2];
        const double dc = sqrt(dcx * dcx + dcy * dcy + dcz * dcz);
        double P = 1.0;
        for (int b = 0; b < nat; ++b) {
            if (b == c) continue;
            const double dbx = px - xyz[3 * b], dby = py - xyz[3 * b + 1], dbz = pz - xyz[3 * b + 2];
            const double db = sqrt(dbx * dbx + dby * dby + dbz * dbz);
            const double ex = xyz[3 * c] - xyz[3 * b], ey = xyz[3 * c + 1] - xyz[3 * b + 1],
                         ez = xyz[3 * c + 2] - xyz[3 * b + 2];
            const double R = sqrt(ex * ex + ey * ey + ez * ez);
            P *= becke_s((dc - db) / R);
        }
        Psum += P;
        if (c == a) Pown = P;
    }
    xyzw[4 * g] = px;
    xyzw[4 * g + 1] = py;
    xyzw[4 * g + 2] = pz;
    xyzw[4 * g + 3] = wr * ang[4 * ia + 3] * (Pown / Psum);
}

// PhiT[mu][g]: one thread per point, loop over shells.  Contraction
// coefficients are those of the (l,0,0) component; mixed d components carry
// the factor sqrt(3).
__global__ void k_basis_values(int nsh, const XcShell *__restrict__ sh, const double *__restrict__ alpha,
                               const double *__restrict__ ct, int64_t npts, int64_t G,
                               const double *__restrict__ xyzw, double *__restrict__ phiT) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= G) return;
    const bool live = g < npts;
    const double px = xyzw[4 * g], py = xyzw[4 * g + 1], pz = xyzw[4 * g + 2];
    for (int s = 0; s < nsh; ++s) {
        const XcShell S = sh[s];
        const double dx = px - S.x, dy = py - S.y, dz = pz - S.z;
        const double r2 = dx * dx + dy * dy + dz * dz;
        double rad = 0.0;
        if (live)
            for (int p = 0; p < S.nprim; ++p) {
                const double e = alpha[S.prim0 + p] * r2;
                if (e < 745.0) rad += ct[S.prim0 + p] * exp(-e);
            }
        double *o = phiT + (int64_t)S.bf0 * G + g;
        if (S.l == 0) {
            o[0] = rad;
        } else if (S.l == 1) {
            o[0] = dx * rad;
            o[G] = dy * rad;
            o[2 * G] = dz * rad;
        } else {
            // xx, xy, xz, yy, yz, zz
            o[0] = dx * dx * rad;
            o[G] = kSqrt3 * dx * dy * rad;
            o[2 * G] = kSqrt3 * dx * dz * rad;
            o[3 * G] = dy * dy * rad;
            o[4 * G] = kSqrt3 * dy * dz * rad;
            o[5 * G] = dz * dz * rad;
        }
    }
}

// dPhiT[k][mu][g] = d phi_mu / d r_k at point g: one thread per point, loop
// over shells; for x^a y^b z^c R(r^2), R = sum c_p e^{-alpha_p r^2},
// d/dx = a x^(a-1) y^b z^c R - 2 x (x^a y^b z^c) sum c_p alpha_p e^{-alpha_p r^2}.
__global__ void k_basis_grad(int nsh, const XcShell *__restrict__ sh, const double *__restrict__ alpha,
                             const double *__restrict__ ct, int64_t npts, int64_t G, int nbf,
                             const double *__restrict__ xyzw, double *__restrict__ dphiT) {
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= G) return;
    const bool live = g < npts;
    const double px = xyzw[4 * g], py = xyzw[4 * g + 1], pz = xyzw[4 * g + 2];
    const int64_t plane = (int64_t)nbf * G;
    for (int s = 0; s < nsh; ++s) {
        const XcShell S = sh[s];
        const double d[3] = {px - S.x, py - S.y, pz - S.z};
        const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        double rad = 0.0, drad = 0.0;
        if (live)
            for (int p = 0; p < S.nprim; ++p) {
                const double a = alpha[S.prim0 + p], e = a * r2;
                if (e < 745.0) {
                    const double t = ct[S.prim0 + p] * exp(-e);
                    rad += t;
                    drad += a * t;
                }
            }
        const int nc = (S.l + 1) * (S.l + 2) / 2;
        for (int c = 0; c < nc; ++c) {
            // component exponents in the order x-major (xx, xy, xz, yy, yz, zz)
            int e[3];
            if (S.l == 0) {
                e[0] = e[1] = e[2] = 0;
            } else if (S.l == 1) {
                e[0] = c == 0;
                e[1] = c == 1;
                e[2] = c == 2;
            } else {
                const int tab[6][3] = {{2, 0, 0}, {1, 1, 0}, {1, 0, 1}, {0, 2, 0}, {0, 1, 1}, {0, 0, 2}};
                e[0] = tab[c][0];
                e[1] = tab[c][1];
                e[2] = tab[c][2];
            }
            const double sc = (S.l == 2 && (c == 1 || c == 2 || c == 4)) ? kSqrt3 : 1.0;
            double mono = 1.0;
            for (int k = 0; k < 3; ++k)
                for (int q = 0; q < e[k]; ++q) mono *= d[k];
            for (int k = 0; k < 3; ++k) {
                double lower = 0.0;
                if (e[k] > 0) {
                    lower = e[k];
                    for (int j = 0; j < 3; ++j)
                        for (int q = 0; q < e[j] - (j == k); ++q) lower *= d[j];
                }
                dphiT[k * plane + (int64_t)(S.bf0 + c) * G + g] = sc * (lower * rad - 2.0 * d[k] * mono * drad);
            }
        }
    }
}

// ------------------------------------------------------------ per density

__device__ __forceinline__ void exchange_terms(double rho, double &ex, double &vx) {
    constexpr double kCx = 0.73855876638202240587;   // (3/4)(3/pi)^(1/3)
    constexpr double kVx = 0.98474502184269654116;   // (3/pi)^(1/3)
    if (rho > 0.0) {
        const double c = cbrt(rho);
        ex = -kCx * rho * c;
        vx = -kVx * c;
    } else {
        ex = 0.0;
        vx = 0.0;
    }
}

typedef double xc_d4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ xc_d4 xc_mfma(double a, double b, xc_d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// v_mfma_f64_16x16x4 takes A[l % 16][l / 16] and B[l / 16][l % 16] from lane
// l and returns C[l / 16 + 4 q][l % 16] in element q.  D in that order:
// Dp[row tile][k / 4][lane].  TRI: tiles above the diagonal hold D + D^T (the
// ones below are not read).
template <bool TRI>
__global__ void k_xc_pack_d(int N, int T, const double *__restrict__ D, double *__restrict__ Dp) {
    const int64_t n = (int64_t)T * T * 256;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(e % 64), ks = (int)(e / 64 % (4 * T)), i = (int)(e / 64 / (4 * T));
        const int r = 16 * i + l % 16, k = 4 * ks + l / 16;
        double v = 0.0;
        if (r < N && k < N) {
            v = D[(int64_t)r * N + k];
            if (TRI && ks / 4 > i) v += D[(int64_t)k * N + r];
        }
        Dp[e] = v;
    }
}

// rho (and, GGA, grad rho) over PT points: the basis values of the tile lie in
// LDS ([row][point], points of odd rows exchanged between halves so that the
// four rows of a B operand fall on all banks), a wave takes row tiles of 16
// and streams its rows of D from the L2 in fragment order, four products of
// 16 points an operand.  Bound by the FP64 matrix rate for LDA (the local part needs
// only the upper block triangle: N^2 flops per point) and by the three
// gradient planes read from memory for GGA at small N.  60-atom cluster, 300
// functions (LDA): 17.7 ms on vector FMAs with the whole product, 4.85 here
// (52 TFLOP/s of the matrix unit with the blocks' padding).  Rows beyond one LDS
// panel (RC rows) are taken by pairs of panels.  LDA also leaves f_g and the
// block's sum of w e_x.
template <bool GGA, int PT>
__global__ void __launch_bounds__(512) k_xc_rho(int N, int64_t G, int TC, const double *__restrict__ Dp,
                                                const double *__restrict__ phiT, const double *__restrict__ dphiT,
                                                const double *__restrict__ xyzw, double *__restrict__ rho_out,
                                                double *__restrict__ grad_out, double *__restrict__ f,
                                                double *__restrict__ epart) {
    constexpr int NC = PT / 16, NQ = GGA ? 4 : 1;
    extern __shared__ double xlds[];
    const int T = (N + 15) / 16, W = blockDim.x / 64, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t g0 = blockIdx.x * (int64_t)PT, plane = (int64_t)N * G;
    const bool one = TC >= T;
    double *const pa = xlds, *const pb = one ? xlds : xlds + 16 * TC * PT;
    auto at = [](int row, int pt) { return row * PT + (PT >= 32 ? pt ^ ((row & 1) << 4) : pt); };
    auto load = [&](double *p, int r0, int rows) {
        for (int e = threadIdx.x; e < rows * (PT / 2); e += blockDim.x) {
            const int r = e / (PT / 2), c = 2 * (e % (PT / 2));
            double2 v = make_double2(0.0, 0.0);
            if (r0 + r < N) v = *reinterpret_cast<const double2 *>(phiT + (int64_t)(r0 + r) * G + g0 + c);
            *reinterpret_cast<double2 *>(p + at(r, c)) = v;
        }
    };
    double part[NQ][NC];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int c = 0; c < NC; ++c) part[q][c] = 0.0;
    for (int ta = 0; ta < T; ta += TC) {
        const int na = min(TC, T - ta);
        __syncthreads();
        load(pa, 16 * ta, 16 * na);
        for (int tb = GGA ? 0 : ta; tb < T; tb += TC) {
            const int nb = min(TC, T - tb);
            if (!one) {
                __syncthreads();
                load(pb, 16 * tb, 16 * nb);
            }
            __syncthreads();
            for (int j = 0;; ++j) {
                // row tiles dealt to the waves forwards and backwards (the triangle's rows shorten)
                const int ir = j * W + ((j & 1) ? W - 1 - wave : wave);
                if (j * W >= na) break;
                if (ir >= na) continue;
                const int i = ta + ir, kt0 = GGA || tb > ta ? 0 : ir;
                xc_d4 acc[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] = xc_d4{0.0, 0.0, 0.0, 0.0};
                const double *dp = Dp + ((int64_t)i * 4 * T + 4 * tb) * 64 + lane;
                double a[4], an[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) an[k] = dp[(4 * kt0 + k) * 64];
                for (int kt = kt0; kt < nb; ++kt) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) a[k] = an[k];
                    if (kt + 1 < nb)
#pragma unroll
                        for (int k = 0; k < 4; ++k) an[k] = dp[(4 * (kt + 1) + k) * 64];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int row = 16 * kt + 4 * k + lane / 16;
#pragma unroll
                        for (int c = 0; c < NC; ++c) acc[c] = xc_mfma(a[k], pb[at(row, 16 * c + lane % 16)], acc[c]);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = 16 * ir + lane / 16 + 4 * q;
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        part[0][c] = fma(pa[at(row, 16 * c + lane % 16)], acc[c][q], part[0][c]);
                        if constexpr (GGA) {
                            const int mu = 16 * ta + row;
                            const int64_t o = (int64_t)mu * G + g0 + 16 * c + lane % 16;
                            if (mu < N)
#pragma unroll
                                for (int k = 0; k < 3; ++k) part[1 + k][c] = fma(dphiT[k * plane + o], acc[c][q], part[1 + k][c]);
                        }
                    }
                }
            }
        }
    }
    __syncthreads();  // the panels give way to the waves' sums
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double v = part[q][c];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lane < 16) xlds[(q * W + wave) * PT + 16 * c + lane] = v;
        }
    __syncthreads();
    double e = 0.0;
    if (threadIdx.x < PT) {
        const int64_t g = g0 + threadIdx.x;
        double r[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            r[q] = 0.0;
            for (int w = 0; w < W; ++w) r[q] += xlds[(q * W + w) * PT + threadIdx.x];
        }
        rho_out[g] = r[0];
        if constexpr (GGA) {
#pragma unroll
            for (int k = 0; k < 3; ++k) grad_out[k * G + g] = 2.0 * r[1 + k];
        } else {
            const double w = xyzw[4 * g + 3];
            double ex, vx;
            exchange_terms(r[0], ex, vx);
            f[g] = w * vx;
            e = w * ex;
        }
    }
    if constexpr (!GGA) {
        // block sum of w e_x: the first wave holds all points
        if (wave == 0) {
            for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
            if (lane == 0) epart[blockIdx.x] = e;
        }
    }
}

__global__ void __launch_bounds__(1024) k_sum_partials(int n, const double *__restrict__ part, double *__restrict__ out) {
    __shared__ double red[1024];
    double s = 0.0;
#pragma unroll 8
    for (int i = threadIdx.x; i < n; i += 1024) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

// A group of up to 8 tiles of 64 x 64 of V, one a wave, and the row blocks of
// 64 that they read: blocks of the left factor, then of the right one.
struct VGroup {
    int nsup, na, nb, first;  // tiles, row blocks, index of the first tile
    int a[12], b[12];         // row blocks (left, right)
    int ai[8], bj[8];         // a tile's positions among them
};
static_assert(sizeof(VGroup) % sizeof(int4) == 0, "VGroup is copied as int4");

// pairs of points that a thread loads per step, left and right rows
template <bool GGA>
inline constexpr int kVLoadA = GGA ? 2 : 5;
constexpr int kVLoadB = 4;

// Partial sums over a chunk of points of the tiles (bi, bj) of a group:
//   LDA: sum_g PhiT[mu][g] f_g PhiT[nu][g], bi <= bj;
//   GGA: sum_g PhiT[mu][g] Z[nu][g], Z[nu][g] = f_g PhiT[nu][g] + hv[.][g] . dPhiT[.][nu][g],
// a wave per tile with 4 x 4 products of 16 x 16 in its accumulators.  Steps
// of KP points of the group's rows are staged in LDS ([row][point] with the
// points of a row permuted in fours, so that 16 rows x 4 points fall on all
// banks), the next step's values on their way meanwhile; every tile of a row
// block shares them, which keeps the reads of PhiT near one (LDA: the 15
// tiles of 300 functions are two groups).  Bound by the FP64 matrix rate, and
// for GGA at small N by the four planes read.  60-atom cluster, 2.6e6 points
// x 300 functions (LDA): 13.8 ms on vector FMAs with atomic partial sums, 5.2
// here; 21 atoms x 105 functions (PBE): 10.4 (112 blocks) and 1.2.
template <bool GGA, int KP>
__global__ void __launch_bounds__(512) k_xc_v(int N, int64_t G, int64_t chunk, const double *__restrict__ phiT,
                                              const double *__restrict__ dphiT, const double *__restrict__ f,
                                              const double *__restrict__ hv, const VGroup *__restrict__ groups,
                                              int ntile, double *__restrict__ vpart) {
    constexpr int NPA = kVLoadA<GGA>, NPB = GGA ? kVLoadB : 1;  // pairs of points a thread has on their way
    extern __shared__ double xlds[];
    const VGroup &gr = groups[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nthr = blockDim.x;
    const int ra = 64 * gr.na, rb = GGA ? 64 * gr.nb : 0, rows = ra + rb;
    const int64_t plane = (int64_t)N * G, gs = blockIdx.x * chunk, ge = gs + chunk < G ? gs + chunk : G;
    double *const fl = xlds + 2 * rows * KP;  // LDA: f of the step's points, two buffers
    const int na2 = ra * (KP / 2), nb2 = rb * (KP / 2);
    auto at = [](int row, int pt) { return row * KP + (pt ^ (((row / (32 / KP)) % (KP / 4)) * 4)); };
    // a thread's rows (function index, -1 beyond the last) and its pair of points
    int mua[NPA], mub[NPB];
#pragma unroll
    for (int i = 0; i < NPA; ++i) {
        const int r = (threadIdx.x + i * nthr) / (KP / 2);
        const int mu = r < ra ? 64 * gr.a[r / 64] + r % 64 : N;
        mua[i] = mu < N ? mu : -1;
    }
    if constexpr (GGA)
#pragma unroll
        for (int i = 0; i < NPB; ++i) {
            const int r = (threadIdx.x + i * nthr) / (KP / 2);
            const int mu = r < rb ? 64 * gr.b[r / 64] + r % 64 : N;
            mub[i] = mu < N ? mu : -1;
        }
    const int c2 = 2 * (threadIdx.x % (KP / 2));
    double2 va[NPA], vb[NPB];
    double fv = 0.0;
    auto fetch = [&](int64_t g0) {
#pragma unroll
        for (int i = 0; i < NPA; ++i)
            va[i] = mua[i] >= 0 ? *reinterpret_cast<const double2 *>(phiT + (int64_t)mua[i] * G + g0 + c2) : make_double2(0.0, 0.0);
        if constexpr (GGA) {
            const double2 w = *reinterpret_cast<const double2 *>(f + g0 + c2);
            double2 h[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) h[k] = *reinterpret_cast<const double2 *>(hv + k * G + g0 + c2);
#pragma unroll
            for (int i = 0; i < NPB; ++i) {
                double2 z = make_double2(0.0, 0.0);
                if (mub[i] >= 0) {
                    const int64_t o = (int64_t)mub[i] * G + g0 + c2;
                    const double2 p = *reinterpret_cast<const double2 *>(phiT + o);
                    z.x = w.x * p.x;
                    z.y = w.y * p.y;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double2 d = *reinterpret_cast<const double2 *>(dphiT + k * plane + o);
                        z.x += h[k].x * d.x;
                        z.y += h[k].y * d.y;
                    }
                }
                vb[i] = z;
            }
        } else if (threadIdx.x < KP) {
            fv = f[g0 + threadIdx.x];
        }
    };
    auto put = [&](int buf) {
        double *p = xlds + buf * rows * KP;
#pragma unroll
        for (int i = 0; i < NPA; ++i) {
            const int e = threadIdx.x + i * nthr;
            if (e < na2) *reinterpret_cast<double2 *>(p + at(e / (KP / 2), 2 * (e % (KP / 2)))) = va[i];
        }
        if constexpr (GGA) {
#pragma unroll
            for (int i = 0; i < NPB; ++i) {
                const int e = threadIdx.x + i * nthr;
                if (e < nb2) *reinterpret_cast<double2 *>(p + at(ra + e / (KP / 2), 2 * (e % (KP / 2)))) = vb[i];
            }
        } else if (threadIdx.x < KP) {
            fl[buf * KP + threadIdx.x] = fv;
        }
    };
    const bool work = wave < gr.nsup;
    const int ai = work ? gr.ai[wave] : 0, bj = work ? gr.bj[wave] : 0;
    const bool diag = !GGA && ai == bj;
    const int ar = 64 * ai + lane % 16, br = (GGA ? ra : 0) + 64 * bj + lane % 16;
    xc_d4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = xc_d4{0.0, 0.0, 0.0, 0.0};
    fetch(gs);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int64_t g0 = gs; g0 < ge; g0 += KP, buf ^= 1) {
        const bool more = g0 + KP < ge;
        if (more) fetch(g0 + KP);
        if (work) {
            const double *p = xlds + buf * rows * KP;
#pragma unroll
            for (int k = 0; k < KP / 4; ++k) {
                const int pt = 4 * k + lane / 16;
                double a[4], b[4];
                const double fk = GGA ? 1.0 : fl[buf * KP + pt];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a[i] = p[at(ar + 16 * i, pt)];
                    b[i] = GGA ? p[at(br + 16 * i, pt)] : fk * p[at(br + 16 * i, pt)];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (!(diag && j < i)) acc[i][j] = xc_mfma(a[i], b[j], acc[i][j]);
            }
        }
        if (more) put(buf ^ 1);
        __syncthreads();
    }
    if (!work) return;
    double *o = vpart + ((int64_t)blockIdx.x * ntile + gr.first + wave) * (kXT * kXT);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) o[(16 * i + lane / 16 + 4 * q) * kXT + 16 * j + lane % 16] = acc[i][j][q];
}

// Vacc <- the tiles' partial sums over the chunks, a block per 64 elements of
// a tile (four shares of the chunks, added in order).
template <bool GGA>
__global__ void __launch_bounds__(256) k_xc_v_sum(int N, int nblk, int ntile, int nchunk, const double *__restrict__ vpart,
                                                  double *__restrict__ Vacc) {
    __shared__ double red[4][64];
    const int tile = blockIdx.y, e = blockIdx.x * 64 + threadIdx.x % 64, w = threadIdx.x / 64;
    double s = 0.0;
#pragma unroll 8
    for (int c = w; c < nchunk; c += 4) s += vpart[((int64_t)c * ntile + tile) * (kXT * kXT) + e];
    red[w][threadIdx.x % 64] = s;
    __syncthreads();
    if (w) return;
    s = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
    int bi = 0, bj = tile;
    if (GGA) {
        bi = tile / nblk;
        bj = tile % nblk;
    } else {
        while (bj >= nblk - bi) bj -= nblk - bi, ++bi;
        bj += bi;
    }
    const int r = kXT * bi + e / kXT, c = kXT * bj + e % kXT;
    if (r < N && c < N) Vacc[(int64_t)r * N + c] = s;
}

// V[i][j] from the upper triangle of Vacc (the upper block triangle was
// accumulated; inside a diagonal block only i <= j is taken, so V is exactly
// symmetric).
__global__ void k_lda_mirror(int N, const double *__restrict__ Vacc, double *__restrict__ V) {
    const int64_t NN = (int64_t)N * N;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < NN; idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx / N), j = (int)(idx % N);
        V[idx] = (i <= j) ? Vacc[idx] : Vacc[(int64_t)j * N + i];
    }
}

// ------------------------------------------------------------------ PBE

constexpr double kRhoMin = 1e-10;

// f = rho eps_x^unif F_x + rho (eps_c + H) and its partial derivatives in
// rho and sigma (closed shell, Hartree atomic units).
//   exchange: s^2 = c_s sigma rho^(-8/3), c_s = 1 / (4 (3 pi^2)^(2/3)),
//     F_x = 1 + kappa - kappa / (1 + mu s^2 / kappa);
//   correlation: Perdew-Wang eps_c(r_s), r_s = (3 / (4 pi rho))^(1/3);
//     t^2 = c_t sigma rho^(-7/3), c_t = pi / (16 (3 pi^2)^(1/3));
//     H = gamma ln(1 + (beta/gamma) t^2 R(A t^2)), R(y) = (1 + y)/(1 + y + y^2),
//     A = (beta/gamma) / (exp(-eps_c/gamma) - 1).
__device__ __forceinline__ void pbe_point(double rho, double sigma, double &f, double &fr, double &fs) {
    if (!(rho >= kRhoMin)) {
        f = fr = fs = 0.0;
        return;
    }
    constexpr double kKappa = 0.804, kBeta = 0.06672455060314922;
    constexpr double kMu = kBeta * M_PI * M_PI / 3.0;
    constexpr double kGamma = 0.031090690869654895;  // (1 - ln 2) / pi^2
    constexpr double kA = 0.031091, kA1 = 0.21370, kB1 = 7.5957, kB2 = 3.5876, kB3 = 1.6382, kB4 = 0.49294;
    constexpr double kCx = -0.73855876638202240587;  // -(3/4)(3/pi)^(1/3)
    constexpr double kCs = 0.026121172985233599;     // 1 / (4 (3 pi^2)^(2/3))
    constexpr double kCt = 0.063468206097703704;     // pi / (16 (3 pi^2)^(1/3))
    constexpr double kRs = 0.62035049089940001667;   // (3 / (4 pi))^(1/3)
    const double r13 = cbrt(rho), r43 = rho * r13;
    const double ir43 = 1.0 / r43, ir83 = ir43 * ir43;
    // exchange
    const double x = kCs * sigma * ir83;
    const double den = 1.0 + kMu * x / kKappa;
    const double Fx = 1.0 + kKappa - kKappa / den;
    const double Fxp = kMu / (den * den);
    const double ex = kCx * r43 * Fx;
    const double exr = kCx * r13 * ((4.0 / 3.0) * Fx - (8.0 / 3.0) * x * Fxp);
    const double exs = kCx * Fxp * kCs * ir43;
    // Perdew-Wang correlation of the uniform gas
    const double rs = kRs / r13, sq = sqrt(rs);
    const double Q = 2.0 * kA * (kB1 * sq + kB2 * rs + kB3 * rs * sq + kB4 * rs * rs);
    const double Qp = 2.0 * kA * (0.5 * kB1 / sq + kB2 + 1.5 * kB3 * sq + 2.0 * kB4 * rs);
    const double Lg = log1p(1.0 / Q);
    const double ec = -2.0 * kA * (1.0 + kA1 * rs) * Lg;
    const double dec = -2.0 * kA * kA1 * Lg + 2.0 * kA * (1.0 + kA1 * rs) * Qp / (Q * Q + Q);
    // gradient correction
    const double u = kCt * sigma * ir43 / rho;  // t^2
    const double E1 = expm1(-ec / kGamma);
    const double Ap = (kBeta / kGamma) / E1;
    const double y = Ap * u, d2 = 1.0 + y + y * y;
    const double R = (1.0 + y) / d2, Rp = -y * (2.0 + y) / (d2 * d2);
    const double Nn = (kBeta / kGamma) * u * R;
    const double H = kGamma * log1p(Nn);
    const double dHdN = kGamma / (1.0 + Nn);
    const double dHdu = dHdN * (kBeta / kGamma) * (R + y * Rp);
    const double dHdec = dHdN * (kBeta / kGamma) * u * u * Rp * (Ap * Ap * (E1 + 1.0) / kBeta);
    f = ex + rho * (ec + H);
    fr = exr + ec + H - (rs / 3.0) * dec * (1.0 + dHdec) - (7.0 / 3.0) * u * dHdu;
    fs = exs + dHdu * kCt * ir43;
}

// The functional per point: energy partial sums per 256-point block (fixed
// order), f_g = w f_rho / 2 and hv[k][g] = 2 w f_sigma d_k rho.
__global__ void __launch_bounds__(256) k_pbe_point(int64_t G, const double *__restrict__ xyzw,
                                                   const double *__restrict__ rho, const double *__restrict__ grad,
                                                   double *__restrict__ f, double *__restrict__ hv,
                                                   double *__restrict__ epart) {
    __shared__ double red[256];
    const int64_t g = blockIdx.x * (int64_t)256 + threadIdx.x;
    double e = 0.0;
    if (g < G) {
        const double w = xyzw[4 * g + 3];
        const double gx = grad[g], gy = grad[G + g], gz = grad[2 * G + g];
        double fv, fr, fs;
        pbe_point(rho[g], gx * gx + gy * gy + gz * gz, fv, fr, fs);
        e = w * fv;
        f[g] = 0.5 * w * fr;
        const double h = 2.0 * w * fs;
        hv[g] = h * gx;
        hv[G + g] = h * gy;
        hv[2 * G + g] = h * gz;
    }
    red[threadIdx.x] = e;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) epart[blockIdx.x] = red[0];
}

// V = Vacc + Vacc^T (exactly symmetric)
__global__ void k_gga_sym(int N, const double *__restrict__ Vacc, double *__restrict__ V) {
    const int64_t NN = (int64_t)N * N;
    for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < NN; idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx / N), j = (int)(idx % N);
        V[idx] = Vacc[idx] + Vacc[(int64_t)j * N + i];
    }
}

template <bool GGA>
static int v_prepare(XcGrid *X);

// Grid and basis values, built once per basis (synchronous).
static int get_xc(mess_basis *B, XcGrid **out) {
    if (B->xc) {
        *out = static_cast<XcGrid *>(B->xc);
        return MESS_OK;
    }
    if (B->n_mol != 1) {
        set_error("LDA exchange is built for a single molecule, not a batch of %d", B->n_mol);
        return MESS_E_UNSUPPORTED;
    }
    auto *X = new XcGrid();
    B->xc = X;
    X->npts = (int64_t)B->nat * kPtsPerAtom;
    X->G = (X->npts + kXT - 1) / kXT * kXT;
    X->nbf = B->nbf;
    // radial (r, w) and angular (ux, uy, uz, w) rules
    std::vector<double> rad(2 * kNRad), ang(4 * kNAng);
    for (int i = 1; i <= kNRad; ++i) {
        const double t = i * M_PI / (kNRad + 1), x = std::cos(t);
        const double r = (1.0 + x) / (1.0 - x);
        rad[2 * (i - 1)] = r;
        rad[2 * (i - 1) + 1] = M_PI / (kNRad + 1) * std::sin(t) * 2.0 / ((1.0 - x) * (1.0 - x)) * r * r;
    }
    std::vector<double> u, a;
    gauss_legendre(kNTheta, u, a);
    for (int j = 0; j < kNTheta; ++j)
        for (int k = 0; k < kNPhi; ++k) {
            const double ph = 2.0 * M_PI * k / kNPhi, st = std::sqrt(1.0 - u[j] * u[j]);
            double *d = &ang[4 * (j * kNPhi + k)];
            d[0] = st * std::cos(ph);
            d[1] = st * std::sin(ph);
            d[2] = u[j];
            d[3] = a[j] * (2.0 * M_PI / kNPhi);
        }
    std::vector<XcShell> hs(B->nsh);
    for (int s = 0; s < B->nsh; ++s) {
        const int at = B->sh_atom[s];
        hs[s] = XcShell{B->xyz[3 * at], B->xyz[3 * at + 1], B->xyz[3 * at + 2], B->sh_l[s], B->sh_prim0[s],
                        B->sh_np[s], B->sh_bf0[s]};
    }
    double *d_rad = nullptr, *d_ang = nullptr, *d_alpha = nullptr, *d_ct = nullptr;
    XcShell *d_sh = nullptr;
    auto cleanup = [&]() {
        hipFree(d_rad);
        hipFree(d_ang);
        hipFree(d_alpha);
        hipFree(d_ct);
        hipFree(d_sh);
    };
    const size_t np = B->alpha.size();
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
    chk(hipMalloc(&X->xyzw, sizeof(double) * 4 * X->G));
    chk(hipMalloc(&X->phiT, sizeof(double) * (size_t)X->nbf * X->G));
    chk(hipMalloc(&X->f, sizeof(double) * X->G));
    chk(hipMalloc(&X->rho, sizeof(double) * X->G));
    chk(hipMalloc(&X->epart, sizeof(double) * (X->G / 16)));
    chk(hipMalloc(&X->ex, sizeof(double)));
    chk(hipMalloc(&X->Vacc, sizeof(double) * (size_t)X->nbf * X->nbf));
    const int64_t T = (X->nbf + 15) / 16;
    chk(hipMalloc(&X->Dp, sizeof(double) * 256 * T * T));
    chk(hipMalloc(&d_rad, sizeof(double) * rad.size()));
    chk(hipMalloc(&d_ang, sizeof(double) * ang.size()));
    chk(hipMalloc(&d_alpha, sizeof(double) * np));
    chk(hipMalloc(&d_ct, sizeof(double) * np));
    chk(hipMalloc(&d_sh, sizeof(XcShell) * B->nsh));
    if (e != hipSuccess) {
        cleanup();
        free_xc(B);
        set_error("LDA grid: device allocation failed (%s)", hipGetErrorString(e));
        return MESS_E_NOMEM;
    }
    chk(hipMemcpy(d_rad, rad.data(), sizeof(double) * rad.size(), hipMemcpyHostToDevice));
    chk(hipMemcpy(d_ang, ang.data(), sizeof(double) * ang.size(), hipMemcpyHostToDevice));
    chk(hipMemcpy(d_alpha, B->alpha.data(), sizeof(double) * np, hipMemcpyHostToDevice));
    chk(hipMemcpy(d_ct, B->ctilde.data(), sizeof(double) * np, hipMemcpyHostToDevice));
    chk(hipMemcpy(d_sh, hs.data(), sizeof(XcShell) * B->nsh, hipMemcpyHostToDevice));
    if (e == hipSuccess) {
        const unsigned nb = (unsigned)((X->G + 255) / 256);
        hipLaunchKernelGGL(k_grid, dim3(nb), dim3(256), 0, nullptr, B->nat, B->d_xyz, d_rad, d_ang, X->npts, X->G,
                           X->xyzw);
        hipLaunchKernelGGL(k_basis_values, dim3(nb), dim3(256), 0, nullptr, B->nsh, d_sh, d_alpha, d_ct, X->npts,
                           X->G, X->xyzw, X->phiT);
        chk(hipGetLastError());
        chk(hipDeviceSynchronize());
    }
    cleanup();
    if (e != hipSuccess) {
        free_xc(B);
        set_error("LDA grid construction failed: %s", hipGetErrorString(e));
        return MESS_E_DEVICE;
    }
    const int rc = v_prepare<false>(X);
    if (rc != MESS_OK) {
        free_xc(B);
        return rc;
    }
    *out = X;
    return MESS_OK;
}

// Basis gradients on the grid and the PBE per-point buffers, built on the
// first PBE call (synchronous).
static int ensure_gga(mess_basis *B, XcGrid *X) {
    if (X->dphiT) return MESS_OK;
    MESS_TRY(v_prepare<true>(X));
    std::vector<XcShell> hs(B->nsh);
    for (int s = 0; s < B->nsh; ++s) {
        const int at = B->sh_atom[s];
        hs[s] = XcShell{B->xyz[3 * at], B->xyz[3 * at + 1], B->xyz[3 * at + 2], B->sh_l[s], B->sh_prim0[s],
                        B->sh_np[s], B->sh_bf0[s]};
    }
    const size_t np = B->alpha.size();
    double *d_alpha = nullptr, *d_ct = nullptr;
    XcShell *d_sh = nullptr;
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) {
        if (e == hipSuccess) e = r;
    };
    chk(hipMalloc(&X->dphiT, sizeof(double) * 3 * (size_t)X->nbf * X->G));
    chk(hipMalloc(&X->grad, sizeof(double) * 3 * X->G));
    chk(hipMalloc(&X->hv, sizeof(double) * 3 * X->G));
    chk(hipMalloc(&d_alpha, sizeof(double) * np));
    chk(hipMalloc(&d_ct, sizeof(double) * np));
    chk(hipMalloc(&d_sh, sizeof(XcShell) * B->nsh));
    if (e == hipSuccess) {
        chk(hipMemcpy(d_alpha, B->alpha.data(), sizeof(double) * np, hipMemcpyHostToDevice));
        chk(hipMemcpy(d_ct, B->ctilde.data(), sizeof(double) * np, hipMemcpyHostToDevice));
        chk(hipMemcpy(d_sh, hs.data(), sizeof(XcShell) * B->nsh, hipMemcpyHostToDevice));
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_basis_grad, dim3((unsigned)((X->G + 255) / 256)), dim3(256), 0, nullptr, B->nsh, d_sh,
                           d_alpha, d_ct, X->npts, X->G, X->nbf, X->xyzw, X->dphiT);
        chk(hipGetLastError());
        chk(hipDeviceSynchronize());
    }
    hipFree(d_alpha);
    hipFree(d_ct);
    hipFree(d_sh);
    if (e != hipSuccess) {
        for (double **p : {&X->dphiT, &X->grad, &X->hv}) {
            hipFree(*p);
            *p = nullptr;
        }
        set_error("PBE basis gradients: %s", hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? MESS_E_NOMEM : MESS_E_DEVICE;
    }
    return MESS_OK;
}

// rho (GGA: and grad rho) of density D on the grid.
template <bool GGA>
static int rho_async(XcGrid *X, const double *D, hipStream_t s, int *nblocks) {
    const int N = X->nbf, T = (N + 15) / 16;
    hipLaunchKernelGGL(k_xc_pack_d<!GGA>, dim3((unsigned)std::min<int64_t>((int64_t)T * T, 4096)), dim3(256), 0, s, N, T, D,
                       X->Dp);
    // Point tile: 32, so that two blocks share a CU up to 320 rows (160 KB of
    // LDS) and one loads its panel while the other multiplies (LDA, 300
    // functions: 6.3 ms with 64 points and one block a CU, 4.85 with 32; PBE,
    // 105 functions, whose gradient planes are read as rows finish: 1.25 and
    // 0.83); 64 for LDA to 160 rows, where two such blocks fit as well and a
    // row of D serves four products instead of two; 16 where 32 points do not
    // fit; beyond 1280 rows, panels of 512 rows in pairs.  Few row tiles are
    // dealt to four waves, so that the triangle's rows even out.
    const int W = T <= 10 ? 4 : 8;
    auto go = [&](auto PTc, int TC, int panels) {
        constexpr int PT = decltype(PTc)::value;
        const size_t lds = std::max(sizeof(double) * 16 * TC * PT * panels, sizeof(double) * 4 * W * PT);
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_xc_rho<GGA, PT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) (void)hipGetLastError();  // the launch itself reports a size it cannot take
        *nblocks = (int)(X->G / PT);
        hipLaunchKernelGGL((k_xc_rho<GGA, PT>), dim3((unsigned)*nblocks), dim3(64 * W), lds, s, N, X->G, TC, X->Dp, X->phiT,
                           X->dphiT, X->xyzw, X->rho, X->grad, X->f, X->epart);
    };
    if (!GGA && T <= 10) go(std::integral_constant<int, 64>{}, T, 1);
    else if (T <= 40) go(std::integral_constant<int, 32>{}, T, 1);
    else if (T <= 80) go(std::integral_constant<int, 16>{}, T, 1);
    else go(std::integral_constant<int, 16>{}, 32, 2);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

// The tiles of V in groups of up to 8 (rows of tiles in order).
static std::vector<VGroup> v_groups(int nblk, bool gga) {
    std::vector<VGroup> out;
    int first = 0;
    for (int bi = 0; bi < nblk; ++bi)
        for (int bj = gga ? 0 : bi; bj < nblk; ++bj) {
            auto find = [](int *list, int &n, int v) {
                for (int i = 0; i < n; ++i)
                    if (list[i] == v) return i;
                list[n] = v;
                return n++;
            };
            if (out.empty() || out.back().nsup == 8) {
                out.push_back(VGroup{});
                out.back().first = first;
            }
            VGroup &g = out.back();
            // LDA reads both factors from one panel
            g.ai[g.nsup] = find(g.a, g.na, bi);
            g.bj[g.nsup] = gga ? find(g.b, g.nb, bj) : find(g.a, g.na, bj);
            ++g.nsup;
            ++first;
        }
    return out;
}

// How the tiles of V are shared out.
template <bool GGA>
struct VPlan {
    int nblk, ntile, ngroup, nw, KP;
    int64_t chunk, nchunk;
    explicit VPlan(const XcGrid *X) {
        nblk = (X->nbf + kXT - 1) / kXT;
        ntile = GGA ? nblk * nblk : nblk * (nblk + 1) / 2;
        ngroup = (ntile + 7) / 8;
        // chunks of points: two rounds of blocks where a block takes a CU's
        // registers (8 waves), 2048 waves where it holds fewer
        nw = std::min(8, (ntile + 1) / 2 * 2);
        nchunk = std::max<int64_t>(1, nw > 4 ? 512 / ngroup : 2048 / ntile);
        // a group reads at most 8 tiles' row blocks: all of them up to 5 blocks,
        // at most 10 beyond (GGA: 3 left, 8 right); steps of 16 points where two
        // buffers of their rows fit the LDS, of 8 else
        KP = !GGA && nblk <= 5 ? 16 : 8;
        chunk = ((X->G + nchunk - 1) / nchunk + KP - 1) / KP * KP;
        nchunk = (X->G + chunk - 1) / chunk;
    }
};

// The tile groups and the partial sums' place, made with the grid (PBE: with
// the basis gradients) and kept as long: a call that was captured finds them
// where they were.
template <bool GGA>
static int v_prepare(XcGrid *X) {
    const VPlan<GGA> P(X);
    hipError_t e = hipSuccess;
    if (!X->groups) {
        const std::vector<VGroup> l = v_groups(P.nblk, false), g = v_groups(P.nblk, true);
        // what a group's threads load in a step (see kVLoadA) covers its rows
        bool fits = true;
        for (const VGroup &q : l) fits &= 64 * q.na * (P.nblk <= 5 ? 8 : 4) <= kVLoadA<false> * 64 * std::min(8, ((int)l[0].nsup + 1) / 2 * 2);
        for (const VGroup &q : g) {
            const int thr = 64 * std::min(8, ((int)g[0].nsup + 1) / 2 * 2);
            fits &= 64 * q.na * 4 <= kVLoadA<true> * thr && 64 * q.nb * 4 <= kVLoadB * thr && q.na <= 3;
        }
        if (!fits) {
            set_error("internal: exchange-correlation tile groups of %d row blocks", P.nblk);
            return MESS_E_ARG;
        }
        std::vector<VGroup> all(l);
        all.insert(all.end(), g.begin(), g.end());
        e = hipMalloc(&X->groups, sizeof(VGroup) * all.size());
        if (e == hipSuccess) e = hipMemcpy(X->groups, all.data(), sizeof(VGroup) * all.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            hipFree(X->groups);
            X->groups = nullptr;
        }
    }
    if (e == hipSuccess && !X->vpart[GGA]) {
        e = hipMalloc(&X->vpart[GGA], sizeof(double) * P.nchunk * P.ntile * kXT * kXT);
        if (e != hipSuccess) X->vpart[GGA] = nullptr;
    }
    if (e != hipSuccess) {
        set_error("exchange-correlation tiles: %s", hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? MESS_E_NOMEM : MESS_E_DEVICE;
    }
    return MESS_OK;
}

// Vacc <- sum over the grid (k_xc_v).
template <bool GGA>
static int v_async(XcGrid *X, hipStream_t s) {
    const VPlan<GGA> P(X);
    const int nblk = P.nblk, ntile = P.ntile, ngroup = P.ngroup, nw = P.nw, KP = P.KP, N = X->nbf;
    const int64_t chunk = P.chunk, nchunk = P.nchunk;
    const VGroup *groups = reinterpret_cast<const VGroup *>(X->groups) + (GGA ? (nblk * (nblk + 1) / 2 + 7) / 8 : 0);
    const int na = std::min(nblk, GGA ? 3 : 10), nb = GGA ? std::min(nblk, 8) : 0;
    const size_t lds = sizeof(double) * (2 * (size_t)64 * (na + nb) * KP + 2 * KP);
    auto go = [&](auto kernel) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) (void)hipGetLastError();
        hipLaunchKernelGGL(kernel, dim3((unsigned)nchunk, (unsigned)ngroup), dim3(64 * nw), lds, s, N, X->G, chunk, X->phiT,
                           X->dphiT, X->f, X->hv, groups, ntile, X->vpart[GGA]);
    };
    if constexpr (!GGA) {
        if (KP == 16) go(&k_xc_v<false, 16>);
        else go(&k_xc_v<false, 8>);
    } else {
        go(&k_xc_v<true, 8>);
    }
    hipLaunchKernelGGL(k_xc_v_sum<GGA>, dim3(64, (unsigned)ntile), dim3(256), 0, s, N, nblk, ntile, (int)nchunk, X->vpart[GGA],
                       X->Vacc);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

// PBE: V (device N x N, may be NULL) and the device scalar X->ex (E_xc)
// from density D.
int pbe_xc_async(mess_basis *B, const double *D, double *V, hipStream_t s, const double **ex_dev) {
    XcGrid *X = nullptr;
    MESS_TRY(get_xc(B, &X));
    MESS_TRY(ensure_gga(B, X));
    const unsigned npb = (unsigned)((X->G + 255) / 256);
    int nrho = 0;
    MESS_TRY(rho_async<true>(X, D, s, &nrho));
    hipLaunchKernelGGL(k_pbe_point, dim3(npb), dim3(256), 0, s, X->G, X->xyzw, X->rho, X->grad, X->f, X->hv,
                       X->epart);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1024), 0, s, (int)npb, X->epart, X->ex);
    MESS_LAUNCH_CHECK();
    if (V) {
        MESS_TRY(v_async<true>(X, s));
        hipLaunchKernelGGL(k_gga_sym, dim3(256), dim3(256), 0, s, X->nbf, X->Vacc, V);
        MESS_LAUNCH_CHECK();
    }
    if (ex_dev) *ex_dev = X->ex;
    return MESS_OK;
}

// V (device N x N, may be NULL) and the device scalar X->ex from density D.
int lda_x_async(mess_basis *B, const double *D, double *V, hipStream_t s, const double **ex_dev) {
    XcGrid *X = nullptr;
    MESS_TRY(get_xc(B, &X));
    int nrho = 0;
    MESS_TRY(rho_async<false>(X, D, s, &nrho));
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1024), 0, s, nrho, X->epart, X->ex);
    MESS_LAUNCH_CHECK();
    if (V) {
        MESS_TRY(v_async<false>(X, s));
        hipLaunchKernelGGL(k_lda_mirror, dim3(256), dim3(256), 0, s, X->nbf, X->Vacc, V);
        MESS_LAUNCH_CHECK();
    }
    if (ex_dev) *ex_dev = X->ex;
    return MESS_OK;
}

int64_t lda_points(const mess_basis *B) { return (int64_t)B->nat * kPtsPerAtom; }

}  // namespace mess

using namespace mess;

extern "C" {

int mess_lda_x(const mess_basis *basis, const double *D, double *Vx, double *Ex, double *rho, mess_stream stream) {
    if (!basis || !D) {
        set_error("mess_lda_x: NULL basis or density");
        return MESS_E_ARG;
    }
    auto *B = const_cast<mess_basis *>(basis);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double *ex = nullptr;
    MESS_TRY(lda_x_async(B, D, Vx, s, &ex));
    XcGrid *X = static_cast<XcGrid *>(B->xc);
    if (rho) MESS_HIP(hipMemcpyAsync(rho, X->rho, sizeof(double) * X->npts, hipMemcpyDeviceToDevice, s));
    if (Ex) {
        MESS_HIP(hipMemcpyAsync(Ex, ex, sizeof(double), hipMemcpyDeviceToHost, s));
        MESS_HIP(hipStreamSynchronize(s));
    }
    return MESS_OK;
}

int mess_pbe_xc(const mess_basis *basis, const double *D, double *Vxc, double *Exc, double *rho, double *grad_rho,
                mess_stream stream) {
    if (!basis || !D) {
        set_error("mess_pbe_xc: NULL basis or density");
        return MESS_E_ARG;
    }
    auto *B = const_cast<mess_basis *>(basis);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const double *ex = nullptr;
    MESS_TRY(pbe_xc_async(B, D, Vxc, s, &ex));
    XcGrid *X = static_cast<XcGrid *>(B->xc);
    if (rho) MESS_HIP(hipMemcpyAsync(rho, X->rho, sizeof(double) * X->npts, hipMemcpyDeviceToDevice, s));
    if (grad_rho)
        for (int k = 0; k < 3; ++k)
            MESS_HIP(hipMemcpyAsync(grad_rho + k * X->npts, X->grad + k * X->G, sizeof(double) * X->npts,
                                    hipMemcpyDeviceToDevice, s));
    if (Exc) {
        MESS_HIP(hipMemcpyAsync(Exc, ex, sizeof(double), hipMemcpyDeviceToHost, s));
        MESS_HIP(hipStreamSynchronize(s));
    }
    return MESS_OK;
}

int mess_grid(const mess_basis *basis, double *xyzw, int64_t *npts, mess_stream stream) {
    if (!basis) {
        set_error("mess_grid: NULL basis");
        return MESS_E_ARG;
    }
    auto *B = const_cast<mess_basis *>(basis);
    if (B->n_mol != 1) {
        set_error("mess_grid: LDA grids are built for a single molecule, not a batch of %d", B->n_mol);
        return MESS_E_UNSUPPORTED;
    }
    if (npts) *npts = lda_points(B);
    if (!xyzw) return MESS_OK;
    XcGrid *X = nullptr;
    MESS_TRY(get_xc(B, &X));
    MESS_HIP(hipMemcpyAsync(xyzw, X->xyzw, sizeof(double) * 4 * X->npts, hipMemcpyDeviceToDevice,
                            static_cast<hipStream_t>(stream)));
    return MESS_OK;
}

}  // extern "C"
