// J and K of many densities from a dense ERI tensor (section 3: the Coulomb
// and exchange matrices are contractions of the repulsion integrals with the
// density), as matrix products over the composite indices r = (i, j),
// c = (k, l) of the N^2 x N^2 views of the tensor:
//   J[d][r] = sum_c (ij|kl) D_d[c],     K[d][r] = sum_c (ik|jl) D_d[c],
// so that with many densities the contraction is a dense product whose
// arithmetic intensity grows with the density count.  Two forms:
//   - MFMA (k_dense_mfma): a wave owns 32 or 48 rows x 16, 32 or 64 densities as
//     16 x 16 x 4 products (FP64 or FP32 operands, accumulation in the operand
//     precision), its operands straight from memory: a lane takes four
//     elements of its tensor row and of its density's row per step of 16
//     columns, which four products use one after another, so neither operand
//     passes through LDS and no wave waits for another.  The eight waves of a
//     block share the rows and take every eighth k; their sums meet in LDS in
//     a fixed order.  J and K run in one launch, their blocks in turn, so that
//     the second reader of a part of the tensor finds it in the last cache.
//     Tensors narrower than a load (one function in FP64, three in FP32) take
//     the other form.
//   - VALU (k_dense_valu): 256-thread blocks own 64 rows x 64 densities, stage
//     64 x 32 tensor and 32 x 64 density panels in LDS and accumulate 16
//     densities a lane with FMAs; the column range is split over blockIdx.z
//     when the row and density tiles alone leave the chip's 256 CUs
//     underfilled, and split parts add into the zeroed output with atomics.
// The two forms are compared by rocprof on the same inputs.
#include <algorithm>

#include "mess_internal.hpp"

namespace mess {

constexpr int kDjRows = 64, kDjDens = 64, kDjK = 32;

typedef double dj_double4 __attribute__((ext_vector_type(4)));
typedef float dj_float4 __attribute__((ext_vector_type(4)));

template <typename Real> struct DjVec;
template <> struct DjVec<double> { using type = dj_double4; };
template <> struct DjVec<float> { using type = dj_float4; };

template <typename Real>
__device__ __forceinline__ typename DjVec<Real>::type dj_mfma(Real a, Real b, typename DjVec<Real>::type c) {
    if constexpr (sizeof(Real) == 8)
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

typedef double dj_d2u __attribute__((ext_vector_type(2), aligned(8)));
typedef float dj_f4u __attribute__((ext_vector_type(4), aligned(4)));
template <typename Real> struct DjVecU;  // 16 bytes at an element's alignment
template <> struct DjVecU<double> { using type = dj_d2u; };
template <> struct DjVecU<float> { using type = dj_f4u; };

constexpr int kDjWaves = 8;

// J (even blocks if both are asked for) and K of 16 NDT densities on 16 NRT
// rows (i, j): element (k, l) of a row at i N^3 + j N^2 + k N + l for J and
// i N^3 + k N^2 + j N + l for K.  Bound by the two reads of the tensor with few
// densities; with 64 the matrix rate (0.43 ms for 105 functions in FP64) and
// the loads' latency, which two waves a SIMD and one step of prefetch hide
// about half of.  Staging both panels in LDS between barriers, with split
// columns added by atomics, took 2.1 times as long (18.9 TFLOP/s).
template <typename Real, int NDT, int NRT>
__global__ void __launch_bounds__(64 * kDjWaves) k_dense_mfma(int N, int nd, const Real *__restrict__ eri,
                                                              const Real *__restrict__ D, Real *__restrict__ J,
                                                              Real *__restrict__ K) {
    using V = typename DjVec<Real>::type;
    using VU = typename DjVecU<Real>::type;
    constexpr int E = 16 / sizeof(Real), P = 4 / E;  // elements a load, loads a step
    constexpr int kDjWRows = 16 * NRT;
    __shared__ Real red[kDjWaves / 2][kDjWRows * 16 * NDT];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane / 16;
    const int64_t M = (int64_t)N * N;
    const bool isk = !J || (K && (blockIdx.x & 1));
    const int64_t r0 = (int64_t)(blockIdx.x >> (J && K ? 1 : 0)) * kDjWRows;
    const int d0 = blockIdx.y * 16 * NDT;
    Real *out = isk ? K : J;
    const int64_t ks = isk ? M : N;  // stride of k in the tensor
    const Real *pa[NRT], *pb[NDT];
#pragma unroll
    for (int t = 0; t < NRT; ++t) {
        // rows beyond the last repeat it (not stored)
        const int64_t r = min(r0 + 16 * t + lane % 16, M - 1);
        pa[t] = eri + (isk ? r / N * M * N + r % N * N : r * M);
    }
#pragma unroll
    for (int t = 0; t < NDT; ++t) pb[t] = D + (int64_t)min(d0 + 16 * t + lane % 16, nd - 1) * M;
    V acc[NRT][NDT];
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int u = 0; u < NDT; ++u) acc[t][u] = {0, 0, 0, 0};
    // the lane's four elements of columns l0 .. l0 + 15 of row k, each load
    // moved back to end with the row where it would pass its end
    auto load = [&](const Real *p, int l0) {
        V v;
#pragma unroll
        for (int h = 0; h < P; ++h) {
            const VU u = *reinterpret_cast<const VU *>(p + min(l0 + 4 * E * h + E * g, N - E));
#pragma unroll
            for (int s = 0; s < E; ++s) v[E * h + s] = u[s];
        }
        return v;
    };
    // undoes that: elements to their places, zero beyond the last column
    auto settle = [&](V &v, int l0) {
#pragma unroll
        for (int h = 0; h < P; ++h) {
            const int back = max(l0 + 4 * E * h + E * g - (N - E), 0);
#pragma unroll
            for (int s = 0; s < E; ++s) {
                Real x = 0;
#pragma unroll
                for (int q = s; q < E; ++q) x = back == q - s ? v[E * h + q] : x;
                v[E * h + s] = x;
            }
        }
    };
    V a[NRT], b[NDT], an[NRT], bn[NDT];
    auto fetch = [&](V(&x)[NRT], V(&y)[NDT], int k, int l0) {
#pragma unroll
        for (int t = 0; t < NRT; ++t) x[t] = load(pa[t] + (int64_t)k * ks, l0);
#pragma unroll
        for (int t = 0; t < NDT; ++t) y[t] = load(pb[t] + (int64_t)k * N, l0);
    };
    int k = wave, l0 = 0;
    if (k < N) fetch(an, bn, k, l0);
    while (k < N) {
#pragma unroll
        for (int t = 0; t < NRT; ++t) a[t] = an[t];
#pragma unroll
        for (int t = 0; t < NDT; ++t) b[t] = bn[t];
        const int lc = l0;
        l0 += 16;
        if (l0 >= N) {
            l0 = 0;
            k += kDjWaves;
        }
        fetch(an, bn, min(k, N - 1), l0);
        if (lc + 16 > N) {
#pragma unroll
            for (int t = 0; t < NRT; ++t) settle(a[t], lc);
#pragma unroll
            for (int t = 0; t < NDT; ++t) settle(b[t], lc);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < NRT; ++t)
#pragma unroll
                for (int u = 0; u < NDT; ++u) acc[t][u] = dj_mfma<Real>(a[t][s], b[u][s], acc[t][u]);
    }
    // the waves' sums in LDS: the upper half hands over, three times
#pragma unroll
    for (int h = kDjWaves / 2; h > 0; h /= 2) {
        if (wave >= h && wave < 2 * h)
#pragma unroll
            for (int t = 0; t < NRT; ++t)
#pragma unroll
                for (int u = 0; u < NDT; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) red[wave - h][((t * NDT + u) * 4 + q) * 64 + lane] = acc[t][u][q];
        __syncthreads();
        if (wave < h)
#pragma unroll
            for (int t = 0; t < NRT; ++t)
#pragma unroll
                for (int u = 0; u < NDT; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[t][u][q] += red[wave][((t * NDT + u) * 4 + q) * 64 + lane];
        __syncthreads();
    }
    if (wave) return;
    // result element q of lane l: density l % 16 and, of the tile's 16 rows,
    // row 4 (l / 16) + q for the FP32 product but row l / 16 + 4 q for the
    // FP64 one (measured lane layouts)
#pragma unroll
    for (int t = 0; t < NRT; ++t)
#pragma unroll
        for (int u = 0; u < NDT; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t r = r0 + 16 * t + (sizeof(Real) == 8 ? g + 4 * q : 4 * g + q);
                const int d = d0 + 16 * u + lane % 16;
                if (r < M && d < nd) out[(int64_t)d * M + r] = acc[t][u][q];
            }
}

// KMODE 0: A(r, c) = eri[r M + c] (J); 1: A((i,j), (k,l)) = eri[((i N + k) N + j) N + l] (K)
template <typename Real, int KMODE>
__global__ void __launch_bounds__(256) k_dense_valu(int N, int nd, int64_t chunk, const Real *__restrict__ eri,
                                                  const Real *__restrict__ D, Real *__restrict__ out) {
    __shared__ Real As[kDjRows][kDjK + 1];
    __shared__ Real Bs[kDjK][kDjDens + 1];
    const int64_t M = (int64_t)N * N;
    const int64_t r0 = (int64_t)blockIdx.x * kDjRows;
    const int d0 = blockIdx.y * kDjDens;
    const int t = threadIdx.x, w = t / 64, l = t % 64;
    Real vacc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) vacc[j] = 0;
    const int64_t cb = (int64_t)blockIdx.z * chunk, ce = cb + chunk < M ? cb + chunk : M;
    const bool split = gridDim.z > 1;
    for (int64_t c0 = cb; c0 < ce; c0 += kDjK) {
        // tensor panel: 64 rows x 16 columns, four elements per thread
        for (int e = t; e < kDjRows * kDjK; e += 256) {
            const int rr = e / kDjK, cc = e % kDjK;
            const int64_t r = r0 + rr, c = c0 + cc;
            Real v = 0;
            if (r < M && c < ce) {
                if (KMODE == 0) {
                    v = eri[r * M + c];
                } else {
                    const int64_t i = r / N, j = r % N, k = c / N, ll = c % N;
                    v = eri[((i * N + k) * N + j) * N + ll];
                }
            }
            As[rr][cc] = v;
        }
        // density panel: 16 columns x 64 densities, four elements per thread
        for (int e = t; e < kDjK * kDjDens; e += 256) {
            const int cc = e % kDjK, dd = e / kDjK;
            const int64_t c = c0 + cc;
            Bs[cc][dd] = (c < ce && d0 + dd < nd) ? D[(int64_t)(d0 + dd) * M + c] : Real(0);
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < kDjK; ++kk) {
            const Real a = As[16 * w + l % 16][kk];
#pragma unroll
            for (int j = 0; j < 16; ++j) vacc[j] = fma(a, Bs[kk][16 * (l / 16) + j], vacc[j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int64_t r = r0 + 16 * w + l % 16;
        const int d = d0 + 16 * (l / 16) + j;
        if (r < M && d < nd) {
            if (split) unsafeAtomicAdd(&out[(int64_t)d * M + r], vacc[j]);
            else out[(int64_t)d * M + r] = vacc[j];
        }
    }
}

template <typename Real>
__global__ void k_dj_zero(int64_t n, Real *__restrict__ p) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = Real(0);
}

// 64, 32 or 16 densities a wave: the fewest that hold them all, several tiles
// of 64 beyond.  48 rows a wave with 64 densities where that leaves a block a
// CU, since its 12 accumulators use each loaded element more often (105
// functions, FP64, normally distributed operands: 801 us, 32 rows 901 us); 32
// rows below (30 functions, 70 densities: 27 us, 48 rows 36 us).  Both: 105
// functions 1651 -> 801 us with 64 densities, 1364 -> 490 us with 16, 1297 ->
// 396 us with one (two reads of the tensor at 4.9 TB/s); FP32 with 64 1315 ->
// 450 us.
template <typename Real>
static void launch_mfma(int N, int nd, const Real *eri, const Real *D, Real *J, Real *K, hipStream_t s) {
    auto tiles = [&](int rows) { return (int)(((int64_t)N * N + rows - 1) / rows) * ((J ? 1 : 0) + (K ? 1 : 0)); };
    auto go = [&](auto T, auto R) {
        constexpr int NDT = decltype(T)::value, NRT = decltype(R)::value;
        const dim3 grid((unsigned)tiles(16 * NRT), (unsigned)((nd + 16 * NDT - 1) / (16 * NDT)));
        hipLaunchKernelGGL((k_dense_mfma<Real, NDT, NRT>), grid, dim3(64 * kDjWaves), 0, s, N, nd, eri, D, J, K);
    };
    std::integral_constant<int, 1> one;
    std::integral_constant<int, 2> two;
    std::integral_constant<int, 3> three;
    std::integral_constant<int, 4> four;
    if (nd <= 16) go(one, two);
    else if (nd <= 32) go(two, two);
    else if ((int64_t)tiles(48) * ((nd + 63) / 64) < 256) go(four, two);
    else go(four, three);
}

template <typename Real>
static void launch_valu(int N, int nd, const Real *eri, const Real *D, Real *J, Real *K, hipStream_t s) {
    const int64_t M = (int64_t)N * N;
    const unsigned gx = (unsigned)((M + kDjRows - 1) / kDjRows), gy = (unsigned)((nd + kDjDens - 1) / kDjDens);
    // split the columns until about 2048 blocks (8 per CU), in chunks of at
    // least 64 staging steps
    int64_t nz = 2048 / std::max<int64_t>(1, (int64_t)gx * gy);
    nz = std::max<int64_t>(1, std::min<int64_t>(nz, M / (64 * kDjK)));
    const int64_t chunk = ((M + nz - 1) / nz + kDjK - 1) / kDjK * kDjK;
    nz = (M + chunk - 1) / chunk;
    const dim3 grid(gx, gy, (unsigned)nz);
    const int64_t nout = (int64_t)nd * M;
    const unsigned zb = (unsigned)std::min<int64_t>((nout + 255) / 256, 65536);
    if (J) {
        if (nz > 1) hipLaunchKernelGGL(k_dj_zero<Real>, dim3(zb), dim3(256), 0, s, nout, J);
        hipLaunchKernelGGL((k_dense_valu<Real, 0>), grid, dim3(256), 0, s, N, nd, chunk, eri, D, J);
    }
    if (K) {
        if (nz > 1) hipLaunchKernelGGL(k_dj_zero<Real>, dim3(zb), dim3(256), 0, s, nout, K);
        hipLaunchKernelGGL((k_dense_valu<Real, 1>), grid, dim3(256), 0, s, N, nd, chunk, eri, D, K);
    }
}

}  // namespace mess

using namespace mess;

extern "C" int mess_jk_dense(const void *eri, int32_t n, int32_t ndens, const void *D, void *J, void *K,
                             int32_t prec, int32_t form, mess_stream stream) {
    if (!eri || !D || n < 1 || ndens < 1) {
        set_error("mess_jk_dense: need eri, D, n >= 1 and ndens >= 1");
        return MESS_E_ARG;
    }
    if ((prec != MESS_FP64 && prec != MESS_FP32) || (form != MESS_DENSE_VALU && form != MESS_DENSE_MFMA)) {
        set_error("mess_jk_dense: prec must be MESS_FP64 or MESS_FP32, form MESS_DENSE_VALU or MESS_DENSE_MFMA");
        return MESS_E_ARG;
    }
    if ((int64_t)n * n > ((int64_t)1 << 31) / 2 || ndens > 65535 * kDjDens) {
        set_error("mess_jk_dense: n or ndens out of range");
        return MESS_E_ARG;
    }
    if (!J && !K) return MESS_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool mf = form == MESS_DENSE_MFMA;
    if (prec == MESS_FP64) {
        auto *e = static_cast<const double *>(eri);
        auto *d = static_cast<const double *>(D);
        if (mf && n >= 16 / (int)sizeof(*e)) launch_mfma<double>(n, ndens, e, d, static_cast<double *>(J), static_cast<double *>(K), s);
        else launch_valu<double>(n, ndens, e, d, static_cast<double *>(J), static_cast<double *>(K), s);
    } else {
        auto *e = static_cast<const float *>(eri);
        auto *d = static_cast<const float *>(D);
        if (mf && n >= 16 / (int)sizeof(*e)) launch_mfma<float>(n, ndens, e, d, static_cast<float *>(J), static_cast<float *>(K), s);
        else launch_valu<float>(n, ndens, e, d, static_cast<float *>(J), static_cast<float *>(K), s);
    }
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}
