// Learned initial density guess: atom-pair features, a 64 -> 256 -> 256 ->
// 128 perceptron (SiLU hidden layers) whose outputs are density blocks,
// assembly into a packed block-diagonal density, and training by masked
// mean-squared error with Adam.  Every layer product runs on the BF16
// matrix cores (v_mfma_f32_16x16x16_bf16): operands are rounded to BF16
// (nearest, ties to even), products accumulate in FP32, and biases,
// pre-activations, gradients and the Adam state stay FP32.
//
// Pair rows: for each molecule, atoms A <= B in A-major order.  Features
// (42 of 64 used): one-hot element of A and B over (H, C, N, O); 16
// Gaussian radial functions of R_AB (centres k 10/15, width 10/15 bohr);
// the unit vector A -> B and its six products; per-element neighbour counts
// of A and B with the cutoff (cos(pi R/6) + 1)/2 below 6 bohr; a self-pair
// flag.  Output 11 i + j is the density element between function i of A and
// function j of B.
#include <algorithm>
#include <cmath>
#include <vector>

#include "mess_internal.hpp"

namespace mess {

constexpr int kIn = 64, kHid = 256, kOut = 128, kBlk = 11;
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kHid * kIn, kOffW2 = kOffB1 + kHid,
                  kOffB2 = kOffW2 + kHid * kHid, kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kOut * kHid,
                  kNParam = kOffB3 + kOut;
static_assert(kNParam == MESS_MLP_NPARAM, "parameter layout");

struct PairRow {
    int64_t moff;    // packed block of the molecule
    int n;           // functions of the molecule
    int fa, na;      // first function (within the molecule) and count of atom A
    int fb, nb;      // same for atom B
    int self, pad;
};

struct GuessTables {
    int64_t nrows = 0;
    std::vector<PairRow> rows;
    std::vector<float> feat;   // [nrows][64]
    PairRow *d_rows = nullptr;
};

void free_guess_tables(mess_basis *B) {
    auto *T = static_cast<GuessTables *>(B->guess);
    if (!T) return;
    hipFree(T->d_rows);
    delete T;
    B->guess = nullptr;
}

static int element_index(int Z) { return Z == 1 ? 0 : Z == 6 ? 1 : Z == 7 ? 2 : Z == 8 ? 3 : -1; }

static int get_tables(mess_basis *B, GuessTables **out) {
    if (B->guess) {
        *out = static_cast<GuessTables *>(B->guess);
        return MESS_OK;
    }
    auto *T = new GuessTables();
    for (int m = 0; m < B->n_mol; ++m) {
        const int a0 = B->mol_atom0[m], na = B->mol_natom[m];
        std::vector<int> first(na, -1), count(na, 0), el(na);
        int last = -1;
        for (int s = B->mol_sh0[m]; s < B->mol_sh0[m] + B->mol_nsh[m]; ++s) {
            const int a = B->sh_atom[s] - a0;
            if (first[a] < 0) {
                if (a < last) goto noncontig;
                first[a] = B->sh_bf0[s] - B->mol_bf0[m];
            } else if (a != last) {
                goto noncontig;
            }
            last = a;
            count[a] += ncart(B->sh_l[s]);
        }
        for (int a = 0; a < na; ++a) {
            el[a] = element_index(B->Z[a0 + a]);
            if (el[a] < 0 || count[a] == 0 || count[a] > kBlk) {
                delete T;
                set_error("learned guess: atom %d of molecule %d has Z=%d and %d functions (H, C, N, O with 1..11 "
                          "functions are supported)",
                          a, m, B->Z[a0 + a], count[a]);
                return MESS_E_UNSUPPORTED;
            }
        }
        {
            const double *X = &B->xyz[3 * a0];
            std::vector<double> cnt(4 * na, 0.0);
            for (int a = 0; a < na; ++a)
                for (int c = 0; c < na; ++c) {
                    if (c == a) continue;
                    const double dx = X[3 * a] - X[3 * c], dy = X[3 * a + 1] - X[3 * c + 1],
                                 dz = X[3 * a + 2] - X[3 * c + 2];
                    const double r = std::sqrt(dx * dx + dy * dy + dz * dz);
                    if (r < 6.0) cnt[4 * a + el[c]] += 0.5 * (std::cos(M_PI * r / 6.0) + 1.0);
                }
            for (int a = 0; a < na; ++a)
                for (int b = a; b < na; ++b) {
                    PairRow pr{B->mol_moff[m], B->mol_nbf[m], first[a], count[a], first[b], count[b], a == b, 0};
                    T->rows.push_back(pr);
                    double f[kIn] = {0.0};
                    f[el[a]] = 1.0;
                    f[4 + el[b]] = 1.0;
                    const double dx = X[3 * b] - X[3 * a], dy = X[3 * b + 1] - X[3 * a + 1],
                                 dz = X[3 * b + 2] - X[3 * a + 2];
                    const double r = std::sqrt(dx * dx + dy * dy + dz * dz);
                    const double sig = 10.0 / 15.0;
                    for (int k = 0; k < 16; ++k) {
                        const double t = (r - k * sig) / sig;
                        f[8 + k] = std::exp(-(t * t));
                    }
                    if (a != b) {
                        const double u[3] = {dx / r, dy / r, dz / r};
                        f[24] = u[0];
                        f[25] = u[1];
                        f[26] = u[2];
                        f[27] = u[0] * u[0];
                        f[28] = u[0] * u[1];
                        f[29] = u[0] * u[2];
                        f[30] = u[1] * u[1];
                        f[31] = u[1] * u[2];
                        f[32] = u[2] * u[2];
                    }
                    for (int e = 0; e < 4; ++e) {
                        f[33 + e] = cnt[4 * a + e];
                        f[37 + e] = cnt[4 * b + e];
                    }
                    f[41] = a == b ? 1.0 : 0.0;
                    for (int k = 0; k < kIn; ++k) T->feat.push_back((float)f[k]);
                }
        }
        continue;
    noncontig:
        delete T;
        set_error("learned guess: the shells of an atom of molecule %d are not contiguous", m);
        return MESS_E_UNSUPPORTED;
    }
    T->nrows = (int64_t)T->rows.size();
    if (hipMalloc(&T->d_rows, sizeof(PairRow) * std::max<int64_t>(T->nrows, 1)) != hipSuccess ||
        hipMemcpy(T->d_rows, T->rows.data(), sizeof(PairRow) * T->nrows, hipMemcpyHostToDevice) != hipSuccess) {
        hipFree(T->d_rows);
        delete T;
        set_error("learned guess: cannot allocate pair tables");
        return MESS_E_NOMEM;
    }
    B->guess = T;
    *out = T;
    return MESS_OK;
}

// T[r][11 i + j] = D block element, M = 1 inside the block (0 elsewhere).
__global__ void k_guess_targets(int64_t nrows, const PairRow *__restrict__ rows, const double *__restrict__ D,
                                float *__restrict__ T, float *__restrict__ M) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= nrows * kOut) return;
    const int64_t r = t / kOut;
    const int k = (int)(t % kOut), i = k / kBlk, j = k % kBlk;
    const PairRow p = rows[r];
    const bool in = k < kBlk * kBlk && i < p.na && j < p.nb;
    if (T) T[t] = in ? (float)D[p.moff + (int64_t)(p.fa + i) * p.n + p.fb + j] : 0.0f;
    if (M) M[t] = in ? 1.0f : 0.0f;
}

// D[A_i][B_j] = D[B_j][A_i] = Y[r][11 i + j]; diagonal blocks symmetrised.
__global__ void k_guess_assemble(int64_t nrows, const PairRow *__restrict__ rows, const float *__restrict__ Y,
                                 double *__restrict__ D) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= nrows * kBlk * kBlk) return;
    const int64_t r = t / (kBlk * kBlk);
    const int k = (int)(t % (kBlk * kBlk)), i = k / kBlk, j = k % kBlk;
    const PairRow p = rows[r];
    if (i >= p.na || j >= p.nb) return;
    const float *y = Y + r * kOut;
    const double v = p.self ? 0.5 * ((double)y[kBlk * i + j] + (double)y[kBlk * j + i]) : (double)y[kBlk * i + j];
    D[p.moff + (int64_t)(p.fa + i) * p.n + p.fb + j] = v;
    D[p.moff + (int64_t)(p.fb + j) * p.n + p.fa + i] = v;
}

// ------------------------------------------------------------ BF16 MFMA

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short to_bf16(float x) {
    unsigned u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// Fragment order.  v_mfma_f32_16x16x16_bf16 takes from lane l the four
// elements A[l % 16][4 (l / 16) + 0..3] and B[4 (l / 16) + 0..3][l % 16] and
// returns in lane l the rows 4 (l / 16) + 0..3 of column l % 16.  A matrix
// whose contracted index is r and whose other index is c is kept as
// [c / 16][r / 16][lane][r % 4], lane = c % 16 + 16 ((r % 16) / 4), so a
// wave reads one operand as 512 consecutive bytes, and an accumulator tile
// rounded to BF16 is, lane by lane, an operand of a product contracted over
// its rows: what the row kernel writes is what the weight gradient reads.
//
// Weights are held in fragment order with the fragments of two consecutive
// contraction steps side by side (16 bytes a lane), once for the forward
// products (contracted over inputs) and, for layers 2 and 3, once for the
// backward ones (contracted over outputs).
constexpr int kW1f = 0, kW2f = kW1f + kHid * kIn, kW3f = kW2f + kHid * kHid, kW2b = kW3f + kOut * kHid,
              kW3b = kW2b + kHid * kHid, kNPacked = kW3b + kOut * kHid;

// Place of element (c, r) of a weight operand contracted over R values of r.
__host__ __device__ __forceinline__ int packed_at(int c, int r, int R) {
    const int lane = c % 16 + 16 * ((r % 16) / 4);
    return (((c / 16) * (R / 32) + r / 32) * 64 + lane) * 8 + ((r / 16) % 2) * 4 + r % 4;
}

// Writes parameter i (a weight) to its packed places.
__device__ __forceinline__ void pack_weight(int64_t i, float x, unsigned short *__restrict__ pk) {
    const unsigned short v = to_bf16(x);
    if (i < kOffB1) {
        pk[kW1f + packed_at((int)i / kIn, (int)i % kIn, kIn)] = v;
    } else if (i >= kOffW2 && i < kOffB2) {
        const int o = (int)(i - kOffW2) / kHid, k = (int)(i - kOffW2) % kHid;
        pk[kW2f + packed_at(o, k, kHid)] = v;
        pk[kW2b + packed_at(k, o, kHid)] = v;
    } else if (i >= kOffW3 && i < kOffB3) {
        const int o = (int)(i - kOffW3) / kHid, k = (int)(i - kOffW3) % kHid;
        pk[kW3f + packed_at(o, k, kHid)] = v;
        pk[kW3b + packed_at(k, o, kOut)] = v;
    }
}

__global__ void k_pack(const float *__restrict__ p, unsigned short *__restrict__ pk) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < kNParam) pack_weight(i, p[i], pk);
}

constexpr int kMaskBlocks = 256;
constexpr int kRowBlocksMax = 1024;  // blocks of the row kernel (bias and loss partials)
constexpr int kBias = 2 * kHid + kOut;
constexpr int kLdsRow = kHid + 8;    // BF16 elements of an activation row in LDS: 4 banks from row to row

// Partial sums of the mask, one per block.
__global__ void __launch_bounds__(256) k_mask_sum(int64_t n, const float *__restrict__ M, double *__restrict__ part) {
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)kMaskBlocks * 256) s += M[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// acc[i][j] += A (rows 16 i.., R values of r, LDS) times NT column tiles of
// a packed weight operand starting at column tile ct0.
template <int RT, int NT, int R>
__device__ __forceinline__ void row_product(const unsigned short *__restrict__ As, int lda,
                                            const unsigned short *__restrict__ W, int ct0, int lane,
                                            v4f (&acc)[RT][NT]) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // four steps of loads in flight; unrolled further, the loads of all five
    // products are hoisted to the top and spill
#pragma unroll RT == 1 ? 4 : 2
    for (int s2 = 0; s2 < R / 32; ++s2) {
        struct alignas(16) Pair { v4s f[2]; } b[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
            b[j] = *reinterpret_cast<const Pair *>(W + (((ct0 + j) * (R / 32) + s2) * 64 + lane) * 8);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const v4s a = *reinterpret_cast<const v4s *>(As + (16 * i + lane % 16) * lda + 32 * s2 + 16 * h + 4 * (lane / 16));
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b[j].f[h], acc[i][j], 0, 0, 0);
            }
    }
}

// Activations and back-propagated gradients kept for the weight gradients,
// in fragment order over the rows (ns steps of 16 rows).
struct RowFrags {
    unsigned short *X, *H1, *H2, *dY, *dZ2, *dZ1;
    int64_t ns;
};

__device__ __forceinline__ void put_frag(unsigned short *__restrict__ F, int64_t ns, int ct, int64_t rs, int lane, v4s v) {
    *reinterpret_cast<v4s *>(F + (((int64_t)ct * ns + rs) * 64 + lane) * 4) = v;
}

// The whole network over 16 RT rows a block: the three layers and, with
// GRAD, the loss, both hidden gradients and the partial sums of the bias
// gradients and of the loss.  The chain of five products is short and every
// layer needs all of the one before it, so what bounds it is latency, then
// the 416 KB of weights that every block reads from the L2: the rows stay in
// one block, the activations in LDS, the pre-activations in the registers of
// the lanes that need them again (the tile of Z that a lane computes is the
// tile of dZ that it computes later), and a wave owns 64 of the 256 hidden
// columns, its weight fragments as 1 KB loads.  Each product accumulates in
// ascending contraction order.  Before, every layer was a launch of its own
// that read and wrote its operands in global memory (gradient call of 4096
// rows, all kernels: 1480 -> 68 us, of which the one-block mask sum was 525,
// the three split weight products with FP32 atomics 410, the three column
// sums with one row group a block 360).
template <int RT, bool GRAD>
__global__ void __launch_bounds__(256) k_mlp_rows(int64_t n, const float *__restrict__ X, const float *__restrict__ p,
                                                  const unsigned short *__restrict__ pk, float *__restrict__ Y,
                                                  const float *__restrict__ T, const float *__restrict__ M,
                                                  const double *__restrict__ mpart, RowFrags fr,
                                                  double *__restrict__ lpart, float *__restrict__ bpart) {
    __shared__ __align__(16) unsigned short Xs[16 * RT][kIn + 8];
    __shared__ __align__(16) unsigned short Ha[16 * RT][kLdsRow];
    __shared__ __align__(16) unsigned short Hb[16 * RT][kLdsRow];
    __shared__ double red[256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, rq = 4 * (lane >> 4);
    float inv = 0.0f;
    if constexpr (GRAD) {
        red[threadIdx.x] = mpart[threadIdx.x];
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        inv = 2.0f / (float)red[0];
        __syncthreads();
    }
    double loss = 0.0;
    float db1[4] = {}, db2[4] = {}, db3[2] = {};
    const int64_t ntile = (n + 16 * RT - 1) / (16 * RT);
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t r0 = tile * 16 * RT;
#pragma unroll
        for (int t = threadIdx.x; t < 16 * RT * kIn; t += 256) {
            const int64_t r = r0 + t / kIn;
            Xs[t / kIn][t % kIn] = r < n ? to_bf16(X[r * kIn + t % kIn]) : 0;
        }
        __syncthreads();
        if constexpr (GRAD)
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                v4s v;
                for (int q = 0; q < 4; ++q) v[q] = (short)Xs[16 * i + rq + q][16 * wave + col];
                put_frag(fr.X, fr.ns, wave, tile * RT + i, lane, v);
            }
        // Z = A W^T + b into z, silu(Z) as BF16 to the next layer's rows
        v4f z1[RT][4], z2[RT][4];
        auto hidden = [&](v4f(&z)[RT][4], const float *bias, unsigned short (*H)[kLdsRow], unsigned short *F) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = 64 * wave + 16 * j + col;
                const float b = bias[c];
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    v4s h;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        z[i][j][q] += b;
                        h[q] = (short)to_bf16(silu_f(z[i][j][q]));
                        H[16 * i + rq + q][c] = (unsigned short)h[q];
                    }
                    if constexpr (GRAD) put_frag(F, fr.ns, 4 * wave + j, tile * RT + i, lane, h);
                }
            }
        };
        row_product<RT, 4, kIn>(&Xs[0][0], kIn + 8, pk + kW1f, 4 * wave, lane, z1);
        hidden(z1, p + kOffB1, Ha, fr.H1);
        __syncthreads();
        row_product<RT, 4, kHid>(&Ha[0][0], kLdsRow, pk + kW2f, 4 * wave, lane, z2);
        hidden(z2, p + kOffB2, Hb, fr.H2);
        __syncthreads();
        v4f y[RT][2];
        row_product<RT, 2, kHid>(&Hb[0][0], kLdsRow, pk + kW3f, 2 * wave, lane, y);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = 32 * wave + 16 * j + col;
            const float b = p[kOffB3 + c];
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                v4s g4;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t r = r0 + 16 * i + rq + q;
                    const float v = y[i][j][q] + b;
                    if constexpr (GRAD) {
                        // dY = 2 M (Y - T) / sum(M)
                        const float d = r < n ? M[r * kOut + c] * (v - T[r * kOut + c]) : 0.0f;
                        loss += (double)d * d;
                        const float g = d * inv;
                        db3[j] += g;
                        g4[q] = (short)to_bf16(g);
                        Ha[16 * i + rq + q][c] = (unsigned short)g4[q];
                    } else if (r < n) {
                        Y[r * kOut + c] = v;
                    }
                }
                if constexpr (GRAD) put_frag(fr.dY, fr.ns, 2 * wave + j, tile * RT + i, lane, g4);
            }
        }
        __syncthreads();
        if constexpr (GRAD) {
            // dZ = (dOut W) .* silu'(Z)
            auto back = [&](v4f(&acc)[RT][4], const v4f(&z)[RT][4], float(&db)[4], unsigned short (*H)[kLdsRow],
                            unsigned short *F) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        v4s h;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float d = acc[i][j][q] * dsilu_f(z[i][j][q]);
                            db[j] += d;
                            h[q] = (short)to_bf16(d);
                            if (H) H[16 * i + rq + q][64 * wave + 16 * j + col] = (unsigned short)h[q];
                        }
                        put_frag(F, fr.ns, 4 * wave + j, tile * RT + i, lane, h);
                    }
            };
            v4f acc[RT][4];
            row_product<RT, 4, kOut>(&Ha[0][0], kLdsRow, pk + kW3b, 4 * wave, lane, acc);
            back(acc, z2, db2, Hb, fr.dZ2);
            __syncthreads();
            row_product<RT, 4, kHid>(&Hb[0][0], kLdsRow, pk + kW2b, 4 * wave, lane, acc);
            back(acc, z1, db1, nullptr, fr.dZ1);
        }
    }
    if constexpr (GRAD) {
        // column sums over the block's rows: the four row groups of a wave
        float *bp = bpart + (int64_t)blockIdx.x * kBias;
        auto put = [&](float v, int c) {
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lane < 16) bp[c + lane] = v;
        };
#pragma unroll
        for (int j = 0; j < 4; ++j) put(db1[j], 64 * wave + 16 * j);
#pragma unroll
        for (int j = 0; j < 4; ++j) put(db2[j], kHid + 64 * wave + 16 * j);
#pragma unroll
        for (int j = 0; j < 2; ++j) put(db3[j], 2 * kHid + 32 * wave + 16 * j);
        red[threadIdx.x] = loss;
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) lpart[blockIdx.x] = red[0];
    }
}

// Weight gradients dW[o][i] = sum over rows of dOut[row][o] In[row][i]: a
// block takes one of the 28 tiles of 64 x 64 (8 of W3, 16 of W2, 4 of W1)
// and one of gridDim.y chunks of row steps, its four waves every fourth step
// each, summed in LDS; chunks leave partial sums for k_mlp_finish.  Both
// operands are read in fragment order, 512 consecutive bytes a wave.  The
// weights are too few to fill the chip with one block a tile, so the rows are
// split, into at most 32 chunks so that the partial sums stay below 15 MB.
// (FP32 atomics in their place cost 137 us a layer at 4096 rows.)
__global__ void __launch_bounds__(256) k_mlp_wgrad(RowFrags fr, int64_t steps_per, float *__restrict__ part) {
    __shared__ float red[4][64 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int t = blockIdx.x;
    const unsigned short *A, *B;
    int64_t off;
    int ldw, ot, it;
    if (t < 8) {
        A = fr.dY, B = fr.H2, off = kOffW3, ldw = kHid, ot = t / 4, it = t % 4;
    } else if (t < 24) {
        t -= 8;
        A = fr.dZ2, B = fr.H1, off = kOffW2, ldw = kHid, ot = t / 4, it = t % 4;
    } else {
        A = fr.dZ1, B = fr.X, off = kOffW1, ldw = kIn, ot = t - 24, it = 0;
    }
    const int64_t s0 = blockIdx.y * steps_per, s1 = s0 + steps_per < fr.ns ? s0 + steps_per : fr.ns;
    v4f acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
    for (int64_t s = s0 + wave; s < s1; s += 4) {
        v4s a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = *reinterpret_cast<const v4s *>(A + (((4 * ot + i) * fr.ns + s) * 64 + lane) * 4);
            b[i] = *reinterpret_cast<const v4s *>(B + (((4 * it + i) * fr.ns + s) * 64 + lane) * 4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) red[wave][(16 * i + 4 * (lane >> 4) + q) * 64 + 16 * j + (lane & 15)] = acc[i][j][q];
    __syncthreads();
    float *o = part + blockIdx.y * kNParam + off;
    for (int e = threadIdx.x; e < 64 * 64; e += 256)
        o[(64 * ot + e / 64) * ldw + 64 * it + e % 64] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

struct AdamArgs {
    float *p, *m, *v;
    unsigned short *pk;
    float lr, b1, b2, eps, c1, c2;
};

constexpr int kFinishW = (int)((kNParam + 255) / 256), kFinishB = kBias / 16;

// Sums the partial gradients (blocks below kFinishW: 256 weights each; the
// next kFinishB: 16 bias columns each) and the loss (last block); the sums
// go to g (may be NULL) or, with ADAM, into the parameters.
template <bool ADAM>
__global__ void __launch_bounds__(256) k_mlp_finish(int nchunk, const float *__restrict__ part, int nrow,
                                                    const float *__restrict__ bpart, const double *__restrict__ lpart,
                                                    const double *__restrict__ mpart, double *__restrict__ loss,
                                                    float *__restrict__ g, AdamArgs ad) {
    __shared__ double red[256];
    auto put = [&](int64_t i, float gi) {
        if constexpr (ADAM) {
            const float mi = ad.b1 * ad.m[i] + (1.0f - ad.b1) * gi;
            const float vi = ad.b2 * ad.v[i] + (1.0f - ad.b2) * gi * gi;
            ad.m[i] = mi;
            ad.v[i] = vi;
            const float pi = ad.p[i] - ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
            ad.p[i] = pi;
            pack_weight(i, pi, ad.pk);
        } else if (g) {
            g[i] = gi;
        }
    };
    const int t = threadIdx.x;
    if (blockIdx.x < kFinishW) {
        const int64_t i = blockIdx.x * (int64_t)256 + t;
        const bool bias = (i >= kOffB1 && i < kOffW2) || (i >= kOffB2 && i < kOffW3) || i >= kOffB3;
        if (i >= kNParam || bias) return;
        float s = 0.0f;
        for (int c = 0; c < nchunk; ++c) s += part[c * kNParam + i];
        put(i, s);
    } else if (blockIdx.x < kFinishW + kFinishB) {
        const int c = 16 * (blockIdx.x - kFinishW) + t % 16;
        float s = 0.0f;
        for (int b = t / 16; b < nrow; b += 16) s += bpart[(int64_t)b * kBias + c];
        float *rf = reinterpret_cast<float *>(red);
        rf[t] = s;
        __syncthreads();
        if (t >= 16) return;
        s = 0.0f;
        for (int k = 0; k < 16; ++k) s += rf[16 * k + t];
        put(c < kHid ? kOffB1 + c : c < 2 * kHid ? kOffB2 + c - kHid : kOffB3 + c - 2 * kHid, s);
    } else {
        auto total = [&](const double *x, int n) {
            double s = 0.0;
            for (int i = t; i < n; i += 256) s += x[i];
            red[t] = s;
            __syncthreads();
            for (int st = 128; st > 0; st >>= 1) {
                if (t < st) red[t] += red[t + st];
                __syncthreads();
            }
            s = red[0];
            __syncthreads();
            return s;
        };
        const double ls = total(lpart, nrow), ms = total(mpart, kMaskBlocks);
        if (t == 0) loss[0] = ls / (double)(float)ms;
    }
}

}  // namespace mess

// ------------------------------------------------------------ the model

struct mess_mlp {
    float *p = nullptr, *m = nullptr, *v = nullptr;
    unsigned short *pk = nullptr;  // weights as BF16 fragments
    int t = 0;
    int64_t cap = 0;               // rows the workspace holds
    unsigned short *frags = nullptr;
    float *wpart = nullptr, *bpart = nullptr;
    double *mpart = nullptr, *lpart = nullptr, *loss = nullptr;
};

namespace mess {

constexpr int kFragCols = kIn + 4 * kHid + kOut;
constexpr int kMaxChunks = 32;

// Workspace of a gradient over n rows, kept until more rows are asked for.
static int ensure_ws(mess_mlp *L, int64_t n) {
    if (n <= L->cap) return MESS_OK;
    MESS_HIP(hipDeviceSynchronize());
    hipFree(L->frags);
    L->frags = nullptr;
    L->cap = 0;
    const int64_t rows = (n + 31) / 32 * 32;
    const hipError_t e = hipMalloc(&L->frags, sizeof(unsigned short) * kFragCols * rows);
    if (e != hipSuccess) {
        L->frags = nullptr;
        set_error("perceptron workspace for %lld rows: %s", (long long)n, hipGetErrorString(e));
        return MESS_E_NOMEM;
    }
    L->cap = rows;
    return MESS_OK;
}

// Launches the row kernel: 16 rows a block while that leaves at most one
// block a CU (4096 rows: the chip is filled and the chain of layers is as
// short as it gets), 32 above (half the weight traffic from the L2).
template <bool GRAD>
static int mlp_rows(mess_mlp *L, int64_t n, const float *X, float *Y, const float *T, const float *M, RowFrags fr,
                    int *nrow, hipStream_t s) {
    const bool small = n <= 256 * 16;
    const int64_t tiles = small ? (n + 15) / 16 : (n + 31) / 32;
    const unsigned g = (unsigned)std::min<int64_t>(tiles, kRowBlocksMax);
    if (small)
        hipLaunchKernelGGL((k_mlp_rows<1, GRAD>), dim3(g), dim3(256), 0, s, n, X, L->p, L->pk, Y, T, M, L->mpart, fr,
                           L->lpart, L->bpart);
    else
        hipLaunchKernelGGL((k_mlp_rows<2, GRAD>), dim3(g), dim3(256), 0, s, n, X, L->p, L->pk, Y, T, M, L->mpart, fr,
                           L->lpart, L->bpart);
    MESS_LAUNCH_CHECK();
    if (nrow) *nrow = (int)g;
    return MESS_OK;
}

// Forward over n rows of X (FP32): Y (FP32).
static int mlp_forward(mess_mlp *L, int64_t n, const float *X, float *Y, hipStream_t s) {
    return mlp_rows<false>(L, n, X, Y, nullptr, nullptr, RowFrags{}, nullptr, s);
}

// Loss (into L->loss) and gradient of the masked MSE over n rows: into g
// (may be NULL), or into the parameters by one Adam step (ad not NULL).
static int mlp_grad(mess_mlp *L, int64_t n, const float *X, const float *T, const float *M, float *g,
                    const AdamArgs *ad, hipStream_t s) {
    MESS_TRY(ensure_ws(L, n));
    // rows in steps of 16, to a whole block of the row kernel
    const int64_t ns = n <= 256 * 16 ? (n + 15) / 16 : (n + 31) / 32 * 2;
    unsigned short *f = L->frags;
    auto take = [&](int cols) {
        unsigned short *q = f;
        f += ns * 16 * cols;
        return q;
    };
    RowFrags fr;
    fr.X = take(kIn);
    fr.H1 = take(kHid);
    fr.H2 = take(kHid);
    fr.dY = take(kOut);
    fr.dZ2 = take(kHid);
    fr.dZ1 = take(kHid);
    fr.ns = ns;
    int nrow = 0;
    hipLaunchKernelGGL(k_mask_sum, dim3(kMaskBlocks), dim3(256), 0, s, n * kOut, M, L->mpart);
    MESS_TRY(mlp_rows<true>(L, n, X, nullptr, T, M, fr, &nrow, s));
    // chunks of at least 32 steps (512 rows)
    int64_t nchunk = std::max<int64_t>(1, std::min<int64_t>(ns / 32, kMaxChunks));
    const int64_t per = (ns + nchunk - 1) / nchunk;
    nchunk = (ns + per - 1) / per;
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(28, (unsigned)nchunk), dim3(256), 0, s, fr, per, L->wpart);
    const dim3 fg(kFinishW + kFinishB + 1);
    if (ad)
        hipLaunchKernelGGL(k_mlp_finish<true>, fg, dim3(256), 0, s, (int)nchunk, L->wpart, nrow, L->bpart, L->lpart,
                           L->mpart, L->loss, nullptr, *ad);
    else
        hipLaunchKernelGGL(k_mlp_finish<false>, fg, dim3(256), 0, s, (int)nchunk, L->wpart, nrow, L->bpart, L->lpart,
                           L->mpart, L->loss, g, AdamArgs{});
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

static void free_mlp(mess_mlp *L) {
    if (!L) return;
    for (void *q : {(void *)L->p, (void *)L->m, (void *)L->v, (void *)L->pk, (void *)L->frags, (void *)L->wpart,
                    (void *)L->bpart, (void *)L->mpart, (void *)L->lpart, (void *)L->loss})
        hipFree(q);
    delete L;
}

static int check_rows(int64_t n, const char *who) {
    if (n <= 0 || n > (int64_t)1 << 21) {
        set_error("%s: row count %lld out of range (1 .. 2^21)", who, (long long)n);
        return MESS_E_ARG;
    }
    return MESS_OK;
}

int guess_rows(mess_basis *B, int64_t *n) {
    GuessTables *T = nullptr;
    MESS_TRY(get_tables(B, &T));
    *n = T->nrows;
    return MESS_OK;
}

int guess_assemble_async(mess_basis *B, const float *Y, double *D, hipStream_t s) {
    GuessTables *T = nullptr;
    MESS_TRY(get_tables(B, &T));
    int zero_async(double *p, int64_t n, hipStream_t s);
    MESS_TRY(zero_async(D, B->packed, s));
    const int64_t nt = T->nrows * kBlk * kBlk;
    hipLaunchKernelGGL(k_guess_assemble, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, T->nrows, T->d_rows, Y,
                       D);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

int guess_features_async(mess_basis *B, float *X, hipStream_t s) {
    GuessTables *T = nullptr;
    MESS_TRY(get_tables(B, &T));
    MESS_HIP(hipMemcpyAsync(X, T->feat.data(), sizeof(float) * T->feat.size(), hipMemcpyHostToDevice, s));
    MESS_HIP(hipStreamSynchronize(s));  // the host array is pageable
    return MESS_OK;
}

int mlp_forward_ext(mess_mlp *L, int64_t n, const float *X, float *Y, hipStream_t s) {
    return mlp_forward(L, n, X, Y, s);
}

}  // namespace mess

using namespace mess;

extern "C" {

int mess_mlp_create(const float *params, mess_mlp **out) {
    if (!params || !out) {
        set_error("mess_mlp_create: NULL parameters or output");
        return MESS_E_ARG;
    }
    *out = nullptr;
    auto *L = new mess_mlp();
    hipError_t e = hipSuccess;
    auto al = [&](void **q, size_t bytes) {
        if (e == hipSuccess) e = hipMalloc(q, bytes);
    };
    al((void **)&L->p, 4 * kNParam);
    al((void **)&L->m, 4 * kNParam);
    al((void **)&L->v, 4 * kNParam);
    al((void **)&L->pk, 2 * kNPacked);
    al((void **)&L->wpart, 4 * kMaxChunks * kNParam);
    al((void **)&L->bpart, 4 * kRowBlocksMax * kBias);
    al((void **)&L->mpart, 8 * kMaskBlocks);
    al((void **)&L->lpart, 8 * kRowBlocksMax);
    al((void **)&L->loss, 8);
    if (e == hipSuccess) e = hipMemcpy(L->p, params, 4 * kNParam, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemset(L->m, 0, 4 * kNParam);
    if (e == hipSuccess) e = hipMemset(L->v, 0, 4 * kNParam);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_pack, dim3((unsigned)((kNParam + 255) / 256)), dim3(256), 0, nullptr, L->p, L->pk);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        set_error("mess_mlp_create: %s", hipGetErrorString(e));
        free_mlp(L);
        return MESS_E_NOMEM;
    }
    *out = L;
    return MESS_OK;
}

void mess_mlp_destroy(mess_mlp *mlp) { free_mlp(mlp); }

int mess_mlp_params(const mess_mlp *mlp, float *params) {
    if (!mlp || !params) {
        set_error("mess_mlp_params: NULL argument");
        return MESS_E_ARG;
    }
    MESS_HIP(hipDeviceSynchronize());
    MESS_HIP(hipMemcpy(params, mlp->p, 4 * kNParam, hipMemcpyDeviceToHost));
    return MESS_OK;
}

int mess_mlp_forward(mess_mlp *mlp, int64_t n, const float *X, float *Y, mess_stream stream) {
    if (!mlp || !X || !Y) {
        set_error("mess_mlp_forward: NULL argument");
        return MESS_E_ARG;
    }
    MESS_TRY(check_rows(n, "mess_mlp_forward"));
    return mlp_forward(mlp, n, X, Y, static_cast<hipStream_t>(stream));
}

int mess_mlp_grad(mess_mlp *mlp, int64_t n, const float *X, const float *T, const float *M, float *grad,
                  double *loss, mess_stream stream) {
    if (!mlp || !X || !T || !M) {
        set_error("mess_mlp_grad: NULL argument");
        return MESS_E_ARG;
    }
    MESS_TRY(check_rows(n, "mess_mlp_grad"));
    hipStream_t s = static_cast<hipStream_t>(stream);
    MESS_TRY(mlp_grad(mlp, n, X, T, M, grad, nullptr, s));
    if (loss) {
        MESS_HIP(hipMemcpyAsync(loss, mlp->loss, 8, hipMemcpyDeviceToHost, s));
        MESS_HIP(hipStreamSynchronize(s));
    }
    return MESS_OK;
}

int mess_mlp_train_step(mess_mlp *mlp, int64_t n, const float *X, const float *T, const float *M, float lr,
                        double *loss, mess_stream stream) {
    if (!mlp || !X || !T || !M || !(lr > 0.0f)) {
        set_error("mess_mlp_train_step: NULL argument or learning rate <= 0");
        return MESS_E_ARG;
    }
    MESS_TRY(check_rows(n, "mess_mlp_train_step"));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const float b1 = 0.9f, b2 = 0.999f, t = (float)(mlp->t + 1);
    const AdamArgs ad{mlp->p, mlp->m, mlp->v, mlp->pk, lr, b1, b2, 1e-8f, 1.0f - std::pow(b1, t), 1.0f - std::pow(b2, t)};
    MESS_TRY(mlp_grad(mlp, n, X, T, M, nullptr, &ad, s));
    mlp->t += 1;
    if (loss) {
        MESS_HIP(hipMemcpyAsync(loss, mlp->loss, 8, hipMemcpyDeviceToHost, s));
        MESS_HIP(hipStreamSynchronize(s));
    }
    return MESS_OK;
}

int mess_guess_rows(const mess_basis *basis, int64_t *n_rows) {
    if (!basis || !n_rows) {
        set_error("mess_guess_rows: NULL argument");
        return MESS_E_ARG;
    }
    return guess_rows(const_cast<mess_basis *>(basis), n_rows);
}

int mess_guess_features(const mess_basis *basis, float *X, mess_stream stream) {
    if (!basis || !X) {
        set_error("mess_guess_features: NULL argument");
        return MESS_E_ARG;
    }
    return guess_features_async(const_cast<mess_basis *>(basis), X, static_cast<hipStream_t>(stream));
}

int mess_guess_targets(const mess_basis *basis, const double *D, float *T, float *M, mess_stream stream) {
    if (!basis || !D || (!T && !M)) {
        set_error("mess_guess_targets: NULL argument");
        return MESS_E_ARG;
    }
    GuessTables *G = nullptr;
    MESS_TRY(get_tables(const_cast<mess_basis *>(basis), &G));
    const int64_t nt = G->nrows * kOut;
    hipLaunchKernelGGL(k_guess_targets, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), G->nrows, G->d_rows, D, T, M);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

int mess_guess_assemble(const mess_basis *basis, const float *Y, double *D, mess_stream stream) {
    if (!basis || !Y || !D) {
        set_error("mess_guess_assemble: NULL argument");
        return MESS_E_ARG;
    }
    return guess_assemble_async(const_cast<mess_basis *>(basis), Y, D, static_cast<hipStream_t>(stream));
}

}  // extern "C"
