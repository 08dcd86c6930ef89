// Builds of small s and p molecules (MESS_FP64): the lane kernels of the five
// classes below (pp|pp) in one launch, P lanes a quartet (kSplits).
//
// Such a build is a few thousand quartets a class; each class kernel takes
// 12-24 us, most of it one wave's chain (find the row, read the pairs, a few
// primitive quartets a lane, the exchanges, the digestion) with the chip
// partly idle, and they ran one after another (six of them, 106 us, for 30
// functions).  A block takes its class from its number, the costliest first.
// (pp|pp) stays a launch of its own: its 81 integrals would leave the other
// classes half the waves.  Bound by the chain up to a round of waves, then by
// issue.  J/K one launch a class -> this, us: 10 functions 73 -> 28, 30
// functions 109 -> 68, 50 functions 371 -> 248; their tensors 42 -> 25 (10), 66
// -> 35 (30), 134 -> 66 (40).
#include <vector>

#include "eri_kernels.hpp"

namespace mess {

struct ShortList {
    const int64_t *rowstart;
    const int2 *rowmap;
    int bra_off, ket_off, nrow, same, block0;
};
constexpr int kShort = 5;
constexpr int kShortCb[kShort] = {2, 2, 1, 1, 0}, kShortCk[kShort] = {1, 0, 1, 0, 0};
struct ShortArgs {
    ShortList c[kShort];
};

template <class Dm, int P, bool DENSE>
__device__ __forceinline__ void short_quartet(const ShortList &l, const PairInfo *__restrict__ pairs,
                                              const PrimPair *__restrict__ pp, const BoysTabs &bt,
                                              const double *__restrict__ D, int64_t N, double *__restrict__ out0,
                                              double *__restrict__ out1) {
    const int64_t t = ((int64_t)(blockIdx.x - l.block0) * 128 + threadIdx.x) / P;
    if (t >= l.rowstart[l.nrow]) return;
    const int sub = threadIdx.x % P;
    const int2 ij = quartet_pairs(l.rowstart, l.rowmap, l.nrow, t);
    const PairInfo bra = pairs[l.bra_off + ij.x], ket = pairs[l.ket_off + ij.y];
    double out[Dm::NOUT];
    eri_quartet<Dm, double, P>(bra, ket, pp, bt, out, sub);
    if constexpr (DENSE)
        dense_block<Dm, double, P>(out, bra, ket, sub, N, out0);
    else if (sub == 0)
        digest_jk<Dm, double>(out, quartet_factor(bra, ket, l.same && ij.x == ij.y), bra.bfa, bra.bfb, ket.bfa, ket.bfb,
                              D + bra.moff, bra.mN, out0 ? out0 + bra.moff : nullptr, out1 ? out1 + bra.moff : nullptr);
}

template <int P, bool DENSE>
__global__ void __launch_bounds__(128, 3) k_short(ShortArgs A, const PairInfo *__restrict__ pairs,
                                                  const PrimPair *__restrict__ pp, BoysTabs bt,
                                                  const double *__restrict__ D, int64_t N, double *__restrict__ out0,
                                                  double *__restrict__ out1) {
    static_for<0, kShort>([&](auto I) {
        constexpr int c = decltype(I)::value;
        constexpr int next = c + 1 < kShort ? c + 1 : c;
        const bool mine = (int)blockIdx.x >= A.c[c].block0 && (next == c || (int)blockIdx.x < A.c[next].block0);
        if (mine)
            short_quartet<ClassOf<kShortCb[c], kShortCk[c]>, P, DENSE>(A.c[c], pairs, pp, bt, D, N, out0, out1);
    });
}

// Launches the lists of act that it can take together and removes them.  It
// takes them for molecules of s and p shells, with no form asked for, whose
// lists all fit P = 64 or P = 16 lanes a quartet by the rule of the class
// kernels (at most 2^20 lanes, half a primitive quartet a lane): 64 while the
// whole launch is at most about one round of three waves a SIMD (2^18 lanes;
// 30 functions, 9.3e5 lanes of 64: 81 us, of 16: 68), and up to 2^21 lanes in
// all (60 functions, 3.7e6: 394 us in one launch, 386 in five).
int short_launch(const mess_basis *B, std::vector<const ClassList *> &act, bool dense, const double *D, double *out0,
                 double *out1, hipStream_t s) {
    ShortArgs A{};
    const ClassList *pick[kShort] = {};
    int P = 64, found = 0;
    int64_t quartets = 0;
    for (const ClassList *cl : act) {
        if (cl->cb > 2) return MESS_OK;
        for (int c = 0; c < kShort; ++c)
            if (cl->cb == kShortCb[c] && cl->ck == kShortCk[c]) {
                if (!form_is_default(cl->cb, cl->ck)) return MESS_OK;
                while (P >= 16 && (cl->total * P > (int64_t(1) << 20) || cl->prim_quartets < cl->total * P / 2)) P /= 4;
                pick[c] = cl;
                ++found;
                quartets += cl->total;
            }
    }
    if (P == 64 && quartets * P > (int64_t(1) << 18)) P = 16;
    if (found < 2 || P < 16 || quartets * P > (int64_t(1) << 21)) return MESS_OK;
    int64_t blocks = 0;
    for (int c = 0; c < kShort; ++c) {
        ShortList &l = A.c[c];
        l.block0 = (int)blocks;
        if (!pick[c]) continue;
        l.rowstart = pick[c]->d_rowstart;
        l.rowmap = pick[c]->d_rowmap;
        l.bra_off = B->pair_class_off[kShortCb[c]];
        l.ket_off = B->pair_class_off[kShortCk[c]];
        l.nrow = pick[c]->nrow;
        l.same = kShortCb[c] == kShortCk[c];
        blocks += (pick[c]->total * P + 127) / 128;
    }
    const BoysTabs bt{B->d_boys, B->d_boys_exp, B->d_boys_f, B->d_boys_exp_f, B->d_boys_t};
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(128), 0, s, A, B->d_pairs, B->d_pp, bt, D, (int64_t)B->nbf,
                           out0, out1);
    };
    if (P == 64) dense ? go(k_short<64, true>) : go(k_short<64, false>);
    else dense ? go(k_short<16, true>) : go(k_short<16, false>);
    MESS_LAUNCH_CHECK();
    std::vector<const ClassList *> rest;
    for (const ClassList *cl : act)
        if (cl->ck == 2) rest.push_back(cl);
    act.swap(rest);
    return MESS_OK;
}

}  // namespace mess
