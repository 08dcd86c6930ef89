// Per-angular-class launchers.  Each of the 21 unique classes (pair class
// of the bra >= pair class of the ket) is compiled in its own object file
// (eri_class.hip built once per class) and reached through ClassOps.
#pragma once

#include "mess_internal.hpp"

namespace mess {

struct ClassLaunch {
    const PairInfo *pairs;
    const PrimPair *pp;
    const PrimPairF *ppf;
    const double *tab, *etab;
    const float *tabf, *etabf;
    const double *tabt;  // per-order polynomial table
    int bra_off, ket_off, nbra, same_class;  // nbra: rows of the work list
    const int64_t *rowstart;
    const int2 *rowmap;  // per row: {bra index, first ket index}
    int64_t total;
    int64_t prims = 0;   // primitive quartets of the list
    int N;
    hipStream_t stream;
    // stored-block digestion by bra-row segments (NULL: one lane per quartet)
    const int4 *segs = nullptr;  // {first row, first quartet, end quartet, end row}
    int nseg = 0;
    int nmax = 0;                // largest molecule dimension (LDS rows)
    // grouped stored digestion (NULL: by segments)
    const int4 *groups = nullptr, *tiles = nullptr;
    const int *grows = nullptr;
    int ngroups = 0;
    // dense mode: workspace for blocks that share a quartet (NULL: none do)
    double *shares = nullptr;
};

// Direct J/K of class (cb, ck) through its cooperative tables (primitive-
// lane, wave or table-driven kernel; coop.hip).
int coop_jk(int cb, int ck, const ClassLaunch &L, const double *D, double *Gj, double *Gk, int prec);

// Doubles of ClassLaunch::shares that the dense mode of class (cb, ck) takes
// for a list of total quartets (0: its blocks do not share them).
int64_t coop_share_doubles(int cb, int ck, int64_t total, int prec);

// Stored-block layout (coop.hip): true when class (cb, ck) keeps its blocks
// quartet-major for J/K streaming (element e of quartet t at t NOUT + e)
// instead of structure-of-arrays (e total + t); to_aos converts a region.
bool stored_aos_class(int cb, int ck);
int to_aos(const void *soa, void *aos, int nout, int64_t total, int prec, hipStream_t s);

// Lanes that share a shell quartet in the kernels with one lane per quartet
// (FP64).  A lane's loop over the quartet's primitive quartets (up to 1296
// of 6 x 6 x 6 x 6 primitives) is a serial chain, so a list that leaves the
// chip's SIMDs with less than about two waves each is as slow as its longest
// quartet: then P lanes take every P-th primitive quartet and sum the
// contracted intermediates (log2 P exchanges each, a few hundred cycles
// against the chain).  The sum's order depends on the list's size alone.
// FP32 keeps one lane: its sums round where they are taken.
constexpr int kSplits[3] = {64, 16, 4};

// Lanes per quartet (1 or one of kSplits) for a list of total quartets with
// prims primitive quartets in all: as many as 2^20 lanes allow (16 waves a
// SIMD: enough of them that the longest does not end alone), 2^21 for the
// classes without the segment form, with at least half a primitive quartet a
// lane.  Measured on water clusters (n waters; us, one lane -> P): (ss|ss) of
// n = 3 340 -> 52 (16 lanes), (dp|ds) 3214 -> 75 (64), n = 7 3051 -> 217 (16
// lanes; 280 with 64), n = 20 3739 -> 1985 (4 lanes, 0.9e6 lanes; 2511 with
// 16), (pp|ps) of n = 20 1051 -> 543 (4 lanes), but (dd|ss) of n = 20, which
// would take 1.4e6 lanes, 1429 by segments and 2723 with 4 lanes: there the
// global atomics that the segments save outweigh the chain.
inline int split_lanes(int cb, int ck, int64_t total, int64_t prims) {
    const bool segments = !(cb == 4 && ck == 3) && !(cb == 3 && ck == 2);
    const int64_t lanes = segments ? int64_t(1) << 20 : int64_t(1) << 21;
    for (int P : kSplits)
        if (total * P <= lanes && prims >= total * P / 2) return P;
    return 1;
}

template <int CB, int CK>
struct ClassOps {
    // Q[off + i] for the n pairs of class CB (requires CB == CK).
    static int schwarz(const ClassLaunch &L, int off, int n, double *Q);
    // Dense N^4 FP64 store of every quartet in the list.
    static int dense(const ClassLaunch &L, double *eri, int prec);
    // Gj, Gk half-matrices (either may be NULL) from density D.
    static int jk(const ClassLaunch &L, const double *D, double *Gj, double *Gk, int prec);
    // Unique blocks of every quartet into base (FP64 or FP32 by prec),
    // element k of quartet t at base[k * total + t].
    static int store(const ClassLaunch &L, void *base, int prec);
    // Gj, Gk from the stored blocks.
    static int jk_stored(const ClassLaunch &L, const void *base, int prec, const double *D, double *Gj, double *Gk);
};

// Calls f(integral_constant<CB>, integral_constant<CK>) for a runtime
// (cb, ck) with cb >= ck.
template <typename F>
int dispatch_class(int cb, int ck, F &&f) {
    using std::integral_constant;
#define MESS_CASE(B, K) \
    case (B) * 6 + (K): return f(integral_constant<int, B>{}, integral_constant<int, K>{});
    switch (cb * 6 + ck) {
        MESS_CASE(0, 0)
        MESS_CASE(1, 0) MESS_CASE(1, 1)
        MESS_CASE(2, 0) MESS_CASE(2, 1) MESS_CASE(2, 2)
        MESS_CASE(3, 0) MESS_CASE(3, 1) MESS_CASE(3, 2) MESS_CASE(3, 3)
        MESS_CASE(4, 0) MESS_CASE(4, 1) MESS_CASE(4, 2) MESS_CASE(4, 3) MESS_CASE(4, 4)
        MESS_CASE(5, 0) MESS_CASE(5, 1) MESS_CASE(5, 2) MESS_CASE(5, 3) MESS_CASE(5, 4) MESS_CASE(5, 5)
        default: break;
    }
#undef MESS_CASE
    set_error("internal: bad class (%d,%d)", cb, ck);
    return MESS_E_ARG;
}


}  // namespace mess
