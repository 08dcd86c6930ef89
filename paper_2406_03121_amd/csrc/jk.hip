// mess_eri and mess_jk: class-by-class launches over the unique
// shell-quartet work lists, then the symmetrisation J = Gj + Gj^T,
// K = Gk + Gk^T of the half-matrices the digestion accumulates.
#include "class_ops.hpp"
#include "mess_internal.hpp"

#include <algorithm>
#include <mutex>
#include <vector>

namespace mess {

int get_work_lists(mess_basis *B, double tau, hipStream_t s, WorkLists **out);
int fill_class_launch(const mess_basis *B, const ClassList &cl, hipStream_t s, ClassLaunch &L);
int jk_stored(mess_basis *B, const double *D, double *Gj, double *Gk, int prec, double tau, hipStream_t s);
int jk_det(mess_basis *B, const double *D, double *Gj, double *Gk, int prec, double tau, hipStream_t s);
int eri_blocks(mess_basis *B, int prec, double tau, void *out, size_t out_bytes, hipStream_t s);

__global__ void k_fill_zero(double *__restrict__ p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// J = Gj + Gj^T, K = Gk + Gk^T (either may be NULL) for every diagonal block
// of a packed block-diagonal matrix (block m: n_m x n_m at offset moff[m]);
// blockIdx.z strides over blocks.
__global__ void k_symmetrise(const double *__restrict__ Gj, const double *__restrict__ Gk, int nmol,
                             const int64_t *__restrict__ moff, const int *__restrict__ nb, double *__restrict__ J,
                             double *__restrict__ K) {
    const int i = blockIdx.y * blockDim.y + threadIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    for (int m = blockIdx.z; m < nmol; m += gridDim.z) {
        const int n = nb[m];
        if (i < n && j < n) {
            const int64_t o = moff[m], ij = o + (int64_t)i * n + j, ji = o + (int64_t)j * n + i;
            if (J) J[ij] = Gj[ij] + Gj[ji];
            if (K) K[ij] = Gk[ij] + Gk[ji];
        }
    }
}

int zero_async(double *p, int64_t n, hipStream_t s) {
    if (n <= 0) return MESS_OK;
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)g), dim3(256), 0, s, p, n);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

int symmetrise_async(const mess_basis *B, const double *Gj, const double *Gk, double *J, double *K, hipStream_t s) {
    const int N = B->nbf_max;
    dim3 blk(32, 8), grd((N + 31) / 32, (N + 7) / 8, (unsigned)std::min(B->n_mol, 65535));
    hipLaunchKernelGGL(k_symmetrise, grd, blk, 0, s, Gj, Gk, B->n_mol, B->d_mol_moff, B->d_mol_nbf, J, K);
    MESS_LAUNCH_CHECK();
    return MESS_OK;
}

// Clears the half matrices (either may be NULL), in one launch where they are adjacent.
int zero_halves(const mess_basis *B, double *Gj, double *Gk, hipStream_t s) {
    if (Gj && Gk == Gj + B->packed) return zero_async(Gj, 2 * B->packed, s);
    if (Gj) MESS_TRY(zero_async(Gj, B->packed, s));
    if (Gk) MESS_TRY(zero_async(Gk, B->packed, s));
    return MESS_OK;
}

// ------------------------------------------------------- class streams
//
// The classes of a build are independent (they meet in atomics), and most
// leave part of the chip idle: short lists, a long last wave, or a form
// bound by latency.  They run on the caller's stream and kSideStreams
// others between a fork and a join (events on the caller's stream), the
// costliest first, each on the stream with the least work so far.  Sets of
// side streams are kept in a pool, at most kMaxSets a device, each used by
// one call at a time while it enqueues.  A call takes the set that its
// stream's call before had (whose work it queues behind in any case), or a
// new one, so that callers on different streams do not queue behind one
// another; beyond kMaxSets callers it takes the set that was given back
// longest ago.  With none left, and under a caller's capture, the classes run
// one after another on the caller's stream.  The batch's own captures are
// lent a set until they end.

constexpr int kSideStreams = 3, kMaxSets = 8, kMaxDevices = 64;

struct SideSet {
    int device = -1;
    hipStream_t user = nullptr;  // stream of the last call
    hipStream_t s[kSideStreams] = {};
    hipEvent_t fork = nullptr, done[kSideStreams] = {};
};

static std::mutex g_side_mutex;
static std::vector<SideSet *> g_side_free;
static int g_side_made[kMaxDevices] = {};  // sets of each device

static thread_local SideSet *t_capture_set = nullptr;  // lent to this thread's captures

// A set for a call on s (for_capture: to be lent to a capture, which any free
// one serves); a new one only if create.
static SideSet *side_acquire(hipStream_t s, bool create, bool for_capture = false) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_side_mutex);
    int pick = -1;
    for (int i = 0; i < (int)g_side_free.size(); ++i) {
        if (g_side_free[i]->device != dev) continue;
        const bool own = g_side_free[i]->user == s;
        if (pick < 0 || own) pick = i;
        if (own) break;
    }
    const bool more = create && g_side_made[dev] < kMaxSets;
    if (pick >= 0 && (for_capture || !more || g_side_free[pick]->user == s)) {
        SideSet *set = g_side_free[pick];
        g_side_free.erase(g_side_free.begin() + pick);
        if (!for_capture) set->user = s;
        return set;
    }
    if (!more) return nullptr;
    auto *set = new SideSet();
    set->device = dev;
    set->user = s;
    bool ok = hipEventCreateWithFlags(&set->fork, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; i < kSideStreams; ++i)
        ok = ok && hipStreamCreateWithFlags(&set->s[i], hipStreamNonBlocking) == hipSuccess &&
             hipEventCreateWithFlags(&set->done[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        for (int i = 0; i < kSideStreams; ++i) {
            if (set->s[i]) (void)hipStreamDestroy(set->s[i]);
            if (set->done[i]) (void)hipEventDestroy(set->done[i]);
        }
        if (set->fork) (void)hipEventDestroy(set->fork);
        delete set;
        return nullptr;
    }
    ++g_side_made[dev];
    return set;
}

static void side_release(SideSet *set) {
    std::lock_guard<std::mutex> lk(g_side_mutex);
    g_side_free.push_back(set);
}

ForkCapture::ForkCapture() {
    if (!t_capture_set) t_capture_set = side_acquire(nullptr, true, true);
}

ForkCapture::~ForkCapture() {
    if (t_capture_set) side_release(t_capture_set);
    t_capture_set = nullptr;
}

int run_forked(hipStream_t s, const std::vector<double> &cost, const std::function<int(int, hipStream_t)> &work,
               bool create) {
    // few classes with little work each (s and p shells of a small molecule: up
    // to six of 15-25 us) end sooner one after another than the fork and the
    // join take (30-function J/K 109 and 151 us, its tensor 75 and 151); with
    // all 21 classes the fork pays from the smallest molecule on (one water
    // 544 -> 226 us, 3 waters 1190 -> 560, 13 waters 11.5 -> 9.0 ms and 17.2
    // -> 8.0 in FP32, 20 waters 31.8 -> 27.7), as it does for few but long ones
    const int n = (int)cost.size();
    double all = 0.0;
    for (double c : cost) all += c;
    SideSet *set = nullptr;
    bool lent = false;
    if ((n >= 8 || (n > 1 && all >= 1e9)) && !prof_on()) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
            (void)hipGetLastError();
        } else {
            lent = cap != hipStreamCaptureStatusNone;
            set = lent ? t_capture_set : side_acquire(s, create);
        }
    }
    if (!set) {
        for (int i = 0; i < n; ++i) MESS_TRY(work(i, s));
        return MESS_OK;
    }
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    const int ns = std::min(n, kSideStreams + 1);
    double load[kSideStreams + 1] = {};
    int rc = MESS_OK;
    hipError_t e = hipEventRecord(set->fork, s);
    for (int i = 0; i + 1 < ns && e == hipSuccess; ++i) e = hipStreamWaitEvent(set->s[i], set->fork, 0);
    if (e == hipSuccess)
        for (int i = 0; i < n && rc == MESS_OK; ++i) {
            int k = 0;
            for (int j = 1; j < ns; ++j)
                if (load[j] < load[k]) k = j;
            load[k] += cost[order[i]];
            rc = work(order[i], k == 0 ? s : set->s[k - 1]);
        }
    // join, also after an error: nothing of this call may outlast it
    for (int i = 0; i + 1 < ns; ++i) {
        hipError_t d = hipEventRecord(set->done[i], set->s[i]);
        if (d == hipSuccess) d = hipStreamWaitEvent(s, set->done[i], 0);
        if (d != hipSuccess && !lent) (void)hipStreamSynchronize(set->s[i]);
        if (e == hipSuccess) e = d;
    }
    if (!lent) side_release(set);
    if (rc == MESS_OK && e != hipSuccess) {
        set_error("class streams: %s", hipGetErrorString(e));
        rc = MESS_E_DEVICE;
    }
    return rc;
}

// The classes with quartets, and their operation counts.
static std::vector<const ClassList *> active_classes(const WorkLists *W) {
    std::vector<const ClassList *> act;
    for (const ClassList &cl : W->classes)
        if (cl.total > 0) act.push_back(&cl);
    return act;
}

static std::vector<double> class_costs(const std::vector<const ClassList *> &act) {
    std::vector<double> cost;
    for (const ClassList *cl : act) {
        double fp = 0.0, fq = 0.0;
        class_flops(cl->cb, cl->ck, &fp, &fq);
        cost.push_back(fp * (double)cl->prim_quartets + fq * (double)cl->total);
    }
    return cost;
}

int short_launch(const mess_basis *B, std::vector<const ClassList *> &act, bool dense, const double *D, double *out0,
                 double *out1, hipStream_t s);  // short.hip

int coop_prepare(int cb, int ck, int prec);                              // coop.hip
int stored_prepare(mess_basis *B, int prec, double tau, hipStream_t s);  // stored.hip

// Everything that a build of this mode, precision and tolerance allocates, so
// that later ones allocate nothing and can be captured: the work lists, step
// tables and stored blocks.
int jk_prepare(mess_basis *B, int mode, int prec, double tau, hipStream_t s) {
    WorkLists *W = nullptr;
    MESS_TRY(get_work_lists(B, tau, s, &W));
    for (const ClassList *cl : active_classes(W)) MESS_TRY(coop_prepare(cl->cb, cl->ck, prec));
    return mode == MESS_JK_DIRECT ? (int)MESS_OK : stored_prepare(B, prec, tau, s);
}

// Gj, Gk (device, packed block-diagonal, may be NULL) <- half-matrices of J and K.
// create: class streams may be made where none are free.
static int direct_half(mess_basis *B, const double *D, double *Gj, double *Gk, int prec, double tau, hipStream_t s,
                       bool create) {
    WorkLists *W = nullptr;
    MESS_TRY(get_work_lists(B, tau, s, &W));
    MESS_TRY(zero_halves(B, Gj, Gk, s));
    const bool prof = prof_on();
    std::vector<const ClassList *> act = active_classes(W);
    if (prec == MESS_FP64 && !prof) MESS_TRY(short_launch(B, act, false, D, Gj, Gk, s));
    const std::vector<double> cost = class_costs(act);
    return run_forked(s, cost, [&](int i, hipStream_t st) {
        const ClassList &cl = *act[i];
        ClassLaunch L;
        fill_class_launch(B, cl, st, L);
        // arithmetic of this class: a build asked for in FP32 runs a class in
        // FP64 where the FP32 form table says its FP64 kernel is faster
        const int cp = (prec == MESS_FP32 && class_form(cl.cb, cl.ck, MESS_FP32) == kFormFp64) ? MESS_FP64 : prec;
        if (prof) {
            double fp = 0.0, fq = 0.0;
            class_flops(cl.cb, cl.ck, &fp, &fq, cp);
            // FP32 launches are recorded under class index + 64
            prof_record(st, class_index(cl.cb, cl.ck) + (cp == MESS_FP32 ? 64 : 0), true, cl.total,
                        cl.prim_quartets,
                        fp * (double)cl.prim_quartets + fq * (double)cl.total);
        }
        MESS_TRY(dispatch_class(cl.cb, cl.ck, [&](auto CB, auto CK) {
            return ClassOps<decltype(CB)::value, decltype(CK)::value>::jk(L, D, Gj, Gk, cp);
        }));
        if (prof) prof_record(st, 0, false, 0, 0, 0.0);
        return (int)MESS_OK;
    }, create);
}

int jk_direct_half(mess_basis *B, const double *D, double *Gj, double *Gk, int prec, double tau,
                   hipStream_t s) {
    return direct_half(B, D, Gj, Gk, prec, tau, s, true);
}

int jk_full(mess_basis *B, const double *D, double *J, double *K, int mode, int prec, double tau,
            hipStream_t s) {
    double *Gj = J ? static_cast<double *>(B->scratch_jk) : nullptr;
    double *Gk = K ? static_cast<double *>(B->scratch_jk) + B->packed : nullptr;
    if (mode == MESS_JK_DIRECT)
        MESS_TRY(jk_direct_half(B, D, Gj, Gk, prec, tau, s));
    else if (mode == MESS_JK_DETERMINISTIC)
        MESS_TRY(jk_det(B, D, Gj, Gk, prec, tau, s));
    else
        MESS_TRY(jk_stored(B, D, Gj, Gk, prec, tau, s));
    return symmetrise_async(B, Gj, Gk, J, K, s);
}

// Workspace of n doubles of the basis for a call on s, which waits for the
// call before, on whatever stream that was; its user records share_done on s
// when it has enqueued its work.  NULL under a caller's capture, whose replays
// nothing could order, and where it cannot be had.
static double *share_workspace(mess_basis *B, int64_t n, hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    bool ok = hipStreamIsCapturing(s, &cap) == hipSuccess;
    if (ok && cap != hipStreamCaptureStatusNone) return nullptr;
    if (ok && !B->share_done) ok = hipEventCreateWithFlags(&B->share_done, hipEventDisableTiming) == hipSuccess;
    if (ok && n > B->share_doubles) {
        if (B->share_ws) (void)hipEventSynchronize(B->share_done);
        hipFree(B->share_ws);
        B->share_ws = nullptr;
        B->share_doubles = 0;
        ok = hipMalloc(&B->share_ws, sizeof(double) * n) == hipSuccess;
        if (ok) B->share_doubles = n;
        else B->share_ws = nullptr;
    } else if (ok) {
        ok = hipStreamWaitEvent(s, B->share_done, 0) == hipSuccess;
    }
    if (!ok) (void)hipGetLastError();
    return ok ? B->share_ws : nullptr;
}

// Fixed device workspace of the allocation-free J/K entry point: the two
// half matrices Gj, Gk of at most kNoAllocMaxPacked doubles each (8 MB in
// all per device, held until the process ends).  Host code never passes the
// array's name to a kernel: it uses the per-device address below.
constexpr int64_t kNoAllocMaxPacked = int64_t(1) << 19;
static __device__ __align__(256) double scratch[2 * kNoAllocMaxPacked];

static std::mutex g_scratch_mutex;
static double *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device (each device holds its own copy of the array).
static int scratch_address(double **out) {
    int dev = 0;
    MESS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("mess_jk_noalloc: device index %d beyond %d", dev, kMaxDevices);
        return MESS_E_DEVICE;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error("mess_jk_noalloc: hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            return MESS_E_DEVICE;
        }
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return MESS_OK;
}

}  // namespace mess

using namespace mess;

extern "C" {

int mess_eri(const mess_basis *basis, int32_t layout, int32_t prec, double schwarz_tol, void *out,
             size_t out_bytes, mess_stream stream) {
    if (!basis || !out) {
        set_error("mess_eri: NULL basis or output");
        return MESS_E_ARG;
    }
    if (prec != MESS_FP64 && prec != MESS_FP32) {
        set_error("mess_eri: unknown precision %d", prec);
        return MESS_E_UNSUPPORTED;
    }
    if (layout != MESS_ERI_DENSE && layout != MESS_ERI_BLOCKS) {
        set_error("mess_eri: unknown layout %d", layout);
        return MESS_E_UNSUPPORTED;
    }
    auto *B = const_cast<mess_basis *>(basis);
    if (layout == MESS_ERI_BLOCKS)
        return eri_blocks(B, prec, schwarz_tol, out, out_bytes, static_cast<hipStream_t>(stream));
    if (B->n_mol != 1) {
        set_error("mess_eri: the dense tensor is built for a single molecule, not a batch of %d", B->n_mol);
        return MESS_E_UNSUPPORTED;
    }
    const int64_t N = B->nbf;
    const size_t need = sizeof(double) * (size_t)(N * N * N * N);
    if (out_bytes < need) {
        set_error("mess_eri: output holds %zu bytes, %zu needed", out_bytes, need);
        return MESS_E_SIZE;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    WorkLists *W = nullptr;
    MESS_TRY(get_work_lists(B, schwarz_tol, s, &W));
    MESS_TRY(zero_async(static_cast<double *>(out), N * N * N * N, s));
    std::vector<const ClassList *> act = active_classes(W);
    if (prec == MESS_FP64 && !prof_on()) MESS_TRY(short_launch(B, act, true, nullptr, static_cast<double *>(out), nullptr, s));
    // shares of quartets, a part of the workspace for each class that has them
    std::vector<int64_t> off(act.size() + 1, 0);
    for (size_t i = 0; i < act.size(); ++i)
        off[i + 1] = off[i] + coop_share_doubles(act[i]->cb, act[i]->ck, act[i]->total, prec);
    double *shares = off.back() ? share_workspace(B, off.back(), s) : nullptr;
    const std::vector<double> cost = class_costs(act);
    const int rc = run_forked(s, cost, [&](int i, hipStream_t st) {
        ClassLaunch L;
        fill_class_launch(B, *act[i], st, L);
        if (shares && off[i + 1] > off[i]) L.shares = shares + off[i];
        return dispatch_class(act[i]->cb, act[i]->ck, [&](auto CB, auto CK) {
            return ClassOps<decltype(CB)::value, decltype(CK)::value>::dense(L, static_cast<double *>(out), prec);
        });
    });
    if (shares && hipEventRecord(B->share_done, s) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(s);
    }
    return rc;
}

int mess_jk(const mess_basis *basis, const double *D, double *J, double *K, int32_t mode, int32_t prec,
            double schwarz_tol, mess_stream stream) {
    if (!basis || !D) {
        set_error("mess_jk: NULL basis or density");
        return MESS_E_ARG;
    }
    if (mode != MESS_JK_DIRECT && mode != MESS_JK_STORED && mode != MESS_JK_DETERMINISTIC) {
        set_error("mess_jk: unknown mode %d", mode);
        return MESS_E_UNSUPPORTED;
    }
    if (prec != MESS_FP64 && prec != MESS_FP32) {
        set_error("mess_jk: unknown precision %d", prec);
        return MESS_E_UNSUPPORTED;
    }
    if (!J && !K) return MESS_OK;
    return jk_full(const_cast<mess_basis *>(basis), D, J, K, mode, prec, schwarz_tol,
                   static_cast<hipStream_t>(stream));
}

int mess_jk_noalloc(const mess_basis *basis, const double *D, double *J, double *K, int32_t prec,
                    double schwarz_tol, mess_stream stream) {
    if (!basis || !D) {
        set_error("mess_jk_noalloc: NULL basis or density");
        return MESS_E_ARG;
    }
    if (prec != MESS_FP64 && prec != MESS_FP32) {
        set_error("mess_jk_noalloc: unknown precision %d", prec);
        return MESS_E_UNSUPPORTED;
    }
    auto *B = const_cast<mess_basis *>(basis);
    if (B->packed > kNoAllocMaxPacked) {
        set_error("mess_jk_noalloc: %lld matrix elements exceed the fixed workspace of %lld per matrix",
                  (long long)B->packed, (long long)kNoAllocMaxPacked);
        return MESS_E_SIZE;
    }
    if (prof_on()) {
        set_error("mess_jk_noalloc: class profiling is on (it records events); turn it off first");
        return MESS_E_ARG;
    }
    const double tau = schwarz_tol > 0.0 ? schwarz_tol : 0.0;
    auto it = B->lists.find(tau);
    bool ready = it != B->lists.end();
    if (ready)
        for (const ClassList &cl : it->second->classes)
            if (cl.total > 0 && !coop_program_cached(cl.cb, cl.ck)) ready = false;
    if (!ready) {
        set_error("mess_jk_noalloc: the work lists for schwarz_tol %g are not built yet; call mess_jk once "
                  "with this basis, precision and tolerance first", schwarz_tol);
        return MESS_E_ARG;
    }
    if (!J && !K) return MESS_OK;
    double *ws = nullptr;
    MESS_TRY(scratch_address(&ws));
    hipStream_t s = static_cast<hipStream_t>(stream);
    double *Gj = J ? ws : nullptr;
    double *Gk = K ? ws + B->packed : nullptr;
    MESS_TRY(direct_half(B, D, Gj, Gk, prec, tau, s, false));
    return symmetrise_async(B, Gj, Gk, J, K, s);
}

}  // extern "C"
