// Multi-pass engine: one operator product A v = d * v + C v in three HBM
// passes over the pruned half spectrum W (L rows x M/2 packed columns).
//
//   row_fwd  (gather + forward R2C along rows)   v rows -> W
//   col      (forward FFT, * ghat/M^2, inverse FFT along columns, in place)
//   row_inv  (C2R along rows + crop + epilogue)   W -> q = d*v + Cv, partials
//
// Eq. (3) of the paper: C is diagonal in Fourier space, so one product is a
// forward 2-D transform, a pointwise multiply by the static spectrum and an
// inverse transform (Listing 4), the scaling of Listing 3 being folded into
// the stored spectrum.  Listing 4 copies the real input into a complex buffer
// and back; here the real input is packed two-per-complex (z[n] = v[2n] +
// i v[2n+1]) so the row transforms have length M/2 and the column pass
// touches only the M/2 non-redundant column frequencies.  The Nyquist column
// k = M/2 is real for every row, as is k = 0, so both ride in packed column 0
// (real part k = 0, imaginary part k = M/2).
//
// On the zero-padded grid (M = 2L) rows >= L and inputs >= L are zero, so the
// row pass transforms only L rows and the first radix-16 stage of every
// forward transform sees only its lower 8 inputs; outputs >= L are cropped,
// so the last inverse stage stores only its lower 8 outputs.
//
// W layout: tiles of TT columns, W[((kt * L) + i) * TT + kk] for column
// k = kt * TT + kk, so a column tile is one contiguous block and each row
// writes runs of RPW * TT complex values.
#pragma once
#include <stddef.h>
#include <type_traits>
#include "fftcg_dev.hpp"
#include "fftcg_types.hpp"

namespace fftcg {
inline namespace FFTCG_RADIX_NS {

#ifndef FFTCG_STATUS_CODES
#define FFTCG_STATUS_CODES
enum { ST_OK = 0, ST_EINVAL = -1, ST_ENOCONV = -4, ST_EBREAKDOWN = -5 };
#endif

__host__ __device__ constexpr int cmin(int a, int b) { return a < b ? a : b; }
__host__ __device__ constexpr int cmax(int a, int b) { return a > b ? a : b; }

template <typename T, int M, int PAD>
struct Geo {
    static constexpr int L = PAD ? M / 2 : M;
    static constexpr int N = M / 2;  // complex row length = number of packed columns
    // row passes
    static constexpr int ER = fft_elems(N);
    static constexpr int PR = N / ER;
    static constexpr int ROW_WORDS = LdsLay<T, 1, 4, 1>::words(N);
    // LDS budget per workgroup: 72 KB (two workgroups per CU); on the largest
    // grid (M = 8192) one workgroup of twice the size takes 144 KB, so that
    // rows and column tiles still come in pairs and W moves in 32-byte runs
    static constexpr int LDS_CAP_BYTES = M >= 8192 ? 147456 : 73728;
    static constexpr int ROW_LDS_CAP = LDS_CAP_BYTES / (int)sizeof(cx<T>);
#ifndef FFTCG_ROW_NT
#define FFTCG_ROW_NT 256
#endif
    static constexpr int ROW_NT = M >= 8192 ? 2 * FFTCG_ROW_NT : FFTCG_ROW_NT;
    static constexpr int RPW0 = cmin(L, cmax(1, ROW_NT / PR));
    static constexpr int RPW_fit(int r) { return (r > 1 && r * ROW_WORDS > ROW_LDS_CAP) ? RPW_fit(r / 2) : r; }
    static constexpr int RPW = RPW_fit(RPW0);
    static constexpr int ROW_THREADS = RPW * PR;
    static constexpr int ROW_BLOCKS = L / RPW;
    // Sums over the row blocks (grid_sums) in the resident kernel's order,
    // where the grid has one: by groups of its workgroups per XCD (one group
    // up to 64 workgroups, eight above).  0: no such order.
    static constexpr int SUM_GROUPS = (M > 1024 || ROW_BLOCKS > 512) ? 0 : (ROW_BLOCKS <= 64 ? 1 : 8);
    // column pass
    static constexpr int EC = fft_elems(M);
    static constexpr int PC = M / EC;
    static constexpr int COL_LDS_CAP = LDS_CAP_BYTES / (int)sizeof(cx<T>);
    static constexpr int TT_fit(int t) {
        return (t > 1 && (t * M + (t * M) / 16 + t > COL_LDS_CAP || t * PC > 1024)) ? TT_fit(t / 2) : t;
    }
#ifndef FFTCG_COL_TTMAX
#define FFTCG_COL_TTMAX 4
#endif
#ifndef FFTCG_W_TT
#define FFTCG_W_TT 2
#endif
    static constexpr int TT = (M >= 8192 && sizeof(T) == 4) ? FFTCG_W_TT : TT_fit(cmin(N, FFTCG_COL_TTMAX));
    // columns per workgroup: a whole tile, but one column of the pair on the
    // largest grid, where a tile takes 140 KB of LDS and leaves one workgroup
    // per CU, whose loads, transform and stores then run one after another.
    // Two workgroups of a column each overlap them (M = 8192 FP32: column
    // pass 137 -> 115 us; at M = 4096, where two workgroups of a tile fit, 24.5 ->
    // 26.4, so not there); W keeps its pairs, for the row passes' 32-byte
    // runs (with tiles of one column the row passes lost 33 us).
    static constexpr int CT = (M >= 8192 && TT > 1) ? 1 : TT;
    // a tile of W; on the largest grid with 128 bytes behind it: a row's
    // elements lie a tile apart, a power of two without them (row-forward
    // pass at M = 8192 FP32 113 -> 101 us, FP64 174 -> 148; at M = 4096 no
    // gain, FP64 37.4 us with, 35.0 without)
    static constexpr int WT = L * TT + (M >= 8192 ? 128 / (int)sizeof(cx<T>) : 0);
    static_assert((N / TT) * (size_t)WT * sizeof(cx<T>) <= w_bytes(L, M), "W holds the padded tiles");
    static constexpr int COL_SH = ilog2c(16 * CT);
    static constexpr int COL_THREADS = CT * PC;
    static constexpr int NTILE = N / TT;
    static constexpr int COL_BLOCKS = N / CT;
    static constexpr int MH = M / 2 + 1;
};

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Row blocks that share 128-byte lines of W must run on the same XCD,
// so block b works on logical block (b % 8) * (G / 8) + b / 8: each XCD gets
// a contiguous range of rows, visited in order.
__device__ __forceinline__ int xcd_remap(int b, int G) {
    if (G < 16 || (G & 7)) return b;
    return (b & 7) * (G >> 3) + (b >> 3);
}

// Status words for the host (pinned, device-visible): [1] status, [2] the
// iteration of the last FP64 check, [3] iterations, then [0] = 2 *
// generation + done with release order.  Done and the solve's generation
// travel in one word, so a host polling a reused slot can never pair a stale
// done of the previous occupant with the new generation; a host that sees
// done also sees the status.
__device__ __forceinline__ void publish_status(const SlotDesc& sd, int done, int status, int gen, int iters,
                                               int last_check) {
    if (!sd.host_status) return;
    auto* hs = gbl(sd.host_status);
    __hip_atomic_store(hs + 1, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(hs + 2, last_check, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(hs + 3, iters, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(hs, 2 * gen + (done ? 1 : 0), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- CG control shared by both engines --------------------------------------

// Whether an FP64 check must come before the next iteration, given the
// recursive r.r: at maxit; every `refresh` iterations (mixed mode); when the
// recursive residual meets the stop rule; or, as a reliable update, once it
// has fallen by sqrt(delta2) since the last replacement (past that point the
// working-precision recursion may drift from the true residual).  The last
// two need an iteration since the previous check, so checks alternate with
// progress.
// iters: the iteration count the decision is for (st->iters, unless the
// caller has counted an iteration whose store to st it cannot read back)
// What the decision depends on besides r.r, read all at once (each read of
// the state costs an L2 round trip when a branch separates it from the next)
struct CheckIn {
    double trigger_rr, delta2, rho_ref;
    int iters, last_check_iter, refresh, maxit;
};
template <class St>
__device__ __forceinline__ CheckIn check_in(const St* st) {
    return CheckIn{st->trigger_rr, st->delta2, st->rho_ref, st->iters, st->last_check_iter, st->refresh, st->maxit};
}
__device__ __forceinline__ bool check_due(const CheckIn& c, double rr, int iters) {
    const int since = iters - c.last_check_iter;
    const bool progressed = since > 0;
    const bool periodic = (c.refresh > 0) & (since >= c.refresh);
    const bool candidate = progressed & !(rr > c.trigger_rr);
    // a reliable update is skipped when the convergence trigger lies within
    // a factor 100 (10 in the residual norm) below its threshold: the check at
    // candidate convergence comes soon and replaces the residual as well
    const double rel = c.delta2 * c.rho_ref;
    const bool reliable = progressed & (rr <= rel) & (c.trigger_rr < 1e-2 * rel);
    return (iters >= c.maxit) | candidate | periodic | reliable;
}
__device__ __forceinline__ bool check_due(const SolveState* st, double rr, int iters) {
    return check_due(check_in(st), rr, iters);
}
__device__ __forceinline__ bool check_due(const SolveState* st, double rr) { return check_due(st, rr, st->iters); }

// Outcome of an FP64 check from its reductions: |b - A x|^2 (R), |x|^2 (X),
// |b|^2 (B), |r_working|^2 (RW), invalid-input count (BAD), drift of the
// recursive residual (DIFF), min d.  Updates the state (one thread); returns
// 1 when CG continues with the replaced residual (r.r = RW), 0 when done.
__device__ inline int check_decide(SolveState* st, double R, double X, double B, double RW, double BAD,
                                   double DIFF, double dmin) {
    const bool first = st->checks == 0;
    st->checks += 1;
    if (first) {
        st->bnorm = sqrt(B);
        st->lam_lb = dmin + st->gmin;
    }
    const double rt = sqrt(R), xn = sqrt(X), bn = st->bnorm;
    if (first && BAD > 0.0) {
        st->status = ST_EINVAL;
        st->done = 1;
        return 0;
    }
    if (first && bn == 0.0) {
        st->status = ST_OK;
        st->done = 1;
        st->bzero = 1;
        st->true_relres = 0.0;
        st->bound = 0.0;
        return 0;
    }
    if (!isfinite(rt) || !isfinite(xn)) {
        st->status = ST_EBREAKDOWN;
        st->done = 1;
        return 0;
    }
    const double tau = st->tau, lam = st->lam_lb;
    const bool lit = rt <= st->tol * bn;
    const double cert_target = tau * lam * xn / (1.0 + tau);
    const bool cert = rt <= cert_target;
    const double e = rt / lam;
    st->true_relres = rt / bn;
    st->bound = xn > e ? e / (xn - e) : 1.0e300;
    if (lit && st->iters_literal < 0) st->iters_literal = st->iters;
    if (lit && cert) {
        st->status = ST_OK;
        st->done = 1;
        return 0;
    }
    if (st->iters >= st->maxit) {
        st->status = ST_ENOCONV;
        st->done = 1;
        return 0;
    }
    double trig = st->tol * bn;
    if (xn > 0.0 && cert_target < trig) trig = cert_target;
    st->trigger_rr = trig * trig;
    if (first) {
        st->worse = 0;
        st->best_rt = rt;
    } else if (rt >= st->best_rt) {
        st->worse += 1;
    } else {
        st->worse = 0;
        st->best_rt = rt;
    }
    if (st->worse >= 2) {
        st->restart = 1;
        st->worse = 0;
    }
    // Keeping p after the replacement is sound only while the recursive
    // residual still tracked the true one; past 10% drift the old direction
    // is no longer conjugate, so restart.
    if (!first && !(DIFF <= 0.01 * R)) st->restart = 1;
    st->rho_ref = RW;
    st->alpha = 0.0;
    st->last_check_iter = st->iters;
    st->last_rt = rt;
    st->xnorm = xn;
    st->pause = 0;
    return 1;
}

// ---- slot access policies -------------------------------------------------
struct ByPtr {
    const SlotDesc* p;
    // a copy, read once: the kernels' stores cannot alias it, so its fields
    // stay in registers instead of being read again after every store
    __device__ __forceinline__ SlotDesc get() const { return p[blockIdx.y]; }
};
struct ByVal {
    SlotDesc s;
    __device__ __forceinline__ const SlotDesc& get() const { return s; }
};

// gates: which slots a kernel works on (inactive slots first, then the
// solve's state; pause and done are adjacent words, read with one load).
__device__ __forceinline__ typename VecT<int, 2>::type pause_done(const SolveState* st) {
    static_assert(offsetof(SolveState, done) == offsetof(SolveState, pause) + sizeof(int) &&
                      offsetof(SolveState, pause) % 8 == 0,
                  "pause and done form one aligned 8-byte word");
    return *gbl(reinterpret_cast<const typename VecT<int, 2>::type*>(&st->pause));
}
struct GateAlways {
    static __device__ __forceinline__ bool ok(const SlotDesc&) { return true; }
};
struct GateIter {  // CG iteration kernels
    static __device__ __forceinline__ bool ok(const SlotDesc& sd) {
        if (!sd.active) return false;
        const auto pd = pause_done(sd.st);
        return (pd.x | pd.y) == 0;
    }
};
struct GateCheck {  // FP64 check kernels
    static __device__ __forceinline__ bool ok(const SlotDesc& sd) {
        if (!sd.active) return false;
        const auto pd = pause_done(sd.st);
        return pd.x != 0 && pd.y == 0;
    }
};
struct GatePre {  // preconditioner after a check that continues the solve
    static __device__ __forceinline__ bool ok(const SlotDesc& sd) {
        if (!sd.active) return false;
        const int done = *gbl(&sd.st->done), need = *gbl(&sd.st->need_pre);
        return (done == 0) & (need != 0);
    }
};

template <typename T>
struct Tab {
    const cx<T>* tw;   // exp(-2 pi i m / M), m in [0, M)
    const T* ghq;      // quarter spectrum / M^2 in tile layout
    const T* ghN;      // ghat(m, M/2) / M^2, m in [0, M/2]
};

template <typename T, int N>
struct PairT;
template <>
struct PairT<float, 2> { using type = float2; };
template <>
struct PairT<double, 2> { using type = double2; };

// a pair of consecutive elements (even index) of a device array
template <typename T>
__device__ __forceinline__ cx<T> ld2(const T* p) {
    return gld(reinterpret_cast<const cx<T>*>(p));
}
template <typename T>
__device__ __forceinline__ void st2(T* p, cx<T> c) {
    gst(reinterpret_cast<cx<T>*>(p), c);
}
// The same at element idx of a base that is the same in every thread: a 32-bit
// byte offset beside a base in scalar registers (every array is under 4 GB),
// instead of a 64-bit address per element (an eighth of the turn pass's
// vector instructions were address arithmetic and sign extensions).
template <typename V, typename T>
__device__ __forceinline__ typename GlobalT<V>::type* at_byte(T* base, unsigned bytes) {
    typedef typename GlobalT<char>::type C;
    return (typename GlobalT<V>::type*)((C*)base + bytes);
}
template <typename T>
__device__ __forceinline__ cx<T> ld2(const T* base, unsigned idx) {
    const auto v = *at_byte<const typename VecT<T, 2>::type>(const_cast<T*>(base), idx * (unsigned)sizeof(T));
    return mkc(v.x, v.y);
}
template <typename T>
__device__ __forceinline__ void st2(T* base, unsigned idx, cx<T> c) {
    typename VecT<T, 2>::type v;
    v.x = c.x;
    v.y = c.y;
    *at_byte<typename VecT<T, 2>::type>(base, idx * (unsigned)sizeof(T)) = v;
}
// Pairs of the grid's vectors (r, p, q, x, ...; L: the grid).  On the largest
// grids an iteration's data (470 MB at L = 4096 FP32) exceeds the 256 MB
// last-level cache; the vectors then pass through it without being kept, and
// W, which is written and read by three passes in a row, stays (mixed solve of
// L = 4096: 79.9 ms kept, 68.8 passing; column pass 133 -> 110 us, row passes
// 133 and 89 -> 113 and 76).  Not q's store: the update reads it next (68.8
// against 69.3 ms).  The periodic grid of L = 4096 (half of W, a quarter of
// the columns' work) gains as well: whole solves FP32 18.8 -> 17.5 ms, FP64
// 36.3 -> 27.9, preconditioned 7.1 -> 6.6 and 11.8 -> 9.4.  Below, everything
// fits (L = 2048: 117 MB FP32, 235 MB FP64), and passing costs: FP32 13.8 ->
// 14.4 ms, FP64 16.0 -> 18.7.
template <int L>
constexpr bool kStream = L >= 4096;
template <typename T, int L>
__device__ __forceinline__ cx<T> ldv(const T* base, unsigned idx) {
    const auto* p = at_byte<const typename VecT<T, 2>::type>(const_cast<T*>(base), idx * (unsigned)sizeof(T));
    typename VecT<T, 2>::type v;
    if constexpr (kStream<L>)
        v = __builtin_nontemporal_load(p);
    else
        v = *p;
    return mkc(v.x, v.y);
}
template <typename T, int L>
__device__ __forceinline__ void stv(T* base, unsigned idx, cx<T> c) {
    typename VecT<T, 2>::type v;
    v.x = c.x;
    v.y = c.y;
    auto* p = at_byte<typename VecT<T, 2>::type>(base, idx * (unsigned)sizeof(T));
    if constexpr (kStream<L>)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}
template <typename T>
__device__ __forceinline__ cx<T> gld(const cx<T>* base, unsigned idx) {
    return ld2<T>(reinterpret_cast<const T*>(base), 2 * idx);
}
template <typename T>
__device__ __forceinline__ void gst(cx<T>* base, unsigned idx, cx<T> c) {
    st2<T>(reinterpret_cast<T*>(base), 2 * idx, c);
}
__device__ __forceinline__ cx<double> ld2f(const float* base, unsigned idx) {
    const cx<float> v = ld2<float>(base, idx);
    return mkc((double)v.x, (double)v.y);
}
__device__ __forceinline__ cx<double> ld2f(const float* p) {
    const cx<float> v = gld(reinterpret_cast<const cx<float>*>(p));
    return mkc((double)v.x, (double)v.y);
}
// Projection onto the intact entries of a masked solve: (m0, m1) in {0, 1}
// for the pair at idx (both 1 without a mask).
struct Mask2 {
    double m0, m1;
};
__device__ __forceinline__ Mask2 mask2(const SlotDesc& sd, unsigned idx) {
    if (!sd.mask) return Mask2{1.0, 1.0};
    const auto* m = gbl(sd.mask + idx);
    return Mask2{(double)m[0], (double)m[1]};
}

// The resident kernel's order of a sum over row blocks (Geo::SUM_GROUPS, NG
// here): block b is member b / NG of group b % NG, a group is a wave sum and
// the groups are added as a tree.  By one wave; the result in every lane.
__device__ __forceinline__ double group_tree(double v) {  // over lane & 7, in rows of 16 lanes holding them twice
    return wave_sum<4>(v);
}
template <int NG, bool MIN = false, class GET>
__device__ __forceinline__ double group_sum(unsigned int n, double none, GET get) {
    const unsigned int lane = threadIdx.x & 63;
    double mine = none;  // the lane's group (lane & 7)
    double v[NG];        // all of them requested together (n > 0)
#pragma unroll
    for (unsigned int g = 0; g < NG; ++g) {
        const unsigned int i = g + NG * lane;
        v[g] = get(i < n ? i : 0u);
        v[g] = i < n ? v[g] : none;
    }
#pragma unroll
    for (unsigned int g = 0; g < NG; ++g) {
        const double t = MIN ? wave_min(v[g]) : wave_sum(v[g]);
        if (NG == 1 || (lane & 7) == g) mine = t;
    }
    if (NG == 1) return mine;
    return MIN ? wave_min<4>(mine) : group_tree(mine);
}
// Sum of n partials, in that order or (NG = 0, or a block without whole
// waves) in sum_partials'; result in every thread.  sh: NT / 64 doubles.
template <int NT, int NG>
__device__ __forceinline__ double sum_blocks(const double* p, int n, double* sh) {
    if constexpr (NG > 0 && NT % 64 == 0) {
        // every wave adds them up by itself
        return group_sum<NG>(n, 0.0, [&](unsigned int i) { return gbl(p)[i]; });
    } else {
        return sum_partials<NT>(p, n, sh);
    }
}

// ==== prologues of the row-forward pass ====================================
//
// begin() decides whether the pass runs and fills the scalars (Sc, the same
// in every thread; Sh: LDS for its reductions).  A pair's input then comes in
// two steps, fetch (reads only) and combine (arithmetic and stores): a pass
// fetches all pairs of a thread, up to eight at a time, before it combines
// them.  In one step each pair's store held up the next pair's reads, which
// may alias it as far as the compiler knows, and a read behind a store also
// waits for that store to complete.  PREF: the fetch comes before begin's
// reductions (FP32).

// fftcg_apply: transform x (FP64 in memory), rounded to T.
template <typename T>
struct ProApply {
    static constexpr int NACC = 0;
    static constexpr bool PREF = false;
    struct Sh {};
    struct Sc {};
    using Gate = GateAlways;
    using Raw = cx<double>;
    static __device__ __forceinline__ bool begin(const SlotDesc&, Sh&, Sc&, int, int) { return true; }
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        return ldv<double, L>(sd.x, (unsigned)row * L + col);
    }
    template <int L>
    static __device__ __forceinline__ cx<T> combine(const SlotDesc&, const Sc&, const Raw& v, int, int, double*) {
        return mkc((T)v.x, (T)v.y);
    }
};

// CG iteration: x_acc += alpha p_old (pending update of the last iteration),
// p = r + beta p_old (or p = r on restart), then transform p.
// W: working precision of r, p; XA: accumulator (double: x itself; float: e).
// FOLD: r.r comes from the state, where the folded update (EpiCGU) or the
// check left it, instead of from the update kernel's partials.
template <typename W, typename XA, int NT, bool FOLD = false>
struct ProCG {
    static constexpr int NACC = 0;
    struct Sh {
        double red[(NT + 63) / 64];
    };
    struct Sc {
        W alpha, beta;
        int restart;
    };
    using Gate = GateIter;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd, Sh& sh, Sc& sc, int npart_rr, int stride) {
        if (!GateIter::ok(sd)) return false;
        auto* st = gbl(sd.st);
        const CheckIn ci = check_in(st);
        const double alpha = st->alpha, rho_prev = st->rho_prev, rho_next = st->rho_next;
        sc.restart = st->restart;
        const double rr = FOLD ? rho_next : sum_partials<NT>(sd.part + PS_RR * stride, npart_rr, sh.red);
        if (check_due(ci, rr, ci.iters)) {
            if (blockIdx.x == 0 && threadIdx.x == 0) st->pause = 1;
            return false;
        }
        sc.alpha = (W)alpha;
        sc.beta = (W)(sc.restart ? 0.0 : rr / rho_prev);
        if (blockIdx.x == 0 && threadIdx.x == 0) st->rho_cur = rr;
        return true;
    }
    static constexpr bool PREF = sizeof(W) == 4;
    // The pending x update (late) runs after the transform (FP32): its reads
    // then overlap the W writes instead of lengthening the pass's first,
    // read-only phase (p stays in registers until then, within the pass's
    // register budget)
#ifndef FFTCG_LATE_X
#define FFTCG_LATE_X 1
#endif
    static constexpr bool LATE_X = PREF && FFTCG_LATE_X;
    struct Raw {
        cx<W> r, p;
        cx<XA> x;
    };
    static __device__ __forceinline__ XA* xacc(const SlotDesc& sd) {
        return reinterpret_cast<XA*>(sizeof(XA) == 8 ? (void*)sd.x : (void*)sd.e);
    }
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        Raw w;
        w.r = ldv<W, L>(reinterpret_cast<const W*>(sd.r), idx);
        w.p = ldv<W, L>(reinterpret_cast<const W*>(sd.p), idx);
        if constexpr (!LATE_X) w.x = ldv<XA, L>(xacc(sd), idx);
        return w;
    }
    template <int L>
    static __device__ __forceinline__ cx<W> combine(const SlotDesc& sd, const Sc& sc, const Raw& w, int row,
                                                    int col, double*) {
        const unsigned idx = (unsigned)row * L + col;
        const cx<W> po = w.p;
        cx<W> p2 = mkc(w.r.x + sc.beta * po.x, w.r.y + sc.beta * po.y);
        if (sc.restart) p2 = w.r;
        if constexpr (!LATE_X) {
            if (!sc.restart && sc.alpha != W(0)) {
                cx<XA> xv = w.x;
                xv.x += (XA)sc.alpha * (XA)po.x;
                xv.y += (XA)sc.alpha * (XA)po.y;
                stv<XA, L>(xacc(sd), idx, xv);
            }
        }
        stv<W, L>(reinterpret_cast<W*>(sd.p), idx, p2);
        return p2;
    }
    // the pending x update of a pair, after the transform (LATE_X), in two steps
    static __device__ __forceinline__ bool late_due(const Sc& sc) { return !sc.restart && sc.alpha != W(0); }
    template <int L>
    static __device__ __forceinline__ cx<XA> late_fetch(const SlotDesc& sd, int row, int col) {
        return ldv<XA, L>(xacc(sd), (unsigned)row * L + col);
    }
    template <int L>
    static __device__ __forceinline__ void late(const SlotDesc& sd, const Sc& sc, const Raw& w, cx<XA> xv, int row,
                                                int col) {
        xv.x += (XA)sc.alpha * (XA)w.p.x;
        xv.y += (XA)sc.alpha * (XA)w.p.y;
        stv<XA, L>(xacc(sd), (unsigned)row * L + col, xv);
    }
};

// FP64 check: x <- x + e + alpha p (flush of the pending updates), e <- 0,
// transform x in FP64.
template <typename W, int NT>
struct ProCheck {
    static constexpr int NACC = 0;
    static constexpr bool PREF = false;
    struct Sh {};
    struct Sc {
        double alpha;
    };
    using Gate = GateCheck;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd, Sh&, Sc& sc, int, int) {
        if (!GateCheck::ok(sd)) return false;
        sc.alpha = gbl(sd.st)->alpha;
        return true;
    }
    // (the correction e belongs to FP32 solves; p is read whether used or not)
    static constexpr bool HAS_E = sizeof(W) == 4;
    struct Raw {
        cx<double> x;
        cx<float> e;
        cx<W> p;
    };
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        Raw w;
        w.x = ldv<double, L>(sd.x, idx);
        if constexpr (HAS_E) w.e = ldv<float, L>(sd.e, idx);
        w.p = ldv<W, L>(reinterpret_cast<const W*>(sd.p), idx);
        return w;
    }
    template <int L>
    static __device__ __forceinline__ cx<double> combine(const SlotDesc& sd, const Sc& sc, const Raw& w, int row,
                                                         int col, double*) {
        const unsigned idx = (unsigned)row * L + col;
        cx<double> xv = w.x;
        if constexpr (HAS_E) {
            xv.x += (double)w.e.x;
            xv.y += (double)w.e.y;
            stv<float, L>(sd.e, idx, mkc(0.0f, 0.0f));
        }
        if (sc.alpha != 0.0) {
            xv.x += sc.alpha * (double)w.p.x;
            xv.y += sc.alpha * (double)w.p.y;
        }
        const Mask2 mk = mask2(sd, idx);  // broken entries carry no force
        xv.x *= mk.m0;
        xv.y *= mk.m1;
        stv<double, L>(sd.x, idx, xv);
        return xv;
    }
};

// Preconditioned CG (Fourier-space circulant preconditioner), first half of
// an iteration: beta = (r.z) / (r.z)_old from the partials of the
// preconditioner pass, p = z + beta p (p = z on restart), pending x update,
// then transform p.  The stop triggers still use r.r.  NPZ: partial count of
// the r.z sums.
template <typename W, typename XA, int NT, int NPZ, int NG>
struct ProPCG {
    static constexpr int NACC = 0;
    static constexpr bool PREF = sizeof(W) == 4;
    struct Sh {
        double red[2 * ((NT + 63) / 64)];
        double tot[2];
    };
    struct Sc {
        W alpha, beta;
        int restart;
    };
    using Gate = GateIter;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd, Sh& sh, Sc& sc, int npart_rr, int stride) {
        if (!GateIter::ok(sd)) return false;
        auto* st = gbl(sd.st);
        const CheckIn ci = check_in(st);
        const double alpha = st->alpha, rho_prev = st->rho_prev;
        sc.restart = st->restart;
        double rr, rz;
        if constexpr (NG > 0) {
            rr = sum_blocks<NT, NG>(sd.part + PS_RR * stride, npart_rr, sh.red);
            rz = sum_blocks<NT, NG>(sd.part + PS_RZ * stride, NPZ, sh.red);
        } else if constexpr (NT % 64 == 0) {
            // r.r and r.z reduced together (each in sum_partials' order)
            double a2[2] = {0.0, 0.0};
            const auto* prr = gbl(sd.part + PS_RR * stride);
            const auto* prz = gbl(sd.part + PS_RZ * stride);
            for (int i = threadIdx.x; i < npart_rr; i += NT) a2[0] += prr[i];
            for (int i = threadIdx.x; i < NPZ; i += NT) a2[1] += prz[i];
            const double t = block_reduce_n<NT, 2, 0u>(a2, sh.red);
            if (threadIdx.x < 2) sh.tot[threadIdx.x] = t;
            __syncthreads();
            rr = sh.tot[0];
            rz = sh.tot[1];
        } else {
            rr = sum_partials<NT>(sd.part + PS_RR * stride, npart_rr, sh.red);
            rz = sum_partials<NT>(sd.part + PS_RZ * stride, NPZ, sh.red);
        }
        if (check_due(ci, rr, ci.iters)) {
            if (blockIdx.x == 0 && threadIdx.x == 0) st->pause = 1;
            return false;
        }
        sc.alpha = (W)alpha;
        sc.beta = (W)(sc.restart ? 0.0 : rz / rho_prev);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->rho_cur = rz;
            st->need_pre = 0;
        }
        return true;
    }
    struct Raw {
        cx<W> z, p;
        cx<XA> x;
    };
    static __device__ __forceinline__ XA* xacc(const SlotDesc& sd) {
        return reinterpret_cast<XA*>(sizeof(XA) == 8 ? (void*)sd.x : (void*)sd.e);
    }
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        return Raw{ldv<W, L>(reinterpret_cast<const W*>(sd.z), idx), ldv<W, L>(reinterpret_cast<const W*>(sd.p), idx),
                   ldv<XA, L>(xacc(sd), idx)};
    }
    template <int L>
    static __device__ __forceinline__ cx<W> combine(const SlotDesc& sd, const Sc& sc, const Raw& w, int row,
                                                    int col, double*) {
        const unsigned idx = (unsigned)row * L + col;
        const cx<W> po = w.p;
        cx<W> p2 = mkc(w.z.x + sc.beta * po.x, w.z.y + sc.beta * po.y);
        if (sc.restart) p2 = w.z;
        if (!sc.restart && sc.alpha != W(0)) {
            cx<XA> xv = w.x;
            xv.x += (XA)sc.alpha * (XA)po.x;
            xv.y += (XA)sc.alpha * (XA)po.y;
            stv<XA, L>(xacc(sd), idx, xv);
        }
        stv<W, L>(reinterpret_cast<W*>(sd.p), idx, p2);
        return p2;
    }
};

// Preconditioned CG, second half: alpha = (r.z) / (p.q) from the partials of
// the operator's row-inverse pass (breakdown if p.q <= 0), r <- r - alpha q
// with partial r.r, then transform r for z = P^{-1} r.  NPQ: partial count of
// the p.q sums.
template <typename W, int NT, int NPQ, int NG>
struct ProUpdPre {
    static constexpr int NACC = 1;
    static constexpr bool PREF = sizeof(W) == 4;
    static constexpr int SET = PS_RR;
    struct Sh {
        double red[(NT + 63) / 64];
    };
    struct Sc {
        W alpha;
    };
    using Gate = GateIter;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd, Sh& sh, Sc& sc, int, int stride) {
        if (!GateIter::ok(sd)) return false;
        auto* st = gbl(sd.st);
        const double rho = st->rho_cur;
        const double pq = sum_blocks<NT, NG>(sd.part + PS_PQ * stride, NPQ, sh.red);
        if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) {
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                st->status = ST_EBREAKDOWN;
                st->done = 1;
                publish_status(sd, 1, ST_EBREAKDOWN, st->gen, st->iters, st->last_check_iter);
            }
            return false;
        }
        const double alpha = rho / pq;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->alpha = alpha;
            st->rho_prev = rho;
            st->iters += 1;
            st->restart = 0;
        }
        sc.alpha = (W)alpha;
        return true;
    }
    struct Raw {
        cx<W> r, q;
    };
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        return Raw{ldv<W, L>(reinterpret_cast<const W*>(sd.r), idx), ldv<W, L>(reinterpret_cast<const W*>(sd.q), idx)};
    }
    template <int L>
    static __device__ __forceinline__ cx<W> combine(const SlotDesc& sd, const Sc& sc, const Raw& w, int row,
                                                    int col, double* acc) {
        const unsigned idx = (unsigned)row * L + col;
        const cx<W> rn = mkc(w.r.x - sc.alpha * w.q.x, w.r.y - sc.alpha * w.q.y);
        stv<W, L>(reinterpret_cast<W*>(sd.r), idx, rn);
        acc[0] += (double)rn.x * (double)rn.x + (double)rn.y * (double)rn.y;
        return rn;
    }
};

// Preconditioner after a check that continues the solve: transform the
// replaced residual r.
template <typename W>
struct ProPre {
    static constexpr int NACC = 0;
    static constexpr bool PREF = false;
    struct Sh {};
    struct Sc {};
    using Gate = GatePre;
    using Raw = cx<W>;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd, Sh&, Sc&, int, int) { return GatePre::ok(sd); }
    template <int L>
    static __device__ __forceinline__ Raw fetch(const SlotDesc& sd, int row, int col) {
        return ldv<W, L>(reinterpret_cast<const W*>(sd.r), (unsigned)row * L + col);
    }
    template <int L>
    static __device__ __forceinline__ cx<W> combine(const SlotDesc&, const Sc&, const Raw& w, int, int, double*) {
        return w;
    }
};

// ==== epilogues of the row-inverse pass ====================================

// As the prologues, in two steps: pre (a pair's operands) and out2p.  PREF:
// the operands are requested with the spectrum, before the transform (FP32);
// otherwise after it, up to eight pairs together.

// fftcg_apply: y = d * x (FP64) + C x.
template <typename T>
struct EpiApply {
    static constexpr int NACC = 0;
    static constexpr bool PREF = false;
    using Gate = GateAlways;
    static __device__ __forceinline__ bool begin(const SlotDesc&) { return true; }
    struct Pre {
        cx<double> d, x;
    };
    template <int L>
    static __device__ __forceinline__ Pre pre(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        return Pre{ldv<double, L>(sd.d, idx), ldv<double, L>(sd.x, idx)};
    }
    template <int L>
    static __device__ __forceinline__ void out2p(const SlotDesc& sd, int row, int col, T c0, T c1, const Pre& pr,
                                                 double*) {
        st2<double>(sd.y, (unsigned)row * L + col,
                    mkc(pr.d.x * pr.x.x + (double)c0, pr.d.y * pr.x.y + (double)c1));
    }
};

// CG iteration: q = d p + C p; partial p . q (FP64 accumulation).
template <typename W>
struct EpiCG {
    static constexpr int NACC = 1;
    static constexpr int SET = PS_PQ;
    using Gate = GateIter;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd) { return GateIter::ok(sd); }
    // FP32: p and d of every output are requested before the transform, so
    // their reads neither wait behind the q stores (which may alias them as
    // far as the compiler knows) nor expose their latency after it
    static constexpr bool PREF = sizeof(W) == 4;
    struct Pre {
        cx<W> p, d;
    };
    template <int L>
    static __device__ __forceinline__ Pre pre(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        Pre v;
        v.p = ldv<W, L>(reinterpret_cast<const W*>(sd.p), idx);
        if constexpr (sizeof(W) == 4) {
            v.d = ldv<float, L>(sd.d32, idx);
        } else {
            v.d = ldv<double, L>(sd.d, idx);
        }
        return v;
    }
    template <int L>
    static __device__ __forceinline__ void out2p(const SlotDesc& sd, int row, int col, W c0, W c1, const Pre& pr,
                                                 double* acc) {
        const unsigned idx = (unsigned)row * L + col;
        W* q = reinterpret_cast<W*>(sd.q);
        const cx<W> pv = pr.p, dv = pr.d;
        cx<W> qv = mkc(dv.x * pv.x + c0, dv.y * pv.y + c1);
        if (sd.mask) {
            const Mask2 mk = mask2(sd, idx);
            qv = mkc(qv.x * (W)mk.m0, qv.y * (W)mk.m1);
        }
        st2<W>(q, idx, qv);
        acc[0] += (double)pv.x * (double)qv.x + (double)pv.y * (double)qv.y;
    }
    // q of a pair without storing it (the grid-synchronised update below)
    template <int L>
    static __device__ __forceinline__ cx<W> outq(const SlotDesc& sd, int row, int col, W c0, W c1, const Pre& pr,
                                                 double* acc) {
        const cx<W> pv = pr.p, dv = pr.d;
        cx<W> qv = mkc(dv.x * pv.x + c0, dv.y * pv.y + c1);
        if (sd.mask) {
            const Mask2 mk = mask2(sd, (unsigned)row * L + col);
            qv = mkc(qv.x * (W)mk.m0, qv.y * (W)mk.m1);
        }
        acc[0] += (double)pv.x * (double)qv.x + (double)pv.y * (double)qv.y;
        return qv;
    }
};

// The CG epilogue with the residual update folded in: q = A p never leaves
// registers.  Every workgroup reduces four sums over its own rows, p.q, r.r,
// r.q and q.q (FP64), meets the others at a grid-wide barrier that returns
// the totals (grid_sums; the host launches this only where the whole grid
// fits the device at once), forms alpha = r.r / p.q and updates r <- r -
// alpha q on its own rows.  r.r of the updated residual, which the next beta
// and the check decision need, follows from the same totals:
//   |r - a q|^2 = r.r - 2 a (r.q) + a^2 (q.q),
// so that no second barrier is needed for it.  It replaces the separate
// update kernel: one pass over q fewer, and one kernel fewer.
template <typename W>
struct EpiCGU : EpiCG<W> {
    static constexpr int NACC = 4;
    static constexpr bool UPD = true;
};
// The preconditioned iteration's two turns, each a row-inverse pass that goes
// on into a forward row pass on the same rows behind one barrier:
// EpiTurnR: q = A p, the sum p.q; then alpha, r <- r - alpha q, and r's
//   transform (EpiCG's pass followed by ProUpdPre's).
// EpiTurnZ: z = P^-1 r, the sums r.z and r.r; then beta, the check decision,
//   p <- z + beta p, the pending x update, and p's transform (EpiPre's pass
//   followed by ProPCG's).
// q and z never reach memory.
template <typename W>
struct EpiTurnR : EpiCG<W> {
    static constexpr int TURN = 1;
};
template <class E, class = void>
struct EpiUpd {
    static constexpr bool value = false;
};
template <class E>
struct EpiUpd<E, decltype((void)E::UPD)> {
    static constexpr bool value = E::UPD;
};
template <class E, class = void>
struct EpiTurn {
    static constexpr int value = 0;
};
template <class E>
struct EpiTurn<E, decltype((void)E::TURN)> {
    static constexpr int value = E::TURN;
};

// r.r after the update from the totals t = {p.q, r.r, r.q, q.q} (a: alpha in
// the working precision, as the update uses it).  Where the residual falls
// by so much that the difference cancels (below a hundredth of a^2 q.q; an
// ordinary iteration leaves a tenth or more) the caller sums it anew behind
// a second barrier.  So in FP64 the relative error stays below 1e-12 (the
// terms are at most 441 times the result; a few 1e-15 in ordinary
// iterations); in FP32 the stored residual differs by its rounding after the
// update, which the sums do not see: at most 2^-23 of r.r, about 2^-23 / L
// where the residual is spread over the grid.  False also for NaN.
__device__ __forceinline__ bool next_rr(const double* t, double a, double* rr) {
    *rr = fma(a, fma(a, t[3], -2.0 * t[2]), t[1]);
    return *rr > 0.01 * (a * a * t[3]);
}

// The sums of N per-thread values over the whole grid, in every thread
// (tot), with a grid-wide barrier on the way, without read-modify-write
// traffic on one address (1,024 atomic additions to one counter serialise
// where they are performed and cost tens of microseconds).  Each call
// carries a token that no other call on the same partial-sum buffer uses.  A
// workgroup stores its N partials (set a at part[sets[a] stride + block]),
// waits for them to complete and arrives by storing the token to its own
// word flags[b]; workgroup 0 waits until every flag holds the token, sums
// the partials (thread t takes t, t + NT, ..., then the block sum), stores
// the totals and then the token to the release line rel, which the others
// wait for (rel[0] the token, rel[1 + a] the totals).  One workgroup summing
// for all keeps the traffic at the coherence point to one read of the
// partials: with every workgroup reading all of them, 1,024 workgroups would
// move 33 MB per barrier.  All of these are agent-scope atomics, performed
// where every XCD sees them, and each step waits for the previous step's
// value, so no cache-wide fence is needed (a release/acquire pair at agent
// scope writes back and invalidates the L2 of every workgroup's XCD, which
// costs more than the whole update).  Waits are bounded: after `limit` ticks
// of the 100 MHz constant clock the workgroup gives up and false is returned
// (a grid that is not resident as a whole cannot complete the barrier).
// Called by every thread of the workgroup; returns the same value in all.
// sh must hold N * (NT + 63) / 64 doubles.
// NG: the summation order (group_sum), 0: thread t takes t, t + NT, ..., then
// the block sum.
template <int NT, int N, int NG>
__device__ inline bool grid_sums(const double* acc, double* part, int stride, unsigned long long token,
                                 long long limit, double* sh, double* tot) {
    // (N = 2, the preconditioned turn: r.z and r.r)
    constexpr int sets[4] = {PS_PQ, N == 2 ? PS_RZ : PS_RR, PS_RQ, PS_QQ};
    static_assert(N <= 4, "four sets");
    __shared__ double s_tot[N];
    __shared__ int s_ok;
    const int tid = threadIdx.x;
    const unsigned int nb = gridDim.x;
    auto* flags = reinterpret_cast<unsigned long long*>(part + PS_BAR * stride);
    auto* rel = reinterpret_cast<unsigned long long*>(part + PS_BARREL * stride);
    auto put = [](unsigned long long* p, double v) {
        (void)__hip_atomic_exchange(gbl(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    };
    auto get = [](const unsigned long long* p) {
        return __builtin_bit_cast(double, __hip_atomic_load(gbl(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    auto setp = [&](int a) {  // partials of set a (a small: no table in memory)
        const int ps = a == 0 ? sets[0] : (a == 1 ? sets[1] : (a == 2 ? sets[2] : sets[3]));
        return reinterpret_cast<unsigned long long*>(part + ps * stride);
    };
    block_sums<NT, N>(acc, sh, s_tot);
    __syncthreads();
    for (int a = tid; a < N; a += NT) put(setp(a) + blockIdx.x, s_tot[a]);
    __builtin_amdgcn_s_waitcnt(0);  // the first wave's exchanges are complete
    if (tid == 0) __hip_atomic_store(gbl(flags + blockIdx.x), token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
    int ok = 1;
    if (blockIdx.x == 0) {
        for (;;) {
            int here = 1;
            for (unsigned int i = tid; i < nb; i += NT)
                here &= __hip_atomic_load(gbl(flags + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == token;
            const int expired = (long long)(__builtin_amdgcn_s_memrealtime() - t0) > limit;
            // both decisions are taken by the whole workgroup
            if (__syncthreads_and(here)) break;
            if (__syncthreads_or(expired)) {
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (ok) {
            if constexpr (NG > 0 && NT % 64 == 0) {
                if (tid < 64) {
#pragma unroll
                    for (int a = 0; a < N; ++a) {
                        const double t = group_sum<NG>(nb, 0.0, [&](unsigned int i) { return get(setp(a) + i); });
                        if (tid == 0) s_tot[a] = t;
                    }
                }
            } else {
                double s[N];
#pragma unroll
                for (int a = 0; a < N; ++a) s[a] = 0.0;
                for (unsigned int i = tid; i < nb; i += NT)
#pragma unroll
                    for (int a = 0; a < N; ++a) s[a] += get(setp(a) + i);
                block_sums<NT, N>(s, sh, s_tot);
            }
            __syncthreads();
            for (int a = tid; a < N; a += NT) put(rel + 1 + a, s_tot[a]);
            __builtin_amdgcn_s_waitcnt(0);
            if (tid == 0) __hip_atomic_store(gbl(rel), token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
    } else {
        if (tid < cmin(N, NT)) {
            // the lanes that fetch the totals wait together, and give up together
            for (;;) {
                const bool here = __hip_atomic_load(gbl(rel), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == token;
                if (__all(here)) break;
                if (__any((long long)(__builtin_amdgcn_s_memrealtime() - t0) > limit)) {
                    ok = 0;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (ok)
                for (int a = tid; a < N; a += NT) s_tot[a] = get(rel + 1 + a);
            if (tid == 0) s_ok = ok;
        }
        __syncthreads();
        ok = s_ok;
    }
#pragma unroll
    for (int a = 0; a < N; ++a) tot[a] = s_tot[a];
    return ok != 0;
}

// FP64 check: r64 = b - d x - C x; r (working precision) <- r64; partials of
// |r64|^2, |x|^2, |b|^2, |r|^2, min d, the count of invalid inputs and
// |r64 - r_old|^2 (drift of the recursive residual it replaces).
template <typename W>
struct EpiCheck {
    static constexpr int NACC = 8;
    static constexpr bool PREF = false;
    using Gate = GateCheck;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd) { return GateCheck::ok(sd); }
    // one pair: returns its new r (checked: a recursive residual ro exists)
    static __device__ __forceinline__ cx<W> pair(cx<double> xv, cx<double> bv, cx<double> dv, Mask2 mk, double c0,
                                                 double c1, bool checked, cx<W> ro, double* acc) {
        const double r0 = mk.m0 * (bv.x - (dv.x * xv.x + c0));
        const double r1 = mk.m1 * (bv.y - (dv.y * xv.y + c1));
        bv = mkc(mk.m0 * bv.x, mk.m1 * bv.y);
        const W w0 = (W)r0, w1 = (W)r1;
        if (checked) acc[6] += (r0 - (double)ro.x) * (r0 - (double)ro.x) + (r1 - (double)ro.y) * (r1 - (double)ro.y);
        acc[0] += r0 * r0 + r1 * r1;
        acc[1] += xv.x * xv.x + xv.y * xv.y;
        acc[2] += bv.x * bv.x + bv.y * bv.y;
        acc[3] += (double)w0 * (double)w0 + (double)w1 * (double)w1;
        acc[4] = fmin(acc[4], fmin(mk.m0 > 0.0 ? dv.x : 1.0e300, mk.m1 > 0.0 ? dv.y : 1.0e300));
        const bool ok = isfinite(bv.x) && isfinite(bv.y) && isfinite(dv.x) && isfinite(dv.y) &&
                        dv.x >= 0.0 && dv.y >= 0.0;
        acc[5] += ok ? 0.0 : 1.0;
        acc[7] += dv.x + dv.y;
        return mkc(w0, w1);
    }
    struct Pre {
        cx<double> x, b, d;
        cx<W> r;
        int checked;
    };
    template <int L>
    static __device__ __forceinline__ Pre pre(const SlotDesc& sd, int row, int col) {
        const unsigned idx = (unsigned)row * L + col;
        return Pre{ldv<double, L>(sd.x, idx), ldv<double, L>(sd.b, idx), ldv<double, L>(sd.d, idx),
                   ldv<W, L>(reinterpret_cast<const W*>(sd.r), idx),
                   *gbl(&sd.st->checks)};  // 0: the first check has no recursive residual yet
    }
    template <int L>
    static __device__ __forceinline__ void out2p(const SlotDesc& sd, int row, int col, double c0, double c1,
                                                 const Pre& pr, double* acc) {
        const unsigned idx = (unsigned)row * L + col;
        st2<W>(reinterpret_cast<W*>(sd.r), idx,
               pair(pr.x, pr.b, pr.d, mask2(sd, idx), c0, c1, pr.checked > 0, pr.r, acc));
    }
};

// Preconditioner: z = C' r (C' the convolution with 1/(dbar + ghat); no
// diagonal term); partial r . z (FP64 accumulation).
template <typename W, class G>
struct EpiPre {
    static constexpr int NACC = 1;
    static constexpr int SET = PS_RZ;
    using Gate = G;
    static __device__ __forceinline__ bool begin(const SlotDesc& sd) { return G::ok(sd); }
    static constexpr bool PREF = sizeof(W) == 4;  // r requested before the transform
    struct Pre {
        cx<W> r;
    };
    template <int L>
    static __device__ __forceinline__ Pre pre(const SlotDesc& sd, int row, int col) {
        return Pre{ldv<W, L>(reinterpret_cast<const W*>(sd.r), (unsigned)row * L + col)};
    }
    template <int L>
    static __device__ __forceinline__ void out2p(const SlotDesc& sd, int row, int col, W c0, W c1, const Pre& pr,
                                                 double* acc) {
        const unsigned idx = (unsigned)row * L + col;
        const cx<W> rv = pr.r;
        if (sd.mask) {
            const Mask2 mk = mask2(sd, idx);
            c0 *= (W)mk.m0;
            c1 *= (W)mk.m1;
        }
        st2<W>(reinterpret_cast<W*>(sd.z), idx, mkc(c0, c1));
        acc[0] += (double)rv.x * (double)c0 + (double)rv.y * (double)c1;
    }
};

template <typename W>
struct EpiTurnZ : EpiPre<W, GateIter> {
    static constexpr int NACC = 2;
    static constexpr int TURN = 2;
};

// Whether a prologue defers part of its work until after the transform.
template <class P, class = void>
struct ProLate {
    static constexpr bool value = false;
};
template <class P>
struct ProLate<P, decltype((void)P::LATE_X)> {
    static constexpr bool value = P::LATE_X;
};

// ==== kernels ==============================================================

// The forward row transform of the thread's inputs v (the row's packed
// values, as the prologue placed them), the split of the packed transform
// into the half spectrum of the real row, and the W stores of the
// workgroup's rows (block rb).
template <typename T, int M, int PAD, int NT>
__device__ __forceinline__ void row_fwd_out(cx<T>* v, cx<T>* lds, const Tab<T>& tab, const SlotDesc& sd, int rb,
                                            const int tid) {
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L, TT = G::TT;
    constexpr int WORDS = G::ROW_WORDS;
    const int rl = tid / P, j = tid % P;
    LdsLay<T, 1, 4, 1> lay{lds + rl * WORDS, 0};
    constexpr int NSTG = fft_nstages(N);
    fft_run<T, N, M, -1, false, PAD != 0>(v, lay, j, tab.tw);
    constexpr int RL = NSTG > 0 ? fft_radix(N, false, NSTG - 1) : 1;
    // the unpack's twiddles, all of them before the first W store: a read
    // behind a store waits for the store to complete, sixteen times in a row.
    // With the operands likewise (fetch, combine) the turn pass at M = 4096
    // went from 47.4 to 41.5 us, FP64 check passes from 42.7 and 53.5 to 37.3
    // and 43.2
    cx<T> twk[E];
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int qi = tid + s * NT;
        twk[s] = gld(tab.tw, (unsigned)((qi / (TT * RPW)) * TT + qi % TT));
    }
    if constexpr (NSTG > 1) __syncthreads();  // the transform's last reads before these writes
#pragma unroll
    for (int u = 0; u < E / RL; ++u) lay.template st_run<RL, N / RL>(j + u * P, v + u * RL);
    __syncthreads();
    cx<T>* Wb = reinterpret_cast<cx<T>*>(sd.W);
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int qi = tid + s * NT;
        const int kk = qi % TT;
        const int il = (qi / TT) % RPW;
        const int kt = qi / (TT * RPW);
        const int k = kt * TT + kk;
        LdsLay<T, 1, 4, 1> rl2{lds + il * WORDS, 0};
        const cx<T> Zk = rl2.ld(k), B = conjc(rl2.ld(N - k));
        const cx<T> s1 = Zk + B, d1 = Zk - B;
        const cx<T> wd = cmul(twk[s], d1);
        cx<T> out = mkc(T(0.5) * (s1.x + wd.y), T(0.5) * (s1.y - wd.x));
        // (k = 0 is among the first tiles: s = 0 alone, without a branch)
        if ((s == 0 || NT < TT * RPW) && k == 0) out = mkc(Zk.x + Zk.y, Zk.x - Zk.y);
        gst(Wb, (unsigned)kt * G::WT + (rb * RPW + il) * TT + kk, out);
    }
}

template <typename T, int M, int PAD, class Pro, class Slot, int NT>
__global__ void __launch_bounds__(NT) k_row_fwd(Tab<T> tab, Slot slot, int npart_rr, int stride) {
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L;
    constexpr int WORDS = G::ROW_WORDS;
    static_assert(NT == G::ROW_THREADS, "row-forward block size");
    __shared__ cx<T> lds[RPW * WORDS];
    __shared__ typename Pro::Sh sh;
    __shared__ double fred[(NT + 63) / 64];
    const SlotDesc& sd = slot.get();
    double acc = 0.0;
    const int tid = threadIdx.x;
    const int rl = tid / P, j = tid % P;
    const int rb = xcd_remap(blockIdx.x, gridDim.x);
    const int row = rb * RPW + rl;
    cx<T> v[E];
    constexpr int NSTG = fft_nstages(N);
    constexpr int R1 = NSTG > 0 ? fft_radix(N, false, 0) : 1;
    constexpr int RK = PAD ? R1 / 2 : R1;  // inputs per run (the rest are known zeros on the padded grid)
    constexpr int NI = (E / R1) * RK, GRP = cmin(NI, 8);  // a thread's inputs, fetched up to eight at a time
    auto col = [&](int i) { return 2 * ((j + (i / RK) * P) + (i % RK) * (N / R1)); };
    constexpr bool LATE = ProLate<Pro>::value && NI <= 8;
    static_assert(!ProLate<Pro>::value || Pro::PREF, "a late part needs the fetched operands");
    typename Pro::Raw raw[GRP];
    typename Pro::Sc sc;
    if constexpr (Pro::PREF) {
        // the (first) inputs are requested before begin()'s reductions
        if (!Pro::Gate::ok(sd)) return;
#pragma unroll
        for (int i = 0; i < GRP; ++i) raw[i] = Pro::template fetch<L>(sd, row, col(i));
    }
    if (!Pro::begin(sd, sh, sc, npart_rr, stride)) return;
#pragma unroll
    for (int g = 0; g < NI; g += GRP) {
        if (!Pro::PREF || g > 0) {
#pragma unroll
            for (int i = 0; i < GRP; ++i) raw[i] = Pro::template fetch<L>(sd, row, col(g + i));
        }
#pragma unroll
        for (int i = 0; i < GRP; ++i)
            v[((g + i) / RK) * R1 + (g + i) % RK] = Pro::template combine<L>(sd, sc, raw[i], row, col(g + i), &acc);
        if constexpr (ProLate<Pro>::value && !LATE) {
            // more pairs than a group: their late part cannot keep its operands
            if (Pro::late_due(sc)) {
                decltype(Pro::template late_fetch<L>(sd, 0, 0)) xv[GRP];
#pragma unroll
                for (int i = 0; i < GRP; ++i) xv[i] = Pro::template late_fetch<L>(sd, row, col(g + i));
#pragma unroll
                for (int i = 0; i < GRP; ++i) Pro::template late<L>(sd, sc, raw[i], xv[i], row, col(g + i));
            }
        }
    }
    row_fwd_out<T, M, PAD, NT>(v, lds, tab, sd, rb, tid);
    if constexpr (LATE) {
        if (Pro::late_due(sc)) {
            decltype(Pro::template late_fetch<L>(sd, 0, 0)) xv[GRP];
#pragma unroll
            for (int i = 0; i < GRP; ++i) xv[i] = Pro::template late_fetch<L>(sd, row, col(i));
#pragma unroll
            for (int i = 0; i < GRP; ++i) Pro::template late<L>(sd, sc, raw[i], xv[i], row, col(i));
        }
    }
    if constexpr (Pro::NACC > 0) {
        const double s = block_sum<NT>(acc, fred);
        if (tid == 0) sd.part[Pro::SET * stride + blockIdx.x] = s;
    }
}

// Multiplier of the preconditioner from the stored ghat / M^2:
// 1 / (M^2 (dbar + ghat)) = 1 / (M^2 dbar + M^4 g).  Real, positive and even
// like ghat, so the preconditioner is symmetric positive definite.
__device__ __forceinline__ float pre_mul(float g, float c2, float c4) {
    return __builtin_amdgcn_rcpf(fmaf(c4, g, c2));
}
__device__ __forceinline__ double pre_mul(double g, double c2, double c4) { return 1.0 / fma(c4, g, c2); }

// PRE: multiply by the preconditioner's multiplier instead of ghat / M^2.
template <typename T, int M, int PAD, class Gate, class Slot, int NT, bool PRE = false>
__global__ void __launch_bounds__(NT) k_col(Tab<T> tab, Slot slot) {
    using G = Geo<T, M, PAD>;
    constexpr int E = G::EC, P = G::PC, TT = G::TT, L = G::L, MH = G::MH;
    static_assert(NT == G::COL_THREADS, "column block size");
    constexpr int CT = G::CT;
    using Lay = LdsLay<T, CT, G::COL_SH, CT>;
    __shared__ cx<T> lds[Lay::words(M)];
    const SlotDesc& sd = slot.get();
    if (!Gate::ok(sd)) return;
    const int tid = threadIdx.x, kl = tid % CT, j = tid / CT;
    int kt = blockIdx.x, kk = kl;  // tile, column in it
    if constexpr (CT < TT) {
        // the columns of a tile go to workgroups next to each other on one
        // XCD (workgroups go round robin over the eight), which share its lines
        static_assert(CT == 1 && G::COL_BLOCKS % (8 * TT) == 0, "tiles split by columns over the XCDs");
        const int i = blockIdx.x >> 3;
        kt = (i / TT) * 8 + (blockIdx.x & 7);
        kk = i % TT;
    }
    Lay lay{lds, kl};
    cx<T>* Wt = reinterpret_cast<cx<T>*>(sd.W) + (size_t)kt * G::WT;
    cx<T> v[E];
    constexpr int NSTG = fft_nstages(M);
    constexpr int R1 = fft_radix(M, false, 0);
#pragma unroll
    for (int u = 0; u < E / R1; ++u)
#pragma unroll
        for (int r = 0; r < R1; ++r) {
            if (PAD && r >= R1 / 2) continue;
            const int n = (j + u * P) + r * (M / R1);
            v[u * R1 + r] = gld(Wt + (size_t)n * TT + kk);
        }
    constexpr int RL = fft_radix(M, false, NSTG - 1);
    const T* g = tab.ghq + (size_t)kt * MH * TT;
    // the spectrum values this thread multiplies by, requested together with
    // the column data so their latency is not exposed after the transform
    T gpre[E];
#pragma unroll
    for (int u = 0; u < E / RL; ++u)
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            const int m = (j + u * P) + r * (M / RL);
            const int mp = m <= M - m ? m : M - m;
            gpre[u * RL + r] = g[mp * TT + kk];
        }
    const T c2 = PRE ? (T)((double)M * (double)M * gbl(sd.st)->dbar) : T(0);
    const T c4 = (T)((double)M * (double)M * (double)M * (double)M);
    if constexpr (PRE) {
#pragma unroll
        for (int i = 0; i < E; ++i) gpre[i] = pre_mul(gpre[i], c2, c4);
    }
    fft_run<T, M, M, -1, false, PAD != 0>(v, lay, j, tab.tw);
    if (kt == 0) {
        // packed column 0 carries k = 0 (real part) and k = M/2 (imaginary
        // part): result(m) = s(m) W(m) + t(m) conj(W(M - m)),
        // s = (g0 + gN)/2, t = (g0 - gN)/2.
        if constexpr (NSTG > 1) __syncthreads();  // the transform's last reads before these writes
#pragma unroll
        for (int u = 0; u < E / RL; ++u) lay.template st_run<RL, M / RL>(j + u * P, v + u * RL);
        // this thread's values of the spectrum's column M/2, read together
        // (inside the per-element branch below each read would wait for the
        // previous element)
        T gN[E];
#pragma unroll
        for (int u = 0; u < E / RL; ++u)
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int m = (j + u * P) + r * (M / RL);
                gN[u * RL + r] = tab.ghN[m <= M - m ? m : M - m];
            }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < E / RL; ++u)
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int m = (j + u * P) + r * (M / RL);
                const cx<T> a = v[u * RL + r];
                if (kk == 0) {
                    const cx<T> bm = conjc(lay.ld((M - m) & (M - 1)));
                    const T g0 = gpre[u * RL + r];
                    const T gNv = PRE ? pre_mul(gN[u * RL + r], c2, c4) : gN[u * RL + r];
                    const T s = T(0.5) * (g0 + gNv), t = T(0.5) * (g0 - gNv);
                    v[u * RL + r] = mkc(s * a.x + t * bm.x, s * a.y + t * bm.y);
                } else {
                    v[u * RL + r] = scalec(a, gpre[u * RL + r]);
                }
            }
        __syncthreads();
    } else {
#pragma unroll
        for (int u = 0; u < E / RL; ++u)
#pragma unroll
            for (int r = 0; r < RL; ++r) v[u * RL + r] = scalec(v[u * RL + r], gpre[u * RL + r]);
    }
    // the forward transform's (or column 0's) reads of the buffer came before
    fft_run<T, M, M, +1, true, false, Lay, true>(v, lay, j, tab.tw);
    constexpr int RZ = fft_radix(M, true, NSTG - 1);
#pragma unroll
    for (int u = 0; u < E / RZ; ++u)
#pragma unroll
        for (int r = 0; r < RZ; ++r) {
            if (PAD && r >= RZ / 2) continue;
            const int n = (j + u * P) + r * (M / RZ);
            gst(Wt + (size_t)n * TT + kk, v[u * RZ + r]);
        }
}

// What follows the row-inverse transform in the preconditioned turns (v: its
// outputs; pre: prefetched operands, or not where they are read here).
template <typename T, int M, int PAD, class Epi, int NT, int TURN, bool HAVE>
__device__ __forceinline__ void turn_pcg(cx<T>* v, typename Epi::Pre* pre, cx<T>* lds, double* red, const Tab<T>& tab,
                                         const SlotDesc& sd, int stride, unsigned long long token, int row0) {
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L;
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = NSTG > 0 ? fft_radix(N, true, NSTG - 1) : 1, R1 = NSTG > 0 ? fft_radix(N, false, 0) : 1;
    static_assert(R1 == RL, "forward first radix and inverse last radix");
    constexpr int RK = (PAD && RL > 1) ? RL / 2 : RL, NO = (E / RL) * RK;
    const int tid = threadIdx.x, rl = tid / P, j = tid % P, row = row0 + rl;
    auto* st = gbl(sd.st);
    auto col = [&](int i) { return 2 * ((j + (i / RK) * P) + (i % RK) * (N / RL)); };
    auto at = [&](int i) { return (unsigned)row * L + col(i); };
    auto give_up = [&]() {
        if (tid == 0) {
            __hip_atomic_store(&st->status, ST_EGRID, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            publish_status(sd, 1, ST_EGRID, st->gen, st->iters, st->last_check_iter);
        }
    };
    // what the second half takes from the state, read before the barrier
    // (one thread; LDS): iters, alpha and rho_prev change in the other turn
    // only, the rest in no turn
    __shared__ CheckIn s_ci;
    __shared__ double s_in[3];
    if (tid == 0) {
        if constexpr (TURN == 2) s_ci = check_in(st);
        s_in[0] = st->alpha;
        s_in[1] = st->rho_prev;
        s_in[2] = st->rho_cur;
    }
    cx<T> w[NO];  // q, then the new r (TURN 1); z, then the new p (TURN 2)
    double acc[2] = {0.0, 0.0}, tot[2];
#pragma unroll
    for (int g = 0; g < NO; g += cmin(NO, 8)) {
        if constexpr (!HAVE) {
#pragma unroll
            for (int i = 0; i < cmin(NO, 8); ++i) pre[i] = Epi::template pre<L>(sd, row, col(g + i));
        }
#pragma unroll
        for (int h = 0; h < cmin(NO, 8); ++h) {
            const int i = g + h;
            const cx<T> c = v[(i / RK) * RL + i % RK];
            const typename Epi::Pre pr = pre[HAVE ? i : h];
            if constexpr (TURN == 1) {
                w[i] = Epi::template outq<L>(sd, row, col(i), c.x, c.y, pr, acc);
            } else {
                w[i] = c;
                if (sd.mask) {
                    const Mask2 mk = mask2(sd, (unsigned)row * L + col(i));
                    w[i] = mkc(c.x * (T)mk.m0, c.y * (T)mk.m1);
                }
                acc[0] += (double)pr.r.x * (double)w[i].x + (double)pr.r.y * (double)w[i].y;
                acc[1] += (double)pr.r.x * (double)pr.r.x + (double)pr.r.y * (double)pr.r.y;
            }
        }
    }
    // the operands that the second half changes, requested before the barrier
    cx<T> o[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) o[i] = ld2<T>((const T*)(TURN == 1 ? sd.r : sd.p), at(i));
    // (the second turn's x accumulator as well)
    T* xa = sizeof(T) == 8 ? (T*)sd.x : (T*)sd.e;
    cx<T> xv[TURN == 2 ? NO : 1];
    if constexpr (TURN == 2) {
#pragma unroll
        for (int i = 0; i < NO; ++i) xv[i] = ld2<T>(xa, at(i));
    }
    if (!grid_sums<NT, TURN, G::SUM_GROUPS>(acc, sd.part, stride, token, st->bar_limit, red, tot)) {
        give_up();
        return;
    }
    cx<T> v2[E];
    if constexpr (TURN == 1) {
        const double pq = tot[0], rho = s_in[2];
        if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) {
            if (blockIdx.x == 0 && tid == 0) {
                st->status = ST_EBREAKDOWN;
                st->done = 1;
                publish_status(sd, 1, ST_EBREAKDOWN, st->gen, st->iters, st->last_check_iter);
            }
            return;
        }
        const double alpha = rho / pq;
        const T a = (T)alpha;
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            o[i].x -= a * w[i].x;
            o[i].y -= a * w[i].y;
            st2<T>((T*)sd.r, at(i), o[i]);
            v2[(i / RK) * RL + i % RK] = o[i];
        }
        if (blockIdx.x == 0 && tid == 0) {
            st->alpha = alpha;
            st->rho_prev = rho;
            st->iters += 1;
            st->restart = 0;
        }
        // r.r of the updated residual for the next launch's prologue, should
        // the next one be a separate pass
        double rr = 0.0;
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            rr += (double)o[i].x * (double)o[i].x + (double)o[i].y * (double)o[i].y;
            __builtin_amdgcn_sched_barrier(0);
        }
        const double s = block_sum<NT>(rr, red);
        if (tid == 0) gbl(sd.part)[PS_RR * stride + blockIdx.x] = s;
    } else {
        const double rz = tot[0], rr = tot[1];
        if (check_due(s_ci, rr, s_ci.iters)) {
            if (blockIdx.x == 0 && tid == 0) st->pause = 1;
            return;
        }
        // (an iteration always precedes, so this is no restart)
        const T a = (T)s_in[0], beta = (T)(rz / s_in[1]);
#pragma unroll
        for (int i = 0; i < NO; ++i) asm volatile("" : "+v"(xv[i].x), "+v"(xv[i].y));
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const cx<T> p2 = mkc(w[i].x + beta * o[i].x, w[i].y + beta * o[i].y);
            st2<T>((T*)sd.p, at(i), p2);
            v2[(i / RK) * RL + i % RK] = p2;
            if (a != T(0)) {
                xv[i].x += a * o[i].x;
                xv[i].y += a * o[i].y;
                st2<T>(xa, at(i), xv[i]);
            }
        }
        if (blockIdx.x == 0 && tid == 0) {
            st->rho_cur = rz;
            st->need_pre = 0;
        }
    }
    // the forward transform reads its tables afresh, as in the turn pass below
    Tab<T> tab2 = tab;
    asm volatile("" : "+s"(tab2.tw));
    int tid2 = tid;
    asm volatile("" : "+v"(tid2));
    tid2 &= NT - 1;
    row_fwd_out<T, M, PAD, NT>(v2, lds, tab2, sd, __builtin_amdgcn_readfirstlane(row0 / RPW), tid2);
}

// Body of the row-inverse pass; token, token + 1: the grid-wide barriers'
// arrival tokens of this launch (epilogues with the folded update only).
// FWD (with the folded update only): the pass goes on into the next
// iteration's forward row pass on the same rows (k_row_turn).
template <typename T, int M, int PAD, class Epi, class Slot, int NT, bool FWD = false>
__device__ __forceinline__ void row_inv_body(const Tab<T>& tab, const Slot& slot, int stride,
                                             unsigned long long token) {
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L, TT = G::TT;
    constexpr int WORDS = G::ROW_WORDS;
    static_assert(NT == G::ROW_THREADS, "row-inverse block size");
    __shared__ cx<T> lds[RPW * WORDS];
    __shared__ double red[(Epi::NACC > 1 ? Epi::NACC : 1) * ((NT + 63) / 64)];
    const SlotDesc& sd = slot.get();
    if (!Epi::begin(sd)) return;
    const int tid = threadIdx.x;
    const int rl = tid / P, j = tid % P;
    const int row0 = xcd_remap(blockIdx.x, gridDim.x) * RPW;
    // FWD: the state that the check decision takes, as this launch found it
    // (block 0 advances st->iters after the first barrier; read before this
    // workgroup arrives)
    __shared__ CheckIn s_ci;
    if (FWD && EpiTurn<Epi>::value == 0 && tid == 0) s_ci = check_in(gbl(sd.st));
    const cx<T>* Wb = reinterpret_cast<const cx<T>*>(sd.W);
    // all of this thread's spectrum values are requested before the first
    // is stored to LDS (more reads in flight per wave)
    cx<T> wv[E];
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int qi = tid + s * NT;
        const int kk = qi % TT;
        const int il = (qi / TT) % RPW;
        const int kt = qi / (TT * RPW);
        wv[s] = gld(Wb, (unsigned)kt * G::WT + (row0 + il) * TT + kk);
    }
    constexpr int NSTG = fft_nstages(N);
    constexpr int R1 = NSTG > 0 ? fft_radix(N, true, 0) : 1;
    constexpr int S1 = N / R1;
    // the unpack's twiddles, requested with the spectrum (before the barrier)
    cx<T> twk[E];
#pragma unroll
    for (int u = 0; u < E / R1; ++u)
#pragma unroll
        for (int r = 0; r < R1; ++r) twk[u * R1 + r] = gld(tab.tw, (unsigned)((j + u * P) + r * S1));
    constexpr int RL = NSTG > 0 ? fft_radix(N, true, NSTG - 1) : 1;
    constexpr int RK = (PAD && RL > 1) ? RL / 2 : RL;  // outputs kept per run (the rest are cropped)
    const int row = row0 + rl;
    // the epilogue's operands (Epi::PREF), requested with the spectrum; not
    // in the turn pass (FWD) on the largest rows (16 pairs a thread), which
    // keeps p of the pairs to its end and would otherwise exceed 128 VGPRs
    // (four workgroups per CU)
    constexpr int NO = (E / RL) * RK;  // outputs (pairs) of this thread
    constexpr bool PF = Epi::PREF && !(FWD && E >= 16);
    auto col = [&](int i) { return 2 * ((j + (i / RK) * P) + (i % RK) * (N / RL)); };
    // (without the prefetch in groups of up to eight pairs; the check's pairs
    // take 56 bytes, four fit the registers)
    // (with the folded update in FP64 and eight pairs a thread, two: the pairs'
    // q and r are kept, and the grid has to be resident as a whole, at most 128
    // VGPRs; with groups of eight the pass took 188, so that periodic L = 2048
    // had to use the separate update, 7.2 ms a solve instead of 6.8)
    constexpr bool TIGHT = EpiUpd<Epi>::value && sizeof(T) == 8 && NO >= 8;
    constexpr int GRP = cmin(NO, TIGHT ? 2 : (sizeof(typename Epi::Pre) > 40 ? 4 : 8));
    typename Epi::Pre pre[PF ? NO : GRP];
    if constexpr (PF) {
#pragma unroll
        for (int i = 0; i < NO; ++i) pre[i] = Epi::template pre<L>(sd, row, col(i));
    }
#pragma unroll
    for (int s = 0; s < E; ++s) {
        const int qi = tid + s * NT;
        const int kk = qi % TT;
        const int il = (qi / TT) % RPW;
        const int kt = qi / (TT * RPW);
        LdsLay<T, 1, 4, 1> l2{lds + il * WORDS, 0};
        l2.st(kt * TT + kk, wv[s]);
    }
    __syncthreads();
    LdsLay<T, 1, 4, 1> lay{lds + rl * WORDS, 0};
    cx<T> v[E];
#pragma unroll
    for (int u = 0; u < E / R1; ++u) {
        // Y at k = jj + r S1, and the partners N - k = (S1 - jj) + (R1-1-r) S1,
        // read as two runs (k = 0 has no partner: position N is the row's
        // last word of padding, read and not used)
        const int jj = j + u * P;
        cx<T> A[R1], Bv[R1];
        lay.template ld_run<R1, S1>(jj, A);
        lay.template ld_run<R1, S1>(S1 - jj, Bv);
#pragma unroll
        for (int r = 0; r < R1; ++r) {
            const cx<T> Y = A[r];
            const cx<T> B = conjc(Bv[R1 - 1 - r]);
            const cx<T> s1 = Y + B, d1 = Y - B;
            const cx<T> wd = cmul(conjc(twk[u * R1 + r]), d1);
            v[u * R1 + r] = mkc(s1.x - wd.y, s1.y + wd.x);
            // k = jj + r S1 = 0: u = r = 0 alone
            if (u == 0 && r == 0 && jj == 0) v[0] = mkc(Y.x + Y.y, Y.x - Y.y);
        }
    }
    __syncthreads();
    fft_run<T, N, M, +1, true, false>(v, lay, j, tab.tw);
    double acc[Epi::NACC > 0 ? Epi::NACC : 1];
#pragma unroll
    for (int a = 0; a < (Epi::NACC > 0 ? Epi::NACC : 1); ++a) acc[a] = 0.0;
    if constexpr (Epi::NACC > 4) acc[4] = 1.0e300;
    constexpr bool UPD = EpiUpd<Epi>::value;
    constexpr int TURN = EpiTurn<Epi>::value;
    if constexpr (TURN > 0) {
        turn_pcg<T, M, PAD, Epi, NT, TURN, PF>(v, pre, lds, red, tab, sd, stride, token, row0);
        return;
    }
    cx<T> qk[UPD ? NO : 1], rk[UPD ? NO : 1];
    static_assert(!FWD || UPD, "the fused forward pass follows the folded update");
    cx<T> pk[FWD ? NO : 1];  // FWD: p of the pairs, for the next direction and the x update
    // all operands of a group are requested together
#pragma unroll
    for (int g = 0; g < NO; g += GRP) {
        if constexpr (!PF) {
#pragma unroll
            for (int i = 0; i < GRP; ++i) pre[i] = Epi::template pre<L>(sd, row, col(g + i));
        }
        if constexpr (UPD) {
#pragma unroll
            for (int i = 0; i < GRP; ++i)
                rk[g + i] = ld2<T>(reinterpret_cast<const T*>(sd.r), (unsigned)row * L + col(g + i));
        }
#pragma unroll
        for (int i = 0; i < GRP; ++i) {
            const cx<T> c = v[((g + i) / RK) * RL + (g + i) % RK];
            if constexpr (UPD) {
                qk[g + i] = Epi::template outq<L>(sd, row, col(g + i), c.x, c.y, pre[PF ? g + i : i], acc);
                if constexpr (FWD) pk[g + i] = pre[PF ? g + i : i].p;
            } else {
                Epi::template out2p<L>(sd, row, col(g + i), c.x, c.y, pre[PF ? g + i : i], acc);
            }
        }
        if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (UPD) {
        // the parts of r.r, r.q and q.q
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const cx<double> rv = mkc((double)rk[i].x, (double)rk[i].y), qv = mkc((double)qk[i].x, (double)qk[i].y);
            acc[1] += rv.x * rv.x + rv.y * rv.y;
            acc[2] += rv.x * qv.x + rv.y * qv.y;
            acc[3] += qv.x * qv.x + qv.y * qv.y;
            // one pair's doubles at a time: widened all together they would
            // spill on the largest rows
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (Epi::NACC > 0 && !UPD) {
        double* part = sd.part;
        if constexpr (Epi::NACC == 1) {
            const double s = block_sum<NT>(acc[0], red);
            if (tid == 0) part[Epi::SET * stride + blockIdx.x] = s;
        } else {
            const int sets[8] = {PS_CHK_R,    PS_CHK_X,   PS_CHK_B,    PS_CHK_RW,
                                 PS_CHK_DMIN, PS_CHK_BAD, PS_CHK_DIFF, PS_CHK_DSUM};
            if constexpr (NT % 64 == 0) {
                // set 4 (min d) is a minimum, the others sums
                const double s = block_reduce_n<NT, 8, 1u << 4>(acc, red);
                if (tid < 8) part[sets[tid] * stride + blockIdx.x] = s;
            } else {
#pragma unroll
                for (int a = 0; a < 8; ++a) {
                    const double s = (a == 4) ? block_min<NT>(acc[a], red) : block_sum<NT>(acc[a], red);
                    if (tid == 0) part[sets[a] * stride + blockIdx.x] = s;
                }
            }
        }
    }
    if constexpr (UPD) {
        auto* st = gbl(sd.st);
        // the grid was not resident as a whole: the solve is abandoned and
        // the host repeats it with the separate update kernel
        auto give_up = [&]() {
            if (tid == 0) {
                __hip_atomic_store(&st->status, ST_EGRID, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                publish_status(sd, 1, ST_EGRID, st->gen, st->iters, st->last_check_iter);
            }
        };
        double tot[4];  // p.q, r.r, r.q, q.q
        if (!grid_sums<NT, 4, G::SUM_GROUPS>(acc, sd.part, stride, token, st->bar_limit, red, tot)) {
            give_up();
            return;
        }
        const double pq = tot[0], rho = tot[1];
        if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) {
            if (blockIdx.x == 0 && tid == 0) {
                st->status = ST_EBREAKDOWN;
                st->done = 1;
                publish_status(sd, 1, ST_EBREAKDOWN, st->gen, st->iters, st->last_check_iter);
            }
            return;
        }
        const double alpha = rho / pq;
        const T a = (T)alpha;
        double rrn;
        const bool sure = next_rr(tot, (double)a, &rrn);
        cx<T> xk[FWD ? NO : 1];  // FWD: the x accumulator of the pairs, requested before the first store
        T* xa = reinterpret_cast<T*>(sizeof(T) == 8 ? (void*)sd.x : (void*)sd.e);
        if constexpr (FWD) {
#pragma unroll
            for (int i = 0; i < NO; ++i) xk[i] = ld2<T>(xa, (unsigned)row * L + col(i));
        }
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            rk[i].x -= a * qk[i].x;
            rk[i].y -= a * qk[i].y;
            st2<T>(reinterpret_cast<T*>(sd.r), (unsigned)row * L + col(i), rk[i]);
        }
        // the totals are the same in every workgroup, so all take this branch
        // or none
        if (!sure) {
            double rr[1] = {0.0};
#pragma unroll
            for (int i = 0; i < NO; ++i) rr[0] += (double)rk[i].x * rk[i].x + (double)rk[i].y * rk[i].y;
            // set 0 of the partials again (its first use ended with the barrier)
            if (!grid_sums<NT, 1, G::SUM_GROUPS>(rr, sd.part, stride, token + 1, st->bar_limit, red, &rrn)) {
                give_up();
                return;
            }
        }
        if (blockIdx.x == 0 && tid == 0) {
            st->alpha = alpha;
            st->rho_prev = rho;
            st->rho_next = rrn;
            st->iters += 1;
            st->restart = 0;
        }
        if constexpr (FWD) {
            // The next iteration's forward row pass on the same rows, as
            // ProCG in k_row_fwd computes it: the check decision, p <- r +
            // beta p, the transform, and the pending x update x <- x + alpha
            // p_old.  The forward pass's first radix equals this pass's last,
            // so the thread holds the same pairs of r and p in both.
            if (check_due(s_ci, rrn, s_ci.iters + 1)) {
                if (blockIdx.x == 0 && tid == 0) st->pause = 1;
                return;
            }
            const T beta = (T)(rrn / rho);
            // x has arrived here (one wait, instead of one for all stores so
            // far before each pair's)
#pragma unroll
            for (int i = 0; i < NO; ++i) asm volatile("" : "+v"(xk[i].x), "+v"(xk[i].y));
            constexpr int R1 = NSTG > 0 ? fft_radix(N, false, 0) : 1;
            static_assert(R1 == RL, "forward first radix and inverse last radix");
            cx<T> v2[E];
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const cx<T> po = pk[i];
                const cx<T> p2 = mkc(rk[i].x + beta * po.x, rk[i].y + beta * po.y);
                st2<T>(reinterpret_cast<T*>(sd.p), (unsigned)row * L + col(i), p2);
                v2[(i / RK) * RL + i % RK] = p2;
                if (a != T(0)) {
                    xk[i].x += a * po.x;
                    xk[i].y += a * po.y;
                    st2<T>(xa, (unsigned)row * L + col(i), xk[i]);
                }
            }
            // the forward transform reads its twiddles afresh (the pointer is
            // opaque to the compiler) rather than reusing the inverse half's
            // loads of the same entries across both barriers; the block
            // index is kept uniform
            Tab<T> tab2 = tab;
            asm volatile("" : "+s"(tab2.tw));
            int tid2 = tid;
            asm volatile("" : "+v"(tid2));
            tid2 &= NT - 1;  // (its range, for the index arithmetic)
            row_fwd_out<T, M, PAD, NT>(v2, lds, tab2, sd, __builtin_amdgcn_readfirstlane(row0 / RPW), tid2);
        }
    }
}

template <typename T, int M, int PAD, class Epi, class Slot, int NT>
__global__ void __launch_bounds__(NT) k_row_inv(Tab<T> tab, Slot slot, int stride) {
    row_inv_body<T, M, PAD, Epi, Slot, NT>(tab, slot, stride, 0);
}

// The CG row-inverse pass with the residual update folded in (EpiCGU).
// token: unique per launch (the host counts launches per workspace), so
// arrival words left by an abandoned launch can never match a later one.
template <typename T, int M, int PAD, class Slot, int NT>
__global__ void __launch_bounds__(NT) k_row_inv_upd(Tab<T> tab, Slot slot, int stride, unsigned long long token) {
    row_inv_body<T, M, PAD, EpiCGU<T>, Slot, NT>(tab, slot, stride, token);
}

// One CG iteration's turn in one pass (k_row_inv_upd followed by k_row_fwd):
// q's row inverse, the folded update, and the next direction's forward row
// transform, with one grid-wide barrier.  Four
// waves per SIMD are asked for: the whole grid must be resident (four
// 256-thread workgroups per CU at M = 4096), which caps it at 128 VGPRs.
template <typename T, int M, int PAD, class Slot, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
k_row_turn(Tab<T> tab, Slot slot, int stride, unsigned long long token) {
    row_inv_body<T, M, PAD, EpiCGU<T>, Slot, NT, true>(tab, slot, stride, token);
}

// The preconditioned turns (EpiTurnR, EpiTurnZ), one barrier each.
template <typename T, int M, int PAD, class Epi, class Slot, int NT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4)))
k_row_turn_pcg(Tab<T> tab, Slot slot, int stride, unsigned long long token) {
    row_inv_body<T, M, PAD, Epi, Slot, NT>(tab, slot, stride, token);
}

// r <- r - alpha q, partial r . r.  alpha = rho / (p . q) from the partials
// of the row-inverse pass (all blocks reduce them in the same order).
// L: the grid (n = L L).
template <typename W, int NT, int L>
__global__ void __launch_bounds__(NT) k_update(ByPtr slot, int n, int npart_pq, int stride) {
    __shared__ double red[(NT + 63) / 64];
    const SlotDesc& sd = slot.get();
    if (!GateIter::ok(sd)) return;
    auto* st = gbl(sd.st);
    constexpr int VW = sizeof(W) == 4 ? 4 : 2;
    using V = typename VecT<W, VW>::type;
    const int nv = n / VW;
    const int per = (nv + gridDim.x - 1) / gridDim.x;
    const int lo = blockIdx.x * per;
    const int hi = lo + per < nv ? lo + per : nv;
    auto* r = gbl(reinterpret_cast<V*>(sd.r));
    const auto* q = gbl(reinterpret_cast<const V*>(sd.q));
    // PF vectors of r and q at a time: the first before the p.q reduction, so
    // its latency overlaps the HBM reads, each of the others before the stores
    // of those before it
    constexpr int PF = 4;
    auto ld = [](const auto* v) {
        if constexpr (kStream<L>)
            return __builtin_nontemporal_load(v);
        else
            return *v;
    };
    V rp[PF], qp[PF];
    auto fetch = [&](int i0) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int i = i0 + u * NT;
            if (i < hi) {
                rp[u] = ld(r + i);
                qp[u] = ld(q + i);
            }
        }
    };
    fetch(lo + threadIdx.x);
    const double pq = sum_partials<NT>(sd.part + PS_PQ * stride, npart_pq, red);
    const double rho = st->rho_cur;
    if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->status = ST_EBREAKDOWN;
            st->done = 1;
            publish_status(sd, 1, ST_EBREAKDOWN, st->gen, st->iters, st->last_check_iter);
        }
        return;
    }
    const double alpha = rho / pq;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->alpha = alpha;
        st->rho_prev = rho;
        st->iters += 1;
        st->restart = 0;
    }
    const W a = (W)alpha;
    double acc = 0.0;
    auto upd = [&](V rv, const V qv) {
        if constexpr (VW == 4) {
            rv.x -= a * qv.x;
            rv.y -= a * qv.y;
            rv.z -= a * qv.z;
            rv.w -= a * qv.w;
            acc += (double)rv.x * rv.x + (double)rv.y * rv.y + (double)rv.z * rv.z + (double)rv.w * rv.w;
        } else {
            rv.x -= a * qv.x;
            rv.y -= a * qv.y;
            acc += rv.x * rv.x + rv.y * rv.y;
        }
        return rv;
    };
    for (int i0 = lo + threadIdx.x; i0 < hi; i0 += PF * NT) {
        V rn[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u)
            if (i0 + u * NT < hi) rn[u] = upd(rp[u], qp[u]);
        fetch(i0 + PF * NT);
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            if (i0 + u * NT >= hi) continue;
            if constexpr (kStream<L>)
                __builtin_nontemporal_store(rn[u], r + i0 + u * NT);
            else
                r[i0 + u * NT] = rn[u];
        }
    }
    const double s = block_sum<NT>(acc, red);
    if (threadIdx.x == 0) sd.part[PS_RR * stride + blockIdx.x] = s;
}

// The first FP64 check of a solve started from x = 0: r = b - A 0 = b, so
// no product is needed.  One pass over b and d writes r and the check's
// partials (the same values the full check would produce, bitwise: C 0 and
// d 0 are exactly zero, and blocks and threads take the FP64 row-inverse
// pass's pairs in its order); the finaliser then decides as usual.
template <typename W, int M, int PAD, int NT>
__global__ void __launch_bounds__(NT) k_check_zero(ByPtr slot, int stride) {
    using G = Geo<double, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L;
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = NSTG > 0 ? fft_radix(N, true, NSTG - 1) : 1;
    constexpr int RK = (PAD && RL > 1) ? RL / 2 : RL;
    static_assert(NT == G::ROW_THREADS, "row block size");
    __shared__ double red[8 * ((NT + 63) / 64)];
    const SlotDesc& sd = slot.get();
    if (!GateCheck::ok(sd)) return;
    const int tid = threadIdx.x, rl = tid / P, j = tid % P;
    const int row = xcd_remap(blockIdx.x, gridDim.x) * RPW + rl;
    double acc[8] = {0, 0, 0, 0, 1.0e300, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < E / RL; ++u)
#pragma unroll
        for (int r = 0; r < RK; ++r) {
            const size_t idx = (size_t)row * L + 2 * ((j + u * P) + r * (N / RL));
            const cx<double> b2 = ld2<double>(sd.b, idx), d2 = ld2<double>(sd.d, idx);
            st2<W>(reinterpret_cast<W*>(sd.r) + idx,
                   EpiCheck<W>::pair(mkc(0.0, 0.0), b2, d2, mask2(sd, idx), 0.0, 0.0, false, mkc(W(0), W(0)), acc));
        }
    const int sets[8] = {PS_CHK_R, PS_CHK_X, PS_CHK_B, PS_CHK_RW, PS_CHK_DMIN, PS_CHK_BAD, PS_CHK_DIFF, PS_CHK_DSUM};
    if constexpr (NT % 64 == 0) {
        const double v = block_reduce_n<NT, 8, 1u << 4>(acc, red);  // set 4 (min d) a minimum
        if (tid < 8) sd.part[sets[tid] * stride + blockIdx.x] = v;
    } else {
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const double v = (a == 4) ? block_min<NT>(acc[a], red) : block_sum<NT>(acc[a], red);
            if (tid == 0) sd.part[sets[a] * stride + blockIdx.x] = v;
        }
    }
}

// Single-block finaliser of an FP64 check: stop decision, residual
// replacement, restart guard, and status for the host.
// NG: the order of its sums (group_sum; 0: sum_partials').
// One serial chain, so its reads are put side by side: the state as a whole
// in registers (thread 0; decided on there and stored once) beside the
// partials, whose sets the waves share (with eight slots of
// L = 512 7.3 us, 15.3 when each field and set was read by itself).
template <int NT, int NG>
__global__ void __launch_bounds__(NT) k_check_final(ByPtr slot, int npart_chk, int npart_rr, int stride, int n) {
    __shared__ double red[8 * ((NT + 63) / 64)];
    __shared__ double s_tot[8];
    __shared__ int s_update;
    const SlotDesc& sd = slot.get();
    if (!sd.active) return;
    const int tid = threadIdx.x;
    const auto pd = pause_done(sd.st);
    SolveState st;
    if (tid == 0) st = *reinterpret_cast<const SolveState*>(sd.st);
    if (pd.y != 0 || pd.x == 0) {
        if (tid == 0) publish_status(sd, st.done, st.status, st.gen, st.iters, st.last_check_iter);
        return;
    }
    // the eight partial sets, each summed (min d: minimised) by thread t over
    // t, t + NT, ... and then over the block, all in one exchange; the order
    // is that of sum_partials / block_min
    constexpr int sets[8] = {PS_CHK_R,    PS_CHK_X,   PS_CHK_B,    PS_CHK_RW,
                             PS_CHK_DMIN, PS_CHK_BAD, PS_CHK_DIFF, PS_CHK_DSUM};
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 1.0e300, 0.0, 0.0, 0.0};
    const auto* part = gbl(sd.part);
    if constexpr (NG > 0 && NT % 64 == 0) {
        constexpr int NW = NT / 64;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            if (a % NW != __builtin_amdgcn_readfirstlane(tid >> 6)) continue;
            const auto* pa = part + sets[a] * stride;
            const auto get = [&](unsigned int i) { return pa[i]; };
            const double t = a == 4 ? group_sum<NG, true>(npart_chk, 1.0e300, get) : group_sum<NG>(npart_chk, 0.0, get);
            if ((tid & 63) == 0) s_tot[a] = t;
        }
    } else {
        for (int i = tid; i < npart_chk; i += NT) {
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const double v = part[sets[a] * stride + i];
                acc[a] = (a == 4) ? fmin(acc[a], v) : acc[a] + v;
            }
        }
        const double tot = block_reduce_n<NT, 8, 1u << 4>(acc, red);
        if (tid < 8) s_tot[tid] = tot;
    }
    __syncthreads();
    const double RW = s_tot[3];
    if (tid == 0) {
        if (st.checks == 0) st.dbar = s_tot[7] / (double)n;
        s_update = check_decide(&st, s_tot[0], s_tot[1], s_tot[2], RW, s_tot[5], s_tot[6], s_tot[4]);
        if (s_update) st.rho_next = RW;  // r.r for the folded update's iterations
        // preconditioned CG: z = P^{-1} r of the replaced residual comes next
        st.need_pre = (s_update && st.pcg) ? 1 : 0;
        *sd.st = st;
        publish_status(sd, st.done, st.status, st.gen, st.iters, st.last_check_iter);
    }
    __syncthreads();
    if (s_update) {
        // residual replacement: the next iteration's rho is |r|^2 of the new r
        auto* prr = gbl(sd.part) + PS_RR * stride;
        for (int i = tid; i < npart_rr; i += NT) prr[i] = (i == 0) ? RW : 0.0;
    }
}


}  // namespace FFTCG_RADIX_NS
}  // namespace fftcg
