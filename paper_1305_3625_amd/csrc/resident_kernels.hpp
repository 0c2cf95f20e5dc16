// The resident kernel: a single solve, checks and all, in one launch.
//
// On mid-sized grids an iteration's passes take a few microseconds each, most
// of it latency: the launch, the chain of loads (slot descriptor, state, then
// data), reading the vectors that the previous pass has just written.  Here
// every workgroup owns RPW rows and CW columns for the whole launch and keeps
// its parts of r, p, z, the x accumulator and d and its columns' spectrum in
// registers; only the half spectrum W crosses workgroups, and workgroups meet
// three times per iteration:
//   rows forward -> W | columns of W in place | rows inverse of W, the sums
//   p.q, r.r, r.q and q.q over the grid -> alpha, r, beta, p.
// With the preconditioner, z = P^-1 r is three more such phases; an FP64 check
// is the same phases in FP64.  A row or column of up to 64 threads is
// transformed inside one wave, without barriers.  The arithmetic and its
// order are those of the passes (EpiCGU, ProCG; iter_pcg; the check), so the
// iterates are bitwise the same; every workgroup takes the decisions of
// check_decide and check_due by itself from the same sums, on its own copy of
// the state.
//
// What bounds it: the meetings.  On one XCD a meeting takes 0.7 us and the
// sums 1.4 us; an iteration takes 6.2 us at padded M = 256 in FP32 (16 us as
// passes) and 5.9 us at periodic M = 64 in FP64.  Over all XCDs, at padded
// M = 1024, a meeting takes 2.1 to 3 us and the sums 2.8 us of 14.2 us (FP32)
// or 18.7 us (FP64; 27 us as passes).  (Iterations alone, without checks:
// device times of solves that stop a few iterations apart.)
//
// W moves between workgroups inside the launch.  Its accesses go past the
// CUs' L1 caches, and past the L2 caches where they must reach other XCDs
// (gst_all, gld_all), and no cache-wide write-back or invalidation is needed;
// a workgroup waits for its stores to complete before it tells the others.
#pragma once
#include "fftcg_kernels.hpp"

namespace fftcg {
inline namespace FFTCG_RADIX_NS {

template <typename T, int M, int PAD>
struct RGeo {
    using G = Geo<T, M, PAD>;
    static constexpr int L = G::L, N = G::N, RPW = G::RPW, NB = G::ROW_BLOCKS;
    static constexpr int RT = G::ROW_THREADS;  // threads of the row phases
    static constexpr int CW = N / cmin(N, NB);  // columns per workgroup
    // a row (column) whose threads fit a wave is transformed without barriers
    static constexpr bool WVR = G::PR <= 64, WVC = G::PC <= 64;
    // threads of the workgroup: as many as its columns use, except where the
    // row transforms need barriers of all threads; there each thread takes U
    // columns in turn
    static constexpr int NT = WVR ? cmax(RT, CW * G::PC) : RT;
    static constexpr int U = cmax(1, CW * G::PC / NT);
    static constexpr int CU = cmax(1, CW / U);  // columns in flight
    using ColLay = LdsLay<T, 1, 4, 1>;
    static constexpr int CWORDS = ColLay::words(M);
    static constexpr int LDS_WORDS = cmax(RPW * G::ROW_WORDS, CU * CWORDS);
    // waves exchange W rows by themselves where their runs still fill 64 bytes
    static constexpr int RWV = cmax(1, 64 / G::PR);  // rows per wave
    static constexpr bool WROW = WVR && RWV * CW * (int)sizeof(cx<T>) >= 64;
    // workgroups on one XCD (ONEX), or spread over all of them in NG groups,
    // one per XCD
    static constexpr int NG = cmax(1, G::SUM_GROUPS), GM = NB / NG;  // groups, members of a group
    static constexpr bool ONEX = NG == 1;
    static constexpr bool OK = G::SUM_GROUPS > 0 && NB % NG == 0 && GM <= 64 && RT % 64 == 0 && N % NB == 0 && CW * G::PC == U * NT && CU * U == CW && RPW >= 2 &&
                               (size_t)LDS_WORDS * sizeof(cx<T>) <= 140 * 1024;
};

// The thread's index, opaque to the compiler, taken afresh in every phase.
// What the phases derive from it (LDS and W offsets, twiddles, the meetings'
// addresses) does not change from one iteration to the next, and the compiler
// would compute it all once before the loop: several hundred values that end
// in accumulation registers and in scratch memory, whose reads wait behind
// the stores to W.  Afresh, against kept (twiddles with it where they fit),
// us per iteration: M = 64 periodic FP32 7.0, was 7.5; padded L = 128 FP32
// 7.3, was 7.6; M = 256 periodic FP32 8.6, was 9.4; M = 512 periodic FP32
// 15.6, was 18.6, FP64 17.5, was 22.0; M = 1024 periodic FP32 18.8, was 20.2;
// padded L = 512 the same.
__device__ __forceinline__ int fresh_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t & 1023;
}

// ---- accesses between workgroups ----------------------------------------------
// Loads that miss the CU's L1 and see what any XCD has stored with scope
// agent, and what the own XCD has stored at all.  Stores: ALL for every XCD
// (written through), else for the own XCD (they end in its L2, from which the
// loads above are served: 0.2 us from one workgroup to another, against 0.4
// to 0.5 us through the memory side).
template <typename T>
__device__ __forceinline__ cx<T> gld_all(const cx<T>* base, unsigned idx) {
    using U = unsigned long long;
    const auto* w = at_byte<const U>(const_cast<cx<T>*>(base), idx * (unsigned)sizeof(cx<T>));
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(cx<T>, __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    } else {
        const U a = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const U b = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return mkc(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
    }
}
template <bool ALL>
__device__ __forceinline__ void word_put(unsigned long long* p, unsigned long long v) {
    if constexpr (ALL)
        __hip_atomic_store(gbl(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(gbl(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ unsigned long long word_get(const unsigned long long* p) {
    return __hip_atomic_load(gbl(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool ALL, typename T>
__device__ __forceinline__ void gst_all(cx<T>* base, unsigned idx, cx<T> c) {
    using U = unsigned long long;
    auto* w = at_byte<U>(base, idx * (unsigned)sizeof(cx<T>));
    if constexpr (!ALL) {
        gst(base, idx, c);
    } else if constexpr (sizeof(T) == 4) {
        __hip_atomic_store(w, __builtin_bit_cast(U, c), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        __hip_atomic_store(w, __builtin_bit_cast(U, c.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(w + 1, __builtin_bit_cast(U, c.y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The XCD that the workgroup runs on.
__device__ __forceinline__ unsigned xcc_id() {
    unsigned x;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(x));
    return x;
}

// ---- meetings of all workgroups -------------------------------------------------
// The workgroups of one XCD form a group (workgroups go to the XCDs round
// robin; hello() checks it).  Members tell their group's leader through the
// XCD's L2; with more than one group the eight leaders tell each other through
// words that every XCD sees, and then their members.  With 256 workgroups,
// polling by every workgroup of every other's word took 4 us per meeting, and
// polling of the leaders' line by everybody 2.1 us.
// One wave per workgroup polls.  Waits are bounded (`limit` ticks of the
// 100 MHz clock, a thousand times an ordinary wait): a grid that is not
// resident as a whole cannot meet, and the launch then ends.
constexpr unsigned long long kEmpty = 0x7ff8dead5e77e1edull;  // a NaN no sum is stored as

template <int NG_, int GM_>
struct Meet {
    static constexpr int NG = NG_, GM = GM_, NB = NG * GM;
    static constexpr int GS = GM < 16 ? 16 : GM;  // words of a group: lines of its own
    static constexpr bool ALL = NG > 1;
    static_assert(NG == 1 || NG == 8, "one group, or one per XCD");
    static_assert(GM <= 64, "a wave polls a group");
    unsigned long long* base;  // the workspace's words (kMeetWords)
    long long limit;
    int g, i;  // this workgroup: group, member (0 leads)

    // layout in words; sets 0-4 of partial sums belong to the iterations,
    // 5-12 (and 3 with the preconditioner) to the checks
    static constexpr int SETS = 13;
    static constexpr int FLAG = 0, REL = FLAG + NG * GS, HELLO = REL + 16, HREL = HELLO + NG * GS, PART = HREL + 16;
    static constexpr int PART_SET = NG * GS, OUT = PART + 2 * SETS * PART_SET, GO = OUT + 2 * SETS * 16;
    static constexpr int FIN = GO + NG * 16, WORDS = FIN + NG * 32;
    static_assert(WORDS <= kMeetWords, "the words fit");
    __device__ __forceinline__ unsigned long long* part(int ring, int set) const {
        return base + PART + (ring * SETS + set) * PART_SET + g * GS;
    }
    __device__ __forceinline__ unsigned long long* out(int ring, int set) const {
        return base + OUT + (ring * SETS + set) * 16;
    }
    __device__ __forceinline__ unsigned long long* fin(int ring, int set) const {
        return base + FIN + g * 32 + ring * 16 + set;
    }
    template <class F>
    __device__ __forceinline__ bool wave_wait(F done) const {
        const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
        while (!__all(done())) {
            if ((long long)(__builtin_amdgcn_s_memrealtime() - t0) > limit) return false;
            __builtin_amdgcn_s_sleep(1);
        }
        return true;
    }
    // by the workgroup's first wave: arrival with `token`, and the wait until
    // all have arrived (tokens only grow)
    __device__ __forceinline__ bool arrive(unsigned long long token) const {
        const int lane = fresh_tid() & 63;
        if (lane == 0) word_put<false>(base + FLAG + g * GS + i, token);
        auto members = [&] { return lane >= GM || word_get(base + FLAG + g * GS + lane) >= token; };
        if constexpr (NG == 1) {
            return wave_wait(members);
        } else if (i == 0) {
            if (!wave_wait(members)) return false;
            if (lane == 0) word_put<true>(base + REL + g, token);
            if (!wave_wait([&] { return lane >= NG || word_get(base + REL + lane) >= token; })) return false;
            if (lane == 0) word_put<false>(base + GO + g * 16, token);
            return true;
        } else {
            return wave_wait([&] { return word_get(base + GO + g * 16) >= token; });
        }
    }
    // All workgroups' stores to W are complete and seen by gld_all after.
    __device__ __forceinline__ bool meet(unsigned long long token, int* s_ok) const {
        drain();
        __syncthreads();
        if (threadIdx.x < 64) {
            const bool ok = arrive(token);
            if (threadIdx.x == 0) *s_ok = ok;
        }
        __syncthreads();
        return *s_ok != 0;
    }
    // The first meeting of a launch, safe wherever the workgroups run: every
    // member must share its leader's XCD, and no two may be the same member
    // (on one XCD the members are those that run there: two that both were
    // there in every eight would be; the later one leaves, and the one that is
    // missing for it ends the launch).
    __device__ __forceinline__ bool hello(unsigned long long token, int* s_ok) const {
        const unsigned long long mine = token * 256 + xcc_id() % 255;
        drain();
        __syncthreads();
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            bool ok = true;
            if (lane == 0) {
                if constexpr (NG == 1)
                    ok = __hip_atomic_exchange(gbl(base + HELLO + i), mine, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) / 256 != token;
                else
                    word_put<true>(base + HELLO + g * GS + i, mine);
            }
            ok = __all(ok);
            if (ok && i == 0) {
                ok = wave_wait([&] { return lane >= GM || word_get(base + HELLO + g * GS + lane) / 256 == token; });
                const bool same = __all(lane >= GM || word_get(base + HELLO + g * GS + lane) == mine);
                if (ok && lane == 0) word_put<true>(base + HREL + g, token * 256 + (same ? 0 : 255));
            }
            unsigned long long w = 0;
            ok = ok && wave_wait([&] {
                     w = lane < NG ? word_get(base + HREL + lane) : token * 256;
                     return w / 256 == token;
                 });
            ok = ok && __all(w == token * 256);
            if (lane == 0) *s_ok = ok;
        }
        __syncthreads();
        return *s_ok != 0;
    }
    // Empties this workgroup's words of the sets in `mask`, in a ring half.
    __device__ __forceinline__ void empty(int ring, unsigned mask) const {
        const int set = fresh_tid();
        if (set < SETS && ((mask >> set) & 1u)) {
            word_put<false>(part(ring, set) + i, kEmpty);
            if (ALL && i == 0) {
                word_put<true>(out(ring, set) + g, kEmpty);
                word_put<false>(fin(ring, set), kEmpty);
            }
        }
    }
    static __device__ __forceinline__ unsigned long long bits(double v) {
        const unsigned long long w = __builtin_bit_cast(unsigned long long, v);
        return w == kEmpty ? w ^ 1 : w;
    }
    // The sums (minimum where bit a of MINMASK is set) of N per-thread values
    // (of the RT row threads) over the grid, in every thread.  The words hold
    // the values themselves, kEmpty until they arrive, so no separate arrival
    // is needed; halves of the ring are used in turn and emptied between two
    // meetings that every reader of their last use has passed.  Order (as
    // grid_sums): the workgroup's partial, the members of a group as a wave
    // sum, the groups as a tree.  sh: N * RT / 64 doubles, s_tot: N.
    template <int RT, int N, unsigned MINMASK = 0u>
    __device__ __forceinline__ bool sums(const double* acc, int set0, int ring, double* sh, double* s_tot, int* s_ok,
                                         double* tot) const {
        constexpr int NW = RT / 64;
        const int tid = fresh_tid(), lane = tid & 63;
        auto is_min = [](int a) { return ((MINMASK >> a) & 1u) != 0; };
        if (tid < RT) {
            double w[N];
#pragma unroll
            for (int a = 0; a < N; ++a) w[a] = is_min(a) ? wave_min(acc[a]) : wave_sum(acc[a]);
            if (lane == 0) {
#pragma unroll
                for (int a = 0; a < N; ++a) sh[a * NW + (tid >> 6)] = w[a];
            }
        }
        if constexpr (NW > 1)
            __syncthreads();
        else
            xsync<true>();
        if (tid < 64) {
            if (lane < N) {
                double r = is_min(lane) ? sh[lane * NW] : 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) r = is_min(lane) ? fmin(r, sh[lane * NW + w]) : r + sh[lane * NW + w];
                word_put<false>(part(ring, set0 + lane) + i, bits(r));
            }
            bool ok = true;
            double t[N];
            if (NG == 1 || i == 0) {
                unsigned long long w[N];
                ok = wave_wait([&] {
                    bool all = true;
#pragma unroll
                    for (int a = 0; a < N; ++a) {
                        w[a] = lane < GM ? word_get(part(ring, set0 + a) + lane) : bits(is_min(a) ? 1.0e300 : 0.0);
                        all &= w[a] != kEmpty;
                    }
                    return all;
                });
#pragma unroll
                for (int a = 0; a < N; ++a) {
                    const double v = __builtin_bit_cast(double, w[a]);
                    t[a] = is_min(a) ? wave_min(v) : wave_sum(v);
                }
                if (ALL && ok && lane == 0) {
#pragma unroll
                    for (int a = 0; a < N; ++a) word_put<true>(out(ring, set0 + a) + g, bits(t[a]));
                }
            }
            if constexpr (NG > 1) {
                if (i == 0) {
                    // the leaders exchange their groups' sums: row q of the
                    // wave takes set a0 + q, its eight groups twice
#pragma unroll
                    for (int a0 = 0; a0 < N; a0 += 4) {
                        const int a = a0 + (lane >> 4) < N ? a0 + (lane >> 4) : a0;
                        unsigned long long w = 0;
                        ok = ok && wave_wait([&] {
                                 w = word_get(out(ring, set0 + a) + (lane & 7));
                                 return w != kEmpty;
                             });
                        const double u = __builtin_bit_cast(double, w);
                        const double v = is_min(a) ? wave_min<4>(u) : group_tree(u);
                        if ((lane & 15) == 0 && a0 + (lane >> 4) < N) {
                            if (ok) word_put<false>(fin(ring, set0 + a), bits(v));
                            s_tot[a] = v;
                        }
                    }
                } else {
                    unsigned long long w = 0;
                    ok = wave_wait([&] {
                        w = lane < N ? word_get(fin(ring, set0 + lane)) : 0ull;
                        return w != kEmpty;
                    });
                    if (lane < N) s_tot[lane] = __builtin_bit_cast(double, w);
                }
            } else if (lane == 0) {
#pragma unroll
                for (int a = 0; a < N; ++a) s_tot[a] = t[a];
            }
            if (lane == 0) *s_ok = ok;
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < N; ++a) tot[a] = s_tot[a];
        // (s_tot, s_ok and sh are written again only behind a later barrier)
        return *s_ok != 0;
    }
};

// ---- the phases -------------------------------------------------------------
// Offset of column k = kt CW + kk of row i in W: tiles of CW columns.
template <typename T, int M, int PAD>
__device__ __forceinline__ unsigned w_at(int kt, int i, int kk) {
    using R = RGeo<T, M, PAD>;
    return ((unsigned)kt * R::L + i) * R::CW + kk;
}
// Element s of the thread's share of the W rows that its exchange group (the
// wave, or the workgroup) owns: local row il, column tile kt, column kk in it.
template <typename T, int M, int PAD>
struct RowShare {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    static constexpr int THREADS = R::WROW ? 64 : R::NT, ROWS = R::WROW ? R::RWV : R::RPW;
    static constexpr int COUNT = ROWS * G::N / THREADS;
    int il, kt, kk;
    __device__ __forceinline__ RowShare(int tid, int s) {
        const int qi = (R::WROW ? (tid & 63) : tid) + s * THREADS;
        kk = qi % R::CW;
        il = (qi / R::CW) % ROWS + (R::WROW ? (tid >> 6) * R::RWV : 0);
        kt = qi / (R::CW * ROWS);
    }
};

// Forward transforms of the workgroup's rows to W (row_fwd_out's arithmetic).
// Called by the row threads' waves only where rows stay in waves, else by all.
template <typename T, int M, int PAD>
__device__ __forceinline__ void res_rows_fwd(cx<T>* v, cx<T>* lds, const cx<T>* tw, cx<T>* Wb, int rb) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, WORDS = G::ROW_WORDS;
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = fft_radix(N, false, NSTG - 1);
    const int tid = fresh_tid() & (R::NT - 1);
    const int rl = tid / P, j = tid % P;
    // the unpack's twiddles, before the first store to W (a read behind a
    // store waits for it to complete)
    constexpr int CNT = RowShare<T, M, PAD>::COUNT;
    cx<T> twk[CNT];
    if (!R::WVR || tid < R::RT) {
        const LdsLay<T, 1, 4, 1> lay{lds + rl * WORDS, 0};
        fft_run<T, N, M, -1, false, PAD != 0, LdsLay<T, 1, 4, 1>, false, R::WVR>(v, lay, j, tw);
        if constexpr (NSTG > 1) xsync<R::WVR>();
#pragma unroll
        for (int u = 0; u < E / RL; ++u) lay.template st_run<RL, N / RL>(j + u * P, v + u * RL);
    }
    if (!R::WROW || tid < R::RT) {
#pragma unroll
        for (int s = 0; s < CNT; ++s) {
            const RowShare<T, M, PAD> e(tid, s);
            twk[s] = gld(tw + (e.kt * R::CW + e.kk));
        }
    }
    xsync<R::WROW>();
    if (!R::WROW || tid < R::RT) {
#pragma unroll
        for (int s = 0; s < CNT; ++s) {
            const RowShare<T, M, PAD> e(tid, s);
            const int k = e.kt * R::CW + e.kk;
            const LdsLay<T, 1, 4, 1> lay{lds + e.il * WORDS, 0};
            const cx<T> Zk = lay.ld(k), B = conjc(lay.ld(N - k));
            const cx<T> s1 = Zk + B, d1 = Zk - B;
            const cx<T> wd = cmul(twk[s], d1);
            cx<T> out = mkc(T(0.5) * (s1.x + wd.y), T(0.5) * (s1.y - wd.x));
            if (k == 0) out = mkc(Zk.x + Zk.y, Zk.x - Zk.y);
            gst_all<!R::ONEX>(Wb, w_at<T, M, PAD>(e.kt, rb * R::RPW + e.il, e.kk), out);
        }
    }
}

// The column that a thread works on (u-th in turn) and its index within it.
template <typename T, int M, int PAD>
struct ColOf {
    using R = RGeo<T, M, PAD>;
    int kk, j, cl;  // column of the workgroup, thread of the column, LDS region
    __device__ __forceinline__ ColOf(int tid, int u) {
        constexpr int P = R::G::PC;
        cl = R::WVC ? tid / P : tid % R::CU;
        j = R::WVC ? tid % P : tid / R::CU;
        kk = u * R::CU + cl;
    }
};
// The spectrum values of a thread's columns (kept in registers for a launch).
template <typename T, int M, int PAD>
struct ResSpec {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    T g[R::U][G::EC], gN[G::EC];  // gN: the column M/2, for packed column 0
    __device__ __forceinline__ void load(const Tab<T>& tab, int blk) {
        constexpr int E = G::EC, P = G::PC, RL = fft_radix(M, false, fft_nstages(M) - 1), TT = G::TT;
#pragma unroll
        for (int u = 0; u < R::U; ++u) {
            const ColOf<T, M, PAD> c(threadIdx.x, u);
            const int k = blk * R::CW + c.kk;
            const T* gc = tab.ghq + (size_t)(k / TT) * G::MH * TT + k % TT;
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int m = (c.j + (i / RL) * P) + (i % RL) * (M / RL);
                const int mp = m <= M - m ? m : M - m;
                g[u][i] = *gbl(gc + mp * TT);
                if (u == 0) gN[i] = *gbl(tab.ghN + mp);
            }
        }
    }
};

// The workgroup's columns of W in place (k_col's arithmetic): forward
// transform, times ghat / M^2, inverse transform.  All values are requested
// before the first transform.
// PRE: times the preconditioner's multiplier (c2, c4: pre_mul's) instead.
template <typename T, int M, int PAD, bool PRE>
__device__ __forceinline__ void res_cols(cx<T>* lds, const cx<T>* tw, const ResSpec<T, M, PAD>& sp, T c2, T c4, cx<T>* Wb,
                                         int blk) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    using Lay = typename R::ColLay;
    constexpr int E = G::EC, P = G::PC;
    const int tid = fresh_tid() & (R::NT - 1);
    constexpr int NSTG = fft_nstages(M);
    constexpr int R1 = fft_radix(M, false, 0), RL = fft_radix(M, false, NSTG - 1), RZ = fft_radix(M, true, NSTG - 1);
    auto mul = [&](T g) {
        if constexpr (PRE)
            return pre_mul(g, c2, c4);
        else
            return g;
    };
    cx<T> v[R::U][E];
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
        const ColOf<T, M, PAD> c(tid, u);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if (PAD && i % R1 >= R1 / 2) continue;
            const int n = (c.j + (i / R1) * P) + (i % R1) * (M / R1);
            v[u][i] = gld_all(Wb, w_at<T, M, PAD>(blk, n, c.kk));
        }
    }
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
        const ColOf<T, M, PAD> c(tid, u);
        const Lay lay{lds + c.cl * R::CWORDS, 0};
        // (LEAD: the column before may still be read)
        fft_run<T, M, M, -1, false, PAD != 0, Lay, (R::U > 1), R::WVC>(v[u], lay, c.j, tw);
        if (u == 0 && blk == 0) {
            // packed column 0 (k = 0 and k = M/2), as in k_col
            if constexpr (NSTG > 1) xsync<R::WVC>();
#pragma unroll
            for (int i = 0; i < E / RL; ++i) lay.template st_run<RL, M / RL>(c.j + i * P, v[u] + i * RL);
            xsync<R::WVC>();
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const int m = (c.j + (i / RL) * P) + (i % RL) * (M / RL);
                const cx<T> a = v[u][i];
                const cx<T> bm = conjc(lay.ld((M - m) & (M - 1)));
                const T g0 = mul(sp.g[u][i]), gN = mul(sp.gN[i]);
                const T s = T(0.5) * (g0 + gN), t = T(0.5) * (g0 - gN);
                v[u][i] = c.kk == 0 ? mkc(s * a.x + t * bm.x, s * a.y + t * bm.y) : scalec(a, g0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i) v[u][i] = scalec(v[u][i], mul(sp.g[u][i]));
        }
        fft_run<T, M, M, +1, true, false, Lay, true, R::WVC>(v[u], lay, c.j, tw);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if (PAD && i % RZ >= RZ / 2) continue;
            const int n = (c.j + (i / RZ) * P) + (i % RZ) * (M / RZ);
            gst_all<!R::ONEX>(Wb, w_at<T, M, PAD>(blk, n, c.kk), v[u][i]);
        }
    }
}

// Inverse transforms of the workgroup's rows (row_inv_body's arithmetic):
// v[u RL + r] holds the pair at n = (j + u P) + r N / RL.  Called as
// res_rows_fwd.
template <typename T, int M, int PAD>
__device__ __forceinline__ void res_rows_inv(cx<T>* v, cx<T>* lds, const cx<T>* tw, const cx<T>* Wb, int rb) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, WORDS = G::ROW_WORDS;
    constexpr int R1 = fft_radix(N, true, 0), S1 = N / R1;
    constexpr int COUNT = RowShare<T, M, PAD>::COUNT;
    const int tid = fresh_tid() & (R::NT - 1);
    const int rl = tid / P, j = tid % P;
    if (!R::WROW || tid < R::RT) {
        cx<T> wv[COUNT];
#pragma unroll
        for (int s = 0; s < COUNT; ++s) {
            const RowShare<T, M, PAD> e(tid, s);
            wv[s] = gld_all(Wb, w_at<T, M, PAD>(e.kt, rb * R::RPW + e.il, e.kk));
        }
#pragma unroll
        for (int s = 0; s < COUNT; ++s) {
            const RowShare<T, M, PAD> e(tid, s);
            const LdsLay<T, 1, 4, 1> l2{lds + e.il * WORDS, 0};
            l2.st(e.kt * R::CW + e.kk, wv[s]);
        }
    }
    xsync<R::WROW>();
    if (!R::WVR || tid < R::RT) {
        const LdsLay<T, 1, 4, 1> lay{lds + rl * WORDS, 0};
#pragma unroll
        for (int u = 0; u < E / R1; ++u) {
            const int jj = j + u * P;
            cx<T> A[R1], Bv[R1];
            lay.template ld_run<R1, S1>(jj, A);
            lay.template ld_run<R1, S1>(S1 - jj, Bv);
#pragma unroll
            for (int r = 0; r < R1; ++r) {
                const int k = jj + r * S1;
                const cx<T> Y = A[r];
                const cx<T> B = conjc(Bv[R1 - 1 - r]);
                const cx<T> s1 = Y + B, d1 = Y - B;
                const cx<T> wd = cmul(conjc(gld(tw + k)), d1);
                v[u * R1 + r] = mkc(s1.x - wd.y, s1.y + wd.x);
                if (k == 0) v[u * R1 + r] = mkc(Y.x + Y.y, Y.x - Y.y);
            }
        }
        xsync<R::WVR>();
        fft_run<T, N, M, +1, true, false, LdsLay<T, 1, 4, 1>, false, R::WVR>(v, lay, j, tw);
    }
}

// One product: the transform of the rows' pairs v (as the forward transform
// takes them) to the rows of C v (as res_rows_inv leaves them).
template <typename T, int M, int PAD, bool PRE, class MT>
__device__ __forceinline__ bool res_product(cx<T>* v, cx<T>* lds, const cx<T>* tw, const ResSpec<T, M, PAD>& sp, T c2, T c4,
                                            cx<T>* Wb, int rb, int blk, const MT& all, unsigned long long token,
                                            int* s_ok) {
    res_rows_fwd<T, M, PAD>(v, lds, tw, Wb, rb);
    if (!all.meet(token, s_ok)) return false;
    res_cols<T, M, PAD, PRE>(lds, tw, sp, c2, c4, Wb, blk);
    if (!all.meet(token + 1, s_ok)) return false;
    res_rows_inv<T, M, PAD>(v, lds, tw, Wb, rb);
    return true;
}

// ---- the kernel ---------------------------------------------------------------
struct ResArgs {
    SlotDesc sd;
    unsigned long long* words;  // kMeetWords
    unsigned long long token;   // the first of the launch's meetings' tokens
    int xcd;                    // the XCD to run on (one-XCD grids)
    int gen;                    // the launch's mark, which the state it leaves carries
    int K;                      // iterations of this launch at most
    int first;                  // the solve begins: state from the argument, no vectors yet
    int zero;                   // ... from x = 0
};

// A meeting gave up: the solve is abandoned and the host repeats it.
__device__ __forceinline__ void res_give_up(const SlotDesc& sd) {
    if (threadIdx.x == 0) {
        __hip_atomic_store(&sd.st->status, ST_EGRID, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&sd.st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The end of a launch: a last meeting, after which every workgroup's results
// are stored, and then the first workgroup stores the state.  It alone may
// also report that this meeting gave up: another one that does so may be
// late only to see that all have arrived, and would then write into the state
// that the first one stores (a solve stopped at its launch's last iteration
// could be left marked as done, with its status of a solve that goes on).
template <class MT>
__device__ __forceinline__ void res_end(const MT& all, unsigned long long token, int* s_ok, int blk,
                                        const SlotDesc& sd, const SolveState& st) {
    if (!all.meet(token, s_ok)) {
        if (blk == 0) res_give_up(sd);
        return;
    }
    if (blk == 0 && threadIdx.x == 0) {
        *sd.st = st;
        publish_status(sd, st.done, st.status, st.gen, st.iters, st.last_check_iter);
    }
}

// A solve, or up to K of its iterations: FP64 checks (check_decide) and CG
// iterations until the solve is done.  Plain CG repeats the folded passes'
// arithmetic, PCG (circulant preconditioner) that of iter_pcg.
template <typename T, int M, int PAD, int NT, bool PCG>
__global__ void __launch_bounds__(NT) k_solve_resident(Tab<T> tab, Tab<double> tab64, ResArgs ra, SolveState init) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    using R64 = RGeo<double, M, PAD>;
    static_assert(R64::NT == NT && R64::NB == R::NB && R64::RT == R::RT && Geo<double, M, PAD>::RPW == G::RPW,
                  "checks run on the same workgroups");
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L, RT = R::RT;
    static_assert(NT == R::NT, "resident block size");
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = fft_radix(N, true, NSTG - 1), RK = PAD ? RL / 2 : RL, NO = (E / RL) * RK;
    static_assert(RL == fft_radix(N, false, 0), "forward first radix and inverse last radix");
    constexpr bool MIXED = sizeof(T) == 4;
    constexpr unsigned ITER_SETS = PCG ? 0x7u : 0x1fu, CHECK_SETS = (0xffu << 5) | (PCG ? 0x8u : 0u);
    __shared__ cx<double> lds64[MIXED ? (R64::LDS_WORDS > (R::LDS_WORDS + 1) / 2 ? R64::LDS_WORDS : (R::LDS_WORDS + 1) / 2)
                                      : R64::LDS_WORDS];
    cx<T>* lds = reinterpret_cast<cx<T>*>(lds64);
    __shared__ double red[8 * (RT / 64)];
    __shared__ double s_tot[8];
    __shared__ int s_ok, s_go;
    __shared__ SolveState st;
    // one-XCD grids: eight times the workgroups are launched, and those that
    // run on the XCD asked for stay: one of every eight, as workgroups go to the
    // XCDs in turn (from which one on depends on the stream's queue, so the
    // XCD is not known from the index)
    if (R::ONEX && (int)xcc_id() != ra.xcd) return;
    const int blk = R::ONEX ? blockIdx.x >> 3 : blockIdx.x;
    const SlotDesc& sd = ra.sd;
    const int tid = threadIdx.x;
    if (tid == 0) {
        st = ra.first ? init : *sd.st;
        st.gen = ra.gen;
    }
    __syncthreads();
    if (st.done) return;
    const bool rows = tid < RT;  // this thread holds a part of a row
    const int rl = tid / P, j = tid % P;
    const int rb = xcd_remap(blk, R::NB);  // as the passes: an XCD's workgroups share lines of W
    const int row = rows ? rb * RPW + rl : 0;
    const Meet<R::NG, R::GM> all{ra.words, st.bar_limit, blk % R::NG, blk / R::NG};
    cx<T>* Wb = reinterpret_cast<cx<T>*>(sd.W);
    unsigned long long token = ra.token;
    auto give_up = [&]() { res_give_up(sd); };
    // all sums' words are empty before the first meeting
    all.empty(0, ITER_SETS | CHECK_SETS);
    all.empty(1, ITER_SETS | CHECK_SETS);
    // (recomputed where they are used, not kept in registers across the loop)
    auto row0 = [&]() {
        unsigned o = (unsigned)row * L + 2 * j;
        asm volatile("" : "+v"(o));
        return o;
    };
    auto rel = [&](int i) { return 2 * ((i / RK) * P + (i % RK) * (N / RL)); };
    // r, p, d, the x accumulator (x itself, or the FP32 correction e), z
    cx<T> r[NO], p[NO], x[NO], d[NO], z[PCG ? NO : 1];
    T* xa = reinterpret_cast<T*>(MIXED ? (void*)sd.e : (void*)sd.x);
    if (rows) {
        const unsigned o = row0();
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const cx<double> d2 = ld2<double>(sd.d + o + rel(i));
            d[i] = mkc((T)d2.x, (T)d2.y);
            r[i] = p[i] = x[i] = mkc(T(0), T(0));
            if constexpr (PCG) z[i] = mkc(T(0), T(0));
            if (!ra.first) {
                r[i] = ld2<T>(reinterpret_cast<const T*>(sd.r) + o + rel(i));
                p[i] = ld2<T>(reinterpret_cast<const T*>(sd.p) + o + rel(i));
                if constexpr (PCG) z[i] = ld2<T>(reinterpret_cast<const T*>(sd.z) + o + rel(i));
            }
            if (MIXED ? !ra.first : !ra.zero) x[i] = ld2<T>(xa + o + rel(i));
        }
    }
    ResSpec<T, M, PAD> sp;
    sp.load(tab, blk);
    if (!all.hello(token, &s_ok)) return give_up();

    // the scalars that change with an iteration are kept in registers (the
    // same in every thread) and put into the state before a check and at the
    // end
    int iters = st.iters, restart = st.restart, k = 0, nchk = 0;
    double alpha = st.alpha, rho_prev = st.rho_prev, rr = st.rho_next, rz = st.rho_cur;
    auto save = [&]() {  // by thread 0
        st.iters = iters;
        st.restart = restart;
        st.alpha = alpha;
        st.rho_prev = rho_prev;
        st.rho_next = rr;
        st.rho_cur = rz;
    };
    // z = P^-1 r and this thread's part of r.z
    auto precondition = [&](double* acc) {
        cx<T> v[E];
#pragma unroll
        for (int i = 0; i < NO; ++i) v[(i / RK) * RL + i % RK] = r[i];
        const T c2 = (T)((double)M * (double)M * st.dbar);
        const T c4 = (T)((double)M * (double)M * (double)M * (double)M);
        if (!res_product<T, M, PAD, true>(v, lds, tab.tw, sp, c2, c4, Wb, rb, blk, all, token, &s_ok)) return false;
        token += 2;
        if (rows) {
            const unsigned o = row0();
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                cx<T> c = v[(i / RK) * RL + i % RK];
                if (sd.mask) {
                    const Mask2 mk = mask2(sd, o + rel(i));
                    c.x *= (T)mk.m0;
                    c.y *= (T)mk.m1;
                }
                if constexpr (PCG) z[i] = c;
                *acc += (double)r[i].x * (double)c.x + (double)r[i].y * (double)c.y;
            }
        }
        return true;
    };
    for (;;) {
        if (__builtin_expect(st.pause, 0)) {
            // ---- FP64 check: x <- x + e + alpha p, e <- 0, r64 = b - A x ----
            double acc[8] = {0, 0, 0, 0, 1.0e300, 0, 0, 0}, tot[8];
            const bool zero = ra.first && ra.zero && st.checks == 0;  // x = 0: r = b, no product
            constexpr int E64 = Geo<double, M, PAD>::ER;
            static_assert(E64 == E, "the same pairs");
            cx<double> v[E], xv[NO];
            if (rows) {
                const unsigned o = row0();
                if constexpr (MIXED) {
#pragma unroll
                    for (int i = 0; i < NO; ++i) xv[i] = zero ? mkc(0.0, 0.0) : ld2<double>(sd.x + o + rel(i));
                }
#pragma unroll
                for (int i = 0; i < NO; ++i) {
                    if constexpr (MIXED) {
                        xv[i].x += (double)x[i].x;
                        xv[i].y += (double)x[i].y;
                    } else {
                        xv[i] = mkc((double)x[i].x, (double)x[i].y);
                    }
                    if (alpha != 0.0) {
                        xv[i].x += alpha * (double)p[i].x;
                        xv[i].y += alpha * (double)p[i].y;
                    }
                    const Mask2 mk = mask2(sd, o + rel(i));
                    xv[i].x *= mk.m0;
                    xv[i].y *= mk.m1;
                    if constexpr (MIXED) {
                        st2<double>(sd.x + o + rel(i), xv[i]);
                        x[i] = mkc(T(0), T(0));
                    } else {
                        x[i] = mkc((T)xv[i].x, (T)xv[i].y);
                    }
                    v[(i / RK) * RL + i % RK] = xv[i];
                }
            }
            if (!zero) {
                Tab<double> t64 = tab64;
                asm volatile("" : "+s"(t64.tw), "+s"(t64.ghq), "+s"(t64.ghN));
                ResSpec<double, M, PAD> sp64;
                sp64.load(t64, blk);
                if (!res_product<double, M, PAD, false>(v, lds64, t64.tw, sp64, 0.0, 0.0,
                                                        reinterpret_cast<cx<double>*>(sd.W), rb, blk, all, token, &s_ok))
                    return give_up();
                token += 2;
            }
            if (rows) {
                const unsigned o = row0();
#pragma unroll
                for (int i = 0; i < NO; ++i) {
                    const cx<double> c = zero ? mkc(0.0, 0.0) : v[(i / RK) * RL + i % RK];
                    r[i] = EpiCheck<T>::pair(xv[i], ld2<double>(sd.b + o + rel(i)), ld2<double>(sd.d + o + rel(i)),
                                             mask2(sd, o + rel(i)), c.x, c.y, st.checks > 0, r[i], acc);
                }
            }
            if (!all.template sums<RT, 8, 1u << 4>(acc, 5, nchk & 1, red, s_tot, &s_ok, tot)) return give_up();
            if (tid == 0) {
                save();
                if (st.checks == 0) st.dbar = tot[7] / (double)(L * L);
                s_go = check_decide(&st, tot[0], tot[1], tot[2], tot[3], tot[5], tot[6], tot[4]);
            }
            __syncthreads();
            if (!s_go) break;
            rr = tot[3];  // |r|^2 of the replaced residual
            alpha = 0.0;
            restart = st.restart;
            if constexpr (PCG) {
                double a1[1] = {0.0};
                if (!precondition(a1)) return give_up();
                if (!all.template sums<RT, 1>(a1, 3, nchk & 1, red, s_tot, &s_ok, &rz)) return give_up();
            }
            ++nchk;
            all.empty(nchk & 1, CHECK_SETS);
        }
        if (k >= ra.K) {
            if (tid == 0) save();
            break;
        }
        // ---- one CG iteration ----
        if (__builtin_expect(check_due(&st, rr, iters), 0)) {
            __syncthreads();
            if (tid == 0) {
                save();
                st.pause = 1;
            }
            __syncthreads();
            continue;
        }
        const double rho1 = PCG ? rz : rr;
        {
            // p <- r + beta p (z with the preconditioner), the pending x <- x + a p
            const T a = (T)alpha, beta = (T)(restart ? 0.0 : rho1 / rho_prev);
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const cx<T> po = p[i];
                const cx<T> g = [&] {
                    if constexpr (PCG)
                        return z[i];
                    else
                        return r[i];
                }();
                if (restart) {
                    p[i] = g;
                } else {
                    p[i] = mkc(g.x + beta * po.x, g.y + beta * po.y);
                    if (a != T(0)) {
                        x[i].x += a * po.x;
                        x[i].y += a * po.y;
                    }
                }
            }
        }
        cx<T> v[E];
#pragma unroll
        for (int i = 0; i < NO; ++i) v[(i / RK) * RL + i % RK] = p[i];
        if (!res_product<T, M, PAD, false>(v, lds, tab.tw, sp, T(0), T(0), Wb, rb, blk, all, token, &s_ok))
            return give_up();
        token += 2;
        constexpr int NS = PCG ? 1 : 4;
        double acc[4] = {0.0, 0.0, 0.0, 0.0}, tot[4];
        cx<T> q[NO];
        if (rows) {
            int row1 = row, j1 = j;  // (the mask's offsets, as row0)
            asm volatile("" : "+v"(row1), "+v"(j1));
            auto col1 = [&](int i) { return 2 * ((j1 + (i / RK) * P) + (i % RK) * (N / RL)); };
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const cx<T> c = v[(i / RK) * RL + i % RK];
                typename EpiCGU<T>::Pre pr;
                pr.p = p[i];
                pr.d = d[i];
                q[i] = EpiCGU<T>::template outq<L>(sd, row1, col1(i), c.x, c.y, pr, acc);
            }
            if constexpr (!PCG) {
#pragma unroll
                for (int i = 0; i < NO; ++i) {
                    const cx<double> rv = mkc((double)r[i].x, (double)r[i].y), qv = mkc((double)q[i].x, (double)q[i].y);
                    acc[1] += rv.x * rv.x + rv.y * rv.y;
                    acc[2] += rv.x * qv.x + rv.y * qv.y;
                    acc[3] += qv.x * qv.x + qv.y * qv.y;
                }
            }
        }
        if (!all.template sums<RT, NS>(acc, 0, k & 1, red, s_tot, &s_ok, tot)) return give_up();
        const double rho = PCG ? rz : tot[1];
        if (!(tot[0] > 0.0) || !isfinite(tot[0]) || !isfinite(rho)) {
            __syncthreads();
            if (tid == 0) {
                save();
                st.status = ST_EBREAKDOWN;
                st.done = 1;
            }
            break;
        }
        alpha = rho / tot[0];
        const T a = (T)alpha;
        double accr[2] = {0.0, 0.0};
        if (rows) {
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                r[i].x -= a * q[i].x;
                r[i].y -= a * q[i].y;
                accr[0] += (double)r[i].x * (double)r[i].x + (double)r[i].y * (double)r[i].y;
            }
        }
        if constexpr (PCG) {
            if (!precondition(accr + 1)) return give_up();
            double t2[2];
            if (!all.template sums<RT, 2>(accr, 1, k & 1, red, s_tot, &s_ok, t2)) return give_up();
            rr = t2[0];
            rz = t2[1];
        } else if (__builtin_expect(!next_rr(tot, (double)a, &rr), 0)) {
            __syncthreads();  // readers of the first sums
            if (!all.template sums<RT, 1>(accr, 4, k & 1, red, s_tot, &s_ok, &rr)) return give_up();
        }
        rho_prev = rho;
        restart = 0;
        ++iters;
        ++k;
        // the half that the next iteration uses: everybody has passed this
        // one's meetings, hence the sums that used it last
        all.empty(k & 1, ITER_SETS);
    }
    // the results, and a last meeting: the state says done only when every
    // workgroup has stored its rows
    if (rows) {
        const unsigned o = row0();
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            if (!st.done) {
                st2<T>(reinterpret_cast<T*>(sd.r) + o + rel(i), r[i]);
                st2<T>(reinterpret_cast<T*>(sd.p) + o + rel(i), p[i]);
                if constexpr (PCG) st2<T>(reinterpret_cast<T*>(sd.z) + o + rel(i), z[i]);
            }
            if (!MIXED || !st.done) st2<T>(xa + o + rel(i), x[i]);
        }
    }
    res_end(all, token, &s_ok, blk, sd, st);
}

}  // namespace FFTCG_RADIX_NS
}  // namespace fftcg
