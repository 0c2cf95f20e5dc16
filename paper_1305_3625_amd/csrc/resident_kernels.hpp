// Resident CG: the iterations of a single solve in one kernel.
//
// On mid-sized grids an iteration's passes take a few microseconds each, most
// of it latency: the launch, the chain of loads (slot descriptor, state, then
// data), reading the vectors that the previous pass has just written.  Here
// one launch runs until a check falls due.  Every workgroup owns RPW rows and
// CW columns for the whole launch and keeps its parts of r, p, the x
// accumulator and d, its columns' spectrum and (where they fit) all twiddles
// in registers; only the half spectrum W crosses workgroups, and workgroups
// meet three times per iteration:
//   rows forward -> W | columns of W in place | rows inverse of W, the sums
//   p.q, r.r, r.q and q.q over the grid -> alpha, r, beta, p.
// A row or column of up to 64 threads is transformed inside one wave, without
// barriers.  The arithmetic and its order are those of the folded update's
// passes (EpiCGU, ProCG), so the iterates are bitwise the same.
//
// What bounds it: the meetings.  On one XCD a meeting takes 0.6 us and the
// sums 1.2 us; an iteration takes 5.8 us at padded M = 256 in FP32 (16 us as
// passes) and 5.2 us at periodic M = 64 in FP64.  Over all XCDs, at padded
// M = 1024, a meeting takes 2.3 to 3.5 us and the sums 3.5 us of 15 us (FP32)
// or 19.5 us (FP64; 27 us as passes).
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
    // twiddles in registers for the whole launch, where they fit beside the rest
    static constexpr bool HOIST = (int)sizeof(T) * M <= 4096;
    static constexpr bool OK = G::SUM_GROUPS > 0 && NB % NG == 0 && GM <= 64 && RT % 64 == 0 && N % NB == 0 && CW * G::PC == U * NT && CU * U == CW && RPW >= 2 &&
                               (size_t)LDS_WORDS * sizeof(cx<T>) <= 140 * 1024;
};

// ---- accesses between workgroups ----------------------------------------------
// Loads that miss the CU's L1 and see what any XCD has stored with scope
// agent, and what the own XCD has stored at all.  Stores: ALL for every XCD
// (written through), else for the own XCD (they end in its L2, from which the
// loads above are served: 0.2 us from one workgroup to another, against 0.4
// to 0.5 us through the memory side).
template <typename T>
__device__ __forceinline__ cx<T> gld_all(const cx<T>* p) {
    using U = unsigned long long;
    const auto* w = reinterpret_cast<const U*>(p);
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(cx<T>, __hip_atomic_load(gbl(w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    } else {
        const U a = __hip_atomic_load(gbl(w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const U b = __hip_atomic_load(gbl(w + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
__device__ __forceinline__ void gst_all(cx<T>* p, cx<T> c) {
    using U = unsigned long long;
    if constexpr (!ALL) {
        gst(p, c);
    } else if constexpr (sizeof(T) == 4) {
        word_put<true>(reinterpret_cast<U*>(p), __builtin_bit_cast(U, c));
    } else {
        word_put<true>(reinterpret_cast<U*>(p), __builtin_bit_cast(U, c.x));
        word_put<true>(reinterpret_cast<U*>(p) + 1, __builtin_bit_cast(U, c.y));
    }
}
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- meetings of all workgroups -------------------------------------------------
// The workgroups of one XCD form a group (workgroups go to the XCDs round
// robin; hello() checks it).  Members tell their group's leader through the
// XCD's L2; with more than one group the leaders tell everybody through words
// that every XCD sees, eight in one line.  Polling by every workgroup of
// every other's word instead took 4 us per meeting with 256 workgroups.
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

    // layout in words
    static constexpr int FLAG = 0, REL = FLAG + NG * GS, HELLO = REL + 16, HREL = HELLO + NG * GS, PART = HREL + 16;
    static constexpr int PART_SET = NG * GS, OUT = PART + 2 * 5 * PART_SET, OUT_RING = 5 * 16, WORDS = OUT + 2 * OUT_RING;
    static_assert(WORDS <= kMeetWords, "the words fit");
    __device__ __forceinline__ unsigned long long* part(int ring, int set) const {
        return base + PART + (ring * 5 + set) * PART_SET + g * GS;
    }
    __device__ __forceinline__ unsigned long long* out(int ring, int set) const {
        return base + OUT + ring * OUT_RING + set * 16;
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
        const int lane = threadIdx.x & 63;
        if (lane == 0) word_put<false>(base + FLAG + g * GS + i, token);
        auto members = [&] { return lane >= GM || word_get(base + FLAG + g * GS + lane) >= token; };
        if constexpr (NG == 1) {
            return wave_wait(members);
        } else {
            bool ok = true;
            if (i == 0) {
                ok = wave_wait(members);
                if (ok && lane == 0) word_put<true>(base + REL + g, token);
            }
            return ok && wave_wait([&] { return lane >= NG || word_get(base + REL + lane) >= token; });
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
    // member must share its leader's XCD.
    __device__ __forceinline__ bool hello(unsigned long long token, int* s_ok) const {
        unsigned xcc;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
        const unsigned long long mine = token * 256 + xcc % 255;
        drain();
        __syncthreads();
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            if (lane == 0) word_put<true>(base + HELLO + g * GS + i, mine);
            bool ok = true;
            if (i == 0) {
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
    // Empties this workgroup's words of a ring half.
    __device__ __forceinline__ void empty(int ring) const {
        if (threadIdx.x == 0) {
#pragma unroll
            for (int a = 0; a < 5; ++a) word_put<false>(part(ring, a) + i, kEmpty);
            if (ALL && i == 0) {
#pragma unroll
                for (int a = 0; a < 5; ++a) word_put<true>(out(ring, a) + g, kEmpty);
            }
        }
    }
    static __device__ __forceinline__ unsigned long long bits(double v) {
        const unsigned long long w = __builtin_bit_cast(unsigned long long, v);
        return w == kEmpty ? w ^ 1 : w;
    }
    // The sums of N per-thread values (of the RT row threads) over the grid,
    // in every thread.  The words hold the values themselves, kEmpty until
    // they arrive, so no separate arrival is needed; halves of the ring are
    // used in turn and emptied between two meetings that every reader of
    // their last use has passed.  Order (group_total): the workgroup's
    // partial, the members of a group as a wave sum, the groups as a tree.
    template <int RT, int N>
    __device__ __forceinline__ bool sums(const double* acc, int set0, int ring, double* sh, double* s_tot, int* s_ok,
                                         double* tot) const {
        constexpr int NW = RT / 64;
        const int tid = threadIdx.x, lane = tid & 63;
        if (tid < RT) {
            double w[N];
#pragma unroll
            for (int a = 0; a < N; ++a) w[a] = wave_sum(acc[a]);
            if (lane == 0) {
#pragma unroll
                for (int a = 0; a < N; ++a) {
                    if constexpr (NW == 1)
                        word_put<false>(part(ring, set0 + a) + i, bits(0.0 + w[a]));
                    else
                        sh[a * NW + (tid >> 6)] = w[a];
                }
            }
        }
        if constexpr (NW > 1) __syncthreads();
        if (tid < 64) {
            if constexpr (NW > 1) {
                if (lane < N) {
                    double r = 0.0;
#pragma unroll
                    for (int w = 0; w < NW; ++w) r += sh[lane * NW + w];
                    word_put<false>(part(ring, set0 + lane) + i, bits(r));
                }
            }
            bool ok = true;
            double t[N];
            if (NG == 1 || i == 0) {
                unsigned long long w[N];
                ok = wave_wait([&] {
                    bool all = true;
#pragma unroll
                    for (int a = 0; a < N; ++a) {
                        w[a] = lane < GM ? word_get(part(ring, set0 + a) + lane) : 0ull;
                        all &= w[a] != kEmpty;
                    }
                    return all;
                });
#pragma unroll
                for (int a = 0; a < N; ++a) t[a] = wave_sum(__builtin_bit_cast(double, w[a]));
                if (ALL && ok && lane == 0) {
#pragma unroll
                    for (int a = 0; a < N; ++a) word_put<true>(out(ring, set0 + a) + g, bits(t[a]));
                }
            }
            if constexpr (NG > 1) {
                // row a of the wave takes set a: its eight groups twice
                const int a = (lane >> 4) < N ? lane >> 4 : 0;
                unsigned long long w = 0;
                ok = ok && wave_wait([&] {
                         w = word_get(out(ring, set0 + a) + (lane & 7));
                         return w != kEmpty;
                     });
                const double v = group_tree(__builtin_bit_cast(double, w));
                if ((lane & 15) == 0 && (lane >> 4) < N) s_tot[lane >> 4] = v;
            } else if (lane == 0) {
#pragma unroll
                for (int a = 0; a < N; ++a) s_tot[a] = t[a];
            }
            if (lane == 0) *s_ok = ok;
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < N; ++a) tot[a] = s_tot[a];
        const bool ok = *s_ok != 0;
        // (s_tot, s_ok and sh are written again only behind a later barrier)
        return ok;
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
    __device__ __forceinline__ RowShare(int s) {
        const int qi = (R::WROW ? (threadIdx.x & 63) : threadIdx.x) + s * THREADS;
        kk = qi % R::CW;
        il = (qi / R::CW) % ROWS + (R::WROW ? (threadIdx.x >> 6) * R::RWV : 0);
        kt = qi / (R::CW * ROWS);
    }
};

// Forward transforms of the workgroup's rows to W (row_fwd_out's arithmetic).
// Called by the row threads' waves only where rows stay in waves, else by all.
template <typename T, int M, int PAD, class TW>
__device__ __forceinline__ void res_rows_fwd(cx<T>* v, cx<T>* lds, TW tw, cx<T>* Wb, int rb) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, WORDS = G::ROW_WORDS;
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = fft_radix(N, false, NSTG - 1);
    const int tid = threadIdx.x;
    const int rl = tid / P, j = tid % P;
    if (!R::WVR || tid < R::RT) {
        const LdsLay<T, 1, 4, 1> lay{lds + rl * WORDS, 0};
        fft_run<T, N, M, -1, false, PAD != 0, LdsLay<T, 1, 4, 1>, false, R::WVR>(v, lay, j, tw);
        if constexpr (NSTG > 1) xsync<R::WVR>();
#pragma unroll
        for (int u = 0; u < E / RL; ++u) lay.template st_run<RL, N / RL>(j + u * P, v + u * RL);
    }
    xsync<R::WROW>();
    if (!R::WROW || tid < R::RT) {
#pragma unroll
        for (int s = 0; s < RowShare<T, M, PAD>::COUNT; ++s) {
            const RowShare<T, M, PAD> e(s);
            const int k = e.kt * R::CW + e.kk;
            const LdsLay<T, 1, 4, 1> lay{lds + e.il * WORDS, 0};
            const cx<T> Zk = lay.ld(k), B = conjc(lay.ld((N - k) & (N - 1)));
            const cx<T> s1 = Zk + B, d1 = Zk - B;
            const cx<T> wd = cmul(twl(tw, k), d1);
            cx<T> out = mkc(T(0.5) * (s1.x + wd.y), T(0.5) * (s1.y - wd.x));
            if (k == 0) out = mkc(Zk.x + Zk.y, Zk.x - Zk.y);
            gst_all<!R::ONEX>(Wb + w_at<T, M, PAD>(e.kt, rb * R::RPW + e.il, e.kk), out);
        }
    }
}

// The column that a thread works on (u-th in turn) and its index within it.
template <typename T, int M, int PAD>
struct ColOf {
    using R = RGeo<T, M, PAD>;
    int kk, j, cl;  // column of the workgroup, thread of the column, LDS region
    __device__ __forceinline__ ColOf(int u) {
        constexpr int P = R::G::PC;
        cl = R::WVC ? threadIdx.x / P : threadIdx.x % R::CU;
        j = R::WVC ? threadIdx.x % P : threadIdx.x / R::CU;
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
            const ColOf<T, M, PAD> c(u);
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
template <typename T, int M, int PAD, class TW>
__device__ __forceinline__ void res_cols(cx<T>* lds, TW tw, const ResSpec<T, M, PAD>& sp, cx<T>* Wb, int blk) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    using Lay = typename R::ColLay;
    constexpr int E = G::EC, P = G::PC;
    constexpr int NSTG = fft_nstages(M);
    constexpr int R1 = fft_radix(M, false, 0), RL = fft_radix(M, false, NSTG - 1), RZ = fft_radix(M, true, NSTG - 1);
    cx<T> v[R::U][E];
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
        const ColOf<T, M, PAD> c(u);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if (PAD && i % R1 >= R1 / 2) continue;
            const int n = (c.j + (i / R1) * P) + (i % R1) * (M / R1);
            v[u][i] = gld_all(Wb + w_at<T, M, PAD>(blk, n, c.kk));
        }
    }
#pragma unroll
    for (int u = 0; u < R::U; ++u) {
        const ColOf<T, M, PAD> c(u);
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
                const T s = T(0.5) * (sp.g[u][i] + sp.gN[i]), t = T(0.5) * (sp.g[u][i] - sp.gN[i]);
                v[u][i] = c.kk == 0 ? mkc(s * a.x + t * bm.x, s * a.y + t * bm.y) : scalec(a, sp.g[u][i]);
            }
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i) v[u][i] = scalec(v[u][i], sp.g[u][i]);
        }
        fft_run<T, M, M, +1, true, false, Lay, true, R::WVC>(v[u], lay, c.j, tw);
#pragma unroll
        for (int i = 0; i < E; ++i) {
            if (PAD && i % RZ >= RZ / 2) continue;
            const int n = (c.j + (i / RZ) * P) + (i % RZ) * (M / RZ);
            gst_all<!R::ONEX>(Wb + w_at<T, M, PAD>(blk, n, c.kk), v[u][i]);
        }
    }
}

// Inverse transforms of the workgroup's rows (row_inv_body's arithmetic):
// v[u RL + r] holds the pair at n = (j + u P) + r N / RL.  Called as
// res_rows_fwd.
template <typename T, int M, int PAD, class TW>
__device__ __forceinline__ void res_rows_inv(cx<T>* v, cx<T>* lds, TW tw, const cx<T>* Wb, int rb) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, WORDS = G::ROW_WORDS;
    constexpr int R1 = fft_radix(N, true, 0), S1 = N / R1;
    constexpr int COUNT = RowShare<T, M, PAD>::COUNT;
    const int tid = threadIdx.x;
    const int rl = tid / P, j = tid % P;
    if (!R::WROW || tid < R::RT) {
        cx<T> wv[COUNT];
#pragma unroll
        for (int s = 0; s < COUNT; ++s) {
            const RowShare<T, M, PAD> e(s);
            wv[s] = gld_all(Wb + w_at<T, M, PAD>(e.kt, rb * R::RPW + e.il, e.kk));
        }
#pragma unroll
        for (int s = 0; s < COUNT; ++s) {
            const RowShare<T, M, PAD> e(s);
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
            lay.template ld_run<R1, S1>(jj == 0 ? 0 : S1 - jj, Bv);
#pragma unroll
            for (int r = 0; r < R1; ++r) {
                const int k = jj + r * S1;
                const cx<T> Y = A[r];
                const cx<T> B = conjc(jj == 0 ? Bv[(R1 - r) % R1] : Bv[R1 - 1 - r]);
                const cx<T> s1 = Y + B, d1 = Y - B;
                const cx<T> wd = cmul(conjc(twl(tw, k)), d1);
                v[u * R1 + r] = mkc(s1.x - wd.y, s1.y + wd.x);
                if (k == 0) v[u * R1 + r] = mkc(Y.x + Y.y, Y.x - Y.y);
            }
        }
        xsync<R::WVR>();
        fft_run<T, N, M, +1, true, false, LdsLay<T, 1, 4, 1>, false, R::WVR>(v, lay, j, tw);
    }
}

// ---- the kernel ---------------------------------------------------------------
// Barrier tokens token .. token + 2 K - 1.  Ends after K iterations, before
// an iteration that must wait for an FP64 check (st->pause), on breakdown, or
// when a wait gives up.
template <typename T, int M, int PAD, int NT>
__global__ void __launch_bounds__(NT)
    k_cg_resident(Tab<T> tab, SlotDesc sd, unsigned long long* words, int xcd, unsigned long long token, int K) {
    using R = RGeo<T, M, PAD>;
    using G = Geo<T, M, PAD>;
    constexpr int N = G::N, E = G::ER, P = G::PR, RPW = G::RPW, L = G::L;
    static_assert(NT == R::NT, "resident block size");
    constexpr int NSTG = fft_nstages(N);
    constexpr int RL = fft_radix(N, true, NSTG - 1), RK = PAD ? RL / 2 : RL, NO = (E / RL) * RK;
    static_assert(RL == fft_radix(N, false, 0), "forward first radix and inverse last radix");
    __shared__ cx<T> lds[R::LDS_WORDS];
    __shared__ double red[4 * (R::RT / 64)];
    __shared__ double s_tot[4];
    __shared__ int s_ok;
    // ONEX: eight times the workgroups are launched, and those of the XCD
    // asked for stay
    if (R::ONEX && (int)(blockIdx.x & 7) != xcd) return;
    const int blk = R::ONEX ? blockIdx.x >> 3 : blockIdx.x;
    if (!GateIter::ok(sd)) return;
    SolveState* st = sd.st;
    double rho = st->rho_next;
    int iters = st->iters;
    const int tid = threadIdx.x;
    const bool lead = blk == 0 && tid == 0;
    if (check_due(st, rho, iters)) {
        if (lead) st->pause = 1;
        return;
    }
    const bool rows = tid < R::RT;  // this thread holds a part of a row
    const int rl = tid / P, j = tid % P;
    const int rb = xcd_remap(blk, R::NB);  // as the passes: an XCD's workgroups share lines of W
    const int row = rows ? rb * RPW + rl : 0;
    const Meet<R::NG, R::GM> all{words, st->bar_limit, blk % R::NG, blk / R::NG};
    cx<T>* Wb = reinterpret_cast<cx<T>*>(sd.W);
    T* xa = reinterpret_cast<T*>(sizeof(T) == 8 ? (void*)sd.x : (void*)sd.e);
    auto twiddles = [&]() {
        if constexpr (R::HOIST) {
            return ConstTw<T>{tab.tw};
        } else {
            // opaque to the compiler: read afresh in every phase
            const cx<T>* t = tab.tw;
            asm volatile("" : "+s"(t));
            return t;
        }
    };
    auto give_up = [&]() {
        if (tid == 0) {
            __hip_atomic_store(&st->status, ST_EGRID, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            publish_status(sd, 1, ST_EGRID, st->gen, st->iters, st->last_check_iter);
        }
    };
    // both halves of the ring are empty before the first meeting
    all.empty(0);
    all.empty(1);
    auto col = [&](int i) { return 2 * ((j + (i / RK) * P) + (i % RK) * (N / RL)); };
    auto at = [&](int i) { return (size_t)row * L + col(i); };
    cx<T> r[NO], p[NO], x[NO], d[NO];
    if (rows) {
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            r[i] = ld2<T>(reinterpret_cast<const T*>(sd.r) + at(i));
            p[i] = ld2<T>(reinterpret_cast<const T*>(sd.p) + at(i));
            x[i] = ld2<T>(xa + at(i));
            if constexpr (sizeof(T) == 4)
                d[i] = ld2<float>(sd.d32 + at(i));
            else
                d[i] = ld2<double>(sd.d + at(i));
        }
    }
    ResSpec<T, M, PAD> sp;
    sp.load(tab, blk);
    // p <- r + beta p with the pending x <- x + a p
    auto direction = [&](T a, T beta) {
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const cx<T> po = p[i];
            p[i] = mkc(r[i].x + beta * po.x, r[i].y + beta * po.y);
            if (a != T(0)) {
                x[i].x += a * po.x;
                x[i].y += a * po.y;
            }
        }
    };
    if (st->restart) {
#pragma unroll
        for (int i = 0; i < NO; ++i) p[i] = r[i];
    } else {
        direction((T)st->alpha, (T)(rho / st->rho_prev));
    }
    double alpha = 0.0, rrn = 0.0;
    bool stop = false;
    if (!all.hello(token, &s_ok)) return give_up();
    for (int k = 0;;) {
        cx<T> v[E];
#pragma unroll
        for (int i = 0; i < NO; ++i) v[(i / RK) * RL + i % RK] = p[i];
        res_rows_fwd<T, M, PAD>(v, lds, twiddles(), Wb, rb);
        if (!all.meet(token, &s_ok)) return give_up();
        res_cols<T, M, PAD>(lds, twiddles(), sp, Wb, blk);
        if (!all.meet(token + 1, &s_ok)) return give_up();
        res_rows_inv<T, M, PAD>(v, lds, twiddles(), Wb, rb);
        double acc[4] = {0.0, 0.0, 0.0, 0.0}, tot[4];
        cx<T> q[NO];
        if (rows) {
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const cx<T> c = v[(i / RK) * RL + i % RK];
                typename EpiCGU<T>::Pre pr;
                pr.p = p[i];
                pr.d = d[i];
                q[i] = EpiCGU<T>::template outq<L>(sd, row, col(i), c.x, c.y, pr, acc);
            }
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                const cx<double> rv = mkc((double)r[i].x, (double)r[i].y), qv = mkc((double)q[i].x, (double)q[i].y);
                acc[1] += rv.x * rv.x + rv.y * rv.y;
                acc[2] += rv.x * qv.x + rv.y * qv.y;
                acc[3] += qv.x * qv.x + qv.y * qv.y;
            }
        }
        if (!all.template sums<R::RT, 4>(acc, 0, k & 1, red, s_tot, &s_ok, tot)) return give_up();
        rho = tot[1];
        if (!(tot[0] > 0.0) || !isfinite(tot[0]) || !isfinite(rho)) {
            if (lead) {
                st->status = ST_EBREAKDOWN;
                st->done = 1;
                publish_status(sd, 1, ST_EBREAKDOWN, st->gen, iters, st->last_check_iter);
            }
            return;
        }
        alpha = rho / tot[0];
        const T a = (T)alpha;
        const bool sure = next_rr(tot, (double)a, &rrn);
        if (rows) {
#pragma unroll
            for (int i = 0; i < NO; ++i) {
                r[i].x -= a * q[i].x;
                r[i].y -= a * q[i].y;
            }
        }
        if (!sure) {
            double rr[1] = {0.0};
            if (rows) {
#pragma unroll
                for (int i = 0; i < NO; ++i) rr[0] += (double)r[i].x * r[i].x + (double)r[i].y * r[i].y;
            }
            __syncthreads();  // readers of the first sums
            if (!all.template sums<R::RT, 1>(rr, 4, k & 1, red, s_tot, &s_ok, &rrn)) return give_up();
        }
        ++iters;
        ++k;
        token += 2;
        stop = check_due(st, rrn, iters);
        if (stop || k >= K) break;
        // the half that the next sums use: everybody has passed this
        // iteration's meetings, hence the sums that used it last
        all.empty(k & 1);
        if (rows) direction(a, (T)(rrn / rho));
    }
    if (rows) {
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            st2<T>(reinterpret_cast<T*>(sd.r) + at(i), r[i]);
            st2<T>(reinterpret_cast<T*>(sd.p) + at(i), p[i]);
            st2<T>(xa + at(i), x[i]);
        }
    }
    if (lead) {
        st->alpha = alpha;
        st->rho_prev = rho;
        st->rho_next = rrn;
        st->iters = iters;
        st->restart = 0;
        if (stop) st->pause = 1;
    }
}

}  // namespace FFTCG_RADIX_NS
}  // namespace fftcg
