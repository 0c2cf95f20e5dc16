// Instantiates the multi-pass engine for one grid; compiled once per
// (FFTCG_M, FFTCG_PAD) by the build script.
#include <string.h>

#include <hip/hip_ext.h>

#include "engine.hpp"
#include "fftcg_kernels.hpp"
#include "resident_kernels.hpp"

#ifndef FFTCG_M
#error "FFTCG_M must be defined"
#endif
#ifndef FFTCG_PAD
#error "FFTCG_PAD must be defined"
#endif

#define FFTCG_CAT2(a, b, c) a##b##_##c
#define FFTCG_CAT(a, b, c) FFTCG_CAT2(a, b, c)
#define FFTCG_OPS_FN FFTCG_CAT(fftcg_engine_ops_, FFTCG_M, FFTCG_PAD)

namespace fftcg {
namespace {

constexpr int M = FFTCG_M;
constexpr int PAD = FFTCG_PAD;
template <typename T>
using G = Geo<T, M, PAD>;
constexpr int LL = G<float>::L;
constexpr int UPD_NT = 256;
constexpr int g4_blocks() {
    return cmax(1, cmin(1024, LL * LL / 1024));
}

template <typename T>
Tab<T> tab_of(const PlanTabs& t);
template <>
Tab<float> tab_of<float>(const PlanTabs& t) {
    return Tab<float>{(const cx<float>*)t.tw32, (const float*)t.ghq32, (const float*)t.ghN32};
}
template <>
Tab<double> tab_of<double>(const PlanTabs& t) {
    return Tab<double>{(const cx<double>*)t.tw64, (const double*)t.ghq64, (const double*)t.ghN64};
}

template <typename T>
void apply_pass_t(int pass, const PlanTabs& pt, const double* d, const double* x, double* y, void* W,
                  hipStream_t s) {
    constexpr int RT = G<T>::ROW_THREADS, CT = G<T>::COL_THREADS;
    ByVal sv;
    memset(&sv.s, 0, sizeof(SlotDesc));
    sv.s.d = d;
    sv.s.x = const_cast<double*>(x);
    sv.s.y = y;
    sv.s.W = W;
    sv.s.active = 1;
    const Tab<T> tab = tab_of<T>(pt);
    if (pass == 0)
        hipLaunchKernelGGL((k_row_fwd<T, M, PAD, ProApply<T>, ByVal, RT>), dim3(G<T>::ROW_BLOCKS), dim3(RT), 0,
                           s, tab, sv, 0, 0);
    else if (pass == 1)
        hipLaunchKernelGGL((k_col<T, M, PAD, GateAlways, ByVal, CT>), dim3(G<T>::COL_BLOCKS), dim3(CT), 0, s, tab, sv);
    else
        hipLaunchKernelGGL((k_row_inv<T, M, PAD, EpiApply<T>, ByVal, RT>), dim3(G<T>::ROW_BLOCKS), dim3(RT), 0,
                           s, tab, sv, 0);
}

template <typename T>
void apply_t(const PlanTabs& pt, const double* d, const double* x, double* y, void* W, hipStream_t s) {
    for (int pass = 0; pass < 3; ++pass) apply_pass_t<T>(pass, pt, d, x, y, W, s);
}

void apply_pass_fn(int prec, int pass, const PlanTabs& pt, const double* d, const double* x, double* y, void* W,
                   hipStream_t s) {
    if (prec == 0)
        apply_pass_t<double>(pass, pt, d, x, y, W, s);
    else
        apply_pass_t<float>(pass, pt, d, x, y, W, s);
}

void apply_fn(int prec, const PlanTabs& pt, const double* d, const double* x, double* y, void* W,
              hipStream_t s) {
    if (prec == 0)
        apply_t<double>(pt, d, x, y, W, s);
    else
        apply_t<float>(pt, d, x, y, W, s);
}

template <typename W, typename XA>
void iter_t(const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS;
    const ByPtr sp{slots};
    const Tab<W> tab = tab_of<W>(pt);
    hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProCG<W, XA, RT>, ByPtr, RT>), dim3(G<W>::ROW_BLOCKS, nslots),
                       dim3(RT), 0, s, tab, sp, g4_blocks(), stride);
    hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS, nslots), dim3(CT), 0, s, tab,
                       sp);
    hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiCG<W>, ByPtr, RT>), dim3(G<W>::ROW_BLOCKS, nslots), dim3(RT), 0,
                       s, tab, sp, stride);
    hipLaunchKernelGGL((k_update<W, UPD_NT, LL>), dim3(g4_blocks(), nslots), dim3(UPD_NT), 0, s, sp, LL * LL,
                       G<W>::ROW_BLOCKS, stride);
}

void iter_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s);

// The same iteration for one slot with the update inside the row-inverse
// pass (EpiCGU): the row-forward pass then takes r.r from the state.  token
// and token + 1 are the row-inverse pass's.
template <typename W>
void iter_grid_t(const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long token, hipStream_t s) {
    constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS, RB = G<W>::ROW_BLOCKS;
    const ByPtr sp{slot};
    const Tab<W> tab = tab_of<W>(pt);
    hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProCG<W, W, RT, true>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp, 0,
                       stride);
    hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s, tab, sp);
    hipLaunchKernelGGL((k_row_inv_upd<W, M, PAD, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp, stride, token);
}

// The resident kernel is built where the iteration is latency-bound and its
// vectors fit the registers.  Whole solves to 1e-10, folded passes (mode 3) ->
// resident: periodic M = 64 FP64 759 -> 241 us, padded M = 256 mixed 1465 ->
// 596 us, M = 1024 FP64 3250 -> 1968 us, M = 1024 mixed 2660 -> 1680 us;
// preconditioned padded M = 1024 FP64 1697 -> 1047 us.
template <typename W>
constexpr bool kResBuilt = M >= 32 && G<W>::SUM_GROUPS > 0 && RGeo<W, M, PAD>::OK;

// The turn pass saves the reads of r and p and one launch per iteration.
// Against the folded update alone (whole solves, alternating in one process):
// padded L = 1024 mixed 4117 -> 3887 us, FP64 5227 -> 4842; padded L = 2048
// mixed 9076 -> 8289; periodic M = 2048 mixed 4188 -> 3824.
// On the resident kernel's grids it serves solves that find no room for that
// (four threads of FP64 L = 512: 1,153 solves a second, 910 with the folded
// update alone; of mixed L = 256 2,580 and 2,440).
// Built where its grid can be resident at once: not in FP64 on rows of 16
// pairs a thread and more (over 200 VGPRs, two workgroups per CU).
template <typename W>
constexpr bool kTurnBuilt = !(sizeof(W) == 8 && G<W>::ER >= 16);

template <typename W>
void iter_pass_t(int pass, bool grid, const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long token,
                 hipEvent_t e0, hipEvent_t e1, hipStream_t s) {
    constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS, RB = G<W>::ROW_BLOCKS;
    const ByPtr sp{slot};
    const Tab<W> tab = tab_of<W>(pt);
    if (pass == 0) {
        if (grid)
            hipExtLaunchKernelGGL((k_row_fwd<W, M, PAD, ProCG<W, W, RT, true>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s,
                                  e0, e1, 0, tab, sp, 0, stride);
        else
            hipExtLaunchKernelGGL((k_row_fwd<W, M, PAD, ProCG<W, W, RT>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, e0,
                                  e1, 0, tab, sp, g4_blocks(), stride);
    } else if (pass == 1) {
        hipExtLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s, e0, e1, 0,
                              tab, sp);
    } else if (pass == 2) {
        if (grid) {
            hipExtLaunchKernelGGL((k_row_inv_upd<W, M, PAD, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, e0, e1, 0, tab, sp,
                                  stride, token);
            return;
        }
        hipExtLaunchKernelGGL((k_row_inv<W, M, PAD, EpiCG<W>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, e0, e1, 0, tab,
                              sp, stride);
    } else if (pass == 3) {
        if (!grid)
            hipExtLaunchKernelGGL((k_update<W, UPD_NT, LL>), dim3(g4_blocks()), dim3(UPD_NT), 0, s, e0, e1, 0, sp,
                                  LL * LL, RB, stride);
    } else if constexpr (kTurnBuilt<W>) {
        if (grid)
            hipExtLaunchKernelGGL((k_row_turn<W, M, PAD, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, e0, e1, 0, tab, sp,
                                  stride, token);
    }
}

void iter_pass_fn(int prec, int pass, bool grid, const PlanTabs& pt, const SlotDesc* slot, int stride,
                  unsigned long long token, hipEvent_t e0, hipEvent_t e1, hipStream_t s) {
    if (prec == 0)
        iter_pass_t<double>(pass, grid, pt, slot, stride, token, e0, e1, s);
    else
        iter_pass_t<float>(pass, grid, pt, slot, stride, token, e0, e1, s);
}

// how many grids of kernel `kern` (RB workgroups of RT threads) can be
// resident as a whole at once on the current device
template <int RT, int RB>
int whole_grids_resident(const void* kern) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, RT, 0) != hipSuccess) return 0;
    return per_cu * cus / RB;
}

template <typename W>
int grid_capable_t() {
    constexpr int RT = G<W>::ROW_THREADS, RB = G<W>::ROW_BLOCKS;
    return whole_grids_resident<RT, RB>(reinterpret_cast<const void*>(k_row_inv_upd<W, M, PAD, ByPtr, RT>));
}

int grid_capable_fn(int prec) {
    return prec == 0 ? grid_capable_t<double>() : grid_capable_t<float>();
}

template <typename W>
int turn_capable_t() {
    constexpr int RT = G<W>::ROW_THREADS, RB = G<W>::ROW_BLOCKS;
    if constexpr (!kTurnBuilt<W>)
        return 0;
    else
        return cmin(grid_capable_t<W>(),
                    whole_grids_resident<RT, RB>(reinterpret_cast<const void*>(k_row_turn<W, M, PAD, ByPtr, RT>)));
}

int turn_capable_fn(int prec) {
    return prec == 0 ? turn_capable_t<double>() : turn_capable_t<float>();
}

template <typename W>
void iter_grid_chunk_t(const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long* token, int K,
                       bool turn, hipStream_t s) {
    if constexpr (kTurnBuilt<W>) {
        if (turn) {
            constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS, RB = G<W>::ROW_BLOCKS;
            const ByPtr sp{slot};
            const Tab<W> tab = tab_of<W>(pt);
            hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProCG<W, W, RT, true>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s,
                               tab, sp, 0, stride);
            hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s, tab, sp);
            for (int k = 1; k < K; ++k) {
                const unsigned long long t = *token + 1;
                *token += 2;
                hipLaunchKernelGGL((k_row_turn<W, M, PAD, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp, stride, t);
                hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s, tab,
                                   sp);
            }
            hipLaunchKernelGGL((k_row_inv_upd<W, M, PAD, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp, stride,
                               *token + 1);
            *token += 2;
            return;
        }
    }
    for (int k = 0; k < K; ++k, *token += 2) iter_grid_t<W>(pt, slot, stride, *token + 1, s);
}

void iter_grid_chunk_fn(int prec, const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long* token,
                        int K, bool turn, hipStream_t s) {
    if (prec == 0)
        iter_grid_chunk_t<double>(pt, slot, stride, token, K, turn, s);
    else
        iter_grid_chunk_t<float>(pt, slot, stride, token, K, turn, s);
}

template <typename W>
void resident_t(bool pcg, const PlanTabs& pt, const ResidentRun& rr, const SolveState& st, hipStream_t s) {
    if constexpr (kResBuilt<W>) {
        using R = RGeo<W, M, PAD>;
        const ResArgs a{rr.slot, rr.words, rr.token, rr.xcd, rr.gen, rr.K, rr.first, rr.zero};
        const dim3 grid(R::NB * (R::ONEX ? 8 : 1)), block(R::NT);
        if (pcg)
            hipLaunchKernelGGL((k_solve_resident<W, M, PAD, R::NT, true>), grid, block, 0, s, tab_of<W>(pt),
                               tab_of<double>(pt), a, st);
        else
            hipLaunchKernelGGL((k_solve_resident<W, M, PAD, R::NT, false>), grid, block, 0, s, tab_of<W>(pt),
                               tab_of<double>(pt), a, st);
    }
}

void resident_fn(int prec, bool pcg, const PlanTabs& pt, const ResidentRun& rr, const SolveState& st, hipStream_t s) {
    if (prec == 0)
        resident_t<double>(pcg, pt, rr, st, s);
    else
        resident_t<float>(pcg, pt, rr, st, s);
}

template <typename W>
bool resident_capable_t(bool pcg) {
    if constexpr (!kResBuilt<W>)
        return false;
    else {
        using R = RGeo<W, M, PAD>;
        const void* k = pcg ? reinterpret_cast<const void*>(k_solve_resident<W, M, PAD, R::NT, true>)
                            : reinterpret_cast<const void*>(k_solve_resident<W, M, PAD, R::NT, false>);
        // on one XCD: an eighth of the CUs
        return whole_grids_resident<R::NT, R::NB * (R::ONEX ? 8 : 1)>(k) > 0;
    }
}

bool resident_capable_fn(int prec, bool pcg) {
    return prec == 0 ? resident_capable_t<double>(pcg) : resident_capable_t<float>(pcg);
}

int resident_xcds_fn(int prec) {
    return (prec == 0 ? RGeo<double, M, PAD>::ONEX : RGeo<float, M, PAD>::ONEX) ? 1 : 8;
}

void iter_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        iter_t<double, double>(pt, slots, nslots, stride, s);
    else
        iter_t<float, float>(pt, slots, nslots, stride, s);
}

template <typename W>
void check_t(const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    constexpr int RT = G<double>::ROW_THREADS, CT = G<double>::COL_THREADS;
    const ByPtr sp{slots};
    const Tab<double> tab = tab_of<double>(pt);
    hipLaunchKernelGGL((k_row_fwd<double, M, PAD, ProCheck<W, RT>, ByPtr, RT>),
                       dim3(G<double>::ROW_BLOCKS, nslots), dim3(RT), 0, s, tab, sp, 0, stride);
    hipLaunchKernelGGL((k_col<double, M, PAD, GateCheck, ByPtr, CT>), dim3(G<double>::COL_BLOCKS, nslots), dim3(CT), 0,
                       s, tab, sp);
    hipLaunchKernelGGL((k_row_inv<double, M, PAD, EpiCheck<W>, ByPtr, RT>), dim3(G<double>::ROW_BLOCKS, nslots),
                       dim3(RT), 0, s, tab, sp, stride);
    hipLaunchKernelGGL((k_check_final<256, G<double>::SUM_GROUPS>), dim3(1, nslots), dim3(256), 0, s, sp, G<double>::ROW_BLOCKS,
                       g4_blocks(), stride, LL * LL);
}

void check_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        check_t<double>(pt, slots, nslots, stride, s);
    else
        check_t<float>(pt, slots, nslots, stride, s);
}

// Preconditioned CG (Fourier-space circulant preconditioner): the operator
// product with the direction (row_fwd with p = z + beta p, col, row_inv with
// q and p.q), then r <- r - alpha q fused into the row-forward pass of the
// preconditioner product (with r.r), its column pass with 1/(dbar + ghat),
// and its row-inverse pass writing z and r.z.
template <typename W, typename XA>
void iter_pcg_t(const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS, RB = G<W>::ROW_BLOCKS;
    const ByPtr sp{slots};
    const Tab<W> tab = tab_of<W>(pt);
    hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProPCG<W, XA, RT, RB, G<W>::SUM_GROUPS>, ByPtr, RT>), dim3(RB, nslots), dim3(RT), 0, s,
                       tab, sp, RB, stride);
    hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS, nslots), dim3(CT), 0, s, tab,
                       sp);
    hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiCG<W>, ByPtr, RT>), dim3(RB, nslots), dim3(RT), 0, s, tab, sp,
                       stride);
    hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProUpdPre<W, RT, RB, G<W>::SUM_GROUPS>, ByPtr, RT>), dim3(RB, nslots), dim3(RT), 0, s,
                       tab, sp, 0, stride);
    hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT, true>), dim3(G<W>::COL_BLOCKS, nslots), dim3(CT), 0, s,
                       tab, sp);
    hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiPre<W, GateIter>, ByPtr, RT>), dim3(RB, nslots), dim3(RT), 0, s,
                       tab, sp, stride);
}

void iter_pcg_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        iter_pcg_t<double, double>(pt, slots, nslots, stride, s);
    else
        iter_pcg_t<float, float>(pt, slots, nslots, stride, s);
}

// The two turns in place of four row passes per iteration, where their grid is
// resident at once (FP32: 120 VGPRs, four workgroups per CU at M = 4096): whole
// solves, passes -> turns, padded L = 2048 mixed 3200 -> 3072 us, L = 1024 1520
// -> 1495.  At M = 8192 it is not (2,048 workgroups, of which the device holds
// 512).  In FP64 at M = 2048, where it would be, it is not built: 2520 us as
// passes, 2366 with the turns (periodic 2330 and 2140).
template <typename W>
constexpr bool kTurnPcgBuilt = !kResBuilt<W> && sizeof(W) == 4 && M >= 2048 && M <= 4096;

template <typename W>
int turn_pcg_capable_t() {
    if constexpr (!kTurnPcgBuilt<W>) {
        return 0;
    } else {
        constexpr int RT = G<W>::ROW_THREADS, RB = G<W>::ROW_BLOCKS;
        return cmin(whole_grids_resident<RT, RB>(
                        reinterpret_cast<const void*>(k_row_turn_pcg<W, M, PAD, EpiTurnR<W>, ByPtr, RT>)),
                    whole_grids_resident<RT, RB>(
                        reinterpret_cast<const void*>(k_row_turn_pcg<W, M, PAD, EpiTurnZ<W>, ByPtr, RT>)));
    }
}

int turn_pcg_capable_fn(int prec) {
    return prec == 0 ? turn_pcg_capable_t<double>() : turn_pcg_capable_t<float>();
}

template <typename W>
void iter_pcg_chunk_t(const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long* token, int K,
                      hipStream_t s) {
    if constexpr (kTurnPcgBuilt<W>) {
        constexpr int RT = G<W>::ROW_THREADS, CT = G<W>::COL_THREADS, RB = G<W>::ROW_BLOCKS;
        const ByPtr sp{slot};
        const Tab<W> tab = tab_of<W>(pt);
        hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProPCG<W, W, RT, RB, G<W>::SUM_GROUPS>, ByPtr, RT>), dim3(RB),
                           dim3(RT), 0, s, tab, sp, RB, stride);
        for (int k = 0; k < K; ++k) {
            if (k > 0)
                hipLaunchKernelGGL((k_row_turn_pcg<W, M, PAD, EpiTurnZ<W>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab,
                                   sp, stride, ++*token);
            hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s, tab,
                               sp);
            hipLaunchKernelGGL((k_row_turn_pcg<W, M, PAD, EpiTurnR<W>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp,
                               stride, ++*token);
            hipLaunchKernelGGL((k_col<W, M, PAD, GateIter, ByPtr, CT, true>), dim3(G<W>::COL_BLOCKS), dim3(CT), 0, s,
                               tab, sp);
        }
        hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiPre<W, GateIter>, ByPtr, RT>), dim3(RB), dim3(RT), 0, s, tab, sp,
                           stride);
    }
}

void iter_pcg_chunk_fn(int prec, const PlanTabs& pt, const SlotDesc* slot, int stride, unsigned long long* token,
                       int K, hipStream_t s) {
    if (prec == 0)
        iter_pcg_chunk_t<double>(pt, slot, stride, token, K, s);
    else
        iter_pcg_chunk_t<float>(pt, slot, stride, token, K, s);
}

// FP64 check of the preconditioned solve (r.r partial count = the working
// precision's row blocks), then z = P^{-1} r and r.z of the replaced
// residual when the solve continues.
template <typename W>
void check_pcg_t(const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    constexpr int RT = G<double>::ROW_THREADS, CT = G<double>::COL_THREADS;
    constexpr int RTW = G<W>::ROW_THREADS, CTW = G<W>::COL_THREADS, RBW = G<W>::ROW_BLOCKS;
    const ByPtr sp{slots};
    const Tab<double> tab = tab_of<double>(pt);
    const Tab<W> tabw = tab_of<W>(pt);
    hipLaunchKernelGGL((k_row_fwd<double, M, PAD, ProCheck<W, RT>, ByPtr, RT>),
                       dim3(G<double>::ROW_BLOCKS, nslots), dim3(RT), 0, s, tab, sp, 0, stride);
    hipLaunchKernelGGL((k_col<double, M, PAD, GateCheck, ByPtr, CT>), dim3(G<double>::COL_BLOCKS, nslots), dim3(CT), 0,
                       s, tab, sp);
    hipLaunchKernelGGL((k_row_inv<double, M, PAD, EpiCheck<W>, ByPtr, RT>), dim3(G<double>::ROW_BLOCKS, nslots),
                       dim3(RT), 0, s, tab, sp, stride);
    hipLaunchKernelGGL((k_check_final<256, G<double>::SUM_GROUPS>), dim3(1, nslots), dim3(256), 0, s, sp, G<double>::ROW_BLOCKS, RBW,
                       stride, LL * LL);
    hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProPre<W>, ByPtr, RTW>), dim3(RBW, nslots), dim3(RTW), 0, s, tabw, sp,
                       0, stride);
    hipLaunchKernelGGL((k_col<W, M, PAD, GatePre, ByPtr, CTW, true>), dim3(G<W>::COL_BLOCKS, nslots), dim3(CTW), 0, s,
                       tabw, sp);
    hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiPre<W, GatePre>, ByPtr, RTW>), dim3(RBW, nslots), dim3(RTW), 0, s,
                       tabw, sp, stride);
}

void check_pcg_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        check_pcg_t<double>(pt, slots, nslots, stride, s);
    else
        check_pcg_t<float>(pt, slots, nslots, stride, s);
}

// The initial check of a solve started from zero (x = 0, e = 0 already
// written by the host): r = b in one pass, then the finaliser (and, for the
// preconditioned solve, z = P^{-1} r).
template <typename W>
void check0_t(bool pcg, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    constexpr int RTW = G<W>::ROW_THREADS, CTW = G<W>::COL_THREADS, RBW = G<W>::ROW_BLOCKS;
    const ByPtr sp{slots};
    constexpr int RT = G<double>::ROW_THREADS;
    hipLaunchKernelGGL((k_check_zero<W, M, PAD, RT>), dim3(G<double>::ROW_BLOCKS, nslots), dim3(RT), 0, s, sp,
                       stride);
    hipLaunchKernelGGL((k_check_final<256, G<double>::SUM_GROUPS>), dim3(1, nslots), dim3(256), 0, s, sp, G<double>::ROW_BLOCKS,
                       pcg ? RBW : g4_blocks(), stride, LL * LL);
    if (pcg) {
        const Tab<W> tabw = tab_of<W>(pt);
        hipLaunchKernelGGL((k_row_fwd<W, M, PAD, ProPre<W>, ByPtr, RTW>), dim3(RBW, nslots), dim3(RTW), 0, s, tabw,
                           sp, 0, stride);
        hipLaunchKernelGGL((k_col<W, M, PAD, GatePre, ByPtr, CTW, true>), dim3(G<W>::COL_BLOCKS, nslots), dim3(CTW), 0,
                           s, tabw, sp);
        hipLaunchKernelGGL((k_row_inv<W, M, PAD, EpiPre<W, GatePre>, ByPtr, RTW>), dim3(RBW, nslots), dim3(RTW), 0,
                           s, tabw, sp, stride);
    }
}

void check0_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        check0_t<double>(false, pt, slots, nslots, stride, s);
    else
        check0_t<float>(false, pt, slots, nslots, stride, s);
}

void check0_pcg_fn(int prec, const PlanTabs& pt, const SlotDesc* slots, int nslots, int stride, hipStream_t s) {
    if (prec == 0)
        check0_t<double>(true, pt, slots, nslots, stride, s);
    else
        check0_t<float>(true, pt, slots, nslots, stride, s);
}

const EngineOps kOps = {M,
                        PAD,
                        LL,
                        G<float>::TT,
                        G<double>::TT,
                        G<float>::ROW_BLOCKS,
                        G<double>::ROW_BLOCKS,
                        g4_blocks(),
                        &apply_fn,
                        &apply_pass_fn,
                        &iter_fn,
                        &check_fn,
                        &iter_pcg_fn,
                        &check_pcg_fn,
                        &check0_fn,
                        &check0_pcg_fn,
                        &iter_pass_fn,
                        &grid_capable_fn,
                        &iter_grid_chunk_fn,
                        &turn_capable_fn,
                        &iter_pcg_chunk_fn,
                        &turn_pcg_capable_fn,
                        &resident_fn,
                        &resident_xcds_fn,
                        &resident_capable_fn};

}  // namespace

const EngineOps* FFTCG_OPS_FN() { return &kOps; }

}  // namespace fftcg
