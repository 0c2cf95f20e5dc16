// Host-side view of one compiled engine (one FFT grid size M and boundary
// condition).  Each engine_inst_<M>_<pad>.o fills one EngineOps with
// launchers for the multi-pass kernels of that size.
#pragma once
#include <hip/hip_runtime.h>
#include "fftcg_types.hpp"

namespace fftcg {

struct PlanTabs {
    const void* tw32;   // cx<float>[M]
    const void* ghq32;  // float, tile layout of the FP32 column pass
    const void* ghN32;  // float[M/2 + 1]
    const void* tw64;   // cx<double>[M]
    const void* ghq64;  // double, tile layout of the FP64 column pass
    const void* ghN64;  // double[M/2 + 1]
};

// One launch of the resident kernel.
struct ResidentRun {
    SlotDesc slot;              // the descriptor itself
    unsigned long long* words;  // kMeetWords 64-bit words the workgroups meet through
    unsigned long long token;   // first of kResidentTokens tokens that no launch on the words has used (they grow)
    int xcd;                    // the XCD to run on (its hardware number), where resident_xcds is 1
    int gen;                    // mark of this launch: the state it leaves carries it (SolveState::gen)
    int K;                      // iterations at most, <= kResidentIters
    int first;                  // 1: the solve begins; 0: it goes on
    int zero;                   // with first: from x = 0 (slot.x is not read)
};
// Iterations of one launch: a bound on its length (some milliseconds); most
// solves end within one.  Every iteration meets at most four times, and at
// most one check (four meetings) precedes it.
constexpr int kResidentIters = 256;
constexpr unsigned long long kResidentTokens = 8ull * (kResidentIters + 2);

struct EngineOps {
    int M, pad, L;
    int tt32, tt64;          // columns per tile of the column pass
    int rowblk32, rowblk64;  // blocks of the row passes (= partial counts)
    int g4;                  // blocks of the update kernel (= r.r partial count)
    // y = d x + C x, precision 0 = FP64, 1 = FP32 operator
    void (*apply)(int prec, const PlanTabs& t, const double* d, const double* x, double* y,
                  void* W, hipStream_t s);
    // one pass of an operator product: 0 row_fwd, 1 col, 2 row_inv
    void (*apply_pass)(int prec, int pass, const PlanTabs& t, const double* d, const double* x, double* y,
                       void* W, hipStream_t s);
    // one CG iteration for nslots slots (row_fwd, col, row_inv, update)
    void (*iter)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride,
                 hipStream_t s);
    // one FP64 check (row_fwd, col, row_inv on x, then the finaliser)
    void (*check)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride,
                  hipStream_t s);
    // the same two for CG with the Fourier-space (circulant) preconditioner
    void (*iter_pcg)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride,
                     hipStream_t s);
    void (*check_pcg)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride,
                      hipStream_t s);
    // the initial check of a solve started from x = 0 (no product: r = b)
    void (*check0)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride, hipStream_t s);
    void (*check0_pcg)(int prec, const PlanTabs& t, const SlotDesc* slots, int nslots, int stride,
                       hipStream_t s);
    // one pass of a plain-CG iteration of one slot (measurement aid): 0 the
    // forward row pass, 1 the column pass, 2 the row-inverse pass (with the
    // folded update when grid), 3 the separate update (nothing when grid),
    // 4 the turn pass (grid only; tokens token and token + 1); the launch
    // records ev0 as the kernel starts and ev1 as it ends
    void (*iter_pass)(int prec, int pass, bool grid, const PlanTabs& t, const SlotDesc* slot, int stride,
                      unsigned long long token, hipEvent_t ev0, hipEvent_t ev1, hipStream_t s);
    // whether the folded update (below) applies on the current device: how
    // many whole row-inverse grids are resident at once (0: not one)
    int (*grid_capable)(int prec);
    // K (>= 1) CG iterations of a single slot, as a chunk, with the update
    // folded into the row-inverse pass behind a grid-wide barrier.  With
    // turn, the row-inverse pass of every iteration but the last goes on into
    // the next iteration's forward row pass (k_row_turn), so the chunk
    // launches row_fwd, col, (turn, col) x (K - 1), row_inv; without it, K
    // times row_fwd, col, row_inv.  *token is advanced past every token the
    // launches use (each unique on the slot's partial-sum buffer).
    void (*iter_grid_chunk)(int prec, const PlanTabs& t, const SlotDesc* slot, int stride,
                            unsigned long long* token, int K, bool turn, hipStream_t s);
    // the same of the turn pass
    int (*turn_capable)(int prec);
    // K preconditioned iterations of a single slot as a chunk, with the two
    // turns behind grid-wide barriers: row_fwd, (col, turn, col) with a turn
    // between them, row_inv.  *token as above.
    void (*iter_pcg_chunk)(int prec, const PlanTabs& t, const SlotDesc* slot, int stride, unsigned long long* token,
                           int K, hipStream_t s);
    // the same of these two (0 also where they are not built)
    int (*turn_pcg_capable)(int prec);
    // a single solve, or K of its iterations, in one launch
    // (k_solve_resident); pcg: with the circulant preconditioner.  st: the
    // state it begins with (run.first), else taken from the slot's.
    void (*resident)(int prec, bool pcg, const PlanTabs& t, const ResidentRun& run, const SolveState& st,
                     hipStream_t s);
    // the XCDs it occupies: 1 or 8
    int (*resident_xcds)(int prec);
    // whether it applies on the current device (built for this grid and
    // resident as a whole)
    bool (*resident_capable)(int prec, bool pcg);
};

const EngineOps* find_engine(int M, int pad);

}  // namespace fftcg
