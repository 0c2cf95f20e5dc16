// Simulated device for host-only tests of plans and single solves
// (tests/test_host_fake.py).  Linked with the unmodified fftcg_host.cpp and
// fused.hip built by g++ against tests/fake_hip/hip/hip_runtime.h.
//
// * "Device" memory is host memory, filled with a pattern when allocated;
//   every operation runs when it is issued.
// * A fake solve of A x = b ends after its first chunk with x = b / 2.  Every
//   launcher calls the test's hook (kind of launch, grid, precision), which
//   may block: the solve is then in flight until the test lets it go on.
// * The test can have the resident kernel or the grid-wide barriers give up,
//   one memset fail, and recorded events stay pending.
// Not part of the product library.
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <new>

#include "common.hpp"
#include "engine.hpp"
#include "fftcg.h"
#include "fftcg_internal.hpp"
#include "fused.hpp"

using namespace fftcg;

struct FakeEvent {
    std::atomic<int> pending{0};
    std::atomic<int> captured{0};  // last recorded in a capture
};

namespace {
enum Kind { kApply, kResident, kChunk, kSeparate, kFused, kCapturedRecord };
typedef void (*Hook)(int kind, int M, int precision);
std::atomic<Hook> g_hook{nullptr};
// bit 0: the resident kernel, bit 1: the barriers; bit 2: no workgroup of the
// resident kernel runs (it leaves the state as it was)
std::atomic<int> g_give_up{0};
std::atomic<size_t> g_fail_memset{0};  // bytes of the memset that fails (once)
std::atomic<int> g_hold_events{0};
std::atomic<int> g_capture{0};           // whether streams are being captured
std::atomic<int> g_captured_queries{0};  // queries of events last recorded in a capture
std::atomic<int> g_words_clear{-1};  // whether the last resident launch's words held no token

void hook(Kind k, int M, int prec) {
    if (Hook h = g_hook.load()) h(k, M, prec);
}
void finish(const SlotDesc& sd, int L, int status) {
    SolveState* st = sd.st;
    st->done = 1;
    st->status = status;
    st->iters = 3;
    st->pause = 0;
    for (size_t i = 0; i < (size_t)L * L; ++i) sd.x[i] = status == ST_EGRID ? -1.0 : 0.5 * sd.b[i];
    if (sd.host_status) {
        sd.host_status[1] = status;
        sd.host_status[3] = 3;
        __atomic_store_n(sd.host_status, 1, __ATOMIC_RELEASE);
    }
}
}  // namespace

// ---- runtime ---------------------------------------------------------------
hipError_t hipMallocRaw(void** p, size_t n) {
    *p = malloc(n ? n : 1);
    if (*p) memset(*p, 0x7b, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
    free(p);
    return hipSuccess;
}
hipError_t hipHostMallocRaw(void** p, size_t n, unsigned) { return hipMallocRaw(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
    memmove(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(dst, src, n, k);
}
hipError_t hipMemset(void* dst, int v, size_t n) {
    memset(dst, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t) {
    size_t want = n;
    if (g_fail_memset.compare_exchange_strong(want, 0)) return hipErrorInvalidValue;
    return hipMemset(dst, v, n);
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = new (std::nothrow) FakeEvent();
    return *e ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    e->captured.store(g_capture.load());
    e->pending.store(g_hold_events.load());
    if (g_capture.load()) hook(kCapturedRecord, 0, 0);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    if (e->captured.load()) g_captured_queries += 1;
    return e->pending.load() && g_hold_events.load() ? hipErrorNotReady : hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = g_capture.load() ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }

// ---- engines ---------------------------------------------------------------
namespace {
// capabilities as on the device: the resident kernel for 32 <= M <= 1024 (one
// XCD up to M = 256), barriers everywhere, the preconditioned turns at M =
// 2048 and 4096 in FP32; above M = 2048 one grid fills the device, at 2048 four do, below sixteen
template <int M, int PAD>
struct Fake {
    static constexpr int L = PAD ? M / 2 : M;
    static void apply(int prec, const PlanTabs&, const double*, const double* x, double* y, void*, hipStream_t) {
        hook(kApply, M, prec);
        memcpy(y, x, (size_t)L * L * 8);
    }
    static void apply_pass(int, int, const PlanTabs&, const double*, const double*, double*, void*, hipStream_t) {}
    static void iter(int prec, const PlanTabs&, const SlotDesc*, int, int, hipStream_t) { hook(kSeparate, M, prec); }
    static void check(int, const PlanTabs&, const SlotDesc* s, int, int, hipStream_t) {
        if (s->st->checks++ > 0 && !s->st->done) finish(*s, L, FFTCG_OK);
    }
    static void iter_pass(int, int, bool, const PlanTabs&, const SlotDesc*, int, unsigned long long, hipEvent_t,
                          hipEvent_t, hipStream_t) {}
    static void chunk(int prec, const SlotDesc* s) {
        hook(kChunk, M, prec);
        if (g_give_up.load() & 2) finish(*s, L, ST_EGRID);
    }
    static void grid_chunk(int prec, const PlanTabs&, const SlotDesc* s, int, unsigned long long*, int, bool,
                           hipStream_t) {
        chunk(prec, s);
    }
    static void pcg_chunk(int prec, const PlanTabs&, const SlotDesc* s, int, unsigned long long*, int, hipStream_t) {
        chunk(prec, s);
    }
    static void resident(int prec, bool, const PlanTabs&, const ResidentRun& r, const SolveState& st, hipStream_t) {
        if (r.first && !(g_give_up.load() & 4)) *r.slot.st = st;
        int clear = 1;
        for (int i = 0; i < kMeetWords; ++i) clear &= r.words[i] < r.token;
        g_words_clear.store(clear);
        hook(kResident, M, prec);
        if (g_give_up.load() & 4) return;
        r.slot.st->gen = r.gen;
        finish(r.slot, L, g_give_up.load() & 1 ? ST_EGRID : FFTCG_OK);
    }
    static int resident_xcds(int) { return M <= 256 ? 1 : 8; }
    static bool resident_capable(int, bool) { return M >= 32 && M <= 1024; }
    static const EngineOps* get() {
        static const EngineOps ops = [] {
            EngineOps o;
            memset(&o, 0, sizeof o);
            o.M = M;
            o.pad = PAD;
            o.L = L;
            o.tt32 = o.tt64 = 1;
            o.rowblk32 = o.rowblk64 = o.g4 = 64;
            o.apply = apply;
            o.apply_pass = apply_pass;
            o.iter = o.iter_pcg = iter;
            o.check = o.check_pcg = o.check0 = o.check0_pcg = check;
            o.iter_pass = iter_pass;
            o.iter_grid_chunk = grid_chunk;
            o.iter_pcg_chunk = pcg_chunk;
            o.grid_capable = [](int) -> decltype(o.grid_capable(0)) { return M > 2048 ? 1 : (M > 1024 ? 4 : 16); };
            o.turn_capable = [](int) -> decltype(o.turn_capable(0)) { return M > 2048 ? 1 : (M > 1024 ? 4 : 16); };
            o.turn_pcg_capable = [](int prec) -> decltype(o.turn_pcg_capable(0)) {
                return prec != FFTCG_MIXED || M < 2048 || M > 4096 ? 0 : (M > 2048 ? 1 : 4);
            };
            o.resident = resident;
            o.resident_xcds = resident_xcds;
            o.resident_capable = resident_capable;
            return o;
        }();
        return &ops;
    }
};
template <int M, int PAD>
struct FakeFused {
    static void solve(int prec, const FusedTabs&, const SlotDesc* s, int, int, hipStream_t) {
        hook(kFused, M, prec);
        finish(*s, PAD ? M / 2 : M, FFTCG_OK);
    }
    static void apply(int prec, const FusedTabs&, const double*, const double*, double*, void*, hipStream_t) {
        hook(kApply, M, prec);
    }
    static const FusedOps* get() {
        static const FusedOps ops = {M, PAD, 0, solve, apply};
        return &ops;
    }
};
}  // namespace

namespace fftcg {
#define FAKE_ENGINE(M, P) \
    const EngineOps* fftcg_engine_ops_##M##_##P() { return Fake<M, P>::get(); }
#define FAKE_FUSED(M, P) \
    const FusedOps* fftcg_fused_ops_##M##_##P() { return FakeFused<M, P>::get(); }
#define FAKE_SMALL(X) \
    X(2, 0) X(4, 0) X(8, 0) X(16, 0) X(32, 0) X(64, 0) X(128, 0) X(256, 0) X(4, 1) X(8, 1) X(16, 1) X(32, 1) X(64, 1) \
        X(128, 1) X(256, 1)
FAKE_SMALL(FAKE_ENGINE)
FAKE_SMALL(FAKE_FUSED)
FAKE_ENGINE(512, 0)
FAKE_ENGINE(1024, 0)
FAKE_ENGINE(2048, 0)
FAKE_ENGINE(4096, 0)
FAKE_ENGINE(8192, 0)
FAKE_ENGINE(512, 1)
FAKE_ENGINE(1024, 1)
FAKE_ENGINE(2048, 1)
FAKE_ENGINE(4096, 1)
FAKE_ENGINE(8192, 1)

void launch_to_f32(const double*, float*, int, hipStream_t) {}
int loadstep_blocks(int) { return 1; }
void launch_loadstep(const double*, const double*, double*, int, double*, int*, int* out, hipStream_t, const double*,
                     double*) {
    *out = 0;
}
void launch_breakstep(const double*, const double*, uint8_t*, int, double*, int*, int* out, double* out_v,
                      hipStream_t) {
    *out = 0;
    *out_v = 1.0;
}
int loadstep_noalloc(const double*, const double*, double*, int, int* index, hipStream_t) {
    *index = 0;
    return 0;
}
void launch_stream(int, bool, int, void*, const void*, size_t, hipStream_t) {}
void launch_fill(double* a, double v, int n, hipStream_t) {
    for (int i = 0; i < n; ++i) a[i] = v;
}
}  // namespace fftcg

// ---- test controls -----------------------------------------------------------
extern "C" void fake_set_hook(Hook h) { g_hook.store(h); }
extern "C" void fake_give_up(int bits) { g_give_up.store(bits); }
extern "C" void fake_fail_memset(size_t n) { g_fail_memset.store(n); }
extern "C" void fake_hold_events(int h) { g_hold_events.store(h); }
extern "C" void fake_capture(int c) { g_capture.store(c); }
extern "C" int fake_captured_queries(void) { return g_captured_queries.load(); }
extern "C" int fake_words_clear(void) { return g_words_clear.load(); }
extern "C" size_t fake_meet_bytes(void) { return (size_t)kMeetWords * 8; }
