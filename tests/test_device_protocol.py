"""Device functions whose outcome depends on what several threads see when,
run on the CPU: the function's own source text, taken out of the header, with
the few device built-ins it uses replaced by scripted ones (the loads and the
clock answer what the test chooses)."""

import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1305_3625_amd", "csrc")
BUILD = os.path.join(ROOT, "_build", "fake")


def _function(header, start, head="template"):
    """The text of the function whose definition contains `start`, from the
    line before it that begins with `head` to its closing brace."""
    src = open(os.path.join(CSRC, header)).read()
    i = src.rindex("\n" + head, 0, src.index(start)) + 1
    return src[i:src.index("\n}\n", i) + 3]


def _run(name, code):
    os.makedirs(BUILD, exist_ok=True)
    src, exe = os.path.join(BUILD, name + ".cpp"), os.path.join(BUILD, name)
    with open(src, "w") as f:
        f.write(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused", "-I" + CSRC, src, "-o", exe, "-lpthread"],
                   check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=60, check=True).stdout.split()


GRID_SUMS = r"""
#include <pthread.h>
#include <stdio.h>
#include <thread>
#include <vector>
#define __device__
#define __shared__ static
#define __HIP_MEMORY_SCOPE_AGENT 0
typedef unsigned long long u64;
struct Idx { unsigned x; };
static thread_local Idx threadIdx;
static const Idx blockIdx{1}, gridDim{2};
constexpr int cmin(int a, int b) { return a < b ? a : b; }
enum { PS_PQ, PS_RR, PS_RZ, PS_RQ, PS_QQ, PS_BAR, PS_BARREL, SETS };
constexpr int LANES = 4, STRIDE = 64;
static pthread_barrier_t bar;
static int votes[LANES];
static void __syncthreads() { pthread_barrier_wait(&bar); }
static bool vote(int v, bool all) {
    votes[threadIdx.x] = v != 0;
    __syncthreads();
    int n = 0;
    for (int i = 0; i < LANES; ++i) n += votes[i];
    __syncthreads();
    return all ? n == LANES : n > 0;
}
static bool __all(int v) { return vote(v, true); }
static bool __any(int v) { return vote(v, false); }
static bool __syncthreads_and(int v) { return vote(v, true); }
static bool __syncthreads_or(int v) { return vote(v, false); }
static double part[SETS * STRIDE];
static u64 TOKEN = 7;
static int blind;   // lanes that see the token only after the deadline (a bit each)
static int polls_seen;
static thread_local int polls;
template <class T> T* gbl(T* p) { return p; }
// the clock runs with the lane's polls: past the limit after the second
static u64 clk() { return polls * 100; }
#define __builtin_amdgcn_s_memrealtime() clk()
#define __builtin_amdgcn_s_sleep(n)
#define __builtin_amdgcn_s_waitcnt(n)
static u64 load(const u64* p) {
    if (p == (const u64*)(part + PS_BARREL * STRIDE)) {
        ++polls;
        if ((blind >> threadIdx.x) & 1) return polls > 2 ? TOKEN : 0;
        return polls > 1 ? TOKEN : 0;
    }
    return *p;
}
#define __hip_atomic_load(p, o, s) load(p)
#define __hip_atomic_store(p, v, o, s) (void)(*(p) = (v))
#define __hip_atomic_exchange(p, v, o, s) (*(p) = (v))
template <int NT, int N> void block_sums(const double* acc, double*, double* out) {
    if (threadIdx.x == 0) for (int a = 0; a < N; ++a) out[a] = acc[a];
}
template <int NG, class G> double group_sum(unsigned, double, G) { return 0; }
@FUNCTION@
int main() {
    pthread_barrier_init(&bar, nullptr, LANES);
    for (blind = 0; blind < 16; ++blind) {
        for (int a = 0; a < 4; ++a) part[PS_BARREL * STRIDE + 1 + a] = 100.0 + a;  // the totals
        bool ok[LANES];
        double tot[LANES][4];
        std::vector<std::thread> th;
        for (int t = 0; t < LANES; ++t)
            th.emplace_back([&, t] {
                threadIdx.x = t;
                polls = 0;
                const double acc[4] = {1, 2, 3, 4};
                double sh[16];
                ok[t] = grid_sums<LANES, 4, 0>(acc, part, STRIDE, TOKEN, 150, sh, tot[t]);
            });
        for (auto& t : th) t.join();
        bool same = true, right = true;
        for (int t = 0; t < LANES; ++t) {
            same &= ok[t] == ok[0];
            for (int a = 0; a < 4; ++a) right &= tot[t][a] == 100.0 + a;
        }
        printf("%d:%d:%d\n", same, ok[0], right);
    }
}
"""


def test_grid_sums_gives_up_as_one():
    """The lanes that fetch the totals must not decide by themselves whether
    the barrier was met: whichever of them miss the release before the
    deadline, either all threads get all totals or all give up."""
    code = GRID_SUMS.replace("@FUNCTION@", _function("fftcg_kernels.hpp", "inline bool grid_sums("))
    out = [tuple(map(int, line.split(":"))) for line in _run("grid_sums", code)]
    assert len(out) == 16
    for blind, (same, ok, right) in enumerate(out):
        assert same and (right or not ok), (blind, same, ok, right)
    assert out[0] == (1, 1, 1)


RES_END = r"""
#include <stdio.h>
#include <string.h>
#include <functional>
#define __device__
#define __forceinline__ inline
struct Idx { unsigned x; };
static const Idx threadIdx{0};
#include "fftcg_types.hpp"
using namespace fftcg;
static void publish_status(const SlotDesc&, int, int, int, int, int) {}
// runs the other workgroup's part before the n-th store to the state
static int store_no;
static std::function<void(int)> before_store;
template <class T> void store(T* p, T v) {
    before_store(store_no++);
    *p = v;
}
#define __hip_atomic_store(p, v, o, s) store(p, v)
struct Meeting {
    bool met;
    bool meet(unsigned long long, int*) const { return met; }
};
@GIVE_UP@
@END@
int main() {
    // workgroup 0 meets the others; workgroup 1 gives up as they arrive.  The
    // solve goes on (done = 0), or has ended with a status of its own.
    for (int done = 0; done < 2; ++done)
        for (int when = 0; when < 3; ++when) {
            SolveState mem, st;
            memset(&mem, 0, sizeof mem);
            memset(&st, 0, sizeof st);
            st.done = done;
            st.status = done ? -4 : 0;
            SlotDesc sd;
            memset(&sd, 0, sizeof sd);
            sd.st = &mem;
            int s_ok = 0;
            bool ran = false;
            auto first = [&] {
                if (ran) return;
                ran = true;
                auto f = before_store;
                before_store = [](int) {};
                res_end(Meeting{true}, 9, &s_ok, 0, sd, st);
                before_store = f;
            };
            store_no = 0;
            before_store = [&](int n) {
                if (n == when) first();
            };
            res_end(Meeting{false}, 9, &s_ok, 1, sd, st);
            first();
            printf("%d:%d:%d:%d\n", done, when, mem.done, mem.status);
        }
    // and where workgroup 0 gives up
    SolveState mem, st;
    memset(&mem, 0, sizeof mem);
    memset(&st, 0, sizeof st);
    SlotDesc sd;
    memset(&sd, 0, sizeof sd);
    sd.st = &mem;
    int s_ok = 0;
    before_store = [](int) {};
    res_end(Meeting{false}, 9, &s_ok, 0, sd, st);
    printf("2:0:%d:%d\n", mem.done, mem.status == ST_EGRID);
}
"""


def test_end_of_resident_launch():
    """The state after the last meeting is the first workgroup's, or says
    that the solve was abandoned; never parts of both."""
    code = RES_END.replace("@GIVE_UP@", _function("resident_kernels.hpp", "void res_give_up(", "__device__"))
    code = code.replace("@END@", _function("resident_kernels.hpp", "void res_end("))
    for line in _run("res_end", code):
        kind, when, done, status = map(int, line.split(":"))
        if kind == 2:
            assert (done, status) == (1, 1)
        else:
            assert (done, status) in ((kind, -4 if kind else 0), (1, -100)), line
