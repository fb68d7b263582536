// Stand-in for the HIP runtime header that compiles kernels without
// cross-lane operations as C++, for tests of their control flow on the CPU.
//
// A workgroup is an OS thread (so that its __shared__ variables, which become
// thread_local, are its own); each of its threads is a context of its own that
// runs until it reaches a barrier or ends.  The test says which threads run
// and when: any interleaving of wavefronts and workgroups can be played.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static thread_local
#define __launch_bounds__(...)

struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
struct int2 { int x, y; };
inline thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
typedef void* hipStream_t;
enum hipError_t { hipSuccess };
inline hipError_t hipGetLastError() { return hipSuccess; }
#define hipLaunchKernelGGL(...) ((void)0)

using std::isfinite;
using std::isnan;
using std::max;
using std::min;
inline double __dadd_rn(double a, double b) { return a + b; }
inline double __dsub_rn(double a, double b) { return a - b; }
inline double __dmul_rn(double a, double b) { return a * b; }
inline double __ddiv_rn(double a, double b) { return a / b; }
inline long long __double_as_longlong(double v) { long long b; std::memcpy(&b, &v, 8); return b; }
inline double __longlong_as_double(long long b) { double v; std::memcpy(&v, &b, 8); return v; }

// cross-lane operations: not played here
[[noreturn]] inline void hostsim_lanes() { std::fprintf(stderr, "cross-lane operation\n"); std::abort(); }
struct LanePair { unsigned v[2]; unsigned operator[](int k) const { return v[k]; } };
inline LanePair hostsim_swap(unsigned) { hostsim_lanes(); }
inline int hostsim_move(int) { hostsim_lanes(); }
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) hostsim_swap(a)
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) hostsim_swap(a)
#define __builtin_amdgcn_mov_dpp(v, c, r, b, z) hostsim_move(v)
#define __builtin_amdgcn_fence(o, s) hostsim_lanes()
#define __builtin_amdgcn_wave_barrier() hostsim_lanes()
template <typename T>
T __shfl(T, int, int = 64) { hostsim_lanes(); }

// memory: one workgroup runs at a time
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
template <typename T, typename V>
void __hip_atomic_store(T* p, V v, int, int) { *p = v; }
template <typename T>
T __hip_atomic_load(const T* p, int, int) { return *p; }
template <typename T, typename V>
T __hip_atomic_fetch_add(T* p, V v, int, int) { T o = *p; *p = o + v; return o; }
inline unsigned atomicAdd(unsigned* p, unsigned v) { const unsigned o = *p; *p = o + v; return o; }

namespace hostsim {

struct Group;
inline thread_local Group* current = nullptr;

struct Group {
    enum State { READY, BARRIER, DONE };
    struct Thread { ucontext_t ctx; std::unique_ptr<char[]> stack; State state = READY; };
    static constexpr size_t kStack = 128 << 10;

    std::vector<Thread> threads;
    std::function<void()> kernel;
    dim3 block, grid, dim;
    bool divergent = false;                  // a thread ended while others of the group waited at a barrier

    Group(std::function<void()> k, dim3 blk, dim3 grd, unsigned n) : threads(n), kernel(k), block(blk), grid(grd), dim(n) {
        worker = std::thread([this] { loop(); });
    }
    ~Group() { post(0, 0, true); worker.join(); }

    // Runs threads [lo, hi) until each waits at a barrier or has ended.
    void run(unsigned lo, unsigned hi) { post(lo, hi, false); }
    // Runs the group to its end; a barrier opens once all threads that are
    // left wait at it.
    void finish() {
        for (;;) {
            run(0, (unsigned)threads.size());
            bool waiting = false, ended = false;
            for (const Thread& t : threads) (t.state == BARRIER ? waiting : ended) = true;
            if (!waiting) return;
            divergent |= ended;
            for (Thread& t : threads)
                if (t.state == BARRIER) t.state = READY;
        }
    }
    void barrier() {
        Thread& t = threads[at];
        t.state = BARRIER;
        swapcontext(&t.ctx, &home);
        threadIdx = dim3(at, 0, 0);
    }

private:
    std::thread worker;
    std::mutex mu;
    std::condition_variable cv;
    ucontext_t home;
    unsigned at = 0, lo = 0, hi = 0;
    bool work = false, quit = false;

    void post(unsigned l, unsigned h, bool q) {
        std::unique_lock<std::mutex> k(mu);
        lo = l; hi = h; quit = q; work = true;
        cv.notify_all();
        if (!q) cv.wait(k, [this] { return !work; });
    }
    static void entry() {
        current->kernel();
        current->threads[current->at].state = DONE;
    }
    void loop() {
        current = this;
        blockIdx = block; gridDim = grid; blockDim = dim;
        for (Thread& t : threads) {
            t.stack.reset(new char[kStack]);
            getcontext(&t.ctx);
            t.ctx.uc_stack.ss_sp = t.stack.get();
            t.ctx.uc_stack.ss_size = kStack;
            t.ctx.uc_link = &home;
            makecontext(&t.ctx, entry, 0);
        }
        for (;;) {
            std::unique_lock<std::mutex> k(mu);
            cv.wait(k, [this] { return work; });
            if (quit) return;
            for (at = lo; at < hi; ++at)
                if (threads[at].state == READY) {
                    threadIdx = dim3(at, 0, 0);
                    swapcontext(&home, &threads[at].ctx);
                }
            work = false;
            cv.notify_all();
        }
    }
};

}  // namespace hostsim

inline void __syncthreads() { hostsim::current->barrier(); }
