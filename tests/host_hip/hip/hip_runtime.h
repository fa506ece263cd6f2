// Just enough of the HIP language for a kernel to run on the host: one
// workgroup, one thread per work item.  __syncthreads() counts only the live
// threads, as the hardware's barrier does, and notes when one was passed with
// some of the workgroup already gone.
#pragma once

#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define hipLaunchKernelGGL(...) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#define __HIP_MEMORY_SCOPE_SYSTEM 0
// asm volatile("" ::"s"(...)): an empty statement that keeps a scalar load early
#define asm
#define volatile(...)

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct int2 {
    int x, y;
};
struct int4 {
    int x, y, z, w;
};
inline int4 make_int4(int a, int b, int c, int d) { return {a, b, c, d}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline unsigned __float_as_uint(float f)
{
    unsigned u;
    std::memcpy(&u, &f, 4);
    return u;
}
typedef struct hip_stream *hipStream_t;

// a barrier over the live members of a set
struct LiveBarrier {
    std::mutex mu;
    std::condition_variable cv;
    int size = 0, live = 0, arrived = 0;
    long phase = 0;
    bool diverged = false;
    void reset(int n)
    {
        size = live = n;
        arrived = 0;
        diverged = false;
    }
    void pass()
    {
        diverged |= live < size;
        arrived = 0;
        phase++;
        cv.notify_all();
    }
    void wait()
    {
        std::unique_lock<std::mutex> l(mu);
        const long p = phase;
        if (++arrived == live) pass();
        cv.notify_all();
        cv.wait(l, [&] { return phase != p; });
    }
    void leave()
    {
        std::lock_guard<std::mutex> l(mu);
        if (--live > 0 && arrived == live) pass();
        cv.notify_all();
    }
};

namespace host_hip {
inline LiveBarrier group, wave[16];
inline double slot[16][64];
inline thread_local int lane = 0, wid = 0;

// One workgroup of `threads` work items as blockIdx.x = block of `grid`.  The
// wavefront `early` runs alone until it waits for the others or ends; then
// between() runs, and the others start.  Returns whether all wavefronts met at
// every barrier.
bool run(int threads, int block, int grid, int early, const std::function<void()> &between,
         const std::function<void()> &kernel);
}  // namespace host_hip

inline thread_local dim3 threadIdx, blockIdx;
inline dim3 blockDim, gridDim;
inline void __syncthreads() { host_hip::group.wait(); }
template <typename T>
T __shfl_xor(T v, int off, int width = 64)
{
    static_assert(sizeof(T) <= 8, "one slot per lane");
    (void)width;
    using namespace host_hip;
    std::memcpy(&slot[wid][lane], &v, sizeof(T));
    wave[wid].wait();
    T r;
    std::memcpy(&r, &slot[wid][lane ^ off], sizeof(T));
    wave[wid].wait();
    return r;
}

inline bool host_hip::run(int threads, int block, int grid, int early, const std::function<void()> &between,
                          const std::function<void()> &kernel)
{
    blockDim = dim3(threads);
    gridDim = dim3(grid);
    group.reset(threads);
    for (int w = 0; w < threads / 64; w++) wave[w].reset(64);
    std::vector<std::thread> pool;
    auto start = [&](int w) {
        for (int l = 0; l < 64; l++)
            pool.emplace_back([=, &kernel] {
                threadIdx = dim3(64 * w + l);
                blockIdx = dim3(block);
                lane = l;
                wid = w;
                kernel();
                wave[w].leave();
                group.leave();
            });
    };
    start(early);
    {
        std::unique_lock<std::mutex> l(group.mu);
        group.cv.wait(l, [&] { return group.arrived + (threads - group.live) == 64; });
    }
    between();
    for (int w = 0; w < threads / 64; w++)
        if (w != early) start(w);
    for (std::thread &t : pool) t.join();
    return !group.diverged;
}
