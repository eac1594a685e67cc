// Stands in for <hip/hip_runtime.h> where the library's device-side plan headers are built for the
// host: one thread per lane of a workgroup, a barrier per workgroup, and wave shuffles through
// memory shared by the threads.
#pragma once
#include <pthread.h>

#include <algorithm>
#include <cstdint>
#include <thread>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline

using std::max;
using std::min;

struct HostIndex { unsigned x; };
inline thread_local HostIndex threadIdx{0};

namespace hosthip {
inline pthread_barrier_t g_barrier;
inline uint64_t g_lane[1024];

// runs f on nt threads as one workgroup
template <typename F>
void run_workgroup(int nt, F f) {
    pthread_barrier_init(&g_barrier, nullptr, nt);
    std::vector<std::thread> ts;
    for (int t = 0; t < nt; t++)
        ts.emplace_back([&f, t] {
            threadIdx.x = t;
            f();
        });
    for (auto& t : ts) t.join();
    pthread_barrier_destroy(&g_barrier);
}
}  // namespace hosthip

inline void __syncthreads() { pthread_barrier_wait(&hosthip::g_barrier); }

// every thread of the workgroup calls these together (as the plan builders do)
template <typename T>
T hosthip_exchange(T v, int src) {
    hosthip::g_lane[threadIdx.x] = (uint64_t)v;
    __syncthreads();
    const T r = (T)hosthip::g_lane[src];
    __syncthreads();
    return r;
}
template <typename T>
T __shfl_up(T v, unsigned d, int) {
    const unsigned lane = threadIdx.x & 63;
    return hosthip_exchange(v, (int)(lane >= d ? threadIdx.x - d : threadIdx.x));
}
template <typename T>
T __shfl_xor(T v, int m, int) {
    return hosthip_exchange(v, (int)(threadIdx.x ^ (unsigned)m));
}
template <typename T>
T __shfl(T v, int l, int) {
    return hosthip_exchange(v, (int)((threadIdx.x & ~63u) + (unsigned)l));
}
inline int atomicAdd(int* p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
