// The few HIP names that a kernel source needs to run on the CPU, one fiber a
// lane (see run_grid).  Only what coarse_solve.hip uses is here.
//
// Scheduling is the caller's: a wavefront runs until each of its lanes waits (at
// a barrier, for its wavefront's other lanes, or after a poll that found
// nothing), then the policy names the next one.  So an order of the wavefronts
// that a GPU takes once in a long while can be taken every time.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
// workgroup memory: one section of the program, put away and brought back when
// another workgroup runs
#define __shared__ static __attribute__((section("workgroup_memory")))
#define __HIP_MEMORY_SCOPE_AGENT 0

typedef int hipError_t;
typedef void *hipStream_t;
typedef void *hipEvent_t;
constexpr hipError_t hipSuccess = 0;
inline hipError_t hipGetLastError() { return hipSuccess; }

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};

namespace emulated {

enum Wait { kReady, kPolled, kBarrier, kWave, kDone };
struct Lane {
    void *sp = nullptr;
    std::vector<char> stack;
    Wait wait = kReady;
    dim3 thread, block;
    int put[2] = {0, 0}, turn = 0;   // what the lane shows its wavefront
    long long seen = 0;              // stores made before its last poll
};
extern Lane *lane;
extern unsigned blocks;
extern long long stores;             // atomic writes so far: what a poll waits for
void wait(Wait w);
int from_lane(int old, int x, int ctrl, int row_mask);
void run_grid(unsigned grid, unsigned lanes, const std::function<void()> &body);
// which of the wavefronts {workgroup, wavefront} that can go on does
struct Wave {
    int block, wave;
};
extern std::function<size_t(const std::vector<Wave> &)> policy;
extern const void *arguments;        // the first of the kernel's
template <typename First, typename... Rest>
const void *first_of(const First &first, const Rest &...) { return &first; }

}  // namespace emulated

#define threadIdx (emulated::lane->thread)
#define blockIdx (emulated::lane->block)
#define gridDim dim3(emulated::blocks)

#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) ((void)(++emulated::stores, *(p) = (v)))
template <typename T>
inline T emulated_add(T *p, T v) {
    const T old = *p;
    *p = old + v;
    ++emulated::stores;
    return old;
}
#define __hip_atomic_fetch_add(p, v, order, scope) emulated_add(p, v)
template <typename T>
inline bool emulated_cas(T *p, T *expected, T desired) {
    if (*p == *expected) {
        *p = desired;
        ++emulated::stores;
        return true;
    }
    *expected = *p;
    return false;
}
#define __hip_atomic_compare_exchange_strong(p, e, d, o1, o2, scope) emulated_cas(p, e, d)

#define __builtin_amdgcn_s_sleep(n) emulated::wait(emulated::kPolled)
#define __builtin_amdgcn_s_barrier() emulated::wait(emulated::kBarrier)
#define __builtin_amdgcn_sched_barrier(n) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_kernarg_segment_ptr() (emulated::arguments)
#define __syncthreads() emulated::wait(emulated::kBarrier)
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, zero) emulated::from_lane(old, x, ctrl, rows)

#define hipLaunchKernelGGL(kernel, grid, block, bytes, stream, ...) \
    (emulated::arguments = emulated::first_of(__VA_ARGS__), emulated::run_grid((grid).x, (block).x, [&] { kernel(__VA_ARGS__); }))
