// What csrc/tokens.hpp takes from its own includes, for a host build of its rounds: the threads of a
// work-group are fibers that run one at a time from barrier to barrier, in an order the driver chooses.
#pragma once

#include <cstdint>
#include <cstdio>
#include <functional>

#define __device__
#define __host__
#define __global__ [[maybe_unused]] static
#define __forceinline__ inline
#define __shared__
#define __launch_bounds__(...)
#define RWC_LDS
#define RWC_GLOBAL
#define __hip_atomic_load(p, order, scope) (switch_point(), *(p))
#define __hip_atomic_store(p, v, order, scope) (switch_point(), *(p) = (v))

struct Dim {
    uint32_t x;
};
extern Dim threadIdx, blockDim, blockIdx;
void __syncthreads();
void switch_point();   // another fiber may run here

namespace rwc {
namespace {

constexpr int kWave = 64;
extern uint32_t kCntMax;   // a count of this many departures overflows
enum : uint32_t { kErrStepLimit = 16, kErrCountOverflow = 32 };

struct GraphArgs {
    int32_t n, root;
    const uint32_t* rootmask;
    uint64_t guard;
    int64_t stride;
};
struct DumpArgs {};
struct Item {
    int32_t graph, slot0;
};
struct PopArgs {
    uint32_t* slots;
    int64_t slot_stride, sample_begin;
    uint64_t seed;
};

uint32_t draw(uint32_t v, uint32_t k, uint32_t sample);   // node v's k-th arrow
template <bool kStrat>
uint32_t pop_draw(const GraphArgs&, uint32_t v, uint32_t k, uint32_t sample, uint32_t, uint32_t) {
    return draw(v, k, sample);
}
inline uint32_t lds_add(uint32_t* p, uint32_t v) {
    const uint32_t old = *p;
    *p += v;
    return old;
}
inline uint32_t lds_or(uint32_t* p, uint32_t v) {
    const uint32_t old = *p;
    *p |= v;
    return old;
}
template <class T>
T* global_ptr(T* p) {
    return p;
}
template <class... Args>
void finish_tree(Args&&...) {}
template <class Grow>
void pop_items(const PopArgs&, Grow) {}

}  // namespace
}  // namespace rwc
