// Sweep of short lists, several steps at a time: launch description.
#pragma once
#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace rlpt {

struct AheadLaunch {
    const ItemDev* items;  // one copy each, hottest temperature slot first (0 items: another sweep kernel)
    int n_items;
    int max_N;
    int block;   // packed lists: threads per workgroup
    int slots;   // packed lists: entries per lane, half a wave per list
    int chunks;  // chunked lists: chunks per lane of the longest list
};

size_t ahead_lds_bytes(int precision, int block, int max_N);
hipError_t launch_sweep_ahead(int precision, const void* ptrs, const ShapeInfo& sh, const AheadLaunch& L, int n_sweeps,
                              hipStream_t st);

}  // namespace rlpt
