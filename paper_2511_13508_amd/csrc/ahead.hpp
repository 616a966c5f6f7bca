// Sweep of short lists, several steps at a time: launch description.
#pragma once
#include <hip/hip_runtime.h>

#include "internal.hpp"

namespace rlpt {

struct AheadLaunch {
    const ItemDev* items;  // one copy each, hottest temperature slot first (0 items: another sweep kernel)
    int n_items;
    int max_N;
    int block;   // threads per workgroup: 512, with up to kShortSlots entries per lane also 256 or 1024
    int slots;   // packed lists: entries per lane, half a wave per list
    int chunks;  // chunked lists: chunks per lane of the longest list
};

// max_N, block, slots and chunks for lists of up to `longest` entries (packed)
// or chunks; false where no instance of the kernel serves them or its LDS does
// not fit
bool ahead_plan(int precision, int layout, uint32_t longest, int max_N, AheadLaunch* L);
// LDS that the launch asks for
size_t ahead_lds_bytes(int precision, const AheadLaunch& L);
hipError_t launch_sweep_ahead(int precision, const void* ptrs, const ShapeInfo& sh, const AheadLaunch& L, int n_sweeps,
                              hipStream_t st);

}  // namespace rlpt
