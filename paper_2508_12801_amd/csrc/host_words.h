// What a kernel tells the host through pinned memory.
#pragma once

#include <hip/hip_runtime.h>

namespace maxscore {

// Past the caches: the word is there at the latest when the kernel has ended, whatever its end writes back.
template <typename V>
__device__ __forceinline__ void tell_host(V *p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace maxscore
