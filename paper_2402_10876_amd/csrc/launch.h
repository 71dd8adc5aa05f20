// Internal: kernel launches.
#pragma once
#include <hip/hip_runtime.h>

namespace twg {

template <class T> struct same_type { typedef T type; };

// One launch call of the runtime and its own status, where the <<< >>> form pushes and pops a configuration and asks
// for the thread's last error in front and behind (2.70 -> 2.46 us of the host per launch, which is what bounds small
// products).  A failed launch leaves no error behind for the next caller.
template <class... P>
inline hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t stream, typename same_type<P>::type... args) {
  void* list[] = {(void*)&args...};
  const hipError_t e = hipLaunchKernel((const void*)kernel, grid, block, list, 0, stream);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

}  // namespace twg
