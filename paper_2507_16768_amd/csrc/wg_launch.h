// How the launchers start their kernels (HIP translation units only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

namespace wg {

// Launches a kernel and returns that launch's own status: the thread's last error may be somebody
// else's, from before, and a call reported as failed on its account would have run all the same.  With a
// pair of events the kernel's own begin / end timestamps are recorded into them, which times the kernel
// without the queue gaps that events recorded between launches would include.
template <typename T> struct AsIs { using type = T; };
template <typename... P>
inline hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, uint32_t lds, hipStream_t s, hipEvent_t *ev,
                         typename AsIs<P>::type... args)
{
    void *at[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    const void *of = reinterpret_cast<const void *>(kernel);
    const hipError_t e = ev ? hipExtLaunchKernel(of, grid, block, at, lds, s, ev[0], ev[1], 0) : hipLaunchKernel(of, grid, block, at, lds, s);
    if (e != hipSuccess) (void)hipGetLastError();      // reported here, and nowhere else
    return e;
}

}  // namespace wg
