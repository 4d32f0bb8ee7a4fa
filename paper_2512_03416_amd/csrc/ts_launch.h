// Kernel launches that can mark their own end.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

namespace ts {

// Launches a kernel; done (if not NULL) is an event recorded at its end.  The event then rides on the kernel's own packet.
// Recorded behind the kernel it is a packet of its own, which the queue works through before the next kernel may start: a
// 20 us kernel in a row of its kind takes 21.3 us with the event on it or without one, 22.4 with one recorded behind it, and
// the host 2.4 us for 3.6.  (Not for streams that are being captured: the event is not part of the graph.)
template <typename... P, typename... A>
inline int launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t st, hipEvent_t done, A&&... args)
{
    if (done) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, nullptr, done, 0, P(args)...);
    else hipLaunchKernelGGL(kernel, grid, block, 0, st, P(args)...);
    return (int)hipGetLastError();
}

}  // namespace ts
