// launch.hpp — how the host code of the kernel files launches.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mezo {

// Launch a one-argument kernel and return the status of this launch itself
// (not the thread's last HIP error, which may hold an earlier failure of
// another caller's call). done: an event that the kernel's own completion
// signals, or null. An event recorded after the launch instead is a packet of
// its own that the next launch waits behind: back-to-back launches took 7.0 us
// each with one on 1M elements, 4.5 with the launch's own event and 2.9 without
// any; on 128M fp32 elements 164.9 and 162.2 (which sets use which: own_event in
// api.cpp).
template <class Arg>
hipError_t launch1(void (*kernel)(Arg), uint32_t workgroups, uint32_t lanes, hipStream_t stream, Arg arg,
                   hipEvent_t done)
{
    void* params[] = {&arg};
    const void* f = reinterpret_cast<const void*>(kernel);
    if (done) return hipExtLaunchKernel(f, dim3(workgroups), dim3(lanes), params, 0, stream, nullptr, done, 0);
    return hipLaunchKernel(f, dim3(workgroups), dim3(lanes), params, 0, stream);
}

}  // namespace mezo
