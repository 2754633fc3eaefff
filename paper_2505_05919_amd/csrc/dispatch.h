// Kernel launches that can carry start/stop events recorded by the
// dispatch itself: their interval is the kernel's execution alone, the
// duration a profiler's kernel trace reports (events recorded on the stream
// around a launch also take in the command processor's work between them).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <tuple>

namespace cvf {

// Cache policy of the stores that leave a launch's results in memory (the
// builtins' cache-policy bits sc0 | sc1): written through L2 as they are made.
// A launch ends by writing its dirty L2 lines back, up to 32 MB in the eight
// XCDs' caches, with the chip otherwise idle; written through, that traffic
// runs beside the launch's arithmetic instead.  Measured: Metropolis sweeps at
// L = 2048 / 4096 28.3 / 76.8 -> 25.0 / 74.2 us, a Swendsen-Wang step at
// L = 1414 45.3 -> 42.8 us, cubic passes at 260^3 152.8 -> 151.0 us (sc1 alone
// the same, nt no change).  It costs traffic: a line that a launch completes in
// parts goes out in parts (191 MB per batched colour pass of 256 replicas
// instead of 167, 50 MB per tile launch at L = 1414 instead of 44), which large
// lattices pay for.  So unaligned Metropolis rows (met_through) and the tiles'
// local roots (kSwThroughCells) are written through only up to a size, and
// single bytes per lane (the ends of ragged rows, bond masks) and the cubic
// shifts not at all (a cubic cluster step 127.4 us with them, 126.0 without).
constexpr int kThrough = 17, kPlain = 0;

// Null events: a plain launch.
struct DispatchEvents {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};

// Launch of kernel k on stream s; the arguments are converted to the
// kernel's parameter types.  Returns the launch status.
template <typename... A, typename... V>
hipError_t go(void (*k)(A...), dim3 grid, dim3 block, hipStream_t s, const DispatchEvents& ev, V... v)
{
    static_assert(sizeof...(A) == sizeof...(V), "kernel argument count");
    std::tuple<A...> args(v...);
    void* ptr[sizeof...(A)];
    std::apply([&ptr](auto&... x) {
        int i = 0;
        ((ptr[i++] = (void*)&x), ...);
    }, args);
    if (ev.start) return hipExtLaunchKernel((const void*)k, grid, block, ptr, 0, s, ev.start, ev.stop, 0);
    return hipLaunchKernel((const void*)k, grid, block, ptr, 0, s);
}

}  // namespace cvf
