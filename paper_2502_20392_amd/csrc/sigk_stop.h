// sigk_stop.h -- how the waves of a workgroup leave a loop of barriers together.
//
// One wave may give up before the barrier that ends iteration k; every wave
// reads the outcome after it.  With a single flag a wave that is already in the
// next iteration could raise it before a slow one has read it for this one, and
// that one would leave a barrier early.  Iterations alternate between two
// flags: a flag is raised again only after a further barrier, which every wave
// passes after its reading.  (Plain C++: the schedules are checked on the CPU.)
#pragma once

#ifdef __HIPCC__
#define SIGK_STOP_FN __device__ __forceinline__
#else
#define SIGK_STOP_FN inline
#endif

namespace sigk {

struct StopFlags {
    int raised[2];
    SIGK_STOP_FN void clear() { raised[0] = raised[1] = 0; }
    SIGK_STOP_FN void raise(int k) { *(volatile int*)&raised[k & 1] = 1; }
    SIGK_STOP_FN bool test(int k) const { return *(const volatile int*)&raised[k & 1] != 0; }
};

}  // namespace sigk
