// sigk_fwd.hip -- persistent forward kernel: k(x, y) for many pairs.
//
// Work unit ("ticket") = one 64-row strip of one pair.  Workgroups (one
// wavefront each) claim tickets from a global counter in an order in which
// every strip's producer (the strip below it) has a smaller ticket, so a
// waiting wave always waits on a wave that is already running (no deadlock
// for any grid size).  Gram mode interleaves pairs strip-major (all pairs'
// strip 0, then strip 1, ...); table mode takes the host-built order.
//
// Compiled once per (P, D) variant: -DSIGK_P=<order> -DSIGK_D=<channel bucket>;
// -DSIGK_SQ=1 builds the square-truncation variant (the paper's fixed-order
// tile matrix, selected by SIGK_FLAG_SQUARE) under the launcher names
// launch_fwdsq_P_D / occupancy_fwdsq_P_D; -DSIGK_ALT=1 the variant with the
// other frontier chunk width (alt_chunk_cols) as launch_fwdt_P_D /
// occupancy_fwdt_P_D; -DSIGK_LONE=1 the 64-column tile for one wave per SIMD
// (SIGK_FWDL_VARIANTS) as launch_fwdl_P_D / occupancy_fwdl_P_D.
#include "sigk_strip.h"
#include "sigk_team.h"

#ifndef SIGK_P
#define SIGK_P 8
#endif
#ifndef SIGK_D
#define SIGK_D 8
#endif
#ifndef SIGK_SQ
#define SIGK_SQ 0
#endif
#ifndef SIGK_ALT
#define SIGK_ALT 0
#endif
#ifndef SIGK_LONE
#define SIGK_LONE 0
#endif

namespace sigk {

template <int P, int D, bool SQ, int CH, bool LONE = false>
__global__ void __launch_bounds__(kWave)
    __attribute__((amdgpu_waves_per_eu(LONE ? 1 : fwd_tile_waves(P, D, CH)))) fwd_kernel(FwdArgs a) {
    // Two waves per SIMD share the CU's LDS with eight waves: a narrower ring
    // at order 10 where d > 8, the frontier written 32 columns at a time.
    constexpr bool kTwo = !LONE && fwd_tile_waves(P, D, CH) == 2;
    // The 32-column tile of a variant whose default is 64 keeps that one's ring
    // and depths, and the form of one wave per SIMD its depths: launches may
    // take any of them and give the same values.
    constexpr bool kNarrow = CH == 32 && D > 0 && fwd_chunk_cols(P, D) == 64;
    constexpr int INC = kNarrow || LONE ? inc_chunk<64, chunk64_ring(P, D)> : 0;
    constexpr int RB = LONE ? 128 : CH == 64 || kNarrow ? chunk64_ring(P, D) : ring_cols(P);
    constexpr int TC = kTwo ? 32 : CH;
    __shared__ LdsStrip<P, D, CH, RB, TC> L;
    Acc acc;
    const int lane = lane_id();
    for (unsigned round = 0;; ++round) {
        unsigned t = round;
        if (!a.solo) {
            if (lane == 0) t = atomicAdd(&a.hdr->ticket, 1u);
            t = (unsigned)uniform((int)t);
        }
        if ((int64_t)t >= a.ntickets) break;
        if (!a.solo && uniform((int)(load_status(a.hdr) & SIGK_ERR_WATCHDOG))) break;
        int pair, strip;
        if (a.mode == kModeGram) {
            pair = (int)((int64_t)t % a.npairs);
            strip = (int)((int64_t)t / a.npairs);
        } else {
            pair = a.tickets[t].pair;
            strip = a.tickets[t].strip;
            if (pair < 0) break;  // unused slots close a table built on the device
        }
        Geo g = resolve(a, pair, P, 0);
        StripCtx<P, D, CH, RB, SQ, false, TC, INC, (P <= 8 || LONE)> S(a, g, L, acc, strip);
        S.pair = pair;
        S.Fout = a.frontier + g.front;
        S.Fin = S.Fout;
        S.prog = a.progress + g.prog;
        S.ck = nullptr;
        S.ckq = nullptr;
        S.ck_every = 1;
        if (!S.sweep()) break;
    }
    finish_forward(a, acc, true);
}

#define SIGK_CAT3(a, b, c) a##b##_##c
#define SIGK_NAME(pre, P, D) SIGK_CAT3(pre, P, D)

#if SIGK_LONE
#define SIGK_LAUNCH launch_fwdl_
#define SIGK_OCC occupancy_fwdl_
#elif SIGK_SQ
#define SIGK_LAUNCH launch_fwdsq_
#define SIGK_OCC occupancy_fwdsq_
#elif SIGK_ALT
#define SIGK_LAUNCH launch_fwdt_
#define SIGK_OCC occupancy_fwdt_
#else
#define SIGK_LAUNCH launch_fwd_
#define SIGK_OCC occupancy_fwd_
#endif
constexpr int kChunk = SIGK_LONE  ? 64
                       : SIGK_ALT ? alt_chunk_cols(SIGK_P, SIGK_D)
                                  : fwd_chunk_cols(SIGK_P, SIGK_D);

hipError_t SIGK_NAME(SIGK_LAUNCH, SIGK_P, SIGK_D)(const FwdArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((fwd_kernel<SIGK_P, SIGK_D, SIGK_SQ != 0, kChunk, SIGK_LONE != 0>), dim3(grid),
                       dim3(kWave), 0, s, a);
    return hipGetLastError();
}

int SIGK_NAME(SIGK_OCC, SIGK_P, SIGK_D)() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, fwd_kernel<SIGK_P, SIGK_D, SIGK_SQ != 0, kChunk, SIGK_LONE != 0>, kWave, 0) != hipSuccess)
        return 0;
    return nb;
}

#if !SIGK_SQ && !SIGK_ALT && !SIGK_LONE
hipError_t SIGK_NAME(launch_team_, SIGK_P, SIGK_D)(const FwdArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((team_kernel<SIGK_P, SIGK_D>), dim3(grid), dim3(kWave * (a.team + 1)),
                       (team_lds_bytes<SIGK_P, SIGK_D>(a.team)), s, a);
    return hipGetLastError();
}

// (asked once per device and team size, before any launch of that size.  The
// kernel's dynamic LDS limit is shared by all host threads: always the largest
// team's, so that no call lowers it between another's setting and launch)
int SIGK_NAME(occupancy_team_, SIGK_P, SIGK_D)(int waves) {
    constexpr int kMax = team_max_waves<SIGK_P, SIGK_D>;
    if (waves < 0) return kMax;
    int nb = 0;
    if (hipFuncSetAttribute((const void*)team_kernel<SIGK_P, SIGK_D>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)team_lds_bytes<SIGK_P, SIGK_D>(kMax)) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, team_kernel<SIGK_P, SIGK_D>, kWave * (waves + 1),
            team_lds_bytes<SIGK_P, SIGK_D>(waves)) != hipSuccess)
        return 0;
    return nb;
}
#endif

}  // namespace sigk
