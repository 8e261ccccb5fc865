// Which logical workgroup a workgroup of a launch takes. Workgroups are handed
// to the 8 XCDs in turn (workgroup b to XCD b mod 8), and each XCD has its own
// L2: neighbouring groups of cells, which share sources and tree nodes, should
// meet in one. Plain integer code: the tests build it for the host.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define RCB_XCD __host__ __device__ __forceinline__
#else
#define RCB_XCD inline
#endif

namespace rcb {

constexpr uint32_t kXcds = 8;
// the same cells either way: groups of 8 leaves
constexpr uint32_t kXcdLeaves = 64, kXcdGroups = 8;   // run of a launch over leaves, over groups

// Workgroup b of nb: XCD x takes runs of `run` logical workgroups in turn with
// the others, and what is left after the last full round, or all of a launch of
// fewer than 4096 runs, in one contiguous range. A bijection on [0, nb) for any nb.
// Contiguous eighths of an uneven cloud leave XCDs idle for a quarter of the
// launch (25M clumpy particles, contiguous / runs of 16, 64, 128, 256, 1024,
// 4096 leaves: FP64 gravity 52.1 / 41.7, 42.4, 43.4, 43.3, 46.2, 47.3 ms,
// neighbours 17.1 / 14.7, 14.8, 14.8, 15.1, 15.8, 16.0 ms; 1e8, contiguous / 64:
// 250 / 160 ms and 76 / 56 ms; 4M Plummer, mixed gravity in the same order
// 7.1 / 7.1, 7.0, 7.0, 7.1, 7.4, 8.2 ms). Below, the eighths even out within 2%,
// and the L2s hold more of a range than of runs (131,072 leaves: VJP 5.52 / 5.65 ms
// by runs of 64; 8192 of 61 particles: neighbours 0.87 / 0.90 ms).
RCB_XCD uint32_t xcd_slot(uint32_t b, uint32_t nb, uint32_t run) {
    const uint32_t x = b % kXcds, j = b / kXcds;
    const uint32_t full = nb < 4096 * run ? 0 : nb / (kXcds * run);   // rounds of a run per XCD
    if (j < full * run) return (j / run * kXcds + x) * run + j % run;
    const uint32_t o = full * run, rest = nb - o * kXcds, q = rest / kXcds, r = rest % kXcds;
    return o * kXcds + x * q + (x < r ? x : r) + (j - o);
}

}  // namespace rcb
#undef RCB_XCD
