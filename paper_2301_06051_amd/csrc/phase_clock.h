// Optional instrumentation of the layer kernel, compiled in only with -DDSVT_PHASE_CLOCKS (the library that
// `python -m paper_2301_06051_amd.phase_clocks` builds beside the product library; the product build has none of
// it): thread 0 of every workgroup notes the shader clock at the phase boundaries of every tile, and
// dsvt_debug_phase_clocks copies the notes of the last launch to the host.  Not part of the C-ABI in dsvt.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#ifdef DSVT_PHASE_CLOCKS
constexpr int kPhaseSlots = 12, kPhaseTiles = 2048;
__device__ unsigned long long dsvt_phase_clk[kPhaseTiles][kPhaseSlots];
#define DSVT_PHASE(tile, i)                                                              \
  do {                                                                                   \
    if (threadIdx.x == 0 && (tile) < kPhaseTiles) dsvt_phase_clk[tile][i] = clock64();    \
  } while (0)
// out: [kPhaseTiles][kPhaseSlots] shader-clock values (host memory); synchronises the device first.
extern "C" int dsvt_debug_phase_clocks(unsigned long long* out, int32_t* tiles, int32_t* slots) {
  if (!out || !tiles || !slots) return -1;
  *tiles = kPhaseTiles;
  *slots = kPhaseSlots;
  if (hipDeviceSynchronize() != hipSuccess) return -3;
  return hipMemcpyFromSymbol(out, HIP_SYMBOL(dsvt_phase_clk), sizeof(unsigned long long) * kPhaseTiles * kPhaseSlots) == hipSuccess ? 0 : -3;
}
#else
#define DSVT_PHASE(tile, i) do {} while (0)
#endif
