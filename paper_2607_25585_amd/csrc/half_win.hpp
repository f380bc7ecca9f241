// The walk over L2 windows shared by the spin-1/2 and general window kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "ftlm_internal.hpp"

namespace ftlm {

// Scatters the low bits of x to the set bits of mask (ascending).
__device__ __forceinline__ uint32_t scatter_bits(uint32_t x, uint32_t mask) {
  uint32_t r = 0;
  while (mask) {
    const uint32_t low = mask & (0u - mask);
    if (x & 1u) r |= low;
    x >>= 1;
    mask &= mask - 1u;
  }
  return r;
}

// Work-item walk of one L2-window pass.  With at least 8 windows and a grid that
// is a multiple of 8, block b runs on XCD b % 8 (workgroups are dispatched to the
// XCDs round robin); XCD x owns windows x, x+8, ... and its blocks walk the
// items of those windows in order, so the windows an XCD works on at any time
// are consecutive in its list and their rows stay in that XCD's L2 (as many
// windows are in flight as the XCD's blocks cover: nb / nin).  Otherwise the
// items are walked flat.  body(win, item) is called for every item of the pass.
template <typename F>
__device__ __forceinline__ void win_walk(const WinPass &W, F &&body) {
  const bool xcd = W.nwin >= 8 && (gridDim.x & 7u) == 0;
  const uint32_t x = xcd ? (blockIdx.x & 7u) : 0u;
  const uint64_t nwx = xcd ? (uint64_t)((W.nwin - x + 7u) >> 3) : (uint64_t)W.nwin;
  const uint64_t jn = nwx * W.nin;
  const uint64_t jstart = xcd ? (blockIdx.x >> 3) : blockIdx.x;
  const uint64_t jstep = xcd ? (gridDim.x >> 3) : gridDim.x;
  for (uint64_t j = jstart; j < jn; j += jstep) {
    const uint32_t wl = (uint32_t)(j / W.nin);
    const uint32_t item = (uint32_t)(j - (uint64_t)wl * W.nin);
    body(xcd ? x + 8u * wl : wl, item);
  }
}

}  // namespace ftlm
