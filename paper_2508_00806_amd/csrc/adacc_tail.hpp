// The end of a tensor with outliers that its groups do not divide, by one workgroup.
#pragma once

#include "adacc_generic.hpp"

namespace adacc {
namespace ADACC_DT_NS {

// ---- the end of a tensor with outliers: d.tail elements behind d.numel, fewer than the larger group, at most one short
// statistics group cut into quantisation groups the last of which may be short.  A segment of the fallback kernels
// (they know short groups) of two octets per thread, done by a workgroup of its own next to those that place the
// tiles' outliers; its own go behind those of the tiles.  (One wavefront in a launch behind the placement, with plain
// loops over LDS arrays, took 14 us for 141 elements of a statistics group of 512, and 41 us for 1455 of one of 4096;
// now it is hidden behind the placement.)
constexpr int kTailOcts = 2;  // per thread: 4096 elements
constexpr uint32_t kTailLdsBytes = kSegHeadBytes + 4u * (2u * kTailOcts * kSegThreads + 2u * 4096u / 8u);
// before: the number of outliers in the tiles, called by every wavefront of the workgroup; FIRST: together with the loads, else
// behind the selection.
template <bool FIRST, class Before>
__device__ __forceinline__ void compress_tail(const TensorDesc& whole, Before&& before, unsigned char* lds) {
  TensorDesc d = whole;
  d.tile_elems = d.gs;  // the segment is one statistics group
  SegmentShared sh = segment_shared<kTailOcts>(lds, d.tile_elems, d.gq);
  SegmentGeo g;
  g.first_elem = d.numel;
  g.cnt = d.tail;
  g.octs = (d.tail + (uint32_t)kOct - 1u) / (uint32_t)kOct;
  g.full = false;
  uint32_t raw[kTailOcts][4], mask[kTailOcts], omag[kTailOcts];
  const bool works = threadIdx.x < (uint32_t)kSegThreads;  // whole wavefronts
  if (works) segment_load(d, g, raw);
  uint32_t total_main = 0u;
  if constexpr (FIRST) total_main = before();
  if (!works) return;  // wavefronts that only helped with that
#pragma unroll
  for (int j = 0; j < kTailOcts; ++j) omag[j] = octet_magnitude(raw[j]);
  segment_select<kTailOcts, kSegAny>(d, g, sh, raw, omag, mask);
#pragma unroll
  for (int j = 0; j < kTailOcts; ++j)
    if (omag[j] >= kNonfiniteMag) mask[j] |= octet_nonfinite(raw[j]);
  if constexpr (!FIRST) total_main = before();
  const uint32_t total = total_main + segment_emit(g, sh, raw, mask, StreamSink{d.idx, d.val}, total_main, d.cap);
  if (threadIdx.x == 0u) {
    if (d.n_tiles == 0u) d.tile_ptr[0] = 0u;
    d.tile_ptr[d.n_tiles_all] = total;
    d.status[0] = total; d.status[1] = total > d.cap ? 1u : 0u; d.status[2] = 0u; d.status[3] = 0u;
  }
#pragma unroll
  for (int j = 0; j < kTailOcts; ++j) {
    if (mask[j] != 0u) {
      clear_elements(raw[j], mask[j]);
      omag[j] = octet_magnitude(raw[j]);
    }
  }
  if (d.bits == 8u) {
    if (d.asym) segment_quantise<8, true, kTailOcts>(d, g, sh, raw, omag); else segment_quantise<8, false, kTailOcts>(d, g, sh, raw, omag);
  } else {
    if (d.asym) segment_quantise<4, true, kTailOcts>(d, g, sh, raw, omag); else segment_quantise<4, false, kTailOcts>(d, g, sh, raw, omag);
  }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
