// The fallback kernels for group sizes the tile kernels do not take.
#include "adacc_generic.hpp"
#include "adacc_fn.hpp"

namespace adacc {
namespace ADACC_DT_NS {

// several TOPK groups: their segments are of at most 4096 elements, two octets per thread
template <int SL>
static CompressFn pick(uint32_t tile_elems, uint32_t mode, uint32_t gs) {
  if (mode == kModeNone) return compress_generic_kernel<SL, (int)kModeNone>;
  if (mode == kModeAbs) return compress_generic_kernel<SL, (int)kModeAbs>;
  if (mode == kModeStd) return compress_generic_kernel<SL, (int)kModeStd>;
  if constexpr (SL == 2) {
    if (gs < tile_elems) return gs <= kShortGroup ? compress_generic_kernel<SL, (int)kModeTopk> : compress_generic_kernel<SL, kSegTopkLong>;
  }
  return compress_generic_kernel<SL, kSegTopkWhole>;
}
template <int SL>
static CompressFn pick_place(uint32_t tile_elems, uint32_t mode, uint32_t gs) {
  if (mode == kModeAbs) return place_generic_kernel<SL, (int)kModeAbs>;
  if (mode == kModeStd) return place_generic_kernel<SL, (int)kModeStd>;
  if constexpr (SL == 2) {
    if (gs < tile_elems) return gs <= kShortGroup ? place_generic_kernel<SL, (int)kModeTopk> : place_generic_kernel<SL, kSegTopkLong>;
  }
  return place_generic_kernel<SL, kSegTopkWhole>;
}
static uint32_t slices_of(uint32_t tile_elems) {  // octets per thread
  const uint32_t slices = ((tile_elems + 7u) / 8u + kSegThreads - 1u) / kSegThreads;
  return slices <= 2u ? 2u : slices <= 4u ? 4u : slices <= 6u ? 6u : 8u;
}
CompressFn compress_generic_fn(uint32_t tile_elems, uint32_t mode, uint32_t gs) {
  switch (slices_of(tile_elems)) {
    case 2u: return pick<2>(tile_elems, mode, gs);
    case 4u: return pick<4>(tile_elems, mode, gs);
    case 6u: return pick<6>(tile_elems, mode, gs);
    default: return pick<8>(tile_elems, mode, gs);
  }
}
CompressFn place_generic_fn(uint32_t tile_elems, uint32_t mode, uint32_t gs) {
  switch (slices_of(tile_elems)) {
    case 2u: return pick_place<2>(tile_elems, mode, gs);
    case 4u: return pick_place<4>(tile_elems, mode, gs);
    case 6u: return pick_place<6>(tile_elems, mode, gs);
    default: return pick_place<8>(tile_elems, mode, gs);
  }
}
uint32_t generic_threads() { return kSegThreads; }
uint32_t generic_lds_bytes(uint32_t tile_elems, uint32_t gq, bool topk_groups) {
  const uint32_t n_oct = slices_of(tile_elems) * kSegThreads, n_grp = (tile_elems + gq - 1u) / gq;
  const uint32_t words = 8u * n_oct + 8u * n_grp;     // a, b, g0, g1
  const uint32_t patterns = topk_groups ? 24u * n_oct : 0u;  // 16-bit patterns and a byte per element
  return kSegHeadBytes + (words > patterns ? words : patterns);
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
