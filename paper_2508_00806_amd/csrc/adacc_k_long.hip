// The kernels for groups of more than half a segment, a wavefront per group.
#include "adacc_fn.hpp"
#include "adacc_long.hpp"

namespace adacc {
namespace ADACC_DT_NS {

template <int E, bool TOPK>
static CompressFn pick(uint32_t bits, uint32_t asym) {
  if (bits == 4) return asym ? compress_long_kernel<E, TOPK, 4, true> : compress_long_kernel<E, TOPK, 4, false>;
  return asym ? compress_long_kernel<E, TOPK, 8, true> : compress_long_kernel<E, TOPK, 8, false>;
}
CompressFn compress_long_fn(uint32_t tile_elems, uint32_t mode, uint32_t topk, uint32_t bits, uint32_t asym) {
  const uint32_t rows = (tile_elems + (uint32_t)kRow - 1u) / (uint32_t)kRow;
  // (nothing to select: [6144, 4000] 14.2 us by workgroups, 14.7 by wavefronts; [6144, 2200] 11.9 and 9.5)
  if (mode == kModeNone && rows > 6u) return nullptr;
  // (TOPK: more than 8 of the largest take rounds over all elements here, over the octets' largest there; us by workgroups and by
  // wavefronts, k = 9 / 16 / 32: [3072, 2200] 23.0 / 29.7 / 46.4 and 33.7 / 49.7 / 85.8, [8192, 4000] 53.4 / 70.4 / 113 and 76.1 / 117 / 209)
  if (mode == kModeTopk) {
    if (topk > 8u || rows > 22u) return nullptr;
    return rows <= 8u ? pick<8, true>(bits, asym) : rows <= 12u ? pick<12, true>(bits, asym) : rows <= 16u ? pick<16, true>(bits, asym) : pick<22, true>(bits, asym);
  }
  if (rows <= 8u) return pick<8, false>(bits, asym);
  // (ABS: [16000, 4104] 55.0 -> 44.3, [12000, 5160] 46.8 -> 42.2; [8000, 8192] 41.4 and 44.6, [8192, 11008] 61.9 and 59.7)
  if (mode != kModeStd && !(mode == kModeAbs && rows <= 12u)) return nullptr;
  // (STD int8 symmetric over 15 and 16 rows is the one that depends on the data: [8192, 8192] by workgroups and by wavefronts 38.4 and 41.4
  // without outliers, SiLU at 6 sigma 41.9 and 44.4, at 4 sigma 103 and 96, heavy-tailed channels at 6 sigma 50.6 and 46.6)
  if (rows <= 12u) return pick<12, false>(bits, asym);
  if (rows <= 16u) return pick<16, false>(bits, asym);
  if (rows <= 22u) return pick<22, false>(bits, asym);
  return nullptr;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
