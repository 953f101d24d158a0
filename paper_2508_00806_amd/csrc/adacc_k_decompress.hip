// Instantiations of the decompression kernels (single tensor and batch).
#include "adacc_kernels.hpp"

namespace adacc {
namespace ADACC_DT_NS {

template <int BITS, bool ASYM>
static DecompressFn pick(bool f32, bool generic) {
  if (generic) return f32 ? decompress_kernel<BITS, ASYM, true, true> : decompress_kernel<BITS, ASYM, false, true>;
  return f32 ? decompress_kernel<BITS, ASYM, true, false> : decompress_kernel<BITS, ASYM, false, false>;
}
DecompressFn decompress_fn(uint32_t bits, uint32_t asym, bool f32, bool generic) {
  if (bits == 4) return asym ? pick<4, true>(f32, generic) : pick<4, false>(f32, generic);
  return asym ? pick<8, true>(f32, generic) : pick<8, false>(f32, generic);
}

BatchDecompressFn decompress_batch_fn(bool f32) {
  return f32 ? decompress_batch_kernel<true> : decompress_batch_kernel<false>;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
