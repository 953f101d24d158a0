// Instantiations of the decompression kernels (single tensor and batch).
#include "adacc_kernels.hpp"

namespace adacc {
namespace ADACC_DT_NS {

template <int BITS, bool ASYM>
static DecompressFn pick(bool f32, bool generic, uint32_t rows) {
  if (f32) {
    switch (rows) {
      case 2: return generic ? decompress_kernel<BITS, ASYM, true, true, 2> : decompress_kernel<BITS, ASYM, true, false, 2>;
      case 4: return generic ? decompress_kernel<BITS, ASYM, true, true, 4> : decompress_kernel<BITS, ASYM, true, false, 4>;
      default: return generic ? decompress_kernel<BITS, ASYM, true, true, 8> : decompress_kernel<BITS, ASYM, true, false, 8>;
    }
  }
  if (generic) return decompress_kernel<BITS, ASYM, false, true, 4>;  // (no smaller pieces there: piece_rows)
  return rows == 2u ? decompress_kernel<BITS, ASYM, false, false, 2> : decompress_kernel<BITS, ASYM, false, false, 4>;
}
DecompressFn decompress_fn(uint32_t bits, uint32_t asym, bool f32, bool generic, uint32_t rows) {
  if (bits == 4) return asym ? pick<4, true>(f32, generic, rows) : pick<4, false>(f32, generic, rows);
  return asym ? pick<8, true>(f32, generic, rows) : pick<8, false>(f32, generic, rows);
}

BatchDecompressFn decompress_batch_fn(bool f32) {
  return f32 ? decompress_batch_kernel<true> : decompress_batch_kernel<false>;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
