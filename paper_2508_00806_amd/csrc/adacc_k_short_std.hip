// Instantiations of the one-launch compression of short tensors, STD.
#include "adacc_fn.hpp"
#include "adacc_short.hpp"

namespace adacc {
namespace ADACC_DT_NS {

CompressShortFn compress_short_fn_std(bool e8, bool rowwise) {
  if (e8) return compress_short_kernel<kModeStd, 8, false, false>;
  return rowwise ? compress_short_kernel<kModeStd, 4, true, false> : compress_short_kernel<kModeStd, 4, false, false>;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
