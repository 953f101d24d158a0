// Instantiations of the one-launch compression of short tensors, TOPK.
#include "adacc_fn.hpp"
#include "adacc_short.hpp"

namespace adacc {
namespace ADACC_DT_NS {

CompressShortFn compress_short_fn_topk(bool e8, bool whole) {
  if (e8) return whole ? compress_short_kernel<kModeTopk, 8, true> : compress_short_kernel<kModeTopk, 8, false>;
  return whole ? compress_short_kernel<kModeTopk, 4, true> : compress_short_kernel<kModeTopk, 4, false>;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
