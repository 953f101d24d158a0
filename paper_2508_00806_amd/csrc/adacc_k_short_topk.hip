// Instantiations of the one-launch compression of short tensors, TOPK.
#include "adacc_fn.hpp"
#include "adacc_short.hpp"

namespace adacc {
namespace ADACC_DT_NS {

CompressShortFn compress_short_fn_topk(bool e8, bool whole, bool rows) {
  if (e8) return whole ? compress_short_kernel<kModeTopk, 8, false, true> : compress_short_kernel<kModeTopk, 8, false, false>;
  if (rows) return compress_short_kernel<kModeTopk, 4, true, false>;
  return whole ? compress_short_kernel<kModeTopk, 4, false, true> : compress_short_kernel<kModeTopk, 4, false, false>;
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
