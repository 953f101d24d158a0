// Instantiations of the one-launch compression of short tensors, ABS.
#include "adacc_fn.hpp"
#include "adacc_short.hpp"

namespace adacc {
namespace ADACC_DT_NS {

CompressShortFn compress_short_fn_abs(bool e8) { return e8 ? compress_short_kernel<kModeAbs, 8, false> : compress_short_kernel<kModeAbs, 4, false>; }

}  // namespace ADACC_DT_NS
}  // namespace adacc
