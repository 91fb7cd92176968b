// decode_f64.hip -- the retrieval kernels for float64 fields.
#include "decode_device.hpp"

namespace pmc {

template hipError_t launch_decode<double>(const DecArgs<double>&, uint64_t, int, bool, const SplitArgs*, hipStream_t);
template hipError_t launch_decode_box<double>(const DecArgs<double>&, const BoxArgs&, uint64_t, int, bool, const SplitArgs*, hipStream_t);
template hipError_t launch_decode_tiles<double>(const DecArgs<double>&, int, hipStream_t);
template hipError_t launch_decode_queries<double>(const ServeArgs&, uint64_t, int, bool, hipStream_t);

}  // namespace pmc
