// encode_f64.hip -- the compression kernels for float64 fields.
#include "encode_device.hpp"

namespace pmc {

template hipError_t launch_encode<double>(const FieldJob&, hipStream_t);
template hipError_t launch_encode_batch<double>(const BatchArgs&, uint32_t, hipStream_t);

}  // namespace pmc
