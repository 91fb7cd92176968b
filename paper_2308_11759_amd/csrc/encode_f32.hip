// encode_f32.hip -- the compression kernels for float32 fields.
#include "encode_device.hpp"

namespace pmc {

template hipError_t launch_encode<float>(const FieldJob&, hipStream_t);
template hipError_t launch_encode_batch<float>(const BatchArgs&, uint32_t, hipStream_t);

}  // namespace pmc
