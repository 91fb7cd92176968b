// decode_f32.hip -- the retrieval kernels for float32 fields.
#include "decode_device.hpp"

namespace pmc {

uint64_t stage_words() { return kStageWords; }

template hipError_t launch_decode<float>(const DecArgs<float>&, uint64_t, int, bool, const SplitArgs*, hipStream_t);
template hipError_t launch_decode_box<float>(const DecArgs<float>&, const BoxArgs&, uint64_t, int, bool, const SplitArgs*, hipStream_t);
template hipError_t launch_decode_tiles<float>(const DecArgs<float>&, int, hipStream_t);
template hipError_t launch_decode_queries<float>(const ServeArgs&, uint64_t, int, bool, hipStream_t);

}  // namespace pmc
