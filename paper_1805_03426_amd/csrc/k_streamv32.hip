// Instantiation of the streaming step's variants (FP32).
#include "stream_variant.h"

namespace mr {
namespace stream {
template hipError_t launch_stream_var<float>(int, int, dim3, const VarArgs<float>&, hipStream_t);
}  // namespace stream
}  // namespace mr
