// Instantiation of the streaming step's variants (FP64).
#include "stream_variant.h"

namespace mr {
namespace stream {
template hipError_t launch_stream_var<double>(int, int, dim3, const VarArgs<double>&, hipStream_t);
}  // namespace stream
}  // namespace mr
