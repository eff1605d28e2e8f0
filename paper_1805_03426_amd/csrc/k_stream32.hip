// Instantiation of the streaming step's kernels (FP32).
#include "stream_kernel.h"

namespace mr {
namespace stream {
template hipError_t launch_stream<float, false>(int, int, dim3, const StreamArgs<float>&, hipStream_t);
template hipError_t launch_stream<float, true>(int, int, dim3, const StreamArgs<float>&, hipStream_t);
}  // namespace stream
}  // namespace mr
