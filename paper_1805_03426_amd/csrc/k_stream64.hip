// Instantiation of the streaming step's kernels (FP64).
#include "stream_kernel.h"

namespace mr {
namespace stream {
template hipError_t launch_stream<double, false>(int, int, dim3, const StreamArgs<double>&, hipStream_t);
template hipError_t launch_stream<double, true>(int, int, dim3, const StreamArgs<double>&, hipStream_t);
}  // namespace stream
}  // namespace mr
