// The convolution kernels of conv_core.h for one storage type (a source of its own so that the three compile side by side).
#include "conv_core.h"

namespace xc {
hipError_t launch_conv_bf16(const ConvParams &P, hipStream_t st) { return launch_conv_dt<XCONV_BF16>(P, st); }
}  // namespace xc
