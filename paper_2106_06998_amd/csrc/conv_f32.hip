// The convolution kernels of conv_core.h for one storage type (a source of its own so that the three compile side by side).
#include "conv_core.h"

namespace xc {
hipError_t launch_conv_f32(const ConvHead &P, const ConvSub *sub, hipStream_t st) { return launch_conv_dt<XCONV_F32>(P, sub, st); }
}  // namespace xc
