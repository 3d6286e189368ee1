// The fused kernel's INT3 instances for widths between the powers of two (fused_ffn.h).
#include "fused_ffn.h"

namespace floe {

hipError_t launch_fused_between_int3(const FusedArgs& a, hipStream_t stream) { return fused_launch_between<3>(a, stream); }

}  // namespace floe
