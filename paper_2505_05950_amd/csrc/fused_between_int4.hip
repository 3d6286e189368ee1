// The fused kernel's INT4 instances for widths between the powers of two (fused_ffn.h).
#include "fused_ffn.h"

namespace floe {

hipError_t launch_fused_between_int4(const FusedArgs& a, hipStream_t stream) { return fused_launch_between<4>(a, stream); }

}  // namespace floe
