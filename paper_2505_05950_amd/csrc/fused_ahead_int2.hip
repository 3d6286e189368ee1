// The fused small-batch kernel (fused_ffn.h) for INT2 codes, the widest rows with consumers one entry ahead.
#include "fused_ffn.h"

namespace floe {

hipError_t launch_fused_ahead_int2(const FusedArgs& a, hipStream_t stream) { return fused_launch_ahead<2>(a, stream); }

}  // namespace floe
