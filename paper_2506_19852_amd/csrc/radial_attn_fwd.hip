// Forward entry of the library: the kernel template of radial_attn_fwd_kernel.h without trace records.
#include "radial_attn_fwd_kernel.h"
#include "radial_attn_fwd_two.h"

namespace radial {

int launch_fwd(int D, int block, const FwdArgs& a, hipStream_t stream) { return fwd::launch_any<false>(D, block, a, stream); }

}  // namespace radial
