// The block attention kernel at head dim 64 for workgroups of 64 Query rows and 2 key groups.
#include "block_attn_kernel.h"

namespace tr {
template hipError_t launch_attn_shape<64, 2, 2>(const AttnParams&, int, dim3, hipStream_t);
}  // namespace tr
