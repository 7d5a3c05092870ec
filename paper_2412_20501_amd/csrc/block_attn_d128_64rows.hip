// The block attention kernel at head dim 128 for workgroups of 64 Query rows and 2 key groups.
#include "block_attn_kernel.h"

namespace tr {
template hipError_t launch_attn_shape<128, 2, 2>(const AttnParams&, int, dim3, hipStream_t);
}  // namespace tr
