// The block attention kernel at head dim 128 for workgroups of 256 Query rows.
#include "block_attn_kernel.h"

namespace tr {
template hipError_t launch_attn_shape<128, 8, 1>(const AttnParams&, int, dim3, hipStream_t);
}  // namespace tr
