// The block attention kernel at head dim 64 for workgroups of 128 Query rows, with two key groups and with one.
#include "block_attn_kernel.h"

namespace tr {
template hipError_t launch_attn_shape<64, 4, 2>(const AttnParams&, int, dim3, hipStream_t);
template hipError_t launch_attn_shape<64, 4, 1>(const AttnParams&, int, dim3, hipStream_t);
}  // namespace tr
