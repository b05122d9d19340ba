// Stream-K decode kernels for bf16 with head_dim 64 (matrix-core fold) and for
// fp32 (VALU fold).
#include "pa_stream_kernel.h"

namespace pa {

template const void* stream_pick<uint16_t, 64, false>(int, int, int);
template const void* stream_pick<float, 128, false>(int, int, int);
template const void* stream_pick<float, 64, false>(int, int, int);

}  // namespace pa
