// One kernel of each kind of weight staging, compiled to assembly by tests/test_kernel_forms.py.
#include "prom_pw_stream.h"
#include "prom_pw_rows.h"

namespace prom {
template __global__ void pw_stream_kernel<3, 1, 8, false, false, kEpiPlain>(const PwArgs);

__global__ __launch_bounds__(256) void rows_staging(const PwArgs a, v4i *out)
{
    __shared__ v4i frag[24 * 64], lpar[24 * 16];
    stage_weights_rows<6>(a, 0, a.KS, 4, blockDim.x, false, frag, lpar);
    for (int i = threadIdx.x; i < 24 * 64; i += blockDim.x) out[i] = frag[i] + lpar[i & 127];
}
}  // namespace prom
