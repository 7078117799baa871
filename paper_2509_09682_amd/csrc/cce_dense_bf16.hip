// Dense kernels of cce_dense_body.hpp for bf16 inputs.
#include "cce_dense_body.hpp"

namespace cce {
hipError_t launch_dense_bf16(int pass, const DenseArgs &a, hipStream_t stream)
{
    return dense_by_width<uint16_t>(a.d, [&](auto kd) { return launch_dense_kd<uint16_t, decltype(kd)::value>(pass, a, stream); });
}
DenseShape dense_shape_bf16(int pass, int d)
{
    return dense_by_width<uint16_t>(d, [&](auto kd) { return dense_shape_kd<uint16_t, decltype(kd)::value>(pass); });
}
}  // namespace cce
