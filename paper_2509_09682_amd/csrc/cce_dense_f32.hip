// Dense kernels of cce_dense_body.hpp for fp32 inputs.
#include "cce_dense_body.hpp"

namespace cce {
hipError_t launch_dense_f32(int pass, const DenseArgs &a, hipStream_t stream)
{
    return dense_by_width<float>(a.d, [&](auto kd) { return launch_dense_kd<float, decltype(kd)::value>(pass, a, stream); });
}
DenseShape dense_shape_f32(int pass, int d)
{
    return dense_by_width<float>(d, [&](auto kd) { return dense_shape_kd<float, decltype(kd)::value>(pass); });
}
}  // namespace cce
