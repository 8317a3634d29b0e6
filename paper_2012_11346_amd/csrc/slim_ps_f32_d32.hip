// Chunk kernels of the explicit prefix-sum mode: float rows, d = 32.
#include "slim_ps.hpp"

namespace slim {
namespace ps {
template hipError_t launch_rows_t<float, 32>(int which, const PsArgs& a, int nwg, hipStream_t s);
}
}  // namespace slim
