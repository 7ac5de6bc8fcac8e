// The builds of the float32 matrix-core join for the angular distance.
#include "join_gram.hpp"

namespace gnnd {
template void launch_gram_builds<kAngularF32>(const Shape&, const DevState&, int, unsigned, hipStream_t);
}  // namespace gnnd
