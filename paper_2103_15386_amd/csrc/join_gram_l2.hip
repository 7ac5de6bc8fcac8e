// The builds of the float32 matrix-core join for squared L2.
#include "join_gram.hpp"

namespace gnnd {
template void launch_gram_builds<kL2F32>(const Shape&, const DevState&, int, unsigned, hipStream_t);
}  // namespace gnnd
