// Forest speculative walk (kernel templates in forest_impl.hpp).
#include "forest_impl.hpp"

namespace dtree {

const void *forest_spec_kernel(const ForestShape &s) { return forest_spec_kernel_impl(s); }

}  // namespace dtree
