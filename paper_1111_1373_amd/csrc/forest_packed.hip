// Forest data walk with exit codes packed into the windows' bottom slots (kernel templates
// in forest_impl.hpp).
#include "forest_impl.hpp"

namespace dtree {

const void *forest_packed_kernel(const ForestShape &s) { return forest_data_kernel<dev::PackedExits>(s); }

}  // namespace dtree
