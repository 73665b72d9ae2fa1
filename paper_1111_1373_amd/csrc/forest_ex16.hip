// Forest data walk with int16 exit codes (kernel templates in forest_impl.hpp).
#include "forest_impl.hpp"

namespace dtree {

const void *forest_ex16_kernel(const ForestShape &s) { return forest_data_kernel<int16_t>(s); }

}  // namespace dtree
