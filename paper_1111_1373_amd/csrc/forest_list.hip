// Forest data walk over node lists (kernel templates in forest_impl.hpp).
#include "forest_impl.hpp"

namespace dtree {

const void *forest_list_kernel(const ForestShape &s) { return forest_data_kernel<dev::NodeList>(s); }

}  // namespace dtree
