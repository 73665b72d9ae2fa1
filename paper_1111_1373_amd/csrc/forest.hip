// gfx950 forest kernels: majority vote of many trees over every record (kernel templates in
// forest_impl.hpp).  This unit holds the data walk's instances for int32 exit codes, the
// choice among the units and the launch.
#include "forest_impl.hpp"

namespace dtree {

const void *forest_kernel_for(const ForestShape &s) {
    if (s.algo != kAlgoData) return forest_spec_kernel(s);
    switch (s.exit_mode) {
        case kExitInt32: return forest_data_kernel<int32_t>(s);
        case kExitInt16: return forest_ex16_kernel(s);
        case kExitPacked: return forest_packed_kernel(s);
        case kExitList: return forest_list_kernel(s);
        default: return nullptr;
    }
}

hipError_t launch_forest(const void *fn, const FArgs &args, int blocks, int lds_bytes,
                         hipStream_t stream) {
    FArgs a = args;
    void *params[] = {&a};
    return hipLaunchKernel(fn, dim3(unsigned(blocks)), dim3(unsigned(args.waves * 64)), params,
                           size_t(lds_bytes), stream);
}

}  // namespace dtree
