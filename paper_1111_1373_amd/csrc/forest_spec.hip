// Forest speculative walk (kernel templates in forest_impl.hpp).
#include "forest_impl.hpp"

namespace dtree {
namespace {

// The speculative one reads across a record: row-major tiles, which keep no prefetch unless
// they are exact (its registers would not fit 16 wavefronts per CU).
template <class Tile>
const void *spec_tile(const ForestShape &s) {
    if (s.depth == 2) return for_tables<int32_t, Tile, 2>(s.split > 0, s.tables_in_lds, s.vote_words);
    if (s.depth == 4) return for_tables<int32_t, Tile, 4>(s.split > 0, s.tables_in_lds, s.vote_words);
    return nullptr;
}

template <int RS>
const void *spec_exact(const ForestShape &s) {
    return spec_tile<dev::ExactTile<kXF32, RS, dev::kRowMajor, kTileRows>>(s);
}

}  // namespace

const void *forest_spec_kernel(const ForestShape &s) {
    if (s.tile.vecs != 0 && s.tile.mode != kLoadExact) return nullptr;
    if (s.tile.mode == kLoadFlat) return spec_tile<dev::RowTile<kXF32, true, 0, kTileRows>>(s);
    // rows of 61 to 64 features: a constant pitch (the rounds' rows are instruction offsets)
    if (s.tile.mode == kLoadRows && s.tile.lds_pitch == 260)
        return spec_tile<dev::RowTile<kXF32, false, 0, kTileRows, 260>>(s);
    if (s.tile.mode == kLoadRows) return spec_tile<dev::RowTile<kXF32, false, 0, kTileRows>>(s);
    switch (s.tile.row_stride) {
        case 4: return spec_exact<4>(s);
        case 8: return spec_exact<8>(s);
        case 16: return spec_exact<16>(s);
        case 32: return spec_exact<32>(s);
        default: return nullptr;
    }
}

}  // namespace dtree
