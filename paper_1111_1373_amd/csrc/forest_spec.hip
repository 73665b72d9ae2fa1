// Forest speculative walk (kernel templates in forest_impl.hpp).
#include "forest_impl.hpp"
#include "tiles.hpp"

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

template <int PITCH_VECS>
const void *spec_rows(const ForestShape &s) {
    return spec_tile<dev::RowTile<kXF32, false, 0, kTileRows, 16 * PITCH_VECS + 4>>(s);
}

}  // namespace

const void *forest_spec_kernel(const ForestShape &s) {
    if (s.tile.mode == kLoadFlat)
        return s.tile.row_vecs > kMaxForestPitchVecs
                   ? spec_tile<dev::RowTile<kXF32, true, 0, kTileRows>>(s)
                   : nullptr;
    if (s.tile.mode == kLoadRows) {
        switch (s.tile.row_vecs > kMaxForestPitchVecs ? 0 : forest_pitch_vecs(s.tile.row_vecs)) {
            case 0: return spec_tile<dev::RowTile<kXF32, false, 0, kTileRows>>(s);
            case 1: return spec_rows<1>(s);
            case 2: return spec_rows<2>(s);
            case 4: return spec_rows<4>(s);
            case 8: return spec_rows<8>(s);
            case 12: return spec_rows<12>(s);
            case 16: return spec_rows<16>(s);
            default: return nullptr;
        }
    }
    switch (s.tile.row_stride) {
        case 4: return spec_exact<4>(s);
        case 8: return spec_exact<8>(s);
        case 16: return spec_exact<16>(s);
        case 32: return spec_exact<32>(s);
        default: return nullptr;
    }
}

}  // namespace dtree
