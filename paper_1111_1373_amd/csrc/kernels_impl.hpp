// gfx950 kernels for single-tree evaluation, templated on the record element type.  Each
// element type is instantiated in a translation unit of its own (kernels.hip: fp32,
// kernels_f16.hip, kernels_bf16.hip, kernels_u8.hip).
//
// The kernels are persistent: each wavefront owns a private tile of 64 records (32 or 16 of
// wide rows and for wide windows) in the LDS and walks a contiguous range of record tiles,
// keeping the loads of its next tile in flight in registers while it walks the current one,
// and writing its results in bursts from an LDS buffer.  The tree's window tables (see
// encode.hpp) are staged into the LDS once per workgroup, or, for trees whose tables do not
// fit next to the record tiles, read from global memory (L2-resident).  Records stay in their
// own element type in the LDS; every tree step widens the element it reads to fp32 and
// compares it with the fp32 threshold, which is the decision on the stored value.
//
//   data_kernel  (Section 3.2, Procedure 3): lane r evaluates record r of its tile.
//   list_kernel  the same over a list of the tree's nodes instead of windows.
//   spec_kernel  (Sections 3.3-3.4, Procedures 4-5): 2^D lanes evaluate all slots of a
//                record's current window at once; a wavefront ballot gathers the outcomes
//                and the exit is found by walking the bits.  The mask replaces the paper's
//                shared `path` array and its barrier-separated pointer jumping.
#pragma once

#include "device_common.hpp"
#include "tiles.hpp"

namespace dtree {
namespace {

using dev::Slot;

template <int XT, class Tile, bool TAB_LDS>
__global__ void __launch_bounds__(512) data_kernel(KArgs a) {
    extern __shared__ int4 lds[];
    const typename dev::Node<XT>::S *slots;
    const int32_t *exits;
    char *tiles = dev::bind_tables<TAB_LDS>(a, lds, slots, exits);
    const int lane = threadIdx.x & 63;
    float *tile;
    uint8_t *obuf;
    dev::wave_buffers(a, Tile::TR, tiles, tile, obuf);
    const int r = lane & (Tile::TR - 1);     // record walked by this lane
    const auto *row = Tile::row(a.in, tile, r);
    const int sw = Tile::swizzle(r);
    const typename dev::Node<XT>::S root0 = slots[1];   // window 0's root, for every record
    dev::tile_loop<Tile>(a, tile, obuf, lane, lane < Tile::TR ? lane : -1, [&]() -> int32_t {
        return ~dev::walk_data<XT>(slots, exits, a.depth, a.levels, row, sw, root0);
    });
}

// The data walk over a node list (see walk_list).
template <int XT, class Tile>
__global__ void __launch_bounds__(512) list_kernel(KArgs a) {
    extern __shared__ int4 lds[];
    dev::copy_to_lds(lds, a.slots, a.slot_bytes >> 4);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    float *tile;
    uint8_t *obuf;
    dev::wave_buffers(a, Tile::TR, reinterpret_cast<char *>(lds) + a.slot_bytes, tile, obuf);
    const int r = lane & (Tile::TR - 1);     // record walked by this lane
    const auto *row = Tile::row(a.in, tile, r);
    const int sw = Tile::swizzle(r);
    const int2 root = reinterpret_cast<const int2 *>(lds)[1];
    dev::tile_loop<Tile>(a, tile, obuf, lane, lane < Tile::TR ? lane : -1, [&]() -> int32_t {
        return dev::walk_list<XT>(lds, a.slots, a.slot_bytes >> 4, a.want_leaf != 0, row, sw, root);
    });
}

template <int XT, class Tile, bool TAB_LDS, int D>
__global__ void __launch_bounds__(64 * tree_max_waves(kAlgoSpec, D, Tile::TR, Tile::kRegs))
spec_kernel(KArgs a) {
    using NS = typename dev::Node<XT>::S;
    extern __shared__ int4 lds[];
    const NS *slots;
    const int32_t *exits;
    char *tiles = dev::bind_tables<TAB_LDS>(a, lds, slots, exits);
    const int lane = threadIdx.x & 63;
    float *tile;
    uint8_t *obuf;
    dev::wave_buffers(a, Tile::TR, tiles, tile, obuf);
    const dev::Spec<XT, D, Tile> spec(lane);
    const NS root = slots[spec.j];   // window 0 is shared by every record
    dev::tile_loop<Tile>(a, tile, obuf, lane, spec.record(), [&]() -> int32_t {
        return ~spec.run(slots, exits, a.levels, root, a.in, tile);
    });
}

// ---- instance tables ------------------------------------------------------------------
// Exact rows: the tile layout of an algorithm.  The speculative walk's 64- and 32-lane
// groups read one or two record rows per round: flat rows, so that a round's row is its
// group's first row plus a constant (an instruction offset; a per-row swizzle would be a
// per-round register).  Narrower groups read 64/S rows at once, and the swizzle keeps rows
// reading the same feature on distinct banks.
template <int XT, int RS, int D>   // D = 0: data walk
using Exact = dev::ExactTile<XT, RS, D >= 5 ? dev::kRowFlat : dev::kRowMajor,
                             exact_tile_rows(D == 0 ? kAlgoData : kAlgoSpec, D,
                                             RS * int(sizeof(typename dev::Elem<XT>::T)))>;

template <int XT, int RS, bool TAB_LDS>
const void *exact_for(int algo, int depth) {
    // the list kernel stages its list: there is none for tables read in place
    if (algo == kAlgoList) {
        if constexpr (TAB_LDS)
            return reinterpret_cast<const void *>(&list_kernel<XT, Exact<XT, RS, 0>>);
        else
            return nullptr;
    }
    if (algo == kAlgoData)
        return reinterpret_cast<const void *>(&data_kernel<XT, Exact<XT, RS, 0>, TAB_LDS>);
    switch (depth) {
        case 1: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 1>, TAB_LDS, 1>);
        case 2: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 2>, TAB_LDS, 2>);
        case 3: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 3>, TAB_LDS, 3>);
        case 4: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 4>, TAB_LDS, 4>);
        case 5: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 5>, TAB_LDS, 5>);
        case 6: return reinterpret_cast<const void *>(&spec_kernel<XT, Exact<XT, RS, 6>, TAB_LDS, 6>);
        default: return nullptr;
    }
}

template <int XT, int RS>
const void *exact_kernel(int algo, bool tab_lds, int depth) {
    constexpr int words = dev::row_words<XT, RS>();
    if constexpr (words < kMinExactWords || words > kMaxExactWords)
        return nullptr;
    else
        return tab_lds ? exact_for<XT, RS, true>(algo, depth) : exact_for<XT, RS, false>(algo, depth);
}

// One class of row tiles, where rows of some width have it.  (Data walk and node lists share
// their tiles, and so do the speculative windows of depths 1 and 2, 3 and 4, 5 and 6.)
template <int XT, bool FLAT, bool CONST, bool TAB_LDS, int NV, int TR>
const void *row_for(int algo, int depth) {
    using Tile = dev::RowTile<XT, FLAT, NV, TR, CONST ? row_tile_pitch(NV, TR) : 0>;
    if constexpr (row_class_used(kAlgoData, XT, 0, FLAT, CONST, NV, TR)) {
        if constexpr (TAB_LDS)
            if (algo == kAlgoList) return reinterpret_cast<const void *>(&list_kernel<XT, Tile>);
        if (algo == kAlgoData)
            return reinterpret_cast<const void *>(&data_kernel<XT, Tile, TAB_LDS>);
    }
    if (algo != kAlgoSpec) return nullptr;
    if constexpr (row_class_used(kAlgoSpec, XT, 1, FLAT, CONST, NV, TR)) {
        if (depth == 1) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 1>);
        if (depth == 2) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 2>);
    }
    if constexpr (row_class_used(kAlgoSpec, XT, 3, FLAT, CONST, NV, TR)) {
        if (depth == 3) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 3>);
        if (depth == 4) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 4>);
    }
    if constexpr (row_class_used(kAlgoSpec, XT, 5, FLAT, CONST, NV, TR)) {
        if (depth == 5) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 5>);
        if (depth == 6) return reinterpret_cast<const void *>(&spec_kernel<XT, Tile, TAB_LDS, 6>);
    }
    return nullptr;
}

template <int XT, bool FLAT, bool CONST, bool TAB_LDS, int TR>
const void *row_tile_for(int algo, int vecs, int depth) {
    switch (vecs) {
        case 2: return row_for<XT, FLAT, CONST, TAB_LDS, 2, TR>(algo, depth);
        case 3: return row_for<XT, FLAT, CONST, TAB_LDS, 3, TR>(algo, depth);
        case 4: return row_for<XT, FLAT, CONST, TAB_LDS, 4, TR>(algo, depth);
        case 6: return row_for<XT, FLAT, CONST, TAB_LDS, 6, TR>(algo, depth);
        case 8: return row_for<XT, FLAT, CONST, TAB_LDS, 8, TR>(algo, depth);
        case 12: return row_for<XT, FLAT, CONST, TAB_LDS, 12, TR>(algo, depth);
        case 16: return row_for<XT, FLAT, CONST, TAB_LDS, 16, TR>(algo, depth);
        default: return nullptr;
    }
}

template <int XT, bool FLAT, bool CONST, bool TAB_LDS>
const void *row_kernel(int algo, int vecs, int tile_rows, int depth) {
    switch (tile_rows) {
        case 64: return row_tile_for<XT, FLAT, CONST, TAB_LDS, 64>(algo, vecs, depth);
        case 32: return row_tile_for<XT, FLAT, CONST, TAB_LDS, 32>(algo, vecs, depth);
        case 16: return row_tile_for<XT, FLAT, CONST, TAB_LDS, 16>(algo, vecs, depth);
        default: return nullptr;
    }
}

template <int XT, bool FLAT, bool CONST>
const void *row_kernel_of(int algo, const TileShape &shape, bool tab_lds, int depth) {
    return tab_lds ? row_kernel<XT, FLAT, CONST, true>(algo, shape.vecs, shape.tile_rows, depth)
                   : row_kernel<XT, FLAT, CONST, false>(algo, shape.vecs, shape.tile_rows, depth);
}

template <int XT>
const void *single_tree_kernel(int algo, const TileShape &shape, bool tab_lds, int depth) {
    if (shape.mode == kLoadFlat) return row_kernel_of<XT, true, false>(algo, shape, tab_lds, depth);
    if (shape.mode != kLoadExact)
        return constant_pitch(algo, XT, shape.mode, depth)
                   ? row_kernel_of<XT, false, true>(algo, shape, tab_lds, depth)
                   : row_kernel_of<XT, false, false>(algo, shape, tab_lds, depth);
    switch (shape.row_stride) {
        case 4: return exact_kernel<XT, 4>(algo, tab_lds, depth);
        case 8: return exact_kernel<XT, 8>(algo, tab_lds, depth);
        case 16: return exact_kernel<XT, 16>(algo, tab_lds, depth);
        case 32: return exact_kernel<XT, 32>(algo, tab_lds, depth);
        case 64: return exact_kernel<XT, 64>(algo, tab_lds, depth);
        case 128: return exact_kernel<XT, 128>(algo, tab_lds, depth);
        case 256: return exact_kernel<XT, 256>(algo, tab_lds, depth);
        default: return nullptr;
    }
}

}  // namespace
}  // namespace dtree
