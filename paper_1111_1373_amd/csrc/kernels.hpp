// Interface between the host library (dtree.hip) and the gfx950 kernels (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace dtree {

// kAlgoList: the data decomposition over a node list (single trees)
enum KernelAlgo { kAlgoData = 0, kAlgoSpec = 1, kAlgoPath = 2, kAlgoList = 3 };

constexpr int kTileRows = 64;          // records per wavefront tile (one per lane)
constexpr int kMaxRowStride = 256;     // LDS row stride limit in floats (n_features <= 256)
constexpr int kMaxWavesPerBlock = 8;   // kernels are built for <= 512 threads, except:
// forest instances whose registers fit 16 wavefronts per CU without spilling (data walk,
// speculative walk with depth-2 windows), built for <= 1024.  `depth` is the speculative
// window depth (unused for data).
constexpr int kMaxForestWavesPerBlock = 16;
__host__ __device__ constexpr int forest_max_waves(int algo, int depth) {
    return algo == 0 || depth == 2 ? kMaxForestWavesPerBlock : kMaxWavesPerBlock;
}
constexpr int kMaxForestTrees = 255;   // 8-bit vote counters
constexpr int kMaxForestClasses = 64;  // 16 VGPRs of packed counters

// Record element types (values of dt_dtype).  Each widens exactly to fp32.
enum ElemType { kXF32 = 0, kXF16 = 1, kXBF16 = 2, kXU8 = 3, kElemTypes = 4 };

__host__ __device__ constexpr int elem_bytes(int xt) { return xt == kXF32 ? 4 : xt == kXU8 ? 1 : 2; }

// The record matrix a kernel reads.
struct Rows {
    const void *x;           // device records, row-major, elements of the kernel's type
    int64_t n;               // records
    int64_t ld;              // row stride in elements
    int64_t n_tiles;         // tiles of the records
    int32_t n_features;      // F
    uint32_t magic_f;        // ceil(2^32 / F) for F >= 2 (row = idx / F via mulhi)
    // row tiles
    int64_t row_pitch;       // bytes from row to row in the input
    int64_t row_gap;         // row_pitch - 16 * row_vecs
    int32_t row_vecs;        // 16-byte vectors of a row
    uint32_t magic_v;        // ceil(2^32 / row_vecs) for row_vecs >= 2
    int32_t tile_vecs;       // 16-byte vectors of a full tile
    int32_t lds_pitch;       // bytes from row to row in the LDS tile
    int32_t lds_off;         // first byte of row 0 in the LDS tile: x modulo 4
    int32_t short_rows;      // last rows of the input whose last vector would leave it
};

// Single-tree kernel arguments (passed by value).
struct KArgs {
    Rows in;
    const int4 *slots;       // n_slots (threshold, feature) pairs, 8 bytes each; list_kernel:
                             // the node list, slot_bytes of it staged in the LDS
    const int4 *exits;       // n_slots int32 exit codes
    int32_t slot_bytes;      // bytes of the slot region (multiple of 16)
    int32_t exit_bytes;      // bytes of the exit region (multiple of 16)
    int32_t depth;           // window depth D
    int32_t levels;          // windows on the longest path
    int32_t waves;           // wavefronts per workgroup
    int32_t out_kind;        // 0: uint8 output, 1: int32 output
    int32_t out_cap;         // tiles of results each wavefront buffers in the LDS (>= 1)
    int32_t tile_bytes;      // LDS bytes of a wavefront's record tile (multiple of 16)
    int32_t out_vec;         // 1: `out` is 16-byte aligned (flushes use 16-byte stores)
    int32_t want_leaf;       // list_kernel: 1: results are leaf indices, 0: classes
    int32_t hops;            // path-reduction kernel: further entries read per round
    void *out;
};

// Path-reduction kernel: per wavefront, 64/S segments of 2S path entries (S lanes each).
constexpr int kPathIntsPerWave = 128;

// Records per wavefront tile of a kernel on exact rows: 64 (one per lane), except for the
// speculative kernel with 32- and 64-slot windows (depths 5 and 6) on rows of at least 32
// bytes in the LDS.  That kernel reads one or two record rows per round, so a tile of 32
// records serves it as well while taking half the LDS, and twice as many wavefronts then
// fit next to its window tables.  (Rows under 32 bytes keep 64 records: 16-byte staging
// needs one vector per lane.)
__host__ __device__ constexpr int exact_tile_rows(int algo, int depth, int row_bytes) {
    return algo == kAlgoSpec && depth >= 5 && row_bytes >= 32 ? 32 : kTileRows;
}

// Largest workgroup of a single-tree kernel instance, in wavefronts: 8, or 16 for the
// speculative walk of wide windows on small tiles (at most 32 prefetch registers per lane),
// whose registers (at most 128 per lane) fit 16 wavefronts per CU and whose tiles leave the
// LDS room for them.
__host__ __device__ constexpr int tree_max_waves(int algo, int depth, int tile_rows,
                                                 int prefetch_regs) {
    return algo == kAlgoSpec && depth >= 5 && tile_rows < kTileRows && prefetch_regs <= 32
               ? 16
               : kMaxWavesPerBlock;
}

// LDS bytes of one wavefront's result buffer: cap tiles of `tile_rows` results of
// out_bytes each.
__host__ __device__ inline int out_buffer_bytes(int cap, int out_bytes, int tile_rows = kTileRows) {
    return cap * tile_rows * out_bytes;
}

// How a forest's data walk finds its exits: int32 or int16 tables of codes, codes packed
// into the windows' bottom slots, or no windows at all but lists of nodes.
enum ExitMode { kExitInt32 = 0, kExitInt16 = 1, kExitPacked = 2, kExitList = 3 };

// Forest kernel arguments.  Tree k's tables are the bytes [off_k, off_k + slot_bytes_k)
// (slots or nodes) followed by its exit codes, if they are a table, inside `tables`;
// trees[k] = {off_k, slot_bytes_k, levels_k, 0} (node lists: the tree's depth for levels).
// Chunks are runs of consecutive trees staged into the LDS together:
// chunks[c] = {first_tree, end_tree, byte_off, bytes}.
struct FArgs {
    Rows in;
    const int4 *tables;
    const int4 *trees;
    const int2 *roots;       // per tree: the root slot {threshold bits, feature byte offset}
    const int4 *chunks;
    int64_t first_tile;      // tiles [first_tile, end_tile) (forest_kernel: from 0)
    int64_t end_tile;
    int32_t n_chunks;
    int32_t table_lds_bytes; // LDS bytes reserved for one chunk (0: tables read in place)
    int32_t tile_bytes;      // LDS bytes of a record tile (multiple of 16)
    int32_t split;           // 2^split wavefronts per tile (0: forest_kernel)
    int32_t depth;           // window depth D (every tree)
    int32_t n_classes;
    int32_t waves;
    int32_t out_kind;        // 0: uint8 output, 1: int32 output
    void *out;
};

// How record tiles are read from HBM.  Single-tree kernels:
//   kLoadExact  dense rows of a power of two of words (4 to 64), 16-byte aligned base
//   kLoadFlat   other dense rows whose width is no multiple of 16 bytes, 4-byte-aligned base
//   kLoadRows   other rows that all start on 4-byte boundaries
//   kLoadBytes  rows (of narrow records) that start between words
// Narrow fp32 rows of large windows are kLoadRows also where they could be flat (flat_rows).
// Forest kernels use kLoadFlat (the speculative ones for more than 64 features), kLoadRows,
// and kLoadExact for rows of 4 to 32 fp32 features.
enum LoadMode { kLoadFlat = 0, kLoadRows = 1, kLoadExact = 2, kLoadBytes = 3, kLoadModes = 4 };
constexpr int kForestLoadModes = 3;

// Row widths of the exact tiles, in 4-byte words: from one 16-byte vector per row to 64
// (wider rows would need 16 KiB and more of registers per wavefront: row tiles of fewer
// records).
constexpr int kMinExactWords = 4;
constexpr int kMaxExactWords = 64;
constexpr int kMaxVecs = 16;          // prefetch vectors per lane

// LDS bytes from row to row of fp32 row tiles of `vecs` prefetch vectors per lane and
// `tile_rows` records (not flat ones): the widest rows of the class and a word.  0 without
// prefetch, where the width is not a class.
__host__ __device__ constexpr int row_tile_pitch(int vecs, int tile_rows) {
    return vecs > 0 ? 16 * (vecs * 64 / tile_rows) + 4 : 0;
}

// Record tile of a single-tree kernel.
struct TileShape {
    int mode = kLoadRows;
    int row_stride = 0;     // kLoadExact: elements per row
    int tile_rows = 0;      // records per tile
    int row_bytes = 0;      // bytes of a row's features
    int vecs = 0;           // row tiles: prefetch vectors per lane (0: none)
    int row_vecs = 0;       // row tiles: 16-byte vectors of a row
    int tile_vecs = 0;      // row tiles: vectors of a full tile
    int lds_pitch = 0;      // LDS bytes from row to row (kLoadBytes: less the input pitch
                            // modulo 4, known at the call)
    int tile_bytes = 0;     // LDS bytes of the tile (multiple of 16)
    int prefetch_regs = 0;  // registers per lane that hold the next tile
};

// Kernel instance for (algorithm, record element type, record tile, tables staged in the
// LDS or read from global memory, window depth), or nullptr if no such instance exists.
// `depth` is ignored by the data kernel.
const void *kernel_for(int algo, int elem_type, const TileShape &shape, bool tables_in_lds,
                       int depth);

// Per element type (one translation unit each): data and speculative kernel instances.
const void *kernel_for_f32(int algo, const TileShape &shape, bool tables_in_lds, int depth);
const void *kernel_for_f16(int algo, const TileShape &shape, bool tables_in_lds, int depth);
const void *kernel_for_bf16(int algo, const TileShape &shape, bool tables_in_lds, int depth);
const void *kernel_for_u8(int algo, const TileShape &shape, bool tables_in_lds, int depth);

// Path-reduction kernel instance (fp32 records, speculative windows of depth 1..6).
const void *path_kernel_for(const TileShape &shape, bool tables_in_lds, int depth);

// Forest kernel instance.
struct ForestShape {
    int algo = kAlgoData;
    TileShape tile;
    bool tables_in_lds = true;
    int vote_words = 2;      // 32-bit words of packed 8-bit counters: 2, 4 or 16 for up to
                             // 8, 16 or 64 classes
    int depth = 0;           // window depth
    int exit_mode = kExitInt32;   // data walk
    int split = 0;           // 2^split wavefronts per tile
};
const void *forest_kernel_for(const ForestShape &s);
// The instances by kind (translation units of their own).
const void *forest_ex16_kernel(const ForestShape &s);
const void *forest_packed_kernel(const ForestShape &s);
const void *forest_list_kernel(const ForestShape &s);
const void *forest_spec_kernel(const ForestShape &s);

// One-time per-instance setup (raise the dynamic LDS limit to the device maximum).
hipError_t prepare_kernel(const void *fn, int max_lds_bytes);

// Launches: grid of `blocks` workgroups of args.waves wavefronts.
hipError_t launch_kernel(const void *fn, const KArgs &args, int blocks, int lds_bytes,
                         hipStream_t stream);
hipError_t launch_forest(const void *fn, const FArgs &args, int blocks, int lds_bytes,
                         hipStream_t stream);

// Dynamic LDS of a workgroup of `waves` wavefronts: tables, one record tile per wavefront,
// then (single-tree kernels) one result buffer of `out_bytes_per_wave` per wavefront.
inline int lds_bytes_for(int table_bytes, int tile_bytes, int waves, int out_bytes_per_wave = 0) {
    return table_bytes + waves * (tile_bytes + out_bytes_per_wave);
}

}  // namespace dtree
