// Host-side choice of the record tiles (see LoadMode and TileShape in kernels.hpp).
#pragma once

#include <algorithm>
#include <cstdint>

#include "kernels.hpp"

namespace dtree {

constexpr int64_t align16(int64_t b) { return (b + 15) & ~int64_t(15); }

// Whether a single-tree call copies dense rows of `n_features` as one run of bytes (flat
// tiles), from a 4-byte-aligned base.  Not so windows of 8 lanes and more on narrow fp32
// rows: their rounds are the time there, and are shorter where a row's pitch is a constant
// (complete tree of depth 10, 3,000,000 records: depth 4, 3 features 43 us flat and 35 us
// row by row, 19 features 66 and 47 us; depth 6, 3 features 74 and 64 us).  Smaller windows
// and wider rows are bound by the stream (65,536 x 38: 6 us flat, 7 us).
constexpr bool flat_rows(int algo, int elem_type, int n_features, int depth) {
    if (n_features * elem_bytes(elem_type) % 16 == 0) return false;
    return !(algo == kAlgoSpec && elem_type == kXF32 && depth >= 3 && n_features <= 32);
}

// Whether the LDS pitch of a single tree's row tiles is that of the widest rows of the class,
// a constant: fp32 rows, and narrow rows that start on words where the rounds are the time
// (windows of 8 lanes and more: 48 uint8 features, 3,000,000 records, depth 6, 80 us with a
// row's own pitch, 70 us with the class's; 48 fp16 features, depth 4, 60 and 52 us).
constexpr bool constant_pitch(int algo, int elem_type, int mode, int depth) {
    return mode == kLoadRows && (elem_type == kXF32 || (algo == kAlgoSpec && depth >= 3));
}

// Record tile of a single-tree kernel for load mode `mode` (see LoadMode).  Row tiles hold
// 64 records, or, so that a tile stays within kMaxVecs prefetch vectors per lane, 32 or 16
// of wide rows.  The speculative walk of wide windows (depths 5 and 6) starts from 32, as
// on exact rows; the path kernel walks 64 at a time and leaves the prefetch out instead.
constexpr TileShape tile_shape(int algo, int elem_type, int n_features, int mode, int depth) {
    TileShape s;
    s.mode = mode;
    const int es = elem_bytes(elem_type);
    const int row_bytes = n_features * es;
    s.row_bytes = row_bytes;
    if (mode == kLoadExact) {
        s.row_stride = n_features;
        s.tile_rows = exact_tile_rows(algo, depth, row_bytes);
        s.lds_pitch = row_bytes;
        s.tile_bytes = s.tile_rows * row_bytes;
        s.prefetch_regs = s.tile_bytes / 256;
        return s;
    }
    const bool flat = mode == kLoadFlat, bytes = mode == kLoadBytes;
    s.row_vecs = (row_bytes + (bytes ? 3 : 0) + 15) / 16;   // a row starts within its first word
    const auto vecs_of = [&](int rows) { return flat ? rows * row_bytes / 16 : rows * s.row_vecs; };
    s.tile_rows = algo == kAlgoSpec && depth >= 5 ? 32 : kTileRows;
    while (algo != kAlgoPath && vecs_of(s.tile_rows) > 64 * kMaxVecs) s.tile_rows /= 2;
    s.tile_vecs = vecs_of(s.tile_rows);
    for (int v : {2, 3, 4, 6, 8, 12, kMaxVecs}) {
        if (v * 64 < s.tile_vecs) continue;
        s.vecs = v;
        break;
    }
    s.prefetch_regs = 4 * s.vecs;
    s.lds_pitch = flat ? row_bytes
                       : constant_pitch(algo, elem_type, mode, depth) && s.vecs > 0
                           ? row_tile_pitch(s.vecs, s.tile_rows)
                           : 16 * s.row_vecs + 4;
    s.tile_bytes = int(align16(s.tile_rows * (s.lds_pitch + (bytes ? 3 : 0)) + (bytes ? 3 : 0)));
    return s;
}

// Whether tile_shape gives row tiles of this class (flat or not, with a constant pitch or not,
// prefetch vectors, records) for any width of rows: the instances that are compiled.
constexpr bool row_class_used(int algo, int elem_type, int depth, bool flat, bool constant,
                              int vecs, int tile_rows) {
    for (int f = 1; f <= kMaxRowStride; ++f) {
        for (int mode : {kLoadFlat, kLoadRows, kLoadBytes}) {
            if ((mode == kLoadFlat) != flat) continue;
            if (flat && !flat_rows(algo, elem_type, f, depth)) continue;
            if (mode == kLoadBytes && elem_type == kXF32) continue;
            if (constant_pitch(algo, elem_type, mode, depth) != constant) continue;
            const TileShape s = tile_shape(algo, elem_type, f, mode, depth);
            if (s.vecs == vecs && s.tile_rows == tile_rows) return true;
        }
    }
    return false;
}

inline bool exact_rows(int32_t n_features, int elem_bytes) {
    const int words = n_features * elem_bytes / 4;
    return (n_features & (n_features - 1)) == 0 && words >= kMinExactWords &&
           words <= kMaxExactWords;
}

// Load path of a call for the layout of the features (see LoadMode).
inline int load_mode_for(const void *d_x, int elem_type, int64_t ld, int32_t n_features) {
    const int es = elem_bytes(elem_type);
    // fp32 rows start on their own words, also off a base between words (forest calls take
    // those; the loads then are off 4-byte boundaries, which global memory allows)
    const bool words = es == 4 || reinterpret_cast<uintptr_t>(d_x) % 4 == 0;
    if (ld != n_features || !words) return words && ld % 4 * es % 4 == 0 ? kLoadRows : kLoadBytes;
    if ((n_features * es) % 16 != 0) return kLoadFlat;
    return exact_rows(n_features, es) && (reinterpret_cast<uintptr_t>(d_x) & 15u) == 0
               ? kLoadExact
               : kLoadRows;
}

// Load path of a single-tree call with windows of `depth` levels.
inline int tree_load_mode(int algo, const void *d_x, int elem_type, int64_t ld, int32_t n_features,
                          int depth) {
    const int mode = load_mode_for(d_x, elem_type, ld, n_features);
    return mode == kLoadFlat && !flat_rows(algo, elem_type, n_features, depth) ? int(kLoadRows)
                                                                               : mode;
}

inline uint32_t magic_div(int32_t d) {
    return d >= 2 ? uint32_t(((uint64_t(1) << 32) + uint64_t(d) - 1) / uint64_t(d)) : 0u;
}

// A single record's stride is never used and may be any number; more records have none
// whose bytes overflow (no memory holds them), and 2^60 elements stand for such a one.
inline Rows make_rows(const void *d_x, int64_t n, int64_t ld, int32_t n_features,
                      int tile_rows = kTileRows) {
    Rows r{};
    r.x = d_x;
    r.n = n;
    r.ld = n > 1 ? std::min(ld, int64_t(1) << 60) : n_features;
    r.n_tiles = (n + tile_rows - 1) / tile_rows;
    r.n_features = n_features;
    r.magic_f = magic_div(n_features);
    return r;
}

// Records of a single-tree call, for the tile `s`.
inline Rows make_tile_rows(const void *d_x, int elem_type, int64_t n, int64_t ld,
                           int32_t n_features, const TileShape &s) {
    Rows r = make_rows(d_x, n, ld, n_features, s.tile_rows);
    const int es = elem_bytes(elem_type);
    r.row_pitch = r.ld * es;
    r.row_vecs = s.row_vecs;
    r.row_gap = r.row_pitch - 16 * s.row_vecs;
    r.magic_v = magic_div(s.row_vecs);
    r.tile_vecs = s.tile_vecs;
    r.lds_pitch = s.lds_pitch + (s.mode == kLoadBytes ? int32_t(r.row_pitch % 4) : 0);
    r.lds_off = es == 4 ? 0 : int32_t(reinterpret_cast<uintptr_t>(d_x) % 4);
    // bytes that a row's vectors read past its end: row i's stay inside the input when at
    // least that many bytes follow it there, (n - 1 - i) * row_pitch of them
    const int64_t over = s.mode == kLoadRows || s.mode == kLoadBytes
                             ? int64_t(16) * s.row_vecs - n_features * es
                             : 0;
    r.short_rows = int32_t((over + r.row_pitch - 1) / r.row_pitch);
    return r;
}

// Row tiles of the speculative forest walk: 16-byte vectors of the LDS pitch for rows of
// `row_vecs`.  Its rounds read 64 / S rows, a constant number of rows apart, so that with a
// constant pitch a round's row is an instruction offset.  Hence classes, as far as the widest
// class leaves the LDS 8 tiles; wider rows keep their own pitch, a register.  Measured with
// 50 complete trees of depth 7, 1,000,001 records, windows of depth 4 (of depth 2), a row's
// own pitch against the class's: 3 features 380 and 288 us (273 and 249), 20 features 391 and
// 310 us (286 and 256), 36 features 435 and 355 us (323 and 294).
constexpr int kMaxForestPitchVecs = 16;
constexpr int forest_pitch_vecs(int row_vecs) {
    for (int v : {1, 2, 4, 8, 12, kMaxForestPitchVecs})
        if (row_vecs <= v) return v;
    return row_vecs;
}

// Record tile of a forest kernel: 64 fp32 records.  Prefetched tiles (unsplit kernels) take
// up to 8 vectors per lane, as many registers as 16 wavefronts per CU leave; the
// speculative walk has them for exact tiles only.  The data walk's tiles are column-major.
inline TileShape forest_tile_shape(int algo, int n_features, int mode, bool prefetch) {
    TileShape s;
    s.mode = mode;
    s.tile_rows = kTileRows;
    s.row_bytes = n_features * 4;
    if (mode == kLoadExact) {
        s.row_stride = n_features;
        s.tile_bytes = kTileRows * s.row_bytes;
        return s;
    }
    const bool flat = mode == kLoadFlat;
    s.row_vecs = (s.row_bytes + 15) / 16;
    s.tile_vecs = flat ? kTileRows * s.row_bytes / 16 : kTileRows * s.row_vecs;
    if (prefetch && algo == kAlgoData)
        for (int v : {2, 4, 6, 8}) {
            if (v * 64 < s.tile_vecs) continue;
            s.vecs = v;
            break;
        }
    s.lds_pitch = flat ? s.row_bytes : 16 * forest_pitch_vecs(s.row_vecs) + 4;
    s.tile_bytes = kTileRows * (algo == kAlgoData ? s.row_bytes : s.lds_pitch);
    return s;
}

// Load path of a forest call.  The speculative walk takes dense rows of up to 64 features one
// by one too: flat tiles have no constant pitch (see forest_pitch_vecs; 3 features 383 us
// flat, 290 us as rows of one vector).
inline int forest_load_mode(int algo, const void *d_x, int64_t ld, int32_t n_features) {
    const int mode = load_mode_for(d_x, kXF32, ld, n_features);
    if (mode == kLoadExact && n_features > 32) return kLoadRows;
    return mode == kLoadFlat && algo == kAlgoSpec && n_features <= 4 * kMaxForestPitchVecs
               ? int(kLoadRows)
               : mode;
}

}  // namespace dtree
