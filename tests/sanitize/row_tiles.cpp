// The record tiles of any width, stride and alignment (csrc/row_tile.hpp with the shapes of
// csrc/tiles.hpp), built for the host under AddressSanitizer and driven lane by lane: the
// input and the LDS tile are heap blocks of exactly their sizes, so a vector that leaves
// either one ends the run; then every feature of every staged record is read back through
// the addresses the walks use.
//   row_tiles SEED CASES
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <vector>

#include "row_tile.hpp"
#include "tiles.hpp"

using namespace dtree;

namespace {

std::mt19937_64 rng;
int pick(int lo, int hi) { return int(lo + rng() % uint64_t(hi - lo + 1)); }

void fail(const char *what, int xt, int F, int64_t ld, int64_t n, int mode, int off) {
    std::printf("%s: type %d F %d ld %lld n %lld mode %d offset %d\n", what, xt, F, (long long)ld,
                (long long)n, mode, off);
    std::exit(1);
}

template <int XT, bool FLAT, int NV, int TR, int PITCH = row_tile_pitch(NV, TR)>
void drive(const Rows &in, const TileShape &s, int off, int parts = 1) {
    using Tile = dev::RowTile<XT, FLAT, NV, TR, PITCH>;
    using T = typename Tile::T;
    const T *x = static_cast<const T *>(in.x);
    const int64_t end = Tile::prefetch_end(in);
    for (int64_t t = 0; t < in.n_tiles; ++t) {
        for (int way = 0; way < 2; ++way) {
            const bool prefetched = way == 0;
            if (prefetched && (!Tile::kPrefetch || t >= end)) continue;
            std::unique_ptr<dev::f32x4[]> mem(new dev::f32x4[size_t(s.tile_bytes / 16)]);
            float *tile = reinterpret_cast<float *>(mem.get());
            if (prefetched) {
                std::vector<Tile> lanes(64);
                for (int l = 0; l < 64; ++l) lanes[size_t(l)].load(in, t, l);
                for (int l = 0; l < 64; ++l) lanes[size_t(l)].store(in, tile, l);
            } else {
                for (int pass = 0; pass < 2; ++pass)   // lanes of a wavefront run together: the
                    for (int part = 0; part < parts; ++part)   // element loads follow every
                        for (int l = 0; l < 64; ++l)           // vector
                            Tile::stage(in, tile, t, l, part, parts);
            }
            for (int r = 0; r < TR && t * TR + r < in.n; ++r)
                for (int f = 0; f < in.n_features; ++f) {
                    const T want = x[(t * TR + r) * in.ld + f];
                    typename dev::Node<XT>::S slot{};
                    if constexpr (XT == kXF32) slot.f = 4 * f;
                    else slot = uint32_t(f) << 16;
                    const T a = dev::feature_at<XT, 1>(Tile::row(in, tile, r), slot, 0);
                    const T b = Tile::at(in, tile, r / 2, r - r / 2, slot);
                    if (std::memcmp(&a, &want, sizeof(T)) || std::memcmp(&b, &want, sizeof(T)))
                        fail(prefetched ? "prefetched tile" : "staged tile", XT, in.n_features,
                             in.ld, in.n, s.mode, off);
                }
        }
    }
}

// Column-major tiles of the forest kernels, staged by one to four wavefronts.
template <bool FLAT, int NV>
void drive_columns(const Rows &in, const TileShape &s, int off, int parts) {
    using Tile = dev::ColTile<FLAT, NV>;
    const float *x = static_cast<const float *>(in.x);
    const int64_t end = Tile::prefetch_end(in);
    for (int64_t t = 0; t < in.n_tiles; ++t) {
        std::unique_ptr<dev::f32x4[]> mem(new dev::f32x4[size_t(s.tile_bytes / 16)]);
        float *tile = reinterpret_cast<float *>(mem.get());
        if (Tile::kPrefetch && t < end) {
            std::vector<Tile> lanes(64);
            for (int l = 0; l < 64; ++l) lanes[size_t(l)].load(in, t, l);
            for (int l = 0; l < 64; ++l) lanes[size_t(l)].store(in, tile, l);
        } else {
            for (int pass = 0; pass < 2; ++pass)
                for (int part = 0; part < parts; ++part)
                    for (int l = 0; l < 64; ++l) Tile::stage(in, tile, t, l, part, parts);
        }
        for (int r = 0; r < kTileRows && t * kTileRows + r < in.n; ++r)
            for (int f = 0; f < in.n_features; ++f)
                if (std::memcmp(&tile[f * kTileRows + r], &x[(t * kTileRows + r) * in.ld + f], 4))
                    fail("column tile", kXF32, in.n_features, in.ld, in.n, s.mode, off);
    }
}

// Row tiles of the speculative forest kernels, staged by one to sixteen wavefronts: classes of
// a constant pitch, and wide rows with their own.
void forest_rows(const void *x, int64_t n, int64_t ld, int F, int off) {
    int mode = forest_load_mode(kAlgoSpec, x, ld, F);
    if (mode == kLoadExact) mode = kLoadRows;
    const TileShape s = forest_tile_shape(kAlgoSpec, F, mode, false);
    const Rows in = make_tile_rows(x, kXF32, n, ld, F, s);
    const int parts = 1 << pick(0, 4);
    if (s.tile_bytes % 16 != 0) fail("forest tile size", kXF32, F, ld, n, mode, off);
    if (mode == kLoadFlat) {
        if (F <= 4 * kMaxForestPitchVecs) fail("flat forest tile", kXF32, F, ld, n, mode, off);
        drive<kXF32, true, 0, kTileRows>(in, s, off, parts);
    } else if (s.row_vecs > kMaxForestPitchVecs) {
        drive<kXF32, false, 0, kTileRows>(in, s, off, parts);
    } else {
        switch (forest_pitch_vecs(s.row_vecs)) {
            case 1: drive<kXF32, false, 0, kTileRows, 20>(in, s, off, parts); break;
            case 2: drive<kXF32, false, 0, kTileRows, 36>(in, s, off, parts); break;
            case 4: drive<kXF32, false, 0, kTileRows, 68>(in, s, off, parts); break;
            case 8: drive<kXF32, false, 0, kTileRows, 132>(in, s, off, parts); break;
            case 12: drive<kXF32, false, 0, kTileRows, 196>(in, s, off, parts); break;
            case 16: drive<kXF32, false, 0, kTileRows, 260>(in, s, off, parts); break;
            default: fail("no pitch class", kXF32, F, ld, n, mode, off);
        }
    }
}

void columns(const void *x, int64_t n, int64_t ld, int F, int mode, int off) {
    if (mode == kLoadExact) mode = kLoadRows;
    const TileShape s = forest_tile_shape(kAlgoData, F, mode, pick(0, 1) == 0);
    const Rows in = make_tile_rows(x, kXF32, n, ld, F, s);
    const bool flat = mode == kLoadFlat;
    const int parts = s.vecs ? 1 : 1 << pick(0, 2);
    switch (s.vecs) {
        case 0: flat ? drive_columns<true, 0>(in, s, off, parts) : drive_columns<false, 0>(in, s, off, parts); break;
        case 2: flat ? drive_columns<true, 2>(in, s, off, parts) : drive_columns<false, 2>(in, s, off, parts); break;
        case 4: flat ? drive_columns<true, 4>(in, s, off, parts) : drive_columns<false, 4>(in, s, off, parts); break;
        case 6: flat ? drive_columns<true, 6>(in, s, off, parts) : drive_columns<false, 6>(in, s, off, parts); break;
        case 8: flat ? drive_columns<true, 8>(in, s, off, parts) : drive_columns<false, 8>(in, s, off, parts); break;
        default: fail("no column tile class", kXF32, F, ld, n, mode, off);
    }
}

template <int XT, bool FLAT, bool CONST, int NV, int TR>
void drive_class(const Rows &in, const TileShape &s, int off) {
    drive<XT, FLAT, NV, TR, CONST ? row_tile_pitch(NV, TR) : 0>(in, s, off);
}

template <int XT, bool FLAT, bool CONST, int TR>
bool by_vecs(const Rows &in, const TileShape &s, int off) {
    switch (s.vecs) {
        case 0: drive_class<XT, FLAT, CONST, 0, TR>(in, s, off); return true;
        case 2: drive_class<XT, FLAT, CONST, 2, TR>(in, s, off); return true;
        case 3: drive_class<XT, FLAT, CONST, 3, TR>(in, s, off); return true;
        case 4: drive_class<XT, FLAT, CONST, 4, TR>(in, s, off); return true;
        case 6: drive_class<XT, FLAT, CONST, 6, TR>(in, s, off); return true;
        case 8: drive_class<XT, FLAT, CONST, 8, TR>(in, s, off); return true;
        case 12: drive_class<XT, FLAT, CONST, 12, TR>(in, s, off); return true;
        case 16: drive_class<XT, FLAT, CONST, 16, TR>(in, s, off); return true;
        default: return false;
    }
}

template <int XT, bool FLAT, bool CONST>
bool by_rows(const Rows &in, const TileShape &s, int off) {
    switch (s.tile_rows) {
        case 64: return by_vecs<XT, FLAT, CONST, 64>(in, s, off);
        case 32: return by_vecs<XT, FLAT, CONST, 32>(in, s, off);
        case 16: return by_vecs<XT, FLAT, CONST, 16>(in, s, off);
        default: return false;
    }
}

template <int XT>
void one_case() {
    using T = typename dev::Elem<XT>::T;
    const int F = pick(0, 2) ? pick(1, 40) : pick(1, kMaxRowStride);
    int64_t ld = F + (pick(0, 1) ? 0 : pick(0, 5) ? pick(0, 9) : pick(0, 700));
    const int64_t n = pick(0, 3) ? pick(1, 200) : pick(1, 20);
    // a single record may come with any stride, also one whose bytes no 64-bit number holds
    if (n == 1 && pick(0, 1)) ld = std::max<int64_t>(ld, INT64_MAX >> pick(0, 40)) - pick(0, 1);
    // elements before the first record: any, or only those of the word it lies in, whose bytes
    // may be read; of the others none is
    const int per_word = 4 / int(sizeof(T));
    const int off = pick(0, 1) ? 0 : pick(0, 1) ? pick(0, per_word - 1) : pick(0, 15);
    // the block starts on a 16-byte boundary and ends with the last record's last feature
    const size_t count = size_t(off) + size_t((n - 1) * ld + F);
    std::unique_ptr<T[]> block(new T[count]);
    for (size_t i = 0; i < count; ++i) {
        const uint64_t v = rng();
        std::memcpy(&block[i], &v, sizeof(T));
    }
    const void *x = block.get() + off;
    const int algos[] = {kAlgoData, kAlgoSpec, kAlgoPath};
    const int algo = algos[XT == kXF32 ? pick(0, 2) : pick(0, 1)];
    const int depth = pick(1, 6);
    int mode = tree_load_mode(algo, x, XT, ld, F, depth);
    if (XT == kXF32) {
        columns(x, n, ld, F, load_mode_for(x, XT, ld, F), off);
        forest_rows(x, n, ld, F, off);
    }
    if (mode == kLoadExact) mode = kLoadRows;           // such rows come strided, too
    const TileShape s = tile_shape(algo, XT, F, mode, depth);
    if (s.tile_bytes % 16 != 0) fail("tile size", XT, F, ld, n, mode, off);
    const Rows in = make_tile_rows(x, XT, n, ld, F, s);
    const bool ok = mode == kLoadFlat ? by_rows<XT, true, false>(in, s, off)
                    : constant_pitch(algo, XT, mode, depth) ? by_rows<XT, false, true>(in, s, off)
                                                            : by_rows<XT, false, false>(in, s, off);
    if (!ok) fail("no tile class", XT, F, ld, n, mode, off);
}

// Every base of fp32 records, those between words among them, has a plan of a forest, whose
// tiles start at the LDS tile's first word.
void forest_bases() {
    for (int F : {1, 3, 4, 8, 19, 32, 64, 256})
        for (int pad : {0, 1, 4})
            for (uintptr_t base = 4096; base < 4112; ++base) {
                const void *x = reinterpret_cast<const void *>(base);
                for (int algo : {kAlgoData, kAlgoSpec}) {
                    const int mode = forest_load_mode(algo, x, F + pad, F);
                    if (mode < 0 || mode >= kForestLoadModes ||
                        (mode == kLoadFlat && (F % 4 == 0 || (algo == kAlgoSpec && F <= 64))) ||
                        (mode == kLoadExact && (base % 16 != 0 || F > 32)))
                        fail("forest plan", kXF32, F, F + pad, 0, mode, int(base % 16));
                    const TileShape s = forest_tile_shape(algo, F, mode, false);
                    if (make_tile_rows(x, kXF32, 100, F + pad, F, s).lds_off != 0)
                        fail("forest tile base", kXF32, F, F + pad, 0, mode, int(base % 16));
                }
            }
}

}  // namespace

int main(int argc, char **argv) {
    forest_bases();
    rng.seed(argc > 1 ? std::strtoull(argv[1], nullptr, 10) : 1);
    const int cases = argc > 2 ? std::atoi(argv[2]) : 1000;
    for (int i = 0; i < cases; ++i) {
        switch (i % 4) {
            case 0: one_case<kXF32>(); break;
            case 1: one_case<kXF16>(); break;
            case 2: one_case<kXBF16>(); break;
            default: one_case<kXU8>(); break;
        }
    }
    std::printf("ok %d\n", cases);
    return 0;
}
