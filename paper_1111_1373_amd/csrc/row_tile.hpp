// Record elements, window-table slots, and the record tiles for rows of any width, stride
// and alignment.  Plain loads and stores only: the file also compiles for the host, where
// every address a tile stages is checked against the input's and the tile's bounds.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "kernels.hpp"

namespace dtree {
namespace dev {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct alignas(8) Slot {
    float t;
    int32_t f;   // byte offset of the feature in an fp32 row: 4 * feature index
};

// The two children 2p, 2p+1 of a heap slot: one aligned 16-byte LDS read.
struct alignas(16) Slot2 {
    Slot l, r;
};

// Word swizzle of row r for rows of RSW 4-byte words.
template <int RSW>
__device__ __forceinline__ int swz(int r) {
    if constexpr (RSW >= 64) {
        return r;                                  // r < 64 <= RSW
    } else {
        constexpr int sh = __builtin_ctz(64 / RSW);
        return (r >> sh) & (RSW - 1);
    }
}

// Record element types.  widen() is exact for every value (NaN stays NaN, fp16 and bf16
// subnormals become the same fp32 value), so a decision on a widened element is the
// decision on the value the element stores.
template <int XT> struct Elem;
template <> struct Elem<kXF32> {
    using T = float;
    static __device__ __forceinline__ float widen(float v) { return v; }
};
template <> struct Elem<kXF16> {
    using T = uint16_t;   // IEEE binary16 bits
    static __device__ __forceinline__ float widen(uint16_t b) {
        return float(__builtin_bit_cast(_Float16, b));
    }
};
template <> struct Elem<kXBF16> {
    using T = uint16_t;   // bfloat16 bits: the high half of an fp32
    static __device__ __forceinline__ float widen(uint16_t b) {
        return __uint_as_float(uint32_t(b) << 16);
    }
};
template <> struct Elem<kXU8> {
    using T = uint8_t;
    static __device__ __forceinline__ float widen(uint8_t b) { return float(b); }
};

// Window-table slots as the kernels for record type XT read them.
//   fp32 records: Slot {float t; int32 f} (8 bytes), decision !(x < t).
//   Narrow records: one 32-bit word, the feature index in the high half and in the low
//   half a key on the record type's grid (built on the host, see encode.hpp): for fp16 and
//   bf16 the threshold rounded up to the nearest value of the type, for uint8 its integer
//   ceiling clamped to 0..256.  No value of the type lies strictly between t and the key,
//   so !(x < key) on the stored element is the decision !(x < t) on its widened value.
template <int XT> struct Node;
template <> struct Node<kXF32> {
    using S = Slot;
    using Pair = Slot2;
    static __device__ __forceinline__ int feature(const Slot &s) { return s.f >> 2; }
    static __device__ __forceinline__ bool right(float x, const Slot &s) { return !(x < s.t); }
};
template <> struct Node<kXF16> {
    using S = uint32_t;
    struct alignas(8) Pair { uint32_t l, r; };
    static __device__ __forceinline__ int feature(uint32_t s) { return int(s >> 16); }
    static __device__ __forceinline__ bool right(uint16_t x, uint32_t s) {
        return !(Elem<kXF16>::widen(x) < Elem<kXF16>::widen(uint16_t(s)));
    }
};
template <> struct Node<kXBF16> {
    using S = uint32_t;
    struct alignas(8) Pair { uint32_t l, r; };
    static __device__ __forceinline__ int feature(uint32_t s) { return int(s >> 16); }
    static __device__ __forceinline__ bool right(uint16_t x, uint32_t s) {
        return !(Elem<kXBF16>::widen(x) < Elem<kXBF16>::widen(uint16_t(s)));
    }
};
template <> struct Node<kXU8> {
    using S = uint32_t;
    struct alignas(8) Pair { uint32_t l, r; };
    static __device__ __forceinline__ int feature(uint32_t s) { return int(s >> 16); }
    static __device__ __forceinline__ bool right(uint8_t x, uint32_t s) {
        return uint32_t(x) >= (s & 0xFFFFu);
    }
};

// Feature of slot `s` in a record row of the tile: element (feature ^ sw) * STRIDE of `row`.
// fp32 slots carry the feature as a byte offset, so the address is one xor-add.
template <int XT, int STRIDE>
__device__ __forceinline__ typename Elem<XT>::T feature_at(const typename Elem<XT>::T *row,
                                                           const typename Node<XT>::S &s, int sw) {
    if constexpr (XT == kXF32)
        return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(row) +
                                                (s.f ^ (sw << 2)) * STRIDE);
    else
        return row[(Node<XT>::feature(s) ^ sw) * STRIDE];
}

// Element-level position swizzle for rows of RS elements of type XT: the word swizzle,
// scaled to elements (the position of an element within its word is unchanged).
template <int XT, int RS>
__device__ __forceinline__ int swz_el(int r) {
    constexpr int kPerWord = 4 / int(sizeof(typename Elem<XT>::T));
    return swz<RS / kPerWord>(r) * kPerWord;
}

// Records of tile `tile` (tiles of TR records) that exist in the input.
template <int TR = kTileRows>
__device__ __forceinline__ int valid_rows(const Rows &in, int64_t tile) {
    const int64_t left = in.n - tile * TR;
    return left < TR ? int(left) : TR;
}

// A 16-byte vector at any 4-byte-aligned address (one global_load_dwordx4).
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));

__device__ __forceinline__ f32x4 load16(const char *p) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4_a4 *>(p));
}

// Rows of any width, stride and alignment.  What bounded them was the load path: one
// element per load, each waited for (3,000,001 x 19 fp32 rows took 244 us, 0.98 TB/s; now
// 40 us over the same windows and 37.5 us over a node list).  Here 16-byte vectors are loaded and the next tile's stay in flight in registers,
// as for the exact tiles.  Vectors lie on 4-byte boundaries: loads off them measured 1.5
// times the time (rows of 20 of 25 fp16 elements, 15.7 us against 9 us).
//   FLAT: dense rows whose width is no multiple of 16 bytes, 4-byte-aligned base.  A tile of
//     TR rows is one run of TR * row_bytes bytes (a multiple of 16) and is copied as it
//     lies: no division, one 16-byte LDS write per vector.  Row r starts at byte r *
//     row_bytes; a width that is no multiple of 16 bytes puts at most two rows of a fixed
//     column on one bank.
//   Otherwise (strided rows, dense rows of a multiple of 16 bytes that have no exact tile,
//     bases between words): a row is the row_vecs vectors from the word its first element
//     lies in, the last of which may read past its end.  Row r starts at LDS byte lds_off +
//     r * lds_pitch; lds_pitch is 16 row_vecs + 4 (an odd number of words, so the 64 rows of
//     a fixed column are on 64 banks; with the row_vecs of the class, a constant, where
//     constant_pitch in tiles.hpp says so), plus what makes it equal to the input's pitch modulo 4, so that a vector's words stay
//     words in the LDS.
// Wide rows make tiles of TR = 32 or 16 records, so that a tile stays within 16 KiB of
// registers and several fit the LDS: lanes share rows then (lane l walks row l % TR), which
// a stream-bound walk has the time for.  NV: prefetch vectors per lane (a class of sizes;
// vectors past the tile re-read its last one); 0: no prefetch.
// Loads of a tile; Derived says where a vector and an element (f of row r: r n_features + f)
// go in the LDS.
template <class Derived, int XT, bool FLAT, int NV, int TRv>
struct RowLoads {
    using T = typename Elem<XT>::T;
    static constexpr int TR = TRv;
    static constexpr bool kFewArgs = false;
    static constexpr bool kPrefetch = NV > 0;
    static constexpr int kRegs = 4 * NV;
    static constexpr int kES = int(sizeof(T));
    f32x4 v[NV > 0 ? NV : 1];

    // Row of vector q (0 for flat tiles, which are one run of vectors).
    static __device__ __forceinline__ int row_of(const Rows &in, int q) {
        if constexpr (FLAT) return 0;
        return in.row_vecs == 1 ? q : int(__umulhi(uint32_t(q), in.magic_v));
    }
    static __device__ __forceinline__ const char *source(const Rows &in, const char *base, int q) {
        if constexpr (FLAT) {
            return base + uint32_t(q) * 16u;
        } else if constexpr (kES == 4) {
            return base + uint32_t(q) * 16u + int64_t(row_of(in, q)) * in.row_gap;
        } else {
            const int r = row_of(in, q);
            return base + ((in.lds_off + int64_t(r) * in.row_pitch) & ~int64_t(3)) +
                   (q - r * in.row_vecs) * 16;
        }
    }
    // First word of tile t in the input (in.x is lds_off bytes past a word; tiles start a
    // multiple of 16 bytes apart).
    static __device__ __forceinline__ const char *tile_base(const Rows &in, int64_t t) {
        const char *x = static_cast<const char *>(in.x) + t * TR * in.row_pitch;
        if constexpr (FLAT || kES == 4) return x;
        return x - in.lds_off;
    }

    // Tiles whose every vector lies inside the input.
    static __device__ __forceinline__ int64_t prefetch_end(const Rows &in) {
        return (in.n - in.short_rows > 0 ? in.n - in.short_rows : 0) / TR;
    }
    __device__ __forceinline__ void load(const Rows &in, int64_t t, int lane) {
        const char *base = tile_base(in, t);
        const int last = in.tile_vecs - 1;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int q = k * 64 + lane;
            v[k] = load16(source(in, base, q < last ? q : last));
        }
    }
    __device__ __forceinline__ void store(const Rows &in, float *tile, int lane) const {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int q = k * 64 + lane;
            if (q < in.tile_vecs) Derived::put(in, tile, q, v[k]);
        }
    }
    // Any tile, staged by one wavefront or, as part `part` of `parts`, by several.  Vectors
    // that would leave the input are not loaded; the elements they hold of the input are
    // loaded one by one (the last bytes of a flat input's last tile, the last elements of
    // the input's last short_rows rows).
    static __device__ __forceinline__ void stage(const Rows &in, float *tile, int64_t t, int lane,
                                                 int part = 0, int parts = 1) {
        const char *base = tile_base(in, t);
        const int64_t row0 = t * TR;
        const int valid = valid_rows<TR>(in, t);
        const int row_bytes = in.n_features * kES;
        int nvec, safe_rows = TR, full_vecs = 0;
        if constexpr (FLAT) {
            nvec = valid * row_bytes >> 4;
        } else {
            nvec = valid * in.row_vecs;
            const int64_t safe = in.n - in.short_rows - row0;   // rows read to their last vector
            safe_rows = safe < 0 ? 0 : safe < TR ? int(safe) : TR;
            full_vecs = row_bytes >> 4;                          // a short row's
            if (safe_rows == 0 && full_vecs == 0) nvec = 0;
        }
        // batches of loads in flight; a lane without a vector re-reads the tile's first
        constexpr int kBatch = NV == 0 || NV > 8 ? 8 : NV;
#pragma unroll 1
        for (int k0 = part; k0 * 64 < nvec; k0 += kBatch * parts) {
            f32x4 x[kBatch];
            bool ok[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                const int q = (k0 + k * parts) * 64 + lane;
                ok[k] = q < nvec;
                if constexpr (!FLAT) {
                    const int r = row_of(in, q);
                    ok[k] = ok[k] && (r < safe_rows || q - r * in.row_vecs < full_vecs);
                }
                x[k] = load16(source(in, base, ok[k] ? q : 0));
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k)
                if (ok[k]) Derived::put(in, tile, (k0 + k * parts) * 64 + lane, x[k]);
        }
        if (part != 0) return;
        const T *x = static_cast<const T *>(in.x);
        if constexpr (FLAT) {
            const int e = (nvec << 4) / kES + lane;       // fewer than 16 bytes are left
            if (e < valid * in.n_features)
                Derived::put_element(in, tile, e, x[row0 * in.n_features + e]);
        } else {
            // a short row's full vectors start up to 3 bytes before it
            const int e = (full_vecs > 0 ? ((full_vecs << 4) - 4) / kES : 0) + lane;
            for (int r = safe_rows; r < valid; ++r)       // at most short_rows rows
                if (e < in.n_features)
                    Derived::put_element(in, tile, r * in.n_features + e, x[(row0 + r) * in.ld + e]);
        }
    }
};

template <int XT, bool FLAT, int NV, int TRv, int PITCH = row_tile_pitch(NV, TRv)>
struct RowTile : RowLoads<RowTile<XT, FLAT, NV, TRv, PITCH>, XT, FLAT, NV, TRv> {
    using Loads = RowLoads<RowTile<XT, FLAT, NV, TRv, PITCH>, XT, FLAT, NV, TRv>;
    using T = typename Loads::T;
    using Loads::kES;
    using Loads::row_of;
    using Loads::TR;
    // The pitch of the widest rows of the class, so that a row some constant number of rows
    // further is an instruction offset away (rows that start on words); 0: in.lds_pitch.
    static constexpr int kPitch = FLAT ? 0 : PITCH;

    static __device__ __forceinline__ void put(const Rows &in, float *tile, int q, f32x4 x) {
        if constexpr (FLAT) {
            reinterpret_cast<f32x4 *>(tile)[q] = x;
        } else {
            const int r = row_of(in, q);
            float *p;
            if constexpr (kPitch > 0)
                p = tile + q * 4 + r * (kPitch / 4 - in.row_vecs * 4);
            else if constexpr (kES == 4)
                p = tile + q * 4 + r;
            else
                p = tile + ((in.lds_off + r * in.lds_pitch) >> 2) + (q - r * in.row_vecs) * 4;
            p[0] = x.x;
            p[1] = x.y;
            p[2] = x.z;
            p[3] = x.w;
        }
    }
    static __device__ __forceinline__ void put_element(const Rows &in, float *tile, int e, T x) {
        if constexpr (FLAT) {
            reinterpret_cast<T *>(tile)[e] = x;
        } else {
            const int r = e / in.n_features;
            row(in, tile, r)[e - r * in.n_features] = x;
        }
    }
    static __device__ __forceinline__ const T *row(const Rows &in, const float *tile, int r) {
        if constexpr (kPitch > 0)
            return reinterpret_cast<const T *>(tile + r * (kPitch / 4));
        else
            return reinterpret_cast<const T *>(reinterpret_cast<const char *>(tile) + in.lds_off +
                                               r * in.lds_pitch);
    }
    static __device__ __forceinline__ T *row(const Rows &in, float *tile, int r) {
        return const_cast<T *>(row(in, static_cast<const float *>(tile), r));
    }
    static __device__ __forceinline__ int swizzle(int) { return 0; }
    static __device__ __forceinline__ T at(const Rows &in, const float *tile, int r, int g,
                                           const typename Node<XT>::S &s) {
        if constexpr (kPitch > 0) return feature_at<XT, 1>(row(in, tile, r + g), s, 0);
        // r's address is the lane's own, g rows further a wavefront-uniform offset.  Where
        // 16 wavefronts of the walk can share a CU the offset is made anew in every round:
        // as a loop invariant it would become one address register per round (20 fp32
        // features, 64-slot windows: 29 us against 48 us).
        int ofs = g * in.lds_pitch;
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (NV <= 8) asm volatile("" : "+s"(ofs));
#endif
        return feature_at<XT, 1>(
            reinterpret_cast<const T *>(reinterpret_cast<const char *>(row(in, tile, r)) + ofs), s, 0);
    }
};

// Column-major tiles of 64 fp32 records for walks whose lanes each read their own record:
// feature c of row r is word c * 64 + r, so lane r reads bank r whatever feature it asks for.
template <bool FLAT, int NV>
struct ColTile : RowLoads<ColTile<FLAT, NV>, kXF32, FLAT, NV, kTileRows> {
    static __device__ __forceinline__ void put(const Rows &in, float *tile, int q, f32x4 x) {
        const float v[4] = {x.x, x.y, x.z, x.w};
        if constexpr (FLAT) {
            const uint32_t e = uint32_t(q) * 4u;
            int r = in.n_features == 1 ? int(e) : int(__umulhi(e, in.magic_f));
            int c = int(e) - r * in.n_features;
            for (int j = 0; j < 4; ++j) {
                tile[c * kTileRows + r] = v[j];
                if (++c == in.n_features) {
                    c = 0;
                    ++r;
                }
            }
        } else {
            const int r = ColTile::row_of(in, q), c = (q - r * in.row_vecs) * 4;
            float *p = tile + c * kTileRows + r;
            if ((in.n_features & 3) == 0) {
                for (int j = 0; j < 4; ++j) p[j * kTileRows] = v[j];
            } else {                           // a row's last vector reaches past its end
                for (int j = 0; j < 4; ++j)
                    if (c + j < in.n_features) p[j * kTileRows] = v[j];
            }
        }
    }
    static __device__ __forceinline__ void put_element(const Rows &in, float *tile, int e, float x) {
        const int r = e / in.n_features;
        tile[(e - r * in.n_features) * kTileRows + r] = x;
    }
};

}  // namespace dev
}  // namespace dtree
