// gfx950 forest kernel templates, instantiated per kind of exit codes (int32: forest.hip,
// int16: forest_ex16.hip, packed: forest_packed.hip, node lists: forest_list.hip) and for
// the speculative walk (forest_spec.hip): translation units compiled in parallel.
//
// Forests are evaluated tree after tree (the concatenated-trees scheme the paper cites
// in Section 1) and the trees' classes are combined by majority vote, ties going to the
// smallest class id.  Each record's votes live in registers as packed 8-bit counters.
//
// The tables of all trees together usually exceed the LDS, so a workgroup works on one
// group of tiles at a time (one 64-record tile per wavefront, staged once) and streams the
// trees' tables through the LDS in chunks of consecutive trees; every tree of a chunk is
// walked for the whole group before the next chunk replaces it.  All wavefronts of a
// workgroup iterate over the same groups and chunks, so the workgroup barriers around the
// chunk copies are reached uniformly.  Forests whose single trees do not fit the LDS read
// their tables from global memory instead.
#pragma once

#include "device_common.hpp"

namespace dtree {
namespace {

using dev::Slot;

// The tree and chunk descriptors never change during a launch and are read at wavefront-
// uniform indices: read them through the constant address space, which makes them scalar
// loads.  A vector load would share the in-order load counter with the record prefetch, so
// waiting for a descriptor would also wait for the next tile to arrive from HBM.
typedef int v4i __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) v4i ConstV4i;

__device__ __forceinline__ int4 read_const(const int4 *p, int i) {
    const v4i v = ((ConstV4i *)(p))[i];
    return int4{v.x, v.y, v.z, v.w};
}

typedef int v2i __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) v2i ConstV2i;

// Root slot of tree i's window 0 (from the per-tree root array): a scalar load that does
// not wait for the tree's descriptor.
__device__ __forceinline__ Slot read_root(const int2 *p, int i) {
    const v2i v = ((ConstV2i *)(p))[i];
    return Slot{__int_as_float(v.x), v.y};
}

template <int NV>
__device__ __forceinline__ void add_vote(uint32_t (&votes)[NV], int cls) {
    if constexpr (NV == 2) {
        // eight counters in one 64-bit word: a shift and a 64-bit add
        uint64_t v = uint64_t(votes[1]) << 32 | votes[0];
        v += uint64_t(1) << (cls * 8);
        votes[0] = uint32_t(v);
        votes[1] = uint32_t(v >> 32);
    } else {
        const int word = cls >> 2;
        const uint32_t inc = 1u << ((cls & 3) * 8);
#pragma unroll
        for (int r = 0; r < NV; ++r) votes[r] += (word == r) ? inc : 0u;
    }
}

// Class with the most votes; the strict comparison keeps the smallest id on ties.
template <int NV>
__device__ __forceinline__ int majority(const uint32_t (&votes)[NV], int n_classes) {
    int best = 0;
    int best_count = -1;
#pragma unroll
    for (int r = 0; r < NV; ++r) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int c = r * 4 + b;
            const int count = int((votes[r] >> (8 * b)) & 255u);
            if (c < n_classes && count > best_count) {
                best_count = count;
                best = c;
            }
        }
    }
    return best;
}

// The kernel arguments, for the code around the walk.  The walk needs every scalar register,
// and the arguments of row tiles held across it spilled to vector lanes (a 32-tree forest
// 457 us against 373 us): for them the arguments are read again, through a pointer the
// compiler cannot see through, from the kernel-argument segment (scalar loads, three times
// per group).  Exact tiles need few arguments and keep them (373 us against 380 us).
template <class Tile>
__device__ __forceinline__ const FArgs &cold_args(const FArgs &a) {
    if constexpr (Tile::kFewArgs) {
        return a;
    } else {
        typedef const __attribute__((address_space(4))) FArgs ConstArgs;
        ConstArgs *p = (ConstArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return *(const FArgs *)p;
    }
}

// Lane `v`; for row tiles so that the LDS addresses of a tile's vectors, the same for every
// tile, are not kept in registers from group to group.
template <class Tile>
__device__ __forceinline__ int cold_lane(int v) {
    if constexpr (!Tile::kFewArgs) asm volatile("" : "+v"(v));
    return v;
}

// Trees walked together per lane by the data decomposition.
constexpr int kIlp = 4;

// The whole chunk buffer, copied by the workgroup.  (One word per thread at a time: more in
// flight would take registers the prefetched tile needs.  The split kernel, which has none,
// copies with dev::copy_to_lds.)
__device__ __forceinline__ void copy_chunk(const FArgs &a, int4 *tab, const int4 &ch) {
    const int4 *src = a.tables + (ch.z >> 4);
    for (int i = threadIdx.x; i < (ch.w >> 4); i += blockDim.x) tab[i] = src[i];
}

// Chunks of up to kStage * 16 bytes per thread are loaded into registers before the
// barrier that frees the chunk buffer, so the loads' latency overlaps the wait for the
// slowest wavefront; only the LDS writes sit between the two barriers.
constexpr int kStage = 2;

__device__ __forceinline__ void copy_chunk_staged(const FArgs &a, int4 *tab, const int4 &ch) {
    const v4i *src = reinterpret_cast<const v4i *>(a.tables) + (ch.z >> 4);
    v4i *dst = reinterpret_cast<v4i *>(tab);
    const int n16 = ch.w >> 4;                       // >= 1: a chunk holds a tree
    v4i v[kStage];
#pragma unroll
    for (int q = 0; q < kStage; ++q) {
        // unconditional loads (a thread past the end re-reads the last word): no branch
        // between the loads, so they are all in flight before the barrier
        const int i = int(threadIdx.x) + q * int(blockDim.x);
        v[q] = src[i < n16 ? i : n16 - 1];
    }
    __syncthreads();                                 // previous chunk no longer read
    // unconditional writes too (a thread past the end writes the last word again, the same
    // value its owner writes): with no branch around them, every load is waited for on one
    // path, and the compiler needs no catch-all wait later (which, the vector-memory counter
    // being in order, would also wait for the next record tiles' prefetch)
#pragma unroll
    for (int q = 0; q < kStage; ++q) {
        const int i = int(threadIdx.x) + q * int(blockDim.x);
        dst[i < n16 ? i : n16 - 1] = v[q];
    }
}

// Votes of this lane's record for trees [k, end) of a chunk whose tables start at `cbase` and
// at byte `cofs` of the forest's tables.  Data decomposition: `row` is the lane's record in a
// column-major tile; kIlp trees at a time.
template <class EX, int NV>
__device__ __forceinline__ void vote_data(const FArgs &a, const char *cbase, int cofs, int k,
                                          int end, const float *row, uint32_t (&votes)[NV]) {
    // K trees of the chunk walked together from tree k0
    auto walk_group = [&](auto kk, int k0) {
        constexpr int K = decltype(kk)::value;
        const char *base[K];
        Slot root[K];
        int sb[K], lv[K];
        int32_t code[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int4 d = read_const(a.trees, k0 + i);   // {byte_off, slot_bytes, levels, 0}
            root[i] = read_root(a.roots, k0 + i);
            base[i] = cbase + (d.x - cofs);
            sb[i] = d.y;
            lv[i] = d.z;
        }
        // Both kinds of scalar loads complete here, before the walk: one wait
        // for them all, instead of one for the roots and, after the root step,
        // another for the descriptors (which the compiler would otherwise sink
        // to their first use).
#pragma unroll
        for (int i = 0; i < K; ++i)
            asm volatile("" ::"s"(base[i]), "s"(sb[i]), "s"(lv[i]), "s"(root[i].t),
                         "s"(root[i].f));
        if constexpr (std::is_same<EX, dev::NodeList>::value)
            dev::walk_list_k<K>(base, root, lv, row, code);
        else
            dev::walk_data_k<K, kTileRows, EX>(base, root, sb, lv, a.depth, row, 0, code);
#pragma unroll
        for (int i = 0; i < K; ++i) add_vote(votes, ~code[i]);
    };
    for (; k + kIlp <= end; k += kIlp) walk_group(std::integral_constant<int, kIlp>(), k);
    if (end - k == 3)
        walk_group(std::integral_constant<int, 3>(), k);
    else if (end - k == 2)
        walk_group(std::integral_constant<int, 2>(), k);
    else if (end - k == 1)
        walk_group(std::integral_constant<int, 1>(), k);
}

// The same for the speculative decomposition (int32 exit codes), all 64 records of `tile`.
template <class Tile, int NV, int SD>
__device__ __forceinline__ void vote_spec(const FArgs &a, const char *cbase, int cofs, int k,
                                          int end, const float *tile, int lane,
                                          uint32_t (&votes)[NV]) {
    for (; k < end; ++k) {
        const int4 d = read_const(a.trees, k);   // {byte_off, slot_bytes, levels, 0}
        const char *base = cbase + (d.x - cofs);
        const Slot *sl = reinterpret_cast<const Slot *>(base);
        const int32_t *ex = reinterpret_cast<const int32_t *>(base + d.y);
        const dev::Spec<kXF32, SD, Tile> spec(lane);
        const Slot root = sl[spec.j];
        add_vote(votes, ~spec.run(sl, ex, d.z, root, a.in, tile));
    }
}

// SD = 0: data decomposition; SD > 0: speculative decomposition with window depth SD.
// EX: exit codes stored as int32, int16 where every code of the forest fits, or packed
// into the windows' bottom slots (dev::PackedExits) where every code fits 11 bits; or no
// windows but node lists (dev::NodeList).  One wavefront per tile.
template <class EX, class Tile, bool TAB_LDS, int NV, int SD>
__global__ void __launch_bounds__(64 * forest_max_waves(SD == 0 ? 0 : 1, SD)) forest_kernel(FArgs a) {
    extern __shared__ int4 lds[];
    constexpr bool kPrefetch = Tile::kPrefetch;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    float *tile = reinterpret_cast<float *>(lds) + wave * (a.tile_bytes >> 2);
    int4 *tab = lds + (a.waves * a.tile_bytes >> 4);    // chunk buffer after the tiles

    // A forest whose tables form one chunk is copied once: the tables then stay for every
    // group.  Otherwise the chunks are copied in turn for each group.
    if constexpr (TAB_LDS) {
        if (a.n_chunks == 1) {
            copy_chunk(a, tab, read_const(a.chunks, 0));
            __syncthreads();
        }
    }
    const bool staged = a.table_lds_bytes <= kStage * 16 * int(blockDim.x);

    // Tiles are prefetched one group ahead; the input's last ones are staged directly.
    Tile buf;
    auto prefetch = [&](int64_t t) {
        if constexpr (kPrefetch) {
            const FArgs &f = cold_args<Tile>(a);
            if (t < f.end_tile && t < Tile::prefetch_end(f.in)) buf.load(f.in, t, cold_lane<Tile>(lane));
        }
    };
    const int64_t n_groups = (a.end_tile + a.waves - 1) / a.waves;
    int64_t g = blockIdx.x;
    if (g < n_groups) prefetch(g * a.waves + wave);
    for (; g < n_groups; g += gridDim.x) {
        const int64_t t = g * a.waves + wave;        // this wavefront's tile
        const bool active = t < a.end_tile;          // uniform per wavefront
        dev::wave_sync();
        if (active) {
            const FArgs &f = cold_args<Tile>(a);
            if (kPrefetch && t < Tile::prefetch_end(f.in))
                buf.store(f.in, tile, cold_lane<Tile>(lane));
            else
                Tile::stage(f.in, tile, t, cold_lane<Tile>(lane));
        }
        dev::wave_sync();
        // The next group's tiles are prefetched into registers: here, or, when the chunks
        // are copied for every group, after the last chunk's copy (its loads would
        // otherwise queue behind the prefetch on the in-order vector-memory counter, and the
        // first chunk copy would wait for the prefetch to arrive from HBM).
        const bool prefetch_late = TAB_LDS && a.n_chunks > 1;
        if (!prefetch_late) prefetch(t + int64_t(gridDim.x) * a.waves);

        uint32_t votes[NV];
#pragma unroll
        for (int r = 0; r < NV; ++r) votes[r] = 0u;
        for (int c = 0; c < a.n_chunks; ++c) {
            const int4 ch = read_const(a.chunks, c);             // {first, end, byte_off, bytes}
            if constexpr (TAB_LDS) {
                if (a.n_chunks > 1) {
                    if (staged) {
                        copy_chunk_staged(a, tab, ch);
                    } else {
                        __syncthreads();             // previous chunk no longer read
                        copy_chunk(a, tab, ch);
                    }
                    __syncthreads();
                    if (c == a.n_chunks - 1) prefetch(t + int64_t(gridDim.x) * a.waves);
                }
            }
            if (!active) continue;
            // tables of the chunk's trees: in the LDS chunk buffer (which starts at the
            // chunk's byte offset ch.z of the tables), or in place
            const char *cbase = TAB_LDS ? reinterpret_cast<const char *>(tab)
                                        : reinterpret_cast<const char *>(a.tables);
            const int cofs = TAB_LDS ? ch.z : 0;
            if constexpr (SD == 0)
                vote_data<EX>(a, cbase, cofs, ch.x, ch.y, tile + lane, votes);
            else
                vote_spec<Tile, NV, SD>(a, cbase, cofs, ch.x, ch.y, tile, lane, votes);
        }
        if (active) {
            const FArgs &f = cold_args<Tile>(a);
            dev::store_value(f.out, f.out_kind, f.in.n, t * kTileRows + lane,
                             majority(votes, f.n_classes));
        }
    }
}

// The same with 2^split wavefronts per tile, each walking a share of every chunk's trees:
// for inputs whose tiles would leave wavefronts or CUs idle (few records, or the last,
// partly filled round of groups), and for rows so wide that the LDS holds fewer tiles than
// wavefronts.  The fewer tiles also leave the LDS larger chunks.  The wavefronts of a tile
// stage it together and add their votes up in the LDS.
template <class EX, class Tile, bool TAB_LDS, int NV, int SD>
__global__ void __launch_bounds__(64 * forest_max_waves(SD == 0 ? 0 : 1, SD))
forest_split_kernel(FArgs a) {
    extern __shared__ int4 lds[];
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int parts = 1 << a.split, part = wave & (parts - 1), slot = wave >> a.split;
    const int tiles = a.waves >> a.split;               // tiles per group, >= 1
    float *tile = reinterpret_cast<float *>(lds) + slot * (a.tile_bytes >> 2);
    uint32_t *box = reinterpret_cast<uint32_t *>(lds + (tiles * a.tile_bytes >> 4)) +
                    slot * (NV * 64) + lane;            // vote word r of this lane at box[64 r]
    int4 *tab = lds + ((tiles * a.tile_bytes + tiles * NV * 256) >> 4);
    const int64_t n_groups = (a.end_tile - a.first_tile + tiles - 1) / tiles;
    const bool resident = TAB_LDS && a.n_chunks == 1;   // copied once, with the first group
    for (int64_t g = blockIdx.x; g < n_groups; g += gridDim.x) {
        const int64_t t = a.first_tile + g * tiles + slot;
        const bool active = slot < tiles && t < a.end_tile;
        if (active) {
            Tile::stage(cold_args<Tile>(a).in, tile, t, cold_lane<Tile>(lane), part, parts);
            if (part == 0)
#pragma unroll
                for (int r = 0; r < NV; ++r) box[64 * r] = 0u;
        }
        uint32_t votes[NV];
#pragma unroll
        for (int r = 0; r < NV; ++r) votes[r] = 0u;
        for (int c = 0; c < a.n_chunks; ++c) {
            const int4 ch = read_const(a.chunks, c);             // {first, end, byte_off, bytes}
            if constexpr (TAB_LDS) {
                if (c > 0) __syncthreads();              // previous chunk no longer read
                if (!resident || g == int64_t(blockIdx.x))
                    dev::copy_to_lds(tab, a.tables + (ch.z >> 4), ch.w >> 4);
            }
            if (TAB_LDS || c == 0) __syncthreads();      // chunk and (first) tiles visible
            if (!active) continue;
            const char *cbase = TAB_LDS ? reinterpret_cast<const char *>(tab)
                                        : reinterpret_cast<const char *>(a.tables);
            const int cofs = TAB_LDS ? ch.z : 0;
            const int per = (ch.y - ch.x + parts - 1) >> a.split;
            const int k = ch.x + part * per, end = k + per < ch.y ? k + per : ch.y;
            if constexpr (SD == 0)
                vote_data<EX>(a, cbase, cofs, k, end, tile + lane, votes);
            else
                vote_spec<Tile, NV, SD>(a, cbase, cofs, k, end, tile, lane, votes);
        }
        if (active)
#pragma unroll
            for (int r = 0; r < NV; ++r) atomicAdd(&box[64 * r], votes[r]);
        __syncthreads();                                 // votes complete, tables and tiles free
        if (active && part == 0) {
#pragma unroll
            for (int r = 0; r < NV; ++r) votes[r] = box[64 * r];
            const FArgs &f = cold_args<Tile>(a);
            dev::store_value(f.out, f.out_kind, f.in.n, t * kTileRows + lane,
                             majority(votes, f.n_classes));
        }
    }
}

// ---- instance tables ------------------------------------------------------------------
template <class EX, class Tile, bool TAB_LDS, int NV, int SD>
const void *kernel_of(bool split) {
    if constexpr (!Tile::kPrefetch)
        if (split) return reinterpret_cast<const void *>(&forest_split_kernel<EX, Tile, TAB_LDS, NV, SD>);
    return split ? nullptr : reinterpret_cast<const void *>(&forest_kernel<EX, Tile, TAB_LDS, NV, SD>);
}

template <class EX, class Tile, bool TAB_LDS, int SD>
const void *for_votes(bool split, int vote_words) {
    switch (vote_words) {
        case 2: return kernel_of<EX, Tile, TAB_LDS, 2, SD>(split);
        case 4: return kernel_of<EX, Tile, TAB_LDS, 4, SD>(split);
        case 16: return kernel_of<EX, Tile, TAB_LDS, 16, SD>(split);
        default: return nullptr;
    }
}

// Tables read in place: tiles without prefetch only.
template <class EX, class Tile, int SD>
const void *for_tables(bool split, bool tab_lds, int vote_words) {
    if (tab_lds) return for_votes<EX, Tile, true, SD>(split, vote_words);
    if constexpr (!Tile::kPrefetch) return for_votes<EX, Tile, false, SD>(split, vote_words);
    return nullptr;
}

// The data decomposition reads each lane's own record: column-major tiles make every such
// read conflict-free.
template <class EX, bool FLAT>
const void *col_tile(const ForestShape &s) {
    switch (s.tile.vecs) {
        case 0: return for_tables<EX, dev::ColTile<FLAT, 0>, 0>(s.split > 0, s.tables_in_lds, s.vote_words);
        case 2: return for_tables<EX, dev::ColTile<FLAT, 2>, 0>(s.split > 0, s.tables_in_lds, s.vote_words);
        case 4: return for_tables<EX, dev::ColTile<FLAT, 4>, 0>(s.split > 0, s.tables_in_lds, s.vote_words);
        case 6: return for_tables<EX, dev::ColTile<FLAT, 6>, 0>(s.split > 0, s.tables_in_lds, s.vote_words);
        case 8: return for_tables<EX, dev::ColTile<FLAT, 8>, 0>(s.split > 0, s.tables_in_lds, s.vote_words);
        default: return nullptr;
    }
}

template <class EX, int RS>
const void *col_exact(const ForestShape &s) {
    return for_tables<EX, dev::ExactTile<kXF32, RS, dev::kColMajor, kTileRows>, 0>(
        s.split > 0, s.tables_in_lds, s.vote_words);
}

// Kernel instance of the data decomposition for exit codes of type EX.  (A template: only the
// unit that asks for it compiles its instances.)
template <class EX>
const void *forest_data_kernel(const ForestShape &s) {
    if (s.tile.mode == kLoadFlat) return col_tile<EX, true>(s);
    if (s.tile.mode == kLoadRows) return col_tile<EX, false>(s);
    switch (s.tile.row_stride) {
        case 4: return col_exact<EX, 4>(s);
        case 8: return col_exact<EX, 8>(s);
        case 16: return col_exact<EX, 16>(s);
        case 32: return col_exact<EX, 32>(s);
        default: return nullptr;
    }
}

}  // namespace
}  // namespace dtree
