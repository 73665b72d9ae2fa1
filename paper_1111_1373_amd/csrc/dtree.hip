// C ABI of the tree evaluator (include/dtree.h): validation, device upload, launch
// planning and dispatch.  No exception crosses the ABI; errors are status codes plus a
// per-thread message.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "dtree.h"
#include "dtree_probe.h"
#include "encode.hpp"
#include "kernels.hpp"
#include "library.hpp"
#include "tiles.hpp"

namespace {

using dtree::align16;
using dtree::exact_rows;
using dtree::make_tile_rows;
using dtree::tile_shape;

thread_local std::string g_last_error;

dt_status fail(dt_status s, const std::string &msg) {
    g_last_error = msg;
    return s;
}

dt_status hip_fail(hipError_t e, const char *what) {
    return fail(DT_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Device resources of one window encoding: the exits, and the slots once per record
// type (8-byte fp32 slots; 4-byte words on each narrow type's grid).
struct Encoding {
    int32_t depth = 0, n_windows = 0, levels = 0;
    int64_t exit_bytes = 0;                        // padded to 16
    int64_t slot_bytes[dtree::kElemTypes] = {};    // padded to 16
    // [fp32 slots][exit_class][exit_leaf][fp16 slots][bf16 slots][uint8 slots]
    void *d_mem = nullptr;
    const int4 *d_slots[dtree::kElemTypes] = {};
    const int4 *d_exit_class = nullptr;
    const int4 *d_exit_leaf = nullptr;
    // A node list instead of windows (data decomposition, see walk_list): d_slots then hold
    // the lists, of slot_bytes each, and the first list_lds_bytes of one go to the LDS.
    bool list = false;
    int64_t table_bytes(int elem_type) const {
        return list ? std::min(slot_bytes[elem_type], dtree::kListLdsBytes)
                    : slot_bytes[elem_type] + exit_bytes;
    }
    // Sizes of the window tables, and of a node list of n nodes.
    void size_windows(int window_depth, int64_t windows, int32_t window_levels) {
        depth = window_depth;
        n_windows = int32_t(windows);
        levels = window_levels;
        const int64_t n_slots = windows << window_depth;
        exit_bytes = align16(n_slots * 4);
        for (int xt = 0; xt < dtree::kElemTypes; ++xt)
            slot_bytes[xt] = align16(n_slots * (xt == dtree::kXF32 ? 8 : 4));
    }
    void size_list(int32_t n) {
        list = true;
        for (int64_t &b : slot_bytes) b = dtree::list_bytes(n);
    }
};

struct DeviceCaps {
    int device = -1;
    int n_cu = 0;
    int lds_per_block = 0;
    int lds_per_cu = 0;
};

dt_status query_device(DeviceCaps *caps) {
    hipError_t e = hipGetDevice(&caps->device);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    e = hipDeviceGetAttribute(&caps->n_cu, hipDeviceAttributeMultiprocessorCount, caps->device);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute(CU count)");
    e = hipDeviceGetAttribute(&caps->lds_per_block, hipDeviceAttributeMaxSharedMemoryPerBlock,
                              caps->device);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute(LDS)");
    e = hipDeviceGetAttribute(&caps->lds_per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor,
                              caps->device);
    if (e != hipSuccess || caps->lds_per_cu < caps->lds_per_block) caps->lds_per_cu = caps->lds_per_block;
    return DT_OK;
}

dt_status upload_encoding(const dtree::WindowTables &wt, Encoding *enc) {
    enc->size_windows(wt.depth, wt.n_windows, wt.levels);
    const int64_t n_slots = int64_t(wt.n_windows) * wt.slots;
    int64_t off[dtree::kElemTypes];
    int64_t total = 0;
    for (int xt = 0; xt < dtree::kElemTypes; ++xt) {
        off[xt] = total;
        total += enc->slot_bytes[xt] + (xt == dtree::kXF32 ? 2 * enc->exit_bytes : 0);
    }
    std::vector<unsigned char> host(size_t(total), 0);
    for (int64_t i = 0; i < n_slots; ++i) {
        const int32_t fb = 4 * wt.feature[size_t(i)];   // byte offset in an fp32 row
        std::memcpy(&host[size_t(8 * i)], &wt.threshold[size_t(i)], 4);
        std::memcpy(&host[size_t(8 * i + 4)], &fb, 4);
    }
    const int64_t exit_off = enc->slot_bytes[dtree::kXF32];
    std::memcpy(&host[size_t(exit_off)], wt.exit_class.data(), size_t(n_slots * 4));
    std::memcpy(&host[size_t(exit_off + enc->exit_bytes)], wt.exit_leaf.data(),
                size_t(n_slots * 4));
    std::vector<uint32_t> words;
    for (int xt = dtree::kXF16; xt < dtree::kElemTypes; ++xt) {
        dtree::build_narrow_slots(wt, static_cast<dt_dtype>(xt), &words);
        std::memcpy(&host[size_t(off[xt])], words.data(), size_t(n_slots * 4));
    }
    hipError_t e = hipMalloc(&enc->d_mem, size_t(total));
    if (e != hipSuccess) {
        enc->d_mem = nullptr;
        return fail(DT_ERR_NO_MEMORY, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    e = hipMemcpy(enc->d_mem, host.data(), size_t(total), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(tables)");
    auto *base = static_cast<unsigned char *>(enc->d_mem);
    for (int xt = 0; xt < dtree::kElemTypes; ++xt)
        enc->d_slots[xt] = reinterpret_cast<const int4 *>(base + off[xt]);
    enc->d_exit_class = reinterpret_cast<const int4 *>(base + exit_off);
    enc->d_exit_leaf = reinterpret_cast<const int4 *>(base + exit_off + enc->exit_bytes);
    return DT_OK;
}

// Upload the tree as node lists, one per record type (see walk_list).
dt_status upload_list(const dt_node *nodes, int32_t n, Encoding *enc) {
    enc->size_list(n);
    const int64_t size = enc->slot_bytes[0];
    const std::vector<int32_t> order = dtree::breadth_first_order(nodes, n);
    std::vector<uint32_t> host(size_t(size / 4) * dtree::kElemTypes, 0u);
    for (int xt = 0; xt < dtree::kElemTypes; ++xt)
        dtree::build_list(nodes, n, order, static_cast<dt_dtype>(xt),
                          host.data() + size_t(size / 4) * size_t(xt));
    hipError_t e = hipMalloc(&enc->d_mem, host.size() * 4);
    if (e != hipSuccess) {
        enc->d_mem = nullptr;
        return fail(DT_ERR_NO_MEMORY, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    e = hipMemcpy(enc->d_mem, host.data(), host.size() * 4, hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(node lists)");
    for (int xt = 0; xt < dtree::kElemTypes; ++xt)
        enc->d_slots[xt] = reinterpret_cast<const int4 *>(static_cast<unsigned char *>(enc->d_mem) +
                                                          size * xt);
    return DT_OK;
}

void free_encoding(Encoding *enc) {
    if (enc->d_mem) (void)hipFree(enc->d_mem);
    enc->d_mem = nullptr;
}

// Pointer-jumping reach per round of the path kernel: entry <- the entry `hops` further
// along.  Procedure 5 reads two further (path[path[path[i]]]).
constexpr int kDefaultPathHops = 2;
constexpr int kMaxPathHops = 8;

dt_status check_options(const dt_tree_options *opt) {
    if (!opt) return DT_OK;
    if (opt->data_window_depth < 0 || opt->data_window_depth > dtree::kMaxWindowDepth)
        return fail(DT_ERR_INVALID_ARG, "data_window_depth must be 0 (auto) or 1..16");
    if (opt->spec_window_depth < 0 || opt->spec_window_depth > dtree::kMaxSpecWindowDepth)
        return fail(DT_ERR_INVALID_ARG, "spec_window_depth must be 0 (auto) or 1..6");
    if (opt->waves_per_cu < 0 || opt->waves_per_cu > 32)
        return fail(DT_ERR_INVALID_ARG, "waves_per_cu must be 0 (auto) or 1..32");
    if (opt->path_hops < 0 || opt->path_hops > kMaxPathHops)
        return fail(DT_ERR_INVALID_ARG, "path_hops must be 0 (auto) or 1..8");
    return DT_OK;
}

void window_depths(const dt_node *nodes, const dtree::TreeShape &shape, int32_t n_features,
                   const dt_tree_options *opt, int *data_d, int *spec_d) {
    *data_d = (opt && opt->data_window_depth)
                  ? opt->data_window_depth
                  : dtree::choose_data_window_depth(nodes, shape,
                                                    dtree::data_table_budget(n_features));
    *spec_d = (opt && opt->spec_window_depth) ? opt->spec_window_depth
                                              : dtree::choose_spec_window_depth(shape);
}

void fill_info(const dtree::TreeShape &shape, int32_t n_features, int32_t n_classes,
               int data_d, int64_t data_w, int32_t data_lv, int spec_d, int64_t spec_w,
               int32_t spec_lv, dt_tree_info *info) {
    info->n_nodes = shape.n_nodes;
    info->n_internal = shape.n_internal;
    info->n_leaves = shape.n_leaves;
    info->depth = shape.depth;
    info->n_features = n_features;
    info->n_classes = n_classes;
    info->data_window_depth = data_d;
    info->data_windows = int32_t(data_w);
    info->data_levels = data_lv;
    info->spec_window_depth = spec_d;
    info->spec_windows = int32_t(spec_w);
    info->spec_levels = spec_lv;
    info->data_table_bytes = align16(data_w * (int64_t(1) << data_d) * 8) +
                             align16(data_w * (int64_t(1) << data_d) * 4);
    info->spec_table_bytes = align16(spec_w * (int64_t(1) << spec_d) * 8) +
                             align16(spec_w * (int64_t(1) << spec_d) * 4);
}

// Launch plan of one kernel instance: wavefronts per workgroup and resident workgroups.
struct Plan {
    const void *fn = nullptr;
    int waves = 0;
    int blocks_per_cu = 0;
    int lds_bytes = 0;
    int out_cap = 0;          // single-tree kernels: result tiles buffered per wavefront
    dtree::TileShape tile;    // single-tree kernels: the record tile
    int tables_in_lds = 0;
    int enc = 0;              // single-tree kernels: the encoding (dt_tree::enc)
    dt_status status = DT_ERR_UNSUPPORTED;
    std::string why;
};

std::mutex g_prep_mutex;
std::vector<const void *> g_prepared;

// Wavefronts per CU the library aims for (measured on MI355X).  The data decomposition is
// HBM-bound once about 64 KiB of record tiles are in flight per CU; more wavefronts only
// add contention.  The speculative decomposition, which does 2^D times the lane work per
// record, is bound by LDS latency once the tiles are small, and then gains from every
// wavefront up to 16 per CU (uint8 records of 64 features: 207 us with 16 against 282 us
// with 8).  With tiles of 64 fp32 features 64 KiB in flight is again the better point:
// 4 wavefronts of 16 KiB tiles keep a larger result buffer next to the tables (640 us on
// 16,777,216 x 64 records against 674 us with 5), and so do 8 of the 8 KiB tiles of 32
// records that depth-5 and depth-6 windows use (682 us against 726 us with 12 at depth
// 6, 710 against 729 us at depth 5).
// The path reduction is latency-bound and takes as many wavefronts as fit, up to 8.
// Row tiles count as the next power of two: 8 wavefronts of 48 uint8 features run 31.8 us
// and 16 run 32.5 us, where 64 KiB of their 3.3 KiB tiles (24 wavefronts) run 34.3 us.  Tiles
// of 16 records keep 16 lanes walking, and take 8 (250 fp32 features: 79.7 us against 90 us
// with 4).
int target_waves_per_cu(int algo, int tile_rows, int tile_bytes) {
    int size = 256;
    while (size < tile_bytes) size <<= 1;
    const int hbm = tile_rows <= 16 ? 8 : std::max(2, std::min(32, (64 * 1024) / size));
    if (algo == DT_ALGO_DATA || algo == dtree::kAlgoList) return hbm;
    if (algo == DT_ALGO_SPECULATIVE)
        return std::min(16, hbm);
    return 8;
}

void prepare_once(const void *fn, int lds_limit, Plan *plan) {
    std::lock_guard<std::mutex> lock(g_prep_mutex);
    if (std::find(g_prepared.begin(), g_prepared.end(), fn) != g_prepared.end()) return;
    hipError_t e = dtree::prepare_kernel(fn, lds_limit);
    if (e != hipSuccess) {
        plan->why = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
        plan->status = DT_ERR_HIP;
        return;
    }
    g_prepared.push_back(fn);
}

// Tables stay in the LDS when that still leaves room for kMinLdsWaves wavefront tiles per
// workgroup; larger trees read their tables from global memory.
constexpr int kMinLdsWaves = 2;
// A workgroup's LDS is allocated in pieces of this size.  The occupancy query does not count
// them: three workgroups of 54,352 bytes were planned where two fit, and the third ran after
// them (2,500 decision nodes, 1,000,000 x 4 fp32: 13.9 us; three of 53,328 bytes: 10.3 us).
constexpr int kLdsGranule = 1280;
constexpr int kMaxOutCap = 256;

// Single-tree plan: workgroup shape, resident workgroups per CU and the result buffer, for
// records of element type `elem_type` and results of `out_bytes` bytes (1 or 4).  The path
// kernel also keeps its path arrays (kPathIntsPerWave ints per wavefront) after the result
// buffers.
dt_status make_plan(const DeviceCaps &caps, int algo, int elem_type, int n_features,
                    int load_mode, int depth, int64_t table_bytes, int out_bytes,
                    int waves_per_cu, Plan *plan) {
    const int path_bytes = algo == DT_ALGO_PATH ? dtree::kPathIntsPerWave * 4 : 0;
    plan->tile = tile_shape(algo, elem_type, n_features, load_mode, depth);
    const int tile_rows = plan->tile.tile_rows;
    const int record_tile_bytes = plan->tile.tile_bytes;
    const int tile_bytes = record_tile_bytes + path_bytes;
    const int res_bytes = tile_rows * out_bytes;   // one tile of results
    if (tile_bytes + res_bytes > caps.lds_per_block) {
        plan->why = "one record tile exceeds the workgroup LDS";
        return plan->status = DT_ERR_UNSUPPORTED;
    }
    const bool tab_lds =
        table_bytes + int64_t(kMinLdsWaves) * (tile_bytes + res_bytes) <= caps.lds_per_block;
    const int table_lds = tab_lds ? int(table_bytes) : 0;
    plan->tables_in_lds = tab_lds ? 1 : 0;
    plan->fn = dtree::kernel_for(algo, elem_type, plan->tile, tab_lds, depth);
    if (!plan->fn) {
        plan->why = "no kernel instance for this configuration";
        return plan->status = DT_ERR_UNSUPPORTED;
    }
    plan->status = DT_OK;
    prepare_once(plan->fn, caps.lds_per_block, plan);
    if (plan->status != DT_OK) return plan->status;

    const int target =
        waves_per_cu > 0 ? waves_per_cu
                         : target_waves_per_cu(algo, tile_rows, tile_rows * plan->tile.row_bytes);
    // Try every workgroup size and count per CU; keep the shape reaching the most resident
    // wavefronts up to the target (registers and the LDS both limit residency); on ties
    // prefer larger workgroups (fewer table copies), then a larger result buffer.
    int best = 0, best_cap = 0;
    const int max_waves =
        dtree::tree_max_waves(algo, depth, tile_rows, plan->tile.prefetch_regs);
    for (int w = std::min(max_waves, target); w >= 1; --w) {
        for (int bpc = (target + w - 1) / w; bpc >= 1; --bpc) {
            const int budget = std::min(caps.lds_per_block,
                                        caps.lds_per_cu / bpc / kLdsGranule * kLdsGranule);
            if (table_lds + w * (tile_bytes + res_bytes) > budget) continue;
            const int cap =
                std::min(kMaxOutCap, (budget - table_lds - w * tile_bytes) / (w * res_bytes));
            const int lds = dtree::lds_bytes_for(table_lds, record_tile_bytes, w, cap * res_bytes) +
                            w * path_bytes;
            // a shape that cannot beat the best one is not asked for its occupancy
            const int most = std::min(target, bpc * w);
            if (most < best || (most == best && (w != plan->waves || cap <= best_cap))) continue;
            int nb = 0;
            hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, plan->fn, w * 64,
                                                                        size_t(lds));
            if (e != hipSuccess) {
                plan->why = std::string("hipOccupancyMaxActiveBlocksPerMultiprocessor: ") +
                            hipGetErrorString(e);
                return plan->status = DT_ERR_HIP;
            }
            const int blocks = std::min(nb, bpc);
            const int score = std::min(target, blocks * w);
            if (blocks >= 1 && (score > best || (score == best && w == plan->waves && cap > best_cap))) {
                best = score;
                best_cap = cap;
                plan->waves = w;
                plan->blocks_per_cu = blocks;
                plan->lds_bytes = lds;
                plan->out_cap = cap;
            }
        }
    }
    if (best == 0) {
        plan->why = "tables and one record tile exceed the workgroup LDS";
        return plan->status = DT_ERR_UNSUPPORTED;
    }
    plan->why.clear();
    return plan->status = DT_OK;
}

}  // namespace

struct dt_tree {
    DeviceCaps caps;
    dtree::TreeShape shape;
    int32_t n_features = 0, n_classes = 0;
    int path_hops = kDefaultPathHops;
    // data windows, speculative windows (also the path kernel's), node list (data walk); those
    // that a plan uses are uploaded
    Encoding enc[3];
    // [algo][record element type][load mode][uint8 / int32 results]
    Plan plan[3][dtree::kElemTypes][dtree::kLoadModes][2];
};

static bool single_tree_algo(dt_algo algo) {
    return algo == DT_ALGO_DATA || algo == DT_ALGO_SPECULATIVE || algo == DT_ALGO_PATH;
}

namespace {

// Device resources of a forest for one decomposition: all trees' tables back to back (tree
// k: window slots, then class exits where they are a table, each padded to 16 bytes; or the
// node list), the per-tree descriptors {byte_off, slot_bytes, levels, 0} and the LDS chunks
// {first_tree, end_tree, byte_off, bytes} of every launch plan.
struct ForestEncoding {
    int32_t depth = 0;
    void *d_mem = nullptr;
    const int4 *d_tables = nullptr, *d_trees = nullptr, *d_chunks = nullptr;
    const int2 *d_roots = nullptr;
    std::vector<int4> trees;     // host copy of the descriptors
    std::vector<int2> roots;     // per tree: slot 1 of window 0 {threshold bits, feature bytes}
    std::vector<int4> chunks;    // host copy of the chunks, plan after plan
    int64_t table_bytes = 0;
    int64_t max_tree_bytes = 0;
    int32_t max_levels = 0;      // most steps of a path: window levels x depth
    std::vector<double> steps;   // data walks: steps that a wavefront takes in each tree
    int exit_mode = dtree::kExitInt32;
};

// Launch plan of a forest for one load mode and split.
struct ForestPlan {
    const void *fn = nullptr;
    dtree::TileShape tile;
    int waves = 0, tiles = 0;    // wavefronts per workgroup, tiles they share
    int blocks_per_cu = 0;
    int lds_bytes = 0;
    int chunk_lds_bytes = 0;     // LDS reserved for one chunk (0: tables read in place)
    int first_chunk = 0, n_chunks = 0;
    std::vector<double> round_cost;   // estimated cycles of a round with b groups on a CU, at
                                      // b - 1 (b up to blocks_per_cu),
    double first_cost = 0.0;          // and of what comes before the first round
    dt_status status = DT_ERR_UNSUPPORTED;
    std::string why = "no kernel instance for this configuration";
};

constexpr int kForestSplits = 5;   // 1, 2, 4, 8 or 16 wavefronts per tile
constexpr int kForestList = 2;     // the node lists' place among a forest's encodings

void free_forest_encoding(ForestEncoding *e) {
    if (e->d_mem) (void)hipFree(e->d_mem);
    e->d_mem = nullptr;
}

}  // namespace

struct dt_forest {
    DeviceCaps caps;
    int32_t n_trees = 0, n_features = 0, n_classes = 0;
    int vote_words = 0;
    // data windows, speculative windows, node lists (data walk); a forest may have data
    // windows and lists, weighed at each call
    ForestEncoding enc[3];
    ForestPlan plan[3][dtree::kForestLoadModes][kForestSplits];   // [encoding][load mode][log2 split]
};

namespace {

bool valid_elem_type(dt_dtype t) {
    return t == DT_F32 || t == DT_F16 || t == DT_BF16 || t == DT_U8;
}

dt_status classify_impl(const dt_tree *tree, const void *d_x, dt_dtype x_type, int64_t n,
                        int64_t ld, void *d_out, dt_output out_kind, dt_algo algo, void *stream) {
    if (!tree) return fail(DT_ERR_INVALID_ARG, "tree is NULL");
    if (n < 0) return fail(DT_ERR_INVALID_ARG, "n must be >= 0");
    if (!single_tree_algo(algo)) return fail(DT_ERR_INVALID_ARG, "unknown algo");
    if (!valid_elem_type(x_type)) return fail(DT_ERR_INVALID_ARG, "unknown x_type");
    if (out_kind != DT_OUT_CLASS_U8 && out_kind != DT_OUT_CLASS_I32 &&
        out_kind != DT_OUT_LEAF_I32)
        return fail(DT_ERR_INVALID_ARG, "unknown out_kind");
    if (ld < tree->n_features) return fail(DT_ERR_INVALID_ARG, "ld must be >= n_features");
    if (out_kind == DT_OUT_CLASS_U8 && tree->n_classes > 256)
        return fail(DT_ERR_INVALID_ARG, "uint8 output needs n_classes <= 256");
    if (tree->n_features > dtree::kMaxRowStride)
        return fail(DT_ERR_UNSUPPORTED, "n_features > 256");
    if (n > (int64_t(1) << 37)) return fail(DT_ERR_UNSUPPORTED, "n > 2^37");
    if (n == 0) return DT_OK;
    if (!d_x || !d_out) return fail(DT_ERR_INVALID_ARG, "null device pointer");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev != tree->caps.device)
        return fail(DT_ERR_INVALID_ARG, "current device differs from the tree's device");

    if ((reinterpret_cast<uintptr_t>(d_x) % uintptr_t(dtree::elem_bytes(x_type))) != 0)
        return fail(DT_ERR_INVALID_ARG, "d_x is not aligned to its element size");
    const int mode = dtree::tree_load_mode(algo, d_x, x_type, ld, tree->n_features, tree->enc[1].depth);
    const Plan &plan = tree->plan[algo][x_type][mode][out_kind == DT_OUT_CLASS_U8 ? 0 : 1];
    if (plan.status != DT_OK) return fail(plan.status, plan.why);
    const Encoding &enc = tree->enc[plan.enc];

    dtree::KArgs a{};
    a.in = make_tile_rows(d_x, x_type, n, ld, tree->n_features, plan.tile);
    a.slots = enc.d_slots[x_type];
    a.exits = out_kind == DT_OUT_LEAF_I32 ? enc.d_exit_leaf : enc.d_exit_class;
    a.slot_bytes = int32_t(enc.list ? enc.table_bytes(x_type) : enc.slot_bytes[x_type]);
    a.want_leaf = out_kind == DT_OUT_LEAF_I32 ? 1 : 0;
    a.exit_bytes = int32_t(enc.exit_bytes);
    a.depth = enc.depth;
    a.levels = enc.levels;
    a.waves = plan.waves;
    a.out_kind = out_kind == DT_OUT_CLASS_U8 ? 0 : 1;
    a.out_cap = plan.out_cap;
    a.tile_bytes = plan.tile.tile_bytes;
    a.out_vec = (reinterpret_cast<uintptr_t>(d_out) & 15u) == 0 ? 1 : 0;
    a.hops = tree->path_hops;
    a.out = d_out;
    const int64_t want = (a.in.n_tiles + plan.waves - 1) / plan.waves;
    const int64_t resident = int64_t(plan.blocks_per_cu) * tree->caps.n_cu;
    const int blocks = int(std::max<int64_t>(1, std::min(want, resident)));
    e = dtree::launch_kernel(plan.fn, a, blocks, plan.lds_bytes,
                             static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "kernel launch");
    return DT_OK;
}

void destroy_impl(dt_tree *t) {
    if (!t) return;
    for (Encoding &e : t->enc) free_encoding(&e);
    delete t;
}

// Plan of the data decomposition for records of type `xt`: over windows or over the node
// list (data_walk_for has the rule).  `plan_on` plans for one encoding.
template <class PlanOn>
void plan_data(const dt_tree &t, int xt, bool listable, PlanOn plan_on, Plan *plan) {
    const Encoding &windows = t.enc[0];
    const int64_t list_bytes = t.enc[2].slot_bytes[xt];
    const dtree::DataWalk walk =
        listable ? dtree::data_walk_for(t.shape, windows.levels, windows.table_bytes(xt), list_bytes)
                 : dtree::DataWalk::kWindows;
    Plan list;
    if (walk != dtree::DataWalk::kWindows) plan_on(2, dtree::kAlgoList, &list);
    if (walk == dtree::DataWalk::kList && list.status == DT_OK) {
        *plan = list;
        return;
    }
    plan_on(0, DT_ALGO_DATA, plan);
    if (list.status != DT_OK) return;
    if (plan->status != DT_OK || !plan->tables_in_lds ||
        dtree::list_is_faster(t.shape, windows.levels, windows.depth, list_bytes,
                              plan->waves * plan->blocks_per_cu, list.waves * list.blocks_per_cu))
        *plan = list;
}

dt_status create_impl(const dt_node *nodes, int32_t n_nodes, int32_t n_features,
                      int32_t n_classes, const dt_tree_options *opt, dt_tree **out) {
    if (!out) return fail(DT_ERR_INVALID_ARG, "out is NULL");
    dt_status st = check_options(opt);
    if (st != DT_OK) return st;
    std::string msg;
    dtree::TreeShape shape;
    st = dtree::validate_tree(nodes, n_nodes, n_features, n_classes, &shape, &msg);
    if (st != DT_OK) return fail(st, msg);
    dt_tree *t = new (std::nothrow) dt_tree();
    if (!t) return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    st = query_device(&t->caps);
    if (st != DT_OK) { delete t; return st; }
    t->shape = shape;
    t->n_features = n_features;
    t->n_classes = n_classes;
    if (opt && opt->path_hops) t->path_hops = opt->path_hops;
    int depth[2];
    window_depths(nodes, shape, n_features, opt, &depth[0], &depth[1]);
    t->enc[0].size_windows(depth[0], dtree::count_windows(nodes, shape, depth[0]),
                           dtree::count_levels(nodes, shape, depth[0]));
    t->enc[1].size_windows(depth[1], dtree::count_windows(nodes, shape, depth[1]),
                           dtree::count_levels(nodes, shape, depth[1]));
    // lists only with the default window depth
    const bool listable = !(opt && opt->data_window_depth) && n_nodes <= dtree::kMaxTreeListNodes;
    if (listable) t->enc[2].size_list(n_nodes);
    bool used[3] = {false, true, false};
    for (int algo = 0; algo < 3; ++algo) {
        for (int xt = 0; xt < dtree::kElemTypes; ++xt) {
            for (int m = 0; m < dtree::kLoadModes; ++m) {
                Plan *pl = t->plan[algo][xt][m];
                if (n_features > dtree::kMaxRowStride) {
                    pl[0].why = pl[1].why = "n_features > 256";
                    continue;
                }
                if (algo == DT_ALGO_PATH && xt != DT_F32) {
                    pl[0].why = pl[1].why = "the path kernel reads fp32 records only";
                    continue;
                }
                const int es = dtree::elem_bytes(xt);
                if (m == dtree::kLoadExact && !exact_rows(n_features, es)) continue;
                if (m == dtree::kLoadFlat && !dtree::flat_rows(algo, xt, n_features, depth[1])) continue;
                if (m == dtree::kLoadBytes && es == 4) continue;
                for (int o = 0; o < 2; ++o) {
                    const auto plan_on = [&](int e, int kernel_algo, Plan *p) {
                        p->enc = e;
                        make_plan(t->caps, kernel_algo, xt, n_features, m, t->enc[e].depth,
                                  t->enc[e].table_bytes(xt), o == 0 ? 1 : 4,
                                  opt ? opt->waves_per_cu : 0, p);
                    };
                    if (algo == DT_ALGO_DATA)
                        plan_data(*t, xt, listable, plan_on, &pl[o]);
                    else
                        plan_on(1, algo, &pl[o]);
                    used[pl[o].enc] = true;
                }
            }
        }
    }
    if (!used[2]) used[0] = true;
    for (int e = 0; e < 3; ++e) {
        if (!used[e]) continue;
        if (e == 2) {
            st = upload_list(nodes, n_nodes, &t->enc[2]);
        } else {
            dtree::WindowTables wt;
            dtree::build_windows(nodes, shape, depth[e], &wt);
            st = upload_encoding(wt, &t->enc[e]);
        }
        if (st != DT_OK) {
            destroy_impl(t);
            return st;
        }
    }
    *out = t;
    return DT_OK;
}

// ---- forests ---------------------------------------------------------------------------

constexpr int64_t kMaxForestBytes = (int64_t(1) << 31) - 1;   // of tables (int32 offsets)

// Speculative forests use windows of depth 2 (default) or 4.
constexpr int kForestSpecDepth = 2;

int vote_words_for(int32_t n_classes) {
    if (n_classes <= 8) return 2;
    if (n_classes <= 16) return 4;
    return 16;
}

// Encode every tree with window depth `depth` and lay the tables out back to back.
void encode_forest(const dt_node *nodes, const int32_t *offsets, int32_t n_trees,
                   const std::vector<dtree::TreeShape> &shapes, int algo, int depth,
                   std::vector<unsigned char> *bytes, ForestEncoding *enc) {
    enc->depth = depth;
    enc->trees.assign(size_t(n_trees), int4{0, 0, 0, 0});
    enc->roots.assign(size_t(n_trees), int2{0, 0});
    enc->max_tree_bytes = 0;
    bytes->clear();
    std::vector<dtree::WindowTables> wts(static_cast<size_t>(n_trees));
    // Exit codes (next window ids, and results -(class + 1)) of the data decomposition are
    // packed into the spare bits of the windows' bottom slots when every code of the forest
    // fits 11 bits (the feature's byte offset, at most 1020, takes the low 10): the tables
    // then hold slots only, a fifth less than with int16 codes (four complete depth-10
    // trees per 32 KiB chunk instead of three), and the walk reads no exit table.  Failing
    // that they are int16 when every code fits, else int32.  (The speculative walk keeps
    // int32 codes: its narrower instances need more registers than 16 wavefronts per CU
    // leave it.)
    bool fits11 = algo == DT_ALGO_DATA, fits16 = algo == DT_ALGO_DATA;
    for (int32_t k = 0; k < n_trees; ++k) {
        dtree::build_windows(nodes + offsets[k], shapes[size_t(k)], depth, &wts[size_t(k)]);
        for (int32_t c : wts[size_t(k)].exit_class) {
            fits11 = fits11 && c >= -1024 && c <= 1023;
            fits16 = fits16 && c >= INT16_MIN && c <= INT16_MAX;
        }
    }
    enc->exit_mode = fits11 ? dtree::kExitPacked : fits16 ? dtree::kExitInt16 : dtree::kExitInt32;
    const int64_t exit_size = enc->exit_mode == dtree::kExitPacked  ? 0
                              : enc->exit_mode == dtree::kExitInt16 ? 2
                                                                    : 4;
    for (int32_t k = 0; k < n_trees; ++k) {
        const dtree::WindowTables &wt = wts[size_t(k)];
        const int64_t n_slots = int64_t(wt.n_windows) * wt.slots;
        const int64_t sb = align16(n_slots * 8), eb = align16(n_slots * exit_size);
        const int64_t off = int64_t(bytes->size());
        bytes->resize(size_t(off + sb + eb), 0);
        unsigned char *p = bytes->data() + off;
        const int64_t S = wt.slots;
        for (int64_t i = 0; i < n_slots; ++i) {
            int32_t fb = 4 * wt.feature[size_t(i)];   // byte offset in an fp32 row
            const int64_t q = i % S;                  // heap position in the window
            if (enc->exit_mode == dtree::kExitPacked && q >= S / 2) {  // bottom level: its children's exits
                const int64_t e = i - q + 2 * q - S;  // exit of child 2q in this window
                const uint32_t lo = uint32_t(wt.exit_class[size_t(e)]) & 0x7FFu;
                const uint32_t hi = uint32_t(wt.exit_class[size_t(e + 1)]) & 0x7FFu;
                fb = int32_t(uint32_t(fb) | lo << 10 | hi << 21);
            }
            std::memcpy(p + 8 * i, &wt.threshold[size_t(i)], 4);
            std::memcpy(p + 8 * i + 4, &fb, 4);
        }
        if (enc->exit_mode == dtree::kExitInt16) {
            for (int64_t i = 0; i < n_slots; ++i) {
                const int16_t c = int16_t(wt.exit_class[size_t(i)]);
                std::memcpy(p + sb + 2 * i, &c, 2);
            }
        } else if (enc->exit_mode == dtree::kExitInt32) {
            std::memcpy(p + sb, wt.exit_class.data(), size_t(n_slots * 4));
        }
        enc->trees[size_t(k)] = int4{int(off), int(sb), wt.levels, 0};
        int2 root{0, 0};                          // the slot just written for slot 1
        std::memcpy(&root, p + 8, 8);
        enc->roots[size_t(k)] = root;
        enc->max_tree_bytes = std::max(enc->max_tree_bytes, sb + eb);
        enc->max_levels = std::max(enc->max_levels, wt.levels * depth);
        if (algo == DT_ALGO_DATA) {
            // whole windows, and, where there are several, an exit to follow after each
            const int reached = dtree::reached_depth(nodes + offsets[k], shapes[size_t(k)]);
            const int levels = std::min(wt.levels, (reached + depth - 1) / depth);
            enc->steps.push_back(double(levels) * (depth + (wt.levels > 1 ? 1 : 0)));
        }
    }
    enc->table_bytes = int64_t(bytes->size());
}

// Every tree as a node list (see walk_list_k).
void list_forest(const dt_node *nodes, const int32_t *offsets, int32_t n_trees,
                 const std::vector<dtree::TreeShape> &shapes, std::vector<unsigned char> *bytes,
                 ForestEncoding *enc) {
    enc->depth = 0;
    enc->exit_mode = dtree::kExitList;
    std::vector<uint32_t> list;
    for (int32_t k = 0; k < n_trees; ++k) {
        const dt_node *t = nodes + offsets[k];
        const int32_t n = offsets[k + 1] - offsets[k];
        const int64_t off = int64_t(bytes->size()), size = dtree::list_bytes(n);
        bytes->resize(size_t(off + size), 0);
        list.assign(size_t(size / 4), 0u);
        dtree::build_forest_list(t, n, dtree::breadth_first_order(t, n), list.data());
        std::memcpy(bytes->data() + off, list.data(), size_t(size));
        const int32_t depth = shapes[size_t(k)].depth;
        enc->trees.push_back(int4{int(off), int(size), depth, 0});
        enc->roots.push_back(int2{int(list[2]), int(list[3])});
        enc->max_tree_bytes = std::max(enc->max_tree_bytes, size);
        enc->steps.push_back(dtree::reached_depth(t, shapes[size_t(k)]));
    }
    enc->table_bytes = int64_t(bytes->size());
}

// Wavefronts per CU the forest kernel aims for by default (measured: 16 beat 8 by 5% on a
// 32-tree forest; more gained nothing).
constexpr int kForestWavesPerCu = 16;

// Workgroup shape and LDS chunks of consecutive trees for a forest whose tiles take
// `tile_bytes` each, 2^split wavefronts to a tile.
void chunk_forest(const DeviceCaps &caps, int algo, int waves_per_cu, int split, int64_t tile_bytes,
                  ForestEncoding *enc, ForestPlan *plan) {
    const int target = waves_per_cu > 0 ? waves_per_cu : kForestWavesPerCu;
    plan->first_chunk = int(enc->chunks.size());
    plan->chunk_lds_bytes = 0;
    // The most resident wavefronts up to the target whose tiles leave a chunk buffer that
    // holds the largest tree; ties: larger chunk buffers (fewer passes).
    int best_w = 0, best_score = 0;
    int64_t best_budget = 0;
    // Speculative walks of wide rows (more than 9 KiB a tile) keep to 8: a ninth tile would
    // take half of the chunk (64 features, 100 trees: 331 us with 8, 400 us with 9).
    int most = algo == DT_ALGO_SPECULATIVE && split == 0 && tile_bytes > 9 * 1024
                   ? dtree::kMaxWavesPerBlock
                   : dtree::forest_max_waves(algo, enc->depth);
    if (split > 0) most = std::min(most, target);   // (unsplit: fewer waves win the tie)
    for (int bpc = 1; bpc <= 4; ++bpc) {
        const int64_t per_block = std::min<int64_t>(caps.lds_per_block, caps.lds_per_cu / bpc);
        for (int w = most; w >= 1 << split; --w) {
            const int64_t budget = per_block - (w >> split) * tile_bytes;
            if (budget < enc->max_tree_bytes) continue;
            const int score = std::min(target, w * bpc);
            if (score > best_score || (score == best_score && budget > best_budget)) {
                best_w = w;
                best_score = score;
                best_budget = budget;
            }
        }
    }
    plan->waves = best_w;
    if (best_w == 0) {   // single trees too large for the LDS: one pass, tables read in place
        enc->chunks.push_back(int4{0, int(enc->trees.size()), 0, int(enc->table_bytes)});
        plan->n_chunks = 1;
        return;
    }
    int32_t first = 0;
    int64_t max_chunk = 0;
    while (first < int32_t(enc->trees.size())) {
        int32_t end = first;
        int64_t bytes = 0;
        while (end < int32_t(enc->trees.size())) {
            const int64_t off = enc->trees[size_t(end)].x;
            const int64_t next = end + 1 < int32_t(enc->trees.size())
                                     ? int64_t(enc->trees[size_t(end + 1)].x)
                                     : enc->table_bytes;
            if (bytes + (next - off) > best_budget) break;
            bytes += next - off;
            ++end;
        }
        // every wavefront of a tile gets as many trees of the chunk, where it holds enough
        const int32_t parts = 1 << split;
        if (end < int32_t(enc->trees.size()) && end - first > parts) {
            end = first + (end - first) / parts * parts;
            bytes = enc->trees[size_t(end)].x - enc->trees[size_t(first)].x;
        }
        const int32_t off0 = enc->trees[size_t(first)].x;
        enc->chunks.push_back(int4{first, end, off0, int(bytes)});
        max_chunk = std::max(max_chunk, bytes);
        first = end;
    }
    plan->chunk_lds_bytes = int32_t(max_chunk);
    plan->n_chunks = int(enc->chunks.size()) - plan->first_chunk;
}

dt_status upload_forest(const std::vector<unsigned char> &bytes, ForestEncoding *enc) {
    const int64_t tb = align16(int64_t(bytes.size()));
    const int64_t db = int64_t(enc->trees.size()) * 16;
    const int64_t cb = int64_t(enc->chunks.size()) * 16;
    const int64_t rb = int64_t(enc->roots.size()) * 8;
    std::vector<unsigned char> host(size_t(tb + db + cb + rb), 0);
    std::memcpy(host.data(), bytes.data(), bytes.size());
    std::memcpy(host.data() + tb, enc->trees.data(), size_t(db));
    std::memcpy(host.data() + tb + db, enc->chunks.data(), size_t(cb));
    std::memcpy(host.data() + tb + db + cb, enc->roots.data(), size_t(rb));
    hipError_t e = hipMalloc(&enc->d_mem, host.size());
    if (e != hipSuccess) {
        enc->d_mem = nullptr;
        return fail(DT_ERR_NO_MEMORY, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    e = hipMemcpy(enc->d_mem, host.data(), host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpy(forest tables)");
    auto *base = static_cast<unsigned char *>(enc->d_mem);
    enc->d_tables = reinterpret_cast<const int4 *>(base);
    enc->d_trees = reinterpret_cast<const int4 *>(base + tb);
    enc->d_chunks = reinterpret_cast<const int4 *>(base + tb + db);
    enc->d_roots = reinterpret_cast<const int2 *>(base + tb + db + cb);
    return DT_OK;
}

// Estimated time, in cycles, of one round of groups (every resident workgroup, `blocks` to a
// CU, walks its tiles through all trees).  A walk of 64 records takes the CU's LDS some
// cycles per step and tree, and its wavefront at least some more per step (data: of four
// trees together; speculative: of one), whichever is longer with this many wavefronts.
// Tables read in place keep each workgroup waiting, a second one as long again.  Each byte of
// tables copied takes 1/64 cycle, each chunk its barriers, each group its staging, which
// kernels without prefetch wait for.  The constants give the measured order, not the time
// (which is up to half as long again).  Of 876 data walks measured with windows and with lists
// (mixed, irregular and chain-like forests of 6 to 200 trees, 8 to 64 features, 1,000 to
// 600,000 records) the choice was slower than the other by more than 5% in 36 to 45 (three
// runs), 1.26 times at most.  Speculative windows of depth 4, 100,001 x 16 records, 30
// complete trees of depth 8, 16 vote words: 42.4 us with one wavefront per tile, 36.6 us with
// the two that are chosen.
double round_cost(const ForestEncoding &enc, int algo, const ForestPlan &p, int split, int blocks) {
    const bool in_place = p.chunk_lds_bytes == 0, data = algo == DT_ALGO_DATA;
    const double lds_step = data ? (in_place ? 20.0 : 10.0) : (in_place ? 100.0 : 40.0);
    const double chain_step = data ? (in_place ? 650.0 : 260.0) : (in_place ? 750.0 : 400.0);
    const double spec_steps = std::max(1, std::min(enc.max_levels, 16));
    constexpr int kIlp = 4;                                 // trees walked together (data)
    const int parts = 1 << split;
    double walk = 0.0;
    for (int c = p.first_chunk; c < p.first_chunk + p.n_chunks; ++c) {
        const int first = enc.chunks[size_t(c)].x, end = enc.chunks[size_t(c)].y;
        const int share = (end - first + parts - 1) / parts;      // of a wavefront
        double all = 0.0, longest = 0.0;     // steps of the trees, of a wavefront's groups
        if (data) {
            for (int k = first; k < end; ++k) all += enc.steps[size_t(k)];
            for (int part = first; part < end; part += share) {
                double steps = 0.0;
                const int last = std::min(end, part + share);
                for (int k = part; k < last; k += kIlp)
                    steps += *std::max_element(enc.steps.begin() + k,
                                               enc.steps.begin() + std::min(k + kIlp, last));
                longest = std::max(longest, steps);
            }
        } else {
            all = spec_steps * (end - first);
            longest = spec_steps * share;
        }
        walk += std::max(lds_step * all * p.tiles * blocks,
                         chain_step * longest * (in_place ? blocks : 1));
    }
    const double tables =
        in_place || p.n_chunks == 1 ? 0.0 : double(enc.table_bytes) / 64.0 + 800.0 * p.n_chunks;
    const double wait = p.tile.vecs > 0 || p.tile.mode == dtree::kLoadExact ? 1500.0 : 7000.0;
    return walk + blocks * (p.tiles * (p.tile.tile_bytes / 64.0) + tables) + wait;
}

dt_status plan_forest(const DeviceCaps &caps, int algo, int n_features, int load_mode, int split,
                      int vote_words, int waves_per_cu, ForestEncoding *enc, ForestPlan *plan) {
    dtree::ForestShape s;
    s.algo = algo;
    s.vote_words = vote_words;
    s.depth = enc->depth;
    s.exit_mode = enc->exit_mode;
    s.split = split;
    s.tile = dtree::forest_tile_shape(algo, n_features, load_mode, split == 0);
    // a split kernel's tiles each have a box of votes beside them
    const int64_t vote_bytes = split ? int64_t(vote_words) * 256 : 0;
    chunk_forest(caps, algo, waves_per_cu, split, s.tile.tile_bytes + vote_bytes, enc, plan);
    s.tables_in_lds = plan->chunk_lds_bytes > 0;
    if (!s.tables_in_lds && s.tile.mode == dtree::kLoadExact) s.tile.mode = dtree::kLoadRows;
    if (!s.tables_in_lds) s.tile = dtree::forest_tile_shape(algo, n_features, s.tile.mode, false);
    plan->tile = s.tile;
    plan->fn = dtree::forest_kernel_for(s);
    if (!plan->fn) {
        plan->why = "no forest kernel instance for this configuration";
        return plan->status = DT_ERR_UNSUPPORTED;
    }
    {
        std::lock_guard<std::mutex> lock(g_prep_mutex);
        if (std::find(g_prepared.begin(), g_prepared.end(), plan->fn) == g_prepared.end()) {
            hipError_t e = dtree::prepare_kernel(plan->fn, caps.lds_per_block);
            if (e != hipSuccess) {
                plan->why = std::string("hipFuncSetAttribute: ") + hipGetErrorString(e);
                return plan->status = DT_ERR_HIP;
            }
            g_prepared.push_back(plan->fn);
        }
    }
    int best_waves = 0;
    const int planned = plan->waves;
    // a split kernel keeps to the caller's wavefronts per CU
    const int limit = split > 0 && waves_per_cu > 0 ? waves_per_cu : INT_MAX;
    for (int w = std::min(limit, dtree::forest_max_waves(algo, enc->depth)); w >= 1 << split; --w) {
        if (s.tables_in_lds && w != planned) continue;   // the chunks were cut for these
        const int tiles = w >> split;
        const int lds = int(plan->chunk_lds_bytes + tiles * (s.tile.tile_bytes + vote_bytes));
        if (lds > caps.lds_per_block) continue;
        int nb = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, plan->fn, w * 64,
                                                                    size_t(lds));
        if (e != hipSuccess) {
            plan->why = std::string("hipOccupancyMaxActiveBlocksPerMultiprocessor: ") +
                        hipGetErrorString(e);
            return plan->status = DT_ERR_HIP;
        }
        nb = std::min(nb, limit / w);
        if (nb >= 1 && nb * w > best_waves) {
            best_waves = nb * w;
            plan->waves = w;
            plan->tiles = tiles;
            plan->blocks_per_cu = nb;
            plan->lds_bytes = lds;
        }
    }
    if (best_waves == 0) {
        plan->why = "no workgroup shape fits this forest kernel";
        return plan->status = DT_ERR_UNSUPPORTED;
    }
    for (int b = 1; b <= plan->blocks_per_cu; ++b)
        plan->round_cost.push_back(round_cost(*enc, algo, *plan, split, b));
    // tables that stay in the LDS are copied once
    if (plan->chunk_lds_bytes > 0 && plan->n_chunks == 1)
        plan->first_cost = double(enc->table_bytes) / 64.0;
    plan->why.clear();
    return plan->status = DT_OK;
}

// How a call's tiles are spread: the first `lead` by the unsplit kernel, the rest by the
// kernel of 2^split wavefronts per tile (split 0: none of them).
struct ForestSpread {
    int enc = 0;             // the encoding walked
    int64_t lead = 0;
    int split = 0;
    double cost = -1.0;      // estimated cycles (-1: no plan holds)
};

// The unsplit kernel walks a tile per wavefront and is the most efficient with every
// workgroup busy; what it does badly is a round that few workgroups have part in (one
// group of 16 tiles more than there are CUs takes two rounds) and inputs of fewer tiles
// than wavefronts.  Weighed here: all tiles by one of the kernels, or the full rounds by the
// unsplit one and the rest by a split one (a second launch).
ForestSpread spread_forest(const ForestPlan *const (&plan)[kForestSplits], int n_cu,
                           int64_t tiles) {
    ForestSpread best;
    best.lead = tiles;          // where no plan holds, the unsplit one says why
    constexpr double kLaunch = 8000.0;   // a second launch: about 3 us
    const auto rounds = [&](const ForestPlan &p, int64_t t) {
        const int64_t groups = (t + p.tiles - 1) / p.tiles, slots = int64_t(p.blocks_per_cu) * n_cu;
        const int64_t rest = groups % slots;      // on as few to a CU as they go
        return double(groups / slots) * p.round_cost.back() + p.first_cost +
               (rest > 0 ? p.round_cost[size_t((rest - 1) / n_cu)] : 0.0);
    };
    const auto weigh = [&](double cost, int64_t lead, int split) {
        if (best.cost >= 0.0 && cost >= best.cost) return;
        best.cost = cost;
        best.lead = lead;
        best.split = split;
    };
    const ForestPlan &whole = *plan[0];
    int64_t full = 0;
    if (whole.status == DT_OK) {
        weigh(rounds(whole, tiles), tiles, 0);
        const int64_t per_round = int64_t(whole.tiles) * whole.blocks_per_cu * n_cu;
        full = tiles / per_round * per_round;
    }
    for (int s = 1; s < kForestSplits; ++s) {
        if (plan[s]->status != DT_OK) continue;
        weigh(rounds(*plan[s], tiles), 0, s);
        if (full > 0 && full < tiles)
            weigh(rounds(whole, full) + rounds(*plan[s], tiles - full) + kLaunch, full, s);
    }
    return best;
}

void forest_destroy_impl(dt_forest *f) {
    if (!f) return;
    for (ForestEncoding &e : f->enc) free_forest_encoding(&e);
    delete f;
}

dt_status forest_create_impl(const dt_node *nodes, const int32_t *offsets, int32_t n_trees,
                             int32_t n_features, int32_t n_classes, const dt_tree_options *opt,
                             dt_forest **out) {
    if (!out) return fail(DT_ERR_INVALID_ARG, "out is NULL");
    if (!nodes || !offsets) return fail(DT_ERR_INVALID_ARG, "nodes or tree_offsets is NULL");
    if (n_trees < 1) return fail(DT_ERR_INVALID_ARG, "n_trees must be >= 1");
    if (n_features < 1 || n_classes < 1)
        return fail(DT_ERR_INVALID_ARG, "n_features and n_classes must be >= 1");
    dt_status st = check_options(opt);
    if (st != DT_OK) return st;
    if (opt && opt->spec_window_depth != 0 && opt->spec_window_depth != 2 &&
        opt->spec_window_depth != 4)
        return fail(DT_ERR_UNSUPPORTED, "forests use speculative windows of depth 2 or 4");
    if (n_trees > dtree::kMaxForestTrees)
        return fail(DT_ERR_UNSUPPORTED, "forests are limited to 255 trees");
    if (n_classes > dtree::kMaxForestClasses)
        return fail(DT_ERR_UNSUPPORTED, "forests are limited to 64 classes");
    if (offsets[0] != 0) return fail(DT_ERR_INVALID_ARG, "tree_offsets[0] must be 0");
    std::vector<dtree::TreeShape> shapes(static_cast<size_t>(n_trees));
    int max_depth = 0;
    for (int32_t k = 0; k < n_trees; ++k) {
        if (offsets[k + 1] <= offsets[k])
            return fail(DT_ERR_INVALID_ARG, "tree_offsets must increase strictly");
        std::string msg;
        st = dtree::validate_tree(nodes + offsets[k], offsets[k + 1] - offsets[k], n_features,
                                  n_classes, &shapes[size_t(k)], &msg);
        if (st != DT_OK) return fail(st, "tree " + std::to_string(k) + ": " + msg);
        max_depth = std::max(max_depth, shapes[size_t(k)].depth);
    }
    dt_forest *f = new (std::nothrow) dt_forest();
    if (!f) return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    st = query_device(&f->caps);
    if (st != DT_OK) { delete f; return st; }
    f->n_trees = n_trees;
    f->n_features = n_features;
    f->n_classes = n_classes;
    f->vote_words = vote_words_for(n_classes);

    // data windows: the depth that makes the forest's tables smallest; where no depth has
    // every tree in one window, or the windows' slots take more than the nodes, node lists too
    int data_d = opt && opt->data_window_depth ? opt->data_window_depth : 0;
    bool list = false, windows = true;
    if (!data_d) {
        int64_t best = -1, list_bytes = 0;
        bool listable = true;
        for (int d = 1; d <= std::min(dtree::kMaxWindowDepth, std::max(1, max_depth)); ++d) {
            int64_t total = 0;
            for (int32_t k = 0; k < n_trees; ++k)
                total += dtree::table_bytes(
                    dtree::count_windows(nodes + offsets[k], shapes[size_t(k)], d), d);
            if (best < 0 || total <= best) { best = total; data_d = d; }
        }
        for (int32_t k = 0; k < n_trees; ++k) {
            list_bytes += 8 * (int64_t(offsets[k + 1] - offsets[k]) + 1);
            listable = listable && offsets[k + 1] - offsets[k] <= dtree::kMaxForestListNodes;
        }
        list = listable && (max_depth > data_d || best / 12 * 8 > list_bytes);
        windows = !list || best < kMaxForestBytes;
    }
    const int spec_d = opt && opt->spec_window_depth ? opt->spec_window_depth : kForestSpecDepth;
    for (int e = 0; e < 3; ++e) {
        if (e == DT_ALGO_DATA ? !windows : e == kForestList && !list) continue;
        const int algo = e == DT_ALGO_SPECULATIVE ? DT_ALGO_SPECULATIVE : DT_ALGO_DATA;
        ForestEncoding *enc = &f->enc[e];
        std::vector<unsigned char> bytes;
        if (e == kForestList)
            list_forest(nodes, offsets, n_trees, shapes, &bytes, enc);
        else
            encode_forest(nodes, offsets, n_trees, shapes, algo, e == DT_ALGO_DATA ? data_d : spec_d,
                          &bytes, enc);
        if (enc->table_bytes > kMaxForestBytes) {
            forest_destroy_impl(f);
            return fail(DT_ERR_UNSUPPORTED, "forest tables exceed 2 GiB");
        }
        for (int m = 0; m < dtree::kForestLoadModes; ++m) {
            for (int sp = 0; sp < kForestSplits; ++sp) {
                ForestPlan *p = &f->plan[e][m][sp];
                if (n_features > dtree::kMaxRowStride) {
                    p->why = "n_features > 256";
                    continue;
                }
                if (m == dtree::kLoadExact &&
                    (!dtree::exact_rows(n_features, 4) || n_features > 32 || sp > 0))
                    continue;
                if (m == dtree::kLoadFlat &&
                    (n_features % 4 == 0 ||
                     (algo == DT_ALGO_SPECULATIVE && n_features <= 4 * dtree::kMaxForestPitchVecs)))
                    continue;
                const int waves_per_cu = opt ? opt->waves_per_cu : 0;
                if ((1 << sp) > dtree::forest_max_waves(algo, enc->depth)) continue;
                if (waves_per_cu > 0 && (1 << sp) > waves_per_cu) continue;
                plan_forest(f->caps, algo, n_features, m, sp, f->vote_words, waves_per_cu, enc, p);
            }
        }
        st = upload_forest(bytes, enc);
        if (st != DT_OK) { forest_destroy_impl(f); return st; }
    }
    *out = f;
    return DT_OK;
}

// How a call's tiles are spread, over the faster of the forest's encodings, and the plans of
// that encoding for the call's load mode, by split.
ForestSpread spread_call(const dt_forest &f, const float *d_x, int64_t n, int64_t ld, dt_algo algo,
                         const ForestPlan *(&plans)[kForestSplits]) {
    // a split kernel reads exact rows as any others of a multiple of 16 bytes
    const int mode = dtree::forest_load_mode(algo, d_x, ld, f.n_features);
    const int split_mode = mode == dtree::kLoadExact ? int(dtree::kLoadRows) : mode;
    const int64_t tiles = (n + dtree::kTileRows - 1) / dtree::kTileRows;
    ForestSpread best;
    bool any = false;
    for (int e : {int(algo), kForestList}) {
        if (!f.enc[e].d_mem || (e == kForestList && algo != DT_ALGO_DATA)) continue;
        const ForestPlan *of_enc[kForestSplits];
        for (int sp = 0; sp < kForestSplits; ++sp)
            of_enc[sp] = &f.plan[e][sp == 0 ? mode : split_mode][sp];
        ForestSpread s = spread_forest(of_enc, f.caps.n_cu, tiles);
        if (any && (s.cost < 0.0 || (best.cost >= 0.0 && s.cost >= best.cost))) continue;
        any = true;
        best = s;
        best.enc = e;
        std::copy(of_enc, of_enc + kForestSplits, plans);
    }
    return best;
}

dt_status forest_classify_impl(const dt_forest *f, const float *d_x, int64_t n, int64_t ld,
                               void *d_out, dt_output out_kind, dt_algo algo, void *stream) {
    if (!f) return fail(DT_ERR_INVALID_ARG, "forest is NULL");
    if (n < 0) return fail(DT_ERR_INVALID_ARG, "n must be >= 0");
    if (algo == DT_ALGO_PATH)
        return fail(DT_ERR_UNSUPPORTED, "forests run the data and speculative decompositions");
    if (algo != DT_ALGO_DATA && algo != DT_ALGO_SPECULATIVE)
        return fail(DT_ERR_INVALID_ARG, "unknown algo");
    if (out_kind != DT_OUT_CLASS_U8 && out_kind != DT_OUT_CLASS_I32)
        return fail(DT_ERR_INVALID_ARG, "forests output classes (uint8 or int32)");
    if (ld < f->n_features) return fail(DT_ERR_INVALID_ARG, "ld must be >= n_features");
    if (f->n_features > dtree::kMaxRowStride)
        return fail(DT_ERR_UNSUPPORTED, "n_features > 256");
    if (n > (int64_t(1) << 37)) return fail(DT_ERR_UNSUPPORTED, "n > 2^37");
    if (n == 0) return DT_OK;
    if (!d_x || !d_out) return fail(DT_ERR_INVALID_ARG, "null device pointer");
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev != f->caps.device)
        return fail(DT_ERR_INVALID_ARG, "current device differs from the forest's device");
    const ForestPlan *plans[kForestSplits];
    const ForestSpread spread = spread_call(*f, d_x, n, ld, algo, plans);
    const ForestEncoding &enc = f->enc[spread.enc];
    const int64_t tiles = (n + dtree::kTileRows - 1) / dtree::kTileRows;

    for (int part = 0; part < 2; ++part) {
        const int64_t first = part == 0 ? 0 : spread.lead, end = part == 0 ? spread.lead : tiles;
        if (first >= end) continue;
        const int split = part == 0 ? 0 : spread.split;
        const ForestPlan &plan = *plans[split];
        if (plan.status != DT_OK) return fail(plan.status, plan.why);
        dtree::FArgs a{};
        a.in = make_tile_rows(d_x, dtree::kXF32, n, ld, f->n_features, plan.tile);
        a.tables = enc.d_tables;
        a.trees = enc.d_trees;
        a.roots = enc.d_roots;
        a.chunks = enc.d_chunks + plan.first_chunk;
        a.first_tile = first;
        a.end_tile = end;
        a.n_chunks = plan.n_chunks;
        a.table_lds_bytes = plan.chunk_lds_bytes;
        a.tile_bytes = plan.tile.tile_bytes;
        a.split = split;
        a.depth = enc.depth;
        a.n_classes = f->n_classes;
        a.waves = plan.waves;
        a.out_kind = out_kind == DT_OUT_CLASS_U8 ? 0 : 1;
        a.out = d_out;
        const int64_t groups = (end - first + plan.tiles - 1) / plan.tiles;
        const int64_t resident = int64_t(plan.blocks_per_cu) * f->caps.n_cu;
        const int blocks = int(std::max<int64_t>(1, std::min(groups, resident)));
        e = dtree::launch_forest(plan.fn, a, blocks, plan.lds_bytes,
                                 static_cast<hipStream_t>(stream));
        if (e != hipSuccess) return hip_fail(e, "forest kernel launch");
    }
    return DT_OK;
}

}  // namespace

namespace dtree {

dt_status set_error(dt_status s, const std::string &msg) { return fail(s, msg); }
dt_status set_hip_error(hipError_t e, const char *what) { return hip_fail(e, what); }
void clear_error() { g_last_error.clear(); }
int device_of(const dt_tree *t) { return t->caps.device; }
int device_of(const dt_forest *f) { return f->caps.device; }
int32_t features_of(const dt_tree *t) { return t->n_features; }
int32_t features_of(const dt_forest *f) { return f->n_features; }

}  // namespace dtree

extern "C" {

int32_t dt_abi_version(void) { return DT_ABI_VERSION; }

const char *dt_status_string(dt_status s) {
    switch (s) {
        case DT_OK: return "ok";
        case DT_ERR_INVALID_ARG: return "invalid argument";
        case DT_ERR_INVALID_TREE: return "invalid tree";
        case DT_ERR_UNSUPPORTED: return "unsupported";
        case DT_ERR_HIP: return "HIP runtime error";
        case DT_ERR_NO_MEMORY: return "out of memory";
        default: return "unknown status";
    }
}

const char *dt_last_error(void) { return g_last_error.c_str(); }

dt_status dt_tree_check(const dt_node *nodes, int32_t n_nodes, int32_t n_features,
                        int32_t n_classes, const dt_tree_options *opt, dt_tree_info *info) {
    try {
        g_last_error.clear();
        dt_status st = check_options(opt);
        if (st != DT_OK) return st;
        std::string msg;
        dtree::TreeShape shape;
        st = dtree::validate_tree(nodes, n_nodes, n_features, n_classes, &shape, &msg);
        if (st != DT_OK) return fail(st, msg);
        if (info) {
            int dd, sd;
            window_depths(nodes, shape, n_features, opt, &dd, &sd);
            fill_info(shape, n_features, n_classes, dd, dtree::count_windows(nodes, shape, dd),
                      dtree::count_levels(nodes, shape, dd), sd, dtree::count_windows(nodes, shape, sd),
                      dtree::count_levels(nodes, shape, sd), info);
        }
        return DT_OK;
    } catch (const std::bad_alloc &) {
        return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_threshold_keys(const float *thresholds, int64_t n, dt_dtype type, uint16_t *keys) {
    g_last_error.clear();
    if (n < 0) return fail(DT_ERR_INVALID_ARG, "n must be >= 0");
    if (type != DT_F16 && type != DT_BF16 && type != DT_U8)
        return fail(DT_ERR_INVALID_ARG, "type must be DT_F16, DT_BF16 or DT_U8");
    if (n > 0 && (!thresholds || !keys)) return fail(DT_ERR_INVALID_ARG, "null buffer");
    for (int64_t i = 0; i < n; ++i) keys[i] = uint16_t(dtree::narrow_key(thresholds[i], type));
    return DT_OK;
}

dt_status dt_encode_windows(const dt_node *nodes, int32_t n_nodes, int32_t n_features,
                            int32_t n_classes, int32_t window_depth, int32_t capacity_windows,
                            int32_t *features, float *thresholds, int32_t *exit_class,
                            int32_t *exit_leaf, int32_t *n_windows, int32_t *levels) {
    try {
        g_last_error.clear();
        if (window_depth < 1 || window_depth > dtree::kMaxWindowDepth)
            return fail(DT_ERR_INVALID_ARG, "window_depth must be 1..16");
        if (capacity_windows < 0) return fail(DT_ERR_INVALID_ARG, "capacity_windows < 0");
        std::string msg;
        dtree::TreeShape shape;
        dt_status st = dtree::validate_tree(nodes, n_nodes, n_features, n_classes, &shape, &msg);
        if (st != DT_OK) return fail(st, msg);
        const int64_t nw = dtree::count_windows(nodes, shape, window_depth);
        if (nw * (int64_t(1) << window_depth) > (int64_t(1) << 30))
            return fail(DT_ERR_UNSUPPORTED, "window tables too large");
        if (n_windows) *n_windows = int32_t(nw);
        if (levels) *levels = dtree::count_levels(nodes, shape, window_depth);
        if (capacity_windows == 0) return DT_OK;
        if (capacity_windows < nw) return fail(DT_ERR_INVALID_ARG, "capacity_windows too small");
        if (!features || !thresholds || !exit_class || !exit_leaf)
            return fail(DT_ERR_INVALID_ARG, "null output buffer");
        dtree::WindowTables wt;
        dtree::build_windows(nodes, shape, window_depth, &wt);
        const size_t ns = wt.feature.size();
        std::memcpy(features, wt.feature.data(), ns * 4);
        std::memcpy(thresholds, wt.threshold.data(), ns * 4);
        std::memcpy(exit_class, wt.exit_class.data(), ns * 4);
        std::memcpy(exit_leaf, wt.exit_leaf.data(), ns * 4);
        return DT_OK;
    } catch (const std::bad_alloc &) {
        return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_tree_create(const dt_node *nodes, int32_t n_nodes, int32_t n_features,
                         int32_t n_classes, const dt_tree_options *opt, dt_tree **out) {
    try {
        g_last_error.clear();
        return create_impl(nodes, n_nodes, n_features, n_classes, opt, out);
    } catch (const std::bad_alloc &) {
        return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_tree_get_info(const dt_tree *t, dt_tree_info *info) {
    g_last_error.clear();
    if (!t || !info) return fail(DT_ERR_INVALID_ARG, "null argument");
    fill_info(t->shape, t->n_features, t->n_classes, t->enc[0].depth, t->enc[0].n_windows,
              t->enc[0].levels, t->enc[1].depth, t->enc[1].n_windows, t->enc[1].levels, info);
    return DT_OK;
}

void dt_tree_destroy(dt_tree *t) { destroy_impl(t); }

dt_status dt_tree_launch_info(const dt_tree *t, const void *d_x, dt_dtype x_type, int64_t ld,
                              dt_output out_kind, dt_algo algo, dt_launch_info *info) {
    g_last_error.clear();
    if (!t || !info) return fail(DT_ERR_INVALID_ARG, "null argument");
    if (!single_tree_algo(algo)) return fail(DT_ERR_INVALID_ARG, "unknown algo");
    if (!valid_elem_type(x_type)) return fail(DT_ERR_INVALID_ARG, "unknown x_type");
    if (out_kind != DT_OUT_CLASS_U8 && out_kind != DT_OUT_CLASS_I32 && out_kind != DT_OUT_LEAF_I32)
        return fail(DT_ERR_INVALID_ARG, "unknown out_kind");
    if (ld < t->n_features) return fail(DT_ERR_INVALID_ARG, "ld must be >= n_features");
    const int mode = dtree::tree_load_mode(algo, d_x, x_type, ld, t->n_features, t->enc[1].depth);
    const Plan &plan = t->plan[algo][x_type][mode][out_kind == DT_OUT_CLASS_U8 ? 0 : 1];
    if (plan.status != DT_OK) return fail(plan.status, plan.why);
    info->waves_per_workgroup = plan.waves;
    info->workgroups_per_cu = plan.blocks_per_cu;
    info->lds_bytes = plan.lds_bytes;
    info->result_buffer_tiles = plan.out_cap;
    const Encoding &enc = t->enc[plan.enc];
    const bool part = enc.list && enc.table_bytes(x_type) < enc.slot_bytes[x_type];
    info->tables_in_lds = part ? 0 : plan.tables_in_lds;
    info->load_mode = mode;
    info->tile_rows = plan.tile.tile_rows;
    return DT_OK;
}

dt_status dt_classify(const dt_tree *t, const float *d_x, int64_t n, int64_t ld, void *d_out,
                      dt_output out_kind, dt_algo algo, void *stream) {
    try {
        g_last_error.clear();
        return classify_impl(t, d_x, DT_F32, n, ld, d_out, out_kind, algo, stream);
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_classify_typed(const dt_tree *t, const void *d_x, dt_dtype x_type, int64_t n,
                            int64_t ld, void *d_out, dt_output out_kind, dt_algo algo,
                            void *stream) {
    try {
        g_last_error.clear();
        return classify_impl(t, d_x, x_type, n, ld, d_out, out_kind, algo, stream);
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_forest_create(const dt_node *nodes, const int32_t *tree_offsets, int32_t n_trees,
                           int32_t n_features, int32_t n_classes, const dt_tree_options *opt,
                           dt_forest **out) {
    try {
        g_last_error.clear();
        return forest_create_impl(nodes, tree_offsets, n_trees, n_features, n_classes, opt, out);
    } catch (const std::bad_alloc &) {
        return fail(DT_ERR_NO_MEMORY, "host allocation failed");
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

void dt_forest_destroy(dt_forest *f) { forest_destroy_impl(f); }

dt_status dt_forest_classify(const dt_forest *f, const float *d_x, int64_t n, int64_t ld,
                             void *d_out, dt_output out_kind, dt_algo algo, void *stream) {
    try {
        g_last_error.clear();
        return forest_classify_impl(f, d_x, n, ld, d_out, out_kind, algo, stream);
    } catch (...) {
        return fail(DT_ERR_INVALID_ARG, "unexpected internal error");
    }
}

dt_status dt_probe_tree_list(const dt_tree *t, const void *d_x, dt_dtype x_type, int64_t ld,
                             dt_output out_kind, dt_algo algo, int32_t *list) {
    dt_launch_info info;
    const dt_status st = dt_tree_launch_info(t, d_x, x_type, ld, out_kind, algo, &info);
    if (st != DT_OK) return st;
    if (!list) return fail(DT_ERR_INVALID_ARG, "null argument");
    const Plan &plan = t->plan[algo][x_type][info.load_mode][out_kind == DT_OUT_CLASS_U8 ? 0 : 1];
    *list = t->enc[plan.enc].list ? 1 : 0;
    return DT_OK;
}

dt_status dt_probe_forest_spread(const dt_forest *f, const float *d_x, int64_t n, int64_t ld,
                                 dt_algo algo, dt_forest_spread *info) {
    g_last_error.clear();
    if (!f || !info || n < 1 || ld < f->n_features ||
        (algo != DT_ALGO_DATA && algo != DT_ALGO_SPECULATIVE))
        return fail(DT_ERR_INVALID_ARG, "null argument, n < 1, ld < n_features or unknown algo");
    if (f->n_features > dtree::kMaxRowStride) return fail(DT_ERR_UNSUPPORTED, "n_features > 256");
    const ForestPlan *plans[kForestSplits];
    const ForestSpread spread = spread_call(*f, d_x, n, ld, algo, plans);
    *info = dt_forest_spread{};
    info->list = spread.enc == kForestList ? 1 : 0;
    info->whole_tiles = spread.lead;
    info->split_tiles = (n + dtree::kTileRows - 1) / dtree::kTileRows - spread.lead;
    if (info->whole_tiles > 0) {
        info->whole_waves = plans[0]->waves;
        info->whole_blocks_per_cu = plans[0]->blocks_per_cu;
    }
    if (info->split_tiles > 0) {
        info->split_waves = plans[spread.split]->waves;
        info->split_blocks_per_cu = plans[spread.split]->blocks_per_cu;
        info->waves_per_tile = 1 << spread.split;
    }
    return DT_OK;
}

}  // extern "C"
