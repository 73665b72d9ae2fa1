// Host-side tree validation and window encoding shared by both GPU decompositions.
//
// A window is a block of at most D levels of the tree, rooted at a decision node and
// embedded in a complete binary heap stored 1-based: slot p in [1, 2^D) holds heap node p
// (children 2p and 2p+1, so the two children of a node are one aligned 16-byte pair), and
// slot 0 is padding.  Leaving the window at bottom position 2^D + e is exit e.
// This is the "window" of Section 6 of the paper (evaluate a few levels, then continue
// from the node reached), and it gives the speculative decomposition its fixed lane map
// (the processor-node map of Procedure 5): lane h of a record's lane group evaluates
// slot h.  Slots that hold no decision node (below a leaf that ends the path early)
// always send the record right, so a leaf met above the bottom is recorded at the exit
// reached by going right from it; this plays the role of Procedure 5's static leaf
// paths.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "dtree.h"

namespace dtree {

constexpr int kMaxNodes = 1 << 24;
constexpr int kMaxWindowDepth = 16;
constexpr int kMaxSpecWindowDepth = 6;
// Default speculative window depth: 4-lane record groups measured fastest on MI355X (the
// paper's 16-lane groups are depth 4).
constexpr int kDefaultSpecWindowDepth = 2;

// Parsed, validated tree.
struct TreeShape {
    int32_t n_nodes = 0, n_internal = 0, n_leaves = 0, depth = 0;
    std::vector<int32_t> node_depth;   // edges from the root
};

// Validates the layout rules of dtree.h.  Returns DT_OK or an error with `msg` set.
dt_status validate_tree(const dt_node *nodes, int32_t n_nodes, int32_t n_features,
                        int32_t n_classes, TreeShape *shape, std::string *msg);

// Window encoding (see dt_encode_windows in dtree.h).  Slot-major arrays of
// n_windows * 2^depth entries.
struct WindowTables {
    int32_t depth = 0;        // D
    int32_t slots = 0;        // S = 2^D
    int32_t n_windows = 0;
    int32_t levels = 0;       // windows on the longest root-to-leaf path
    int32_t first_depth = 0;  // decision levels of window 0 (d0 <= D; the others have D)
    std::vector<int32_t> feature;
    std::vector<float> threshold;
    std::vector<int32_t> exit_class;
    std::vector<int32_t> exit_leaf;
};

// Slot words of the windows for narrow records (fp16, bf16, uint8): feature index << 16 |
// key, where the key is the threshold moved onto the record type's grid, rounded up: the
// smallest value of the type (as its bits) not below t, and for uint8 the integer ceiling
// of t clamped to 0..256.  No representable record value lies in [t, key), so a stored
// element x satisfies x < key exactly when its widened value is below t.  A NaN threshold
// sends every record right (key NaN, or 0 for uint8).  One word per slot, slot-major.
uint32_t narrow_key(float t, dt_dtype type);
void build_narrow_slots(const WindowTables &wt, dt_dtype type, std::vector<uint32_t> *out);

// Depth d0 of the first window for window depth D: windows are rooted at tree depth 0 and
// at depths d0, d0 + D, d0 + 2D, ...  d0 is D, or the depth that fills the deepest level of
// windows when that needs fewer windows.
int first_window_depth(const dt_node *nodes, const TreeShape &shape, int depth);

// Node lists (see walk_list and walk_list_k in device_common.hpp): entry 0 is unused, node v
// is entry 1 + order[v], 8 bytes each.  The order is breadth-first whatever the order of the
// caller's array, so that the first entries are the tree's upper levels, which every record
// passes: the part of a large list that the LDS holds.
std::vector<int32_t> breadth_first_order(const dt_node *nodes, int32_t n);

// Of single trees, for records of type `type`: decision node {threshold (its bits, or the
// narrow key with the feature above it), index of its children's pair (fp32: << 10 | byte
// offset of the feature)}, leaf {leaf index, ~class}.  Links hold 21 bits of pairs.
constexpr int32_t kMaxTreeListNodes = (1 << 22) - 2;
void build_list(const dt_node *nodes, int32_t n, const std::vector<int32_t> &order, dt_dtype type,
                uint32_t *out);

// Of a forest's tree (fp32 records, classes below 256): decision node {threshold bits, left
// child's entry << 10 | byte offset of the feature}, leaf {NaN with the class in its low
// bits, own entry - 1, << 10}.  Links hold 22 bits of entries.
constexpr int32_t kMaxForestListNodes = (1 << 22) - 2;
void build_forest_list(const dt_node *nodes, int32_t n, const std::vector<int32_t> &order,
                       uint32_t *out);

inline int64_t list_bytes(int32_t n) { return (8 * (int64_t(n) + 1) + 15) & ~int64_t(15); }

// Most LDS a node list takes; the nodes of larger lists' lower levels stay in global memory.
constexpr int64_t kListLdsBytes = 48 * 1024;

// Whether the data decomposition of a single tree walks windows or the node list, for tables
// of these bytes (windows take 12 bytes a slot for fp32 records and 8 for narrow ones, the
// list 8 a node).  Windows pad every path to whole windows and end each with an exit read,
// and sparse trees leave most of their slots empty; the list takes a path's own steps, at a
// slightly longer step (the loop's test and the child's index).  Measured over 1,000,000
// records, the list against the windows:
//   Several levels of windows: the list (300 random decision nodes, 32 fp32 features, 21.3
//     against 21.9 us; 3,500 nodes, 16 features 15.6 against 20.2 us), unless the tree is
//     chain-like, all of whose paths are long (depth of three times log2 of the nodes and
//     more: a chain of 20, 19 features, 18.1 against 16.5 us).
//   One level: the windows, whose tables then are about as large as the list's (a complete
//     tree of depth 12 on 200 fp16 features 61.6 against 81.0 us), unless they take more than
//     four times the list's bytes (20 random nodes, 8 fp32 features 0.84 of the time); chains
//     (depth of twice log2 of the nodes and more: 10 decision nodes 1.05) keep up to 12 KiB.
//   Lists, or one level of windows, of more than 48 KiB (kEither): by list_is_faster.
enum class DataWalk { kWindows, kList, kEither };
DataWalk data_walk_for(const TreeShape &shape, int32_t levels, int64_t window_bytes,
                       int64_t list_bytes);

// Of the two with windows in the LDS, by the steps of a path and the wavefronts that a CU
// holds with each: the part of a list that is not in the LDS costs about four steps for each
// of its levels, and the time of a step falls with about the root of the wavefronts.  The
// choice was within 19% of the better walk on each of 663 trees, widths and types measured
// (1,000,000 records; 651 of them within 3%): a complete tree of depth 13, 64 fp32 features
// 47.9 us with the list and 41.2 with windows, 8 features (half the wavefronts) 11.5 and 13.0;
// depth 14, 4 uint8 features 10.4 and 12.1 (windows taken); 5,000 random nodes, 64 fp32
// features 43.8 and 63.7 us.
bool list_is_faster(const TreeShape &shape, int32_t levels, int window_depth, int64_t list_bytes,
                    int waves_windows, int waves_list);

// Levels of decision nodes that some record of a wavefront's 64 passes, if both branches of
// every node are as likely: at least 1, at most the depth.
int reached_depth(const dt_node *nodes, const TreeShape &shape);

// Number of windows, and window levels on the longest path, for window depth D (without
// building them).
int64_t count_windows(const dt_node *nodes, const TreeShape &shape, int depth);
int32_t count_levels(const dt_node *nodes, const TreeShape &shape, int depth);

void build_windows(const dt_node *nodes, const TreeShape &shape, int depth, WindowTables *out);

// Bytes a workgroup stages in LDS for a table of n_windows windows of 2^depth slots:
// one 8-byte (threshold, feature) pair and one 4-byte exit per slot.
inline int64_t table_bytes(int64_t n_windows, int depth) {
    return n_windows * (int64_t(1) << depth) * 12;
}

// LDS bytes of a gfx950 workgroup, and the most LDS the default data windows may take.
constexpr int64_t kLdsBytes = 160 * 1024;
constexpr int64_t kDataTableBudget = 48 * 1024;

// Table bytes the default data window depth may use for records of n_features: at most
// kDataTableBudget, and room left for two fp32 record tiles (of 64 rows of the next power of
// two of features, whatever tiles a launch then uses: the cut of a tree is the same for every
// record type and layout; data_walk_for decides for each whether it is walked).
int64_t data_table_budget(int32_t n_features);

// Library's default window depths (see dt_tree_options in dtree.h).  Data: the fewest
// window levels among the depths whose tables fit max_bytes (ties: smaller tables), or the
// smallest tables if none fits.
int choose_data_window_depth(const dt_node *nodes, const TreeShape &shape, int64_t max_bytes);
int choose_spec_window_depth(const TreeShape &shape);

}  // namespace dtree
