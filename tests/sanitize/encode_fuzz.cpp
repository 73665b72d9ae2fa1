// Host check of the tree validation and window encoder (encode.cpp) built with
// AddressSanitizer and UndefinedBehaviorSanitizer.  Random full trees in the breadth-first
// layout of Procedure 1 are encoded at every window depth 1..8; walking each record
// through the window tables (D heap steps per window, then the exit) must reach the leaf
// a direct walk of the tree reaches.  So must walks of the node lists, which are breadth-first
// also for arrays in another order.  Corrupted arrays must be rejected, not crash.
// Usage: encode_fuzz SEED TREES
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "encode.hpp"

namespace {

uint64_t g_state;
uint64_t next_u64() {   // splitmix64
    uint64_t z = (g_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
int below(int n) { return int(next_u64() % uint64_t(n)); }
float unit() { return float(next_u64() >> 40) / float(1 << 24); }

float special_or_unit() {
    switch (below(12)) {
        case 0: return std::numeric_limits<float>::quiet_NaN();
        case 1: return std::numeric_limits<float>::infinity();
        case 2: return -std::numeric_limits<float>::infinity();
        case 3: return -0.0f;
        case 4: return std::numeric_limits<float>::denorm_min();
        default: return unit();
    }
}

// Random full binary tree with n_int decision nodes (split random leaves), renumbered
// breadth-first so that every node's right child directly follows its left child.
std::vector<dt_node> random_tree(int n_int, int F, int C) {
    struct Kids { int l = -1; };
    std::vector<Kids> t(1);
    std::vector<int> leaves{0};
    for (int k = 0; k < n_int; ++k) {
        const int pick = below(int(leaves.size()));
        const int v = leaves[size_t(pick)];
        leaves[size_t(pick)] = leaves.back();
        leaves.pop_back();
        const int a = int(t.size());
        t.resize(t.size() + 2);
        t[size_t(v)].l = a;
        leaves.push_back(a);
        leaves.push_back(a + 1);
    }
    std::vector<int> order{0}, id(t.size());
    for (size_t h = 0; h < order.size(); ++h) {
        const int v = order[h];
        id[size_t(v)] = int(h);
        if (t[size_t(v)].l >= 0) {
            order.push_back(t[size_t(v)].l);
            order.push_back(t[size_t(v)].l + 1);
        }
    }
    std::vector<dt_node> out(order.size());
    for (size_t h = 0; h < order.size(); ++h) {
        const int v = order[h];
        if (t[size_t(v)].l >= 0)
            out[h] = dt_node{below(F), special_or_unit(), id[size_t(t[size_t(v)].l)], -1};
        else
            out[h] = dt_node{0, 0.0f, -1, below(C)};
    }
    return out;
}

int direct_leaf(const std::vector<dt_node> &t, const float *x) {
    int i = 0;
    while (t[size_t(i)].cls < 0)
        i = x[t[size_t(i)].feature] < t[size_t(i)].threshold ? t[size_t(i)].left
                                                              : t[size_t(i)].left + 1;
    return i;
}

int window_leaf(const dtree::WindowTables &wt, const float *x) {
    int w = 0;
    for (int level = 0; level < wt.levels; ++level) {
        int p = 1;
        for (int k = 0; k < wt.depth; ++k) {
            const size_t s = size_t(w) * size_t(wt.slots) + size_t(p);
            p = 2 * p + int(!(x[wt.feature[s]] < wt.threshold[s]));
        }
        const int code = wt.exit_leaf[size_t(w) * size_t(wt.slots) + size_t(p - wt.slots)];
        if (code < 0) return -code - 1;
        if (code >= wt.n_windows) return -2;
        w = code;
    }
    return -3;   // more windows on a path than `levels`
}

// The same tree with its nodes in depth-first order (siblings stay neighbours).
std::vector<dt_node> depth_first(const std::vector<dt_node> &t) {
    std::vector<dt_node> out(t.size());
    std::vector<std::pair<int, int>> todo{{0, 0}};   // node, its place
    int next = 1;
    while (!todo.empty()) {
        const auto [v, place] = todo.back();
        todo.pop_back();
        out[size_t(place)] = t[size_t(v)];
        if (t[size_t(v)].cls >= 0) continue;
        out[size_t(place)].left = next;
        todo.emplace_back(t[size_t(v)].left + 1, next + 1);
        todo.emplace_back(t[size_t(v)].left, next);
        next += 2;
    }
    return out;
}

// Leaf index and ~class that a record of `type` reaches in the list of build_list.
std::pair<uint32_t, int32_t> list_leaf(const std::vector<uint32_t> &list, dt_dtype type,
                                       const float *x) {
    size_t at = 1;
    while (int32_t(list.at(2 * at + 1)) >= 0) {
        const uint32_t key = list[2 * at], link = list[2 * at + 1];
        bool right;
        if (type == DT_F32) {
            float t;
            std::memcpy(&t, &key, 4);
            right = !(x[(link & 1023) / 4] < t);
        } else if (type == DT_U8) {
            right = uint32_t(x[key >> 16]) >= (key & 0xFFFF);
        } else {
            const uint32_t bits = key << 16;          // bf16
            float t;
            std::memcpy(&t, &bits, 4);
            right = !(x[key >> 16] < t);
        }
        at = 2 * size_t(type == DT_F32 ? link >> 10 : link) + size_t(right);
    }
    return {list[2 * at], int32_t(list[2 * at + 1])};
}

// Class that the walk of a forest's list ends in after `depth` steps.
int forest_list_class(const std::vector<uint32_t> &list, int depth, const float *x) {
    size_t at = 1;
    float t = 0.0f;
    for (int k = 0; k < depth; ++k) {
        const uint32_t link = list.at(2 * at + 1);
        std::memcpy(&t, &list[2 * at], 4);
        at = size_t(link >> 10) + size_t(!(x[(link & 1023) / 4] < t));
    }
    return int(list.at(2 * at) & 0xFF);
}

int fail(const char *what, int a, int b) {
    std::fprintf(stderr, "FAIL %s (%d, %d)\n", what, a, b);
    return 1;
}

// Lists of one tree, and of the same tree depth-first: the walks, the order, the sizes.
int check_lists(const std::vector<dt_node> &tree, const dtree::TreeShape &shape, int F,
                const std::vector<float> &x) {
    const std::vector<dt_node> orders[] = {tree, depth_first(tree)};
    for (int o = 0; o < 2; ++o) {
        const std::vector<dt_node> &t = orders[o];
        const int n = int(t.size());
        const std::vector<int32_t> order = dtree::breadth_first_order(t.data(), n);
        std::vector<uint32_t> list(size_t(dtree::list_bytes(n) / 4), 0u);
        for (dt_dtype type : {DT_F32, DT_BF16, DT_U8}) {
            dtree::build_list(t.data(), n, order, type, list.data());
            uint32_t pair = 0;       // breadth-first: the decision nodes' pairs in sequence
            for (int i = 1; i <= n; ++i) {
                const uint32_t link = list[size_t(2 * i + 1)];
                if (int32_t(link) >= 0 && (type == DT_F32 ? link >> 10 : link) != ++pair)
                    return fail("list order", o, i);
            }
            for (int r = 0; r < 64; ++r) {
                std::vector<float> row(x.begin() + r * (F + 1), x.begin() + (r + 1) * (F + 1));
                for (float &v : row) {               // records of the type, widened
                    if (type == DT_U8) v = v > 0.0f && v <= 1.0f ? std::floor(v * 255.0f) : 0.0f;
                    uint32_t bits;
                    std::memcpy(&bits, &v, 4);
                    if (type == DT_BF16 && v == v) bits &= 0xFFFF0000u;
                    std::memcpy(&v, &bits, 4);
                }
                const int leaf = direct_leaf(t, row.data());
                const auto got = list_leaf(list, type, row.data());
                if (int(got.first) != leaf || ~got.second != t[size_t(leaf)].cls)
                    return fail("list walk leaf", int(got.first), leaf);
            }
        }
        std::vector<dt_node> small = t;             // forests: at most 64 classes
        for (dt_node &v : small)
            if (v.cls >= 0) v.cls %= 64;
        dtree::build_forest_list(small.data(), n, order, list.data());
        for (int r = 0; r < 64; ++r) {
            const float *row = x.data() + r * (F + 1);
            const int want = small[size_t(direct_leaf(small, row))].cls;
            for (int extra : {0, 3})                // a walk that is over stays at its leaf
                if (forest_list_class(list, std::max(1, shape.depth) + extra, row) != want)
                    return fail("forest list walk class", r, want);
        }
    }
    return 0;
}

// Lists at the largest size that their links can hold: every decision node leads to its
// children.
int check_list_limits() {
    static_assert(dtree::kMaxTreeListNodes == dtree::kMaxForestListNodes, "one tree serves both");
    const int n = dtree::kMaxTreeListNodes - 1;     // a full tree has an odd number of nodes
    std::vector<dt_node> t(static_cast<size_t>(n));
    for (int i = 0; i < n; ++i)
        t[size_t(i)] = 2 * i + 2 < n ? dt_node{255, 0.5f, 2 * i + 1, -1} : dt_node{0, 0.0f, -1, 63};
    const std::vector<int32_t> order = dtree::breadth_first_order(t.data(), n);
    std::vector<uint32_t> list(size_t(dtree::list_bytes(n) / 4), 0u);
    for (dt_dtype type : {DT_F32, DT_U8}) {
        dtree::build_list(t.data(), n, order, type, list.data());
        for (int i = 0; i < n; ++i) {
            const uint32_t link = list[2 * (size_t(i) + 1) + 1];
            if (t[size_t(i)].cls >= 0 ? link != ~63u
                                      : int32_t(link) < 0 ||
                                            (type == DT_F32 ? link >> 10 : link) != uint32_t(i + 1) ||
                                            (type == DT_F32 && (link & 1023) != 1020))
                return fail("list link", int(type), i);
        }
    }
    dtree::build_forest_list(t.data(), n, order, list.data());
    for (int i = 0; i < n; ++i) {
        const uint32_t link = list[2 * (size_t(i) + 1) + 1];
        if (link != (t[size_t(i)].cls >= 0 ? uint32_t(i) << 10 : uint32_t(2 * i + 2) << 10 | 1020))
            return fail("forest list link", i, int(link));
    }
    return 0;
}

// Which trees walk lists: complete trees keep one level of windows while as many wavefronts
// fit beside them, also where the list alone would be over its share of the LDS.
int check_list_rule() {
    struct Want {
        int depth, nodes, levels, window_depth;
        int64_t slots;
        int slot_bytes, waves_windows, waves_list;   // wavefronts of a CU with either
        bool list;
    };
    const Want want[] = {
        {12, 8191, 1, 12, 4096, 12, 6, 6, false},      // complete, 200 fp32 features
        {12, 8191, 1, 12, 4096, 8, 4, 4, false},       // 200 fp16 features
        {13, 16383, 1, 13, 8192, 12, 3, 4, false},     // complete, 64 fp32 features
        {13, 16383, 1, 13, 8192, 12, 8, 14, false},    // 16
        {13, 16383, 1, 13, 8192, 12, 8, 16, true},     // 8: half the wavefronts
        {13, 16383, 1, 13, 8192, 8, 16, 16, false},    // 16 uint8 features
        {14, 32767, 1, 14, 16384, 8, 7, 14, false},    // 64 uint8 features
        {14, 32767, 1, 14, 16384, 8, 3, 8, true},      // 64 fp16 features
        {19, 601, 4, 5, 1920, 12, 8, 8, true},         // 300 random nodes
        {9, 41, 1, 9, 512, 12, 32, 32, true},          // 20 random nodes
        {29, 10001, 15, 2, 9988, 12, 3, 7, true},      // 5,000 random nodes
        {14, 20157, 4, 4, 12000, 8, 4, 4, false},      // grown, 200 fp16 features
        {14, 20157, 4, 4, 12000, 8, 8, 14, true},      // 32
        {10, 21, 1, 10, 1024, 8, 32, 32, false},       // chains
        {20, 41, 2, 10, 2048, 12, 8, 8, false},
        {11, 31, 1, 11, 2048, 12, 16, 16, true},       // 24 KiB of windows for 15 nodes, or
        {11, 31, 1, 11, 2048, 8, 16, 16, true},        // 16
    };
    for (const Want &w : want) {
        dtree::TreeShape shape;
        shape.depth = w.depth;
        shape.n_nodes = w.nodes;
        const int64_t list = dtree::list_bytes(w.nodes);
        const auto walk = dtree::data_walk_for(shape, w.levels, w.slots * w.slot_bytes, list);
        const bool got = walk == dtree::DataWalk::kEither
                             ? dtree::list_is_faster(shape, w.levels, w.window_depth, list,
                                                     w.waves_windows, w.waves_list)
                             : walk == dtree::DataWalk::kList;
        if (got != w.list) return fail("list rule", w.depth, w.nodes);
    }
    return 0;
}

}  // namespace

int main(int argc, char **argv) {
    g_state = argc > 1 ? std::strtoull(argv[1], nullptr, 10) : 1;
    const int trees = argc > 2 ? std::atoi(argv[2]) : 200;
    const int sizes[] = {0, 1, 2, 3, 7, 15, 40, 63, 64, 200, 1000, 3000};
    long checked = 0;
    if (const int bad = check_list_limits()) return bad;
    if (const int bad = check_list_rule()) return bad;
    for (int it = 0; it < trees; ++it) {
        const int F = 1 + below(40), C = 1 + below(300);
        const int n_int = sizes[below(int(sizeof(sizes) / sizeof(sizes[0])))];
        const std::vector<dt_node> t = random_tree(n_int, F, C);
        dtree::TreeShape shape;
        std::string msg;
        if (dtree::validate_tree(t.data(), int32_t(t.size()), F, C, &shape, &msg) != DT_OK)
            return fail("valid tree rejected", it, n_int);
        std::vector<float> x(size_t(64) * size_t(F + 1));
        for (float &v : x) v = special_or_unit();
        for (int r = 0; r < 64 && n_int > 0; ++r) {   // ties on some decision node
            const int node = below(int(t.size()));
            if (t[size_t(node)].cls < 0)
                x[size_t(r) * size_t(F + 1) + size_t(t[size_t(node)].feature)] =
                    t[size_t(node)].threshold;
        }
        for (int D = 1; D <= 8; ++D) {
            dtree::WindowTables wt;
            dtree::build_windows(t.data(), shape, D, &wt);
            if (wt.n_windows != dtree::count_windows(t.data(), shape, D))
                return fail("window count", it, D);
            if (wt.levels != dtree::count_levels(t.data(), shape, D))
                return fail("window levels", it, D);
            for (int32_t e : wt.exit_class)
                if (e < -C || e >= wt.n_windows) return fail("exit code range", it, e);
            for (int r = 0; r < 64; ++r) {
                const float *row = x.data() + size_t(r) * size_t(F + 1);
                const int a = direct_leaf(t, row), b = window_leaf(wt, row);
                if (a != b) return fail("window walk leaf", a, b);
                ++checked;
            }
        }
        if (const int bad = check_lists(t, shape, F, x)) return bad;
        // corrupted copies: validation must reject them
        if (n_int > 0) {
            for (int kind = 0; kind < 5; ++kind) {
                std::vector<dt_node> bad = t;
                int node = below(int(bad.size()));
                while (bad[size_t(node)].cls >= 0) node = below(int(bad.size()));
                switch (kind) {
                    case 0: bad[size_t(node)].left = node; break;                      // back edge
                    case 1: bad[size_t(node)].left = int(bad.size()) - 1; break;       // right out of range
                    case 2: bad[size_t(node)].feature = F; break;
                    case 3: bad[size_t(bad.size()) - 1].cls = C; break;
                    default: bad.pop_back(); break;                                    // truncated
                }
                dtree::TreeShape s2;
                if (dtree::validate_tree(bad.data(), int32_t(bad.size()), F, C, &s2, &msg) == DT_OK)
                    return fail("corrupt tree accepted", it, kind);
            }
        }
        for (int k = 0; k < 64; ++k) {   // narrow threshold keys of arbitrary floats
            const float v = k % 2 ? special_or_unit() : (unit() - 0.5f) * 1e6f;
            if (dtree::narrow_key(v, DT_U8) > 256u) return fail("uint8 key range", it, k);
            (void)dtree::narrow_key(v, DT_F16);
            (void)dtree::narrow_key(v, DT_BF16);
        }
    }
    std::printf("ok %ld walks\n", checked);
    return 0;
}
