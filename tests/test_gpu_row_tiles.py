"""GPU parity on rows of every staging class: dense rows that are no multiple of 16 bytes,
strided rows and bases between words or vectors, rows wide enough for tiles of 32 and 16
records, and record counts around the tile edges.  Integer outputs: exact."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1111_1373_amd import workloads as W
from tests import treeutil as TU

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1111_1373_amd import dtree
    return dtree


class _Spread(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in (
        "list", "whole_waves", "split_waves", "waves_per_tile", "whole_blocks_per_cu",
        "split_blocks_per_cu")] + [(n, ctypes.c_int64) for n in ("whole_tiles", "split_tiles")]


def _spread(dt, forest, x, algo="data"):
    """How a forest call on the records x is spread over kernels."""
    s = _Spread()
    dt._check(dt._lib.dt_probe_forest_spread(
        forest._h, ctypes.c_void_p(x.data_ptr()), ctypes.c_int64(x.shape[0]),
        ctypes.c_int64(x.stride(0)), dt.ALGOS[algo], ctypes.byref(s)), "dt_probe_forest_spread")
    return s


# features, columns beyond them, elements before the first record
LAYOUTS = [(1, 0, 0), (1, 1, 1), (2, 1, 0), (3, 0, 3), (5, 2, 0), (7, 0, 1), (12, 0, 0),
           (19, 0, 0), (19, 3, 2), (48, 0, 0), (65, 0, 0), (96, 1, 0), (97, 0, 1),
           (128, 0, 0), (128, 4, 1), (200, 0, 0), (255, 2, 3), (256, 0, 0), (256, 1, 0)]


@pytest.mark.parametrize("x_type", ["f32", "f16", "bf16", "u8"])
@pytest.mark.parametrize("F,pad,off", LAYOUTS)
def test_row_classes(dt, x_type, F, pad, off):
    r = np.random.Generator(np.random.PCG64(F * 100 + pad * 10 + off))
    ld, n_max = F + pad, 1000
    x = W.uniform_f32(r, (n_max * ld + off + 64,))
    xn = x if x_type == "f32" else W.narrow_records(x, x_type)
    nodes = W.narrow_tree(W.random_full_tree(r, 100, F, 7), x_type)
    t = torch.from_numpy(xn)
    if x_type == "bf16":
        t = t.view(torch.int16).view(torch.bfloat16)
    dev = t.cuda()
    rows = xn[off:off + n_max * ld].reshape(n_max, ld)[:, :F]
    want = oracle.tree_leaves(nodes, np.ascontiguousarray(
        rows if x_type == "f32" else TU.widen(np.ascontiguousarray(rows), x_type)), F)
    for sd in (1, 2, 5, 6):
        tree = dt.Tree(nodes, F, 7, spec_window_depth=sd)
        algos = ["speculative"] + (["data"] if sd == 2 else [])
        algos += ["path"] if x_type == "f32" and sd in (2, 5) else []
        for n in (1, 15, 16, 17, 31, 33, 63, 64, 65, 1000):
            xd = dev[off:off + n * ld].view(n, ld)[:, :F]
            for algo in algos:
                got = tree.classify(xd, algo=algo, out_kind="leaf_i32").cpu().numpy()
                np.testing.assert_array_equal(got, want[:n], err_msg="%s n=%d sd=%d" % (algo, n, sd))


# Forests: every staging class, record counts that take one, a few and all wavefronts per
# tile and leave a last partly filled round, vote words of each size, and trees that are
# walked as packed windows ("complete") and as node lists ("random").
@pytest.mark.parametrize("F,pad,off", [(1, 0, 0), (3, 2, 1), (8, 0, 0), (19, 0, 0), (32, 0, 1),
                                       (33, 0, 0), (64, 0, 0), (100, 5, 0), (200, 0, 0), (256, 0, 3)])
@pytest.mark.parametrize("shape,C", [("complete", 5), ("random", 16), ("random", 60), ("leaf", 3)])
def test_forest_row_classes_and_splits(dt, F, pad, off, shape, C):
    r = np.random.Generator(np.random.PCG64(7000 + F * 100 + C))
    trees = []
    for k in range(37):
        if shape == "leaf" and k % 2:
            leaf = np.zeros(1, dtype=W.NODE_DTYPE)
            leaf[0] = (0, 0.0, -1, int(r.integers(0, C)))
            trees.append(leaf)
        elif shape == "complete":
            trees.append(W.complete_tree(r, 6, F, C))
        else:
            trees.append(W.random_full_tree(r, int(r.integers(1, 150)), F, C))
    nodes = np.concatenate(trees)
    offsets = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    ld, n_max = F + pad, 20_000
    x = W.uniform_f32(r, (n_max * ld + off,))
    x[r.integers(0, x.size, 500)] = np.nan
    rows = x[off:].reshape(n_max, ld)[:, :F]
    want = oracle.forest_classes(nodes, offsets, np.ascontiguousarray(rows), F, C)
    dev = torch.from_numpy(x).cuda()
    f = dt.Forest(nodes, offsets, F, C)
    for n in (1, 63, 65, 1000, 4097, n_max):
        xd = dev[off:off + n * ld].view(n, ld)[:, :F]
        for algo in ("data", "speculative"):
            got = f.classify(xd, algo=algo, out_kind="class_i32").cpu().numpy()
            np.testing.assert_array_equal(got, want[:n], err_msg="%s n=%d" % (algo, n))


@pytest.mark.parametrize("n", [256 * 16 * 64 + 1, 256 * 16 * 64 + 40 * 64])
def test_forest_lead_and_rest(dt, n):
    """A full round of tiles by the unsplit kernel and the rest by a split one."""
    r = np.random.Generator(np.random.PCG64(n))
    trees = [W.random_full_tree(r, 255, 6, 9) for _ in range(60)]
    nodes = np.concatenate(trees)
    offsets = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    x = W.uniform_f32(r, (n, 6))
    f = dt.Forest(nodes, offsets, 6, 9)
    xd = torch.from_numpy(x).cuda()
    s = _spread(dt, f, xd)
    assert s.list == 1 and s.whole_tiles == 256 * 16 and s.split_tiles == -(-n // 64) - 256 * 16
    assert s.waves_per_tile >= 2
    got = f.classify(xd, out_kind="class_i32").cpu().numpy()
    at = np.concatenate([np.arange(0, n, 97), np.arange(n - 3000, n)])
    np.testing.assert_array_equal(got[at], oracle.forest_classes(nodes, offsets, x[at], 6, 9))


@pytest.mark.parametrize("waves", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("algo", ["data", "speculative"])
@pytest.mark.parametrize("shape", ["complete", "random", "large"])
def test_split_forest_keeps_to_the_wavefronts_asked_for(dt, waves, algo, shape):
    """waves_per_cu of the options bounds the resident wavefronts of a split kernel, with tables
    in the LDS and in place."""
    r = np.random.Generator(np.random.PCG64(waves))
    F, C = 19, 5
    make = {"complete": lambda: W.complete_tree(r, 6, F, C),
            "random": lambda: W.random_full_tree(r, 100, F, C),
            "large": lambda: W.random_full_tree(r, 25_000, F, C)}[shape]
    trees = [make() for _ in range(3 if shape == "large" else 40)]
    nodes = np.concatenate(trees)
    offsets = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    x = W.uniform_f32(r, (5000, F))
    want = oracle.forest_classes(nodes, offsets, x, F, C)
    f, xd = dt.Forest(nodes, offsets, F, C, waves_per_cu=waves), torch.from_numpy(x).cuda()
    for n in (64, 5000):
        s = _spread(dt, f, xd[:n], algo)
        assert s.split_waves * s.split_blocks_per_cu <= waves and s.waves_per_tile <= waves
        got = f.classify(xd[:n], algo=algo, out_kind="class_i32").cpu().numpy()
        np.testing.assert_array_equal(got, want[:n])


@pytest.mark.parametrize("deep,size,want_list", [(11, 0, [0, 0, 0]), (14, 0, None), (0, 300, None)])
def test_mixed_forest(dt, deep, size, want_list):
    """Complete trees, which one packed window each holds, beside one that is deeper: windows
    and node lists are weighed at each call (32 features, 1,500,000 records, one tree of depth
    11: 155.6 us with windows, 208.5 us with lists)."""
    r = np.random.Generator(np.random.PCG64(deep + size))
    F, C = 32, 8
    trees = [W.complete_tree(r, 10, F, C) for _ in range(31)]
    trees.append(W.complete_tree(r, deep, F, C) if deep else W.random_full_tree(r, size, F, C))
    nodes = np.concatenate(trees)
    offsets = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    x = W.uniform_f32(r, (300_000, F))
    f, xd = dt.Forest(nodes, offsets, F, C), torch.from_numpy(x).cuda()
    at = np.arange(0, 20_000)
    want = oracle.forest_classes(nodes, offsets, x[at], F, C)
    lists = []
    for n in (1000, 20_000, 300_000):
        lists.append(_spread(dt, f, xd[:n]).list)
        got = f.classify(xd[:n], out_kind="class_i32").cpu().numpy()
        np.testing.assert_array_equal(got[:20_000], want[:n])
    assert want_list is None or lists == want_list


@pytest.mark.parametrize("algo", ["data", "speculative"])
@pytest.mark.parametrize("F,pad", [(3, 0), (19, 2), (32, 0), (64, 0)])
def test_forest_base_between_words(dt, F, pad, algo):
    """The C call takes fp32 records off a base between words."""
    r = np.random.Generator(np.random.PCG64(F))
    trees = [W.random_full_tree(r, 50, F, 5) for _ in range(9)]
    nodes = np.concatenate(trees)
    offsets = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    n, ld = 3000, F + pad
    x = W.uniform_f32(r, (n, ld))
    want = oracle.forest_classes(nodes, offsets, np.ascontiguousarray(x[:, :F]), F, 5)
    block = torch.zeros(n * ld * 4 + 16, dtype=torch.uint8, device="cuda")
    f = dt.Forest(nodes, offsets, F, 5)
    for shift in (1, 2):
        block[shift:shift + n * ld * 4] = torch.from_numpy(x.reshape(-1).view(np.uint8)).cuda()
        out = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        dt._check(dt._lib.dt_forest_classify(
            f._h, block.data_ptr() + shift, n, ld, out.data_ptr(), dt.OUT_KINDS["class_i32"],
            dt.ALGOS[algo], torch.cuda.current_stream().cuda_stream), "dt_forest_classify")
        np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("F", [1, 3, 4, 6, 8, 16, 19, 64, 200])
@pytest.mark.parametrize("size", [30, 1200, 2500, 3500])
def test_planned_workgroups_fit_the_lds(dt, F, size):
    """The workgroups that a plan counts on are resident together: a workgroup's LDS is
    allocated in pieces of 1,280 bytes, of which a CU has 128."""
    r = np.random.Generator(np.random.PCG64(size + F))
    nodes = W.random_full_tree(r, size, F, 9)
    for depth in (0, 4):
        tree = dt.Tree(nodes, F, 9, data_window_depth=depth)
        for x_type in (torch.float32, torch.float16, torch.uint8):
            x = torch.zeros((64, F), dtype=x_type, device="cuda")
            for algo in ("data", "speculative"):
                for out_kind in ("class_u8", "leaf_i32"):
                    li = tree.launch_info(x, algo=algo, out_kind=out_kind)
                    assert li["workgroups_per_cu"] * -(-li["lds_bytes"] // 1280) <= 128, li


@pytest.mark.parametrize("F,depth,mode", [(3, 2, 0), (3, 3, 1), (19, 2, 0), (19, 4, 1), (30, 6, 1),
                                          (33, 6, 0), (100, 4, 1), (101, 4, 0)])
def test_narrow_rows_of_large_windows_are_read_row_by_row(dt, F, depth, mode):
    """Dense fp32 rows of up to 32 features go one by one into tiles of a constant pitch for
    windows of 8 lanes and more, and as one run of bytes otherwise (rows of no multiple of 16
    bytes); the labels are the oracle's either way."""
    r = np.random.Generator(np.random.PCG64(F * 10 + depth))
    nodes = W.random_full_tree(r, 60, F, 5)
    x = W.uniform_f32(r, (1003, F))
    tree, xd = dt.Tree(nodes, F, 5, spec_window_depth=depth), torch.from_numpy(x).cuda()
    assert tree.launch_info(xd, algo="speculative")["load_mode"] == mode
    assert tree.launch_info(xd, algo="data")["load_mode"] == (1 if F == 100 else 0)
    got = tree.classify(xd, algo="speculative", out_kind="leaf_i32").cpu().numpy()
    np.testing.assert_array_equal(got, oracle.tree_leaves(nodes, x, F))


@pytest.mark.parametrize("x_type", ["f32", "f16", "u8"])
@pytest.mark.parametrize("ld", [1 << 40, 1 << 61, 1 << 62, (1 << 63) - 1])
def test_one_record_with_any_stride(dt, x_type, ld):
    """The stride of a single record is never used, also where its bytes overflow 64 bits."""
    r = np.random.Generator(np.random.PCG64(9))
    F, C = 19, 5
    nodes = W.narrow_tree(W.random_full_tree(r, 60, F, C), x_type)
    x = W.uniform_f32(r, (1, F))
    xn = x if x_type == "f32" else W.narrow_records(x, x_type)
    want = oracle.tree_classes(nodes, x if x_type == "f32" else TU.widen(xn, x_type), F)
    tree, xd = dt.Tree(nodes, F, C, spec_window_depth=4), torch.from_numpy(xn).cuda()
    forest = dt.Forest(nodes, [0, len(nodes)], F, C)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for algo in ("data", "speculative"):
        out = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        args = (ctypes.c_int64(1), ctypes.c_int64(ld), ctypes.c_void_p(out.data_ptr()),
                dt.OUT_KINDS["class_i32"], dt.ALGOS[algo], stream)
        dt._check(dt._lib.dt_classify_typed(tree._h, ctypes.c_void_p(xd.data_ptr()),
                                            dt.X_TYPES[x_type], *args), "dt_classify_typed")
        assert int(out[0]) == want[0]
        if x_type == "f32":
            out.fill_(-1)
            dt._check(dt._lib.dt_forest_classify(forest._h, ctypes.c_void_p(xd.data_ptr()), *args),
                      "dt_forest_classify")
            assert int(out[0]) == want[0]
