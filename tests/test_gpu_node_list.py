"""GPU parity of the data decomposition over node lists: trees whose windows need several
levels or do not fit the LDS, with lists that fit it, that end just at its share (48 KiB:
6,143 nodes) and that continue in global memory, every record type and result kind; and
chain-like and complete trees beside them, which keep their windows.  Exact."""
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


def _walks_list(dt, tree, x, out_kind="class_u8"):
    import ctypes
    got = ctypes.c_int32(-1)
    dt._check(dt._lib.dt_probe_tree_list(tree._h, ctypes.c_void_p(x.data_ptr()), dt._x_type(x),
                                         ctypes.c_int64(x.stride(0)), dt.OUT_KINDS[out_kind], 0,
                                         ctypes.byref(got)), "dt_probe_tree_list")
    return got.value == 1


@pytest.mark.parametrize("x_type", ["f32", "f16", "bf16", "u8"])
@pytest.mark.parametrize("shape,size", [("random", 20), ("random", 3070), ("random", 3071),
                                        ("random", 3072), ("random", 3073), ("random", 9000),
                                        ("chain", 70), ("paper", 11), ("complete", 12),
                                        ("complete", 13), ("complete", 14)])
@pytest.mark.parametrize("F,pad", [(16, 0), (19, 0), (150, 3)])
def test_node_lists(dt, x_type, shape, size, F, pad):
    r = np.random.Generator(np.random.PCG64(size * 1000 + F))
    C = 300
    if shape == "random":
        nodes = W.random_full_tree(r, size, F, C, threshold_values=np.concatenate(
            [W.uniform_f32(r, 4000), TU.special_pool()]))
    elif shape == "chain":
        nodes = W.chain_tree(r, size, F, C)
    elif shape == "paper":
        nodes = W.paper_shape_tree(r, 15, size, F, C, spine_p=0.8)
    else:
        nodes = W.complete_tree(r, size, F, C)
    nodes = W.narrow_tree(nodes, x_type) if shape != "random" or x_type == "f32" else nodes
    x = W.uniform_f32(r, (3000, F + pad))
    xn = x if x_type == "f32" else W.narrow_records(x, x_type)
    if x_type in ("f32", "f16"):
        xn[r.integers(0, 3000, 300), r.integers(0, F, 300)] = np.nan
    t = torch.from_numpy(xn)
    if x_type == "bf16":
        t = t.view(torch.int16).view(torch.bfloat16)
    xd = t.cuda()[:, :F]
    rows = np.ascontiguousarray(xn[:, :F])
    rows = rows if x_type == "f32" else TU.widen(rows, x_type)
    leaf, cls = oracle.tree_leaves(nodes, rows, F), oracle.tree_classes(nodes, rows, F)
    tree = dt.Tree(nodes, F, C)
    walks_list = _walks_list(dt, tree, xd)
    if shape == "random" and 3000 < size < 4000:
        assert walks_list
    if shape == "chain" or (shape, size) == ("complete", 12):
        assert not walks_list
    for n in (1, 65, 3000):
        np.testing.assert_array_equal(tree.classify(xd[:n], out_kind="leaf_i32").cpu().numpy(), leaf[:n])
        np.testing.assert_array_equal(tree.classify(xd[:n], out_kind="class_i32").cpu().numpy(), cls[:n])


@pytest.mark.parametrize("x_type", ["f32", "f16", "u8"])
@pytest.mark.parametrize("depth,F", [(12, 200), (13, 64), (13, 16)])
def test_complete_trees_keep_one_window(dt, x_type, depth, F):
    """One level of windows that fits the LDS whole stays, also where the list of the same
    tree is over its share (complete depth 13, 1,000,000 x 64 fp32: 40.0 us against 47.5 us)."""
    r = np.random.Generator(np.random.PCG64(depth))
    tree = dt.Tree(W.narrow_tree(W.complete_tree(r, depth, F, 7), x_type), F, 7)
    x = torch.zeros((64, F), dtype={"f32": torch.float32, "f16": torch.float16,
                                    "u8": torch.uint8}[x_type], device="cuda")
    for out_kind in ("class_u8", "class_i32"):
        assert not _walks_list(dt, tree, x, out_kind)


@pytest.mark.parametrize("size,whole", [(3070, 1), (3071, 1), (3072, 0), (20_000, 0)])
def test_launch_info_of_lists(dt, size, whole):
    """A list of which only the first 48 KiB are staged is not reported as staged."""
    r = np.random.Generator(np.random.PCG64(size))
    tree = dt.Tree(W.random_full_tree(r, size, 16, 7), 16, 7)
    x = torch.zeros((64, 16), device="cuda")
    assert _walks_list(dt, tree, x)
    info = tree.launch_info(x)
    assert info["tables_in_lds"] == whole
    assert info["lds_bytes"] < 160 * 1024
