"""GPU parity on rows of every staging class: dense rows that are no multiple of 16 bytes,
strided rows and bases between words or vectors, rows wide enough for tiles of 32 and 16
records, and record counts around the tile edges.  Integer outputs: exact."""
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
