"""A row of B that is not finite does not answer any query: chamfer_nn_min, which does
not check its inputs, returns what the oracle's float32 search finds among the others,
at sizes that take the matrix-core and the byte-difference passes."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L1, L2 = 1, 2


@pytest.fixture(scope="module")
def ch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03043_amd as lib
    lib.lib()
    return lib


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0")


@pytest.mark.parametrize("metric,d", [(L2, 5), (L2, 10), (L2, 20), (L2, 64), (L2, 200), (L1, 20),
                                      (L1, 100), (L1, 200)])
@pytest.mark.parametrize("row", [1, 1300, 9998])  # sampled rows are those of a sixteenth's start
@pytest.mark.parametrize("value", [np.float32("nan"), -np.float32("nan"), np.inf, -np.inf])
def test_one_row(ch, orc, metric, d, row, value):
    print(f"[case] metric={metric} d={d} row={row} value={value}", flush=True)
    rng = np.random.default_rng(d + row)
    A = rng.standard_normal((800, d)).astype(np.float32)
    B = rng.standard_normal((9999, d)).astype(np.float32)
    B[row, d // 2] = value
    keep = np.delete(np.arange(9999), row)
    m32, a32 = orc.nn_f32(A, B[keep], metric)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), metric)
    torch.cuda.synchronize()
    assert np.array_equal(arg.cpu().numpy(), keep[a32].astype(np.int32))
    assert np.array_equal(mn.cpu().numpy().view(np.uint32), m32.view(np.uint32))
