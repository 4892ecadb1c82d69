"""GPU parity of the l1 exact pass in three dimensions on both sides of its queries
per lane (one, two, eight), of the wavefronts that share a chunk's rows (one to four
groups of queries) and of its passes of eight rows: bit for bit the oracle's float32
search, ties to the lower index."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L1 = 1


@pytest.fixture(scope="module")
def ch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03043_amd as lib
    lib.lib()
    return lib


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0")


@pytest.mark.parametrize("n_a", [1, 64, 65, 128, 129, 256, 300, 511, 1024, 1025, 4096, 4097])
@pytest.mark.parametrize("n_b", [1, 7, 8, 257, 2051, 16384, 16385])
def test_points(ch, orc, n_a, n_b):
    rng = np.random.default_rng(n_a + n_b)
    A = rng.uniform(-1, 1, (n_a, 3)).astype(np.float32)
    B = np.round(rng.uniform(-1, 1, (n_b, 3)), 2).astype(np.float32)  # repeated rows
    A[::2] = np.round(A[::2], 2)
    print(f"[case] n_a={n_a} n_b={n_b}", flush=True)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), L1)
    torch.cuda.synchronize()
    m32, a32 = orc.nn_f32(A, B, L1)
    assert np.array_equal(arg.cpu().numpy(), a32)
    assert np.array_equal(mn.cpu().numpy().view(np.uint32), m32.view(np.uint32))
