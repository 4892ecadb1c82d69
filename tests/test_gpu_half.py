"""GPU parity of the l2 exact pass on the FP16 matrix cores where it can go
wrong: the rows it rules out come from a rounded score, so every result is
compared bit for bit with the oracle's float32 search (canonical minimum,
lower index on ties).  The three-product form (d <= 10) at every dimension and
on tile, chunk and query-block remainders; crowded tiles (more rows within the
bound than the queue holds: duplicates, a large offset, one point repeated);
queries outside FP16's range of the scale chosen for B; tables of 12 <= d <= 256
over several chunks and query blocks; draws seeded with crude distances."""

import numpy as np
import pytest

import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L2 = 2


@pytest.fixture(scope="module")
def ch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03043_amd as lib
    lib.lib()
    return lib


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0")


def same(got_min, got_nn, ref):
    torch.cuda.synchronize()
    m32, a32 = ref
    assert np.array_equal(got_nn.cpu().numpy(), a32)
    assert np.array_equal(got_min.cpu().numpy().view(np.uint32), m32.view(np.uint32))


def check(ch, orc, A, B):
    print(f"[case] n_a={A.shape[0]} n_b={B.shape[0]} d={A.shape[1]}", flush=True)
    ref = orc.nn_f32(A, B, L2)
    _, rmin, rnn = ch.chamfer_exact(dev(A), dev(B), L2)
    same(rmin, rnn, ref)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), L2)
    same(mn, arg, ref)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 9, 10, 11])
def test_low_dimensions(ch, orc, d):
    rng = np.random.default_rng(d)
    A = rng.uniform(-1, 1, (777, d))
    B = np.round(rng.uniform(-1, 1, (1533, d)), 3)  # ties in d = 1, 2
    check(ch, orc, A.astype(np.float32), B.astype(np.float32))


# n_a: query blocks of 32, wavefronts of 128, workgroups of 256; n_b: row blocks
# of 32, tiles of 64 to 256, chunks
@pytest.mark.parametrize("n_a,n_b", [(1, 1), (31, 33), (32, 32), (129, 63), (256, 255),
                                     (257, 256), (100, 257), (300, 4097), (16500, 513)])
@pytest.mark.parametrize("d", [3, 7, 20, 64, 128, 256])
def test_remainders(ch, orc, n_a, n_b, d):
    A, B = workloads.clusters_l2(seed=n_a + n_b + d, n=n_a, d=d, k=7, n_b=n_b)
    check(ch, orc, A, B)


@pytest.mark.parametrize("d", [3, 16, 100, 200])
@pytest.mark.parametrize("kind", ["copies", "one", "offset", "tiny"])
def test_crowded(ch, orc, d, kind):
    rng = np.random.default_rng(7 * d)
    A = rng.standard_normal((400, d))
    B = rng.standard_normal((3000, d))
    if kind == "copies":    # every row 300 times
        B = B[rng.integers(0, 10, 3000)]
    elif kind == "one":     # all rows the same but one
        B[:] = B[0]
        B[1234] = A[5]
    elif kind == "offset":  # far from the origin: the float32 grid itself is coarse
        A, B = A + 1e4, B + 1e4
    else:                   # a dense ball in a wide cloud
        B[:2900] = 1e-4 * B[:2900]
        A[:300] = 1e-4 * A[:300]
        B[2900:] *= 100
    check(ch, orc, A.astype(np.float32), B.astype(np.float32))


@pytest.mark.parametrize("d", [3, 64])
def test_far_queries(ch, orc, d):
    """nn_min scales by B alone: queries 2^20 times B's extent leave FP16's
    range and have every row evaluated; overflowing squares come back as inf."""
    rng = np.random.default_rng(d)
    A = rng.standard_normal((200, d)).astype(np.float32)
    B = rng.standard_normal((700, d)).astype(np.float32)
    A[17] *= 1e6
    A[140] *= 1e25
    check(ch, orc, A, B)


@pytest.mark.parametrize("d,n_b", [(3, 30011), (24, 20011), (128, 9001)])
def test_draws(ch, orc, d, n_b):
    rng = np.random.default_rng(n_b)
    if d == 3:
        A, B = workloads.surface_pair(rng, 5001, n_b)
    else:
        A, B = workloads.clusters_l2(seed=d, n=5001, d=d, k=40, n_b=n_b)
    out = ch.chamfer_estimate(dev(A), dev(B), L2, 0.2, 700, 3)
    torch.cuda.synchronize()
    idx = out["sample_idx"].cpu().numpy()
    same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, L2, rows=idx))


@pytest.mark.parametrize("metric", [1, 2])
@pytest.mark.parametrize("d", [3, 24])
@pytest.mark.parametrize("n_b,T,uniform", [(20, 20000, False), (2000, 300, True), (20, 9000, True)])
def test_draws_without_shared_thresholds(ch, orc, metric, d, n_b, T, uniform):
    """Estimates whose workspace has no room for the thresholds."""
    A, B = workloads.clusters_l2(seed=d, n=600, d=d, k=10, n_b=n_b)
    out = ch.chamfer_estimate(dev(A), dev(B), metric, 0.2, T, 3,
                              sampling=ch.UNIFORM if uniform else ch.IMPORTANCE)
    torch.cuda.synchronize()
    idx = out["sample_idx"].cpu().numpy()
    same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, metric, rows=idx))
