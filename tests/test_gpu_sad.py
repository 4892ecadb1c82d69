"""GPU parity of the l1 exact pass on byte differences where it can go wrong:
rows are ruled out by rounded sums, so every result is compared bit for bit with
the oracle's float32 search (canonical minimum, lower index on ties).  Every
row width with ragged d, tile, chunk and query-block remainders, queues that
fill (duplicates, one point repeated, integers), rows of B far outside the
sampled box (clamped), queries far outside B's, equal rows (no step at all)."""

import numpy as np
import pytest

import workloads

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


def same(got_min, got_nn, ref):
    torch.cuda.synchronize()
    m32, a32 = ref
    assert np.array_equal(got_nn.cpu().numpy(), a32)
    assert np.array_equal(got_min.cpu().numpy().view(np.uint32), m32.view(np.uint32))


def check(ch, orc, A, B):
    A, B = np.asarray(A, np.float32), np.asarray(B, np.float32)
    print(f"[case] n_a={A.shape[0]} n_b={B.shape[0]} d={A.shape[1]}", flush=True)
    ref = orc.nn_f32(A, B, L1)
    _, rmin, rnn = ch.chamfer_exact(dev(A), dev(B), L1)
    same(rmin, rnn, ref)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), L1)
    same(mn, arg, ref)


# both sides of every row width (16, 32, 64, 112, 128, 256) and of the dispatch (8)
@pytest.mark.parametrize("d", [8, 9, 16, 17, 32, 33, 50, 64, 65, 100, 112, 113, 128, 129, 200,
                               256, 257])
def test_dimensions(ch, orc, d):
    A, B = workloads.clusters_l2(seed=d, n=700, d=d, k=9, n_b=1501)
    check(ch, orc, A, B)


# the dimensions that keep the vector-ALU form for small products, on both sides
# of 2e9 coordinates
@pytest.mark.parametrize("d,n_a,n_b", [(16, 11000, 11400), (16, 11000, 11300), (32, 8000, 8001),
                                       (64, 5000, 6301), (128, 4001, 4000)])
def test_large_products(ch, orc, d, n_a, n_b):
    A, B = workloads.clusters_l2(seed=d, n=n_a, d=d, k=50, n_b=n_b)
    check(ch, orc, A, B)


# n_a: 64 lanes, 128 and 256 queries per wavefront, one to four of them per
# workgroup, 512 where four queries per lane begin; n_b: groups of 4, tiles, chunks
@pytest.mark.parametrize("n_a,n_b", [(1, 1), (63, 3), (128, 5), (129, 36), (257, 37), (512, 256),
                                     (513, 255), (1025, 1030), (300, 4097), (5000, 66)])
@pytest.mark.parametrize("d", [12, 40, 60, 100, 120])
def test_remainders(ch, orc, n_a, n_b, d):
    A, B = workloads.clusters_l2(seed=n_a + n_b + d, n=n_a, d=d, k=7, n_b=n_b)
    check(ch, orc, A, B)


@pytest.mark.parametrize("d", [10, 60, 100])
@pytest.mark.parametrize("kind", ["copies", "one", "integers", "offset", "far rows",
                                  "far queries", "equal"])
def test_hard(ch, orc, d, kind):
    rng = np.random.default_rng(3 * d)
    A = rng.standard_normal((600, d))
    B = rng.standard_normal((3000, d))
    if kind == "copies":         # every row 300 times
        B = B[rng.integers(0, 10, 3000)]
    elif kind == "one":          # all rows the same but one
        B[:] = B[0]
        B[1234] = A[5]
    elif kind == "integers":     # ties everywhere
        A, B = np.round(A), np.round(B)
    elif kind == "offset":       # the float32 grid itself is coarse
        A, B = A + 1e4, B + 1e4
    elif kind == "far rows":     # outside the sampled box, one the nearest of a query
        B[7] *= 1e4
        B[2500] += 300.0
        A[11] = B[2500] + 0.1
    elif kind == "far queries":
        A[17] += 5e5
        A[333] *= 1e30
    else:
        B[:] = B[0]
    check(ch, orc, A, B)


@pytest.mark.parametrize("d,n_b", [(30, 30011), (64, 50011), (100, 9001)])
def test_draws(ch, orc, d, n_b):
    A, B = workloads.clusters_l2(seed=d, n=5001, d=d, k=40, n_b=n_b)
    out = ch.chamfer_estimate(dev(A), dev(B), L1, 0.2, 700, 3)
    torch.cuda.synchronize()
    idx = out["sample_idx"].cpu().numpy()
    same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, L1, rows=idx))
