"""GPU parity of the exact passes on both sides of the lines between their forms:
bit for bit the oracle's float32 search, whichever form a size takes."""

import numpy as np
import pytest

import workloads

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


def same(got_min, got_nn, ref):
    torch.cuda.synchronize()
    m32, a32 = ref
    assert np.array_equal(got_nn.cpu().numpy(), a32)
    assert np.array_equal(got_min.cpu().numpy().view(np.uint32), m32.view(np.uint32))


def check(ch, orc, n_a, n_b, d, metric, rows):
    """All rows of A against a sample of the oracle's: the product is large."""
    A, B = workloads.clusters_l2(seed=n_a + n_b + d, n=n_a, d=d, k=20, n_b=n_b)
    print(f"[case] metric={metric} n_a={n_a} n_b={n_b} d={d}", flush=True)
    idx = np.unique(np.random.default_rng(d).integers(0, n_a, rows)).astype(np.int32)
    ref = orc.nn_f32(A, B, metric, rows=idx)
    _, rmin, rnn = ch.chamfer_exact(dev(A), dev(B), metric)
    pick = torch.from_numpy(idx.astype(np.int64)).to("cuda:0")
    same(rmin[pick], rnn[pick], ref)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), metric, rows=torch.from_numpy(idx).to("cuda:0"))
    same(mn, arg, ref)


# the table of B in one pass of 256 units a workgroup and in four (2^18 units of eight
# coordinates), and a small launch's first scan with B of one tile and a little more
@pytest.mark.parametrize("d,n_b", [(20, 65536), (20, 65537), (64, 32768), (64, 32769),
                                   (200, 8192), (200, 8193)])
def test_row_tables(ch, orc, d, n_b):
    check(ch, orc, 70, n_b, d, L2, 70)


@pytest.mark.parametrize("d", [12, 32, 33, 64])
@pytest.mark.parametrize("n_a,n_b", [(300, 127), (300, 129), (2000, 5000)])
def test_first_scan(ch, orc, d, n_a, n_b):
    check(ch, orc, n_a, n_b, d, L2, 300)


# three dimensions, l2: the vector form up to 12288 rows, and on small products
@pytest.mark.parametrize("n_a,n_b", [(73300, 12288), (73300, 12289), (73200, 12289),
                                     (30000, 30000), (30001, 30000), (27000, 32768),
                                     (13000, 32769), (12000, 32769), (4000, 100000),
                                     (4001, 100000), (50, 100001), (50, 100000)])
def test_points(ch, orc, n_a, n_b):
    check(ch, orc, n_a, n_b, 3, L2, 200)


@pytest.mark.parametrize("n_b", [500, 40000])
def test_points_uniform_draws(ch, orc, n_b):
    A, B = workloads.clusters_l2(seed=n_b, n=3000, d=3, k=20, n_b=n_b)
    out = ch.chamfer_estimate(dev(A), dev(B), L2, 0.2, 300, 3, sampling=ch.UNIFORM)
    torch.cuda.synchronize()
    idx = out["sample_idx"].cpu().numpy()
    same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, L2, rows=idx))


# l1 at the dimensions that the vector form is compiled for: bytes from a product on
@pytest.mark.parametrize("d,n_a,n_b", [
    (16, 30600, 16383), (16, 30600, 16384), (16, 30500, 16384),
    (32, 2500, 99999), (32, 2500, 100000),
    (64, 14700, 2047), (64, 14700, 2048), (64, 300, 99999), (64, 300, 100000),
    (128, 160, 99999), (128, 160, 100000)])
def test_l1(ch, orc, d, n_a, n_b):
    check(ch, orc, n_a, n_b, d, L1, 100)


@pytest.mark.parametrize("metric,d", [(L2, 3), (L2, 10), (L2, 20), (L2, 128), (L1, 20), (L1, 64),
                                      (L1, 100)])
@pytest.mark.parametrize("n_a,n_b", [(1, 20000), (256, 19969), (257, 40001), (512, 39936),
                                     (513, 20000), (1024, 20001), (1025, 20001), (2048, 50001)])
def test_few_queries(ch, orc, metric, d, n_a, n_b):
    check(ch, orc, n_a, n_b, d, metric, 40)


@pytest.mark.parametrize("d,n_b", [(3, 1), (3, 20000), (64, 1), (64, 20000)])
@pytest.mark.parametrize("n_a", [63, 1024])
def test_smallest_workspace(ch, orc, d, n_b, n_a):
    """A workspace sized for any entry point with the same options is enough for the
    exact ones, whatever they lay out with a larger one."""
    A, B = workloads.clusters_l2(seed=n_a + d, n=n_a, d=d, k=20, n_b=max(n_b, 20))
    A, B = dev(A), dev(B[:n_b])
    print(f"[case] n_a={n_a} n_b={n_b} d={d}", flush=True)
    ref = orc.nn_f32(A.cpu().numpy(), B.cpu().numpy(), L2)
    size = ch.chamfer_workspace_bytes(n_a, n_b, d, L2, 0.1, 1, sampling=ch.UNIFORM)
    assert size < ch.chamfer_workspace_bytes(n_a, n_b, d, L2, 0.0, 0)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    out = torch.empty(3, dtype=torch.float64, device="cuda:0")
    mn = torch.empty(n_a, dtype=torch.float32, device="cuda:0")
    nn = torch.empty(n_a, dtype=torch.int32, device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    lib = ch.lib()
    rc = lib.chamfer_exact(A.data_ptr(), B.data_ptr(), n_a, n_b, d, L2, out.data_ptr(),
                           mn.data_ptr(), nn.data_ptr(), None, ws.data_ptr(), size, st)
    assert rc == 0
    same(mn, nn, ref)
    rc = lib.chamfer_nn_min(A.data_ptr(), None, n_a, B.data_ptr(), n_b, d, L2, mn.data_ptr(),
                            nn.data_ptr(), None, ws.data_ptr(), size, st)
    assert rc == 0
    same(mn, nn, ref)


@pytest.mark.parametrize("metric,d,n_b", [(L2, 20, 1024), (L2, 32, 1025), (L2, 8, 1024),
                                          (L1, 20, 500), (L1, 12, 500)])
def test_few_rows(ch, orc, metric, d, n_b):
    check(ch, orc, 150001, n_b, d, metric, 100)


@pytest.mark.parametrize("d,n_b,T", [(16, 65535, 3200), (16, 65536, 3200), (32, 69000, 1023),
                                     (32, 69000, 1024), (64, 2000, 15001), (64, 2000, 14999)])
def test_l1_draws(ch, orc, d, n_b, T):
    A, B = workloads.clusters_l2(seed=n_b, n=3000, d=d, k=20, n_b=n_b)
    print(f"[case] draws n_b={n_b} d={d} T={T}", flush=True)
    out = ch.chamfer_estimate(dev(A), dev(B), L1, 0.2, T, 3)
    torch.cuda.synchronize()
    idx = out["sample_idx"].cpu().numpy()[:100]
    same(out["sample_min"][:100], out["sample_nn"][:100], orc.nn_f32(A, B, L1, rows=idx))


# batches: vector form and the other by each batch's draws and sizes
@pytest.mark.parametrize("metric,d", [(L2, 3), (L1, 16), (L1, 32), (L1, 64), (L1, 128), (L1, 20),
                                      (L2, 20), (L2, 128), (L2, 7)])
@pytest.mark.parametrize("T", [40, 310, 1100])
@pytest.mark.parametrize("sizes", [(900, 1500, 33), (700, 9000, 60000, 100)])
def test_batches(ch, metric, d, T, sizes):
    """Every symmetric estimate of a retrieval is that of its own call, bit for bit,
    far points among them."""
    rng = np.random.default_rng(d + T)
    A = rng.standard_normal((800, d)).astype(np.float32)
    clouds = [rng.standard_normal((n, d)).astype(np.float32) for n in sizes]
    clouds[-1][5] *= 1e9
    print(f"[case] metric={metric} d={d} T={T} sizes={sizes}", flush=True)
    Bs = [dev(c) for c in clouds]
    est, top, vals = ch.chamfer_retrieve(dev(A), Bs, metric, 0.2, T, 3, 1, n_scales=12)
    ref = [ch.chamfer_estimate_symmetric(dev(A), B, metric, 0.2, T, 3, n_scales=12)[0].item()
           for B in Bs]
    torch.cuda.synchronize()
    assert est.cpu().tolist() == ref
    exact = [ch.chamfer_exact_symmetric(dev(A), B, metric)[0].item() for B in Bs]
    assert vals[0] == exact[top[0]] and top[0] == int(np.argmin(ref))
