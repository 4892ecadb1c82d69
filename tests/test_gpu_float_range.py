"""GPU parity of the exact passes at the ends of float32's range, where the
canonical sums lose what the passes' own bounds are relative to: squares in the
subnormal range or below it (rows a few quanta apart, ties at zero), squares and
sums that overflow (every row at infinity: the lowest index is the answer), spans that
overflow themselves.  Bit for bit the oracle's float32 search."""

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


def same(got_min, got_nn, ref):
    torch.cuda.synchronize()
    m32, a32 = ref
    assert np.array_equal(got_nn.cpu().numpy(), a32)
    assert np.array_equal(got_min.cpu().numpy().view(np.uint32), m32.view(np.uint32))


def check(ch, orc, A, B, metric):
    print(f"[case] n_a={A.shape[0]} n_b={B.shape[0]} d={A.shape[1]}", flush=True)
    ref = orc.nn_f32(A, B, metric)
    _, rmin, rnn = ch.chamfer_exact(dev(A), dev(B), metric)
    same(rmin, rnn, ref)
    mn, arg = ch.chamfer_nn_min(dev(A), dev(B), metric)
    same(mn, arg, ref)


def clouds(rng, n_a, n_b, d, scale):
    return ((rng.standard_normal((n_a, d)) * scale).astype(np.float32),
            (rng.standard_normal((n_b, d)) * scale).astype(np.float32))


@pytest.mark.parametrize("d", [3, 9, 16, 64, 128, 256])
@pytest.mark.parametrize("scale", [1e-20, 1e-21, 1e-22, 1e-23, 1e-30])
def test_l2_underflow(ch, orc, d, scale):
    """The accumulator of d squares is off by up to d 2^-150 on top of its
    relative error: at 1e-22 that is a few per cent of a distance, at 1e-23 most
    squares are zero."""
    A, B = clouds(np.random.default_rng(d), 700, 3000, d, scale)
    check(ch, orc, A, B, L2)


@pytest.mark.parametrize("d", [3, 16, 128])
@pytest.mark.parametrize("scale", [1e-21, 1e-22])
def test_l2_underflow_draws(ch, orc, d, scale):
    """The draws' passes start from the crude distances, whose squares are
    rounded in the subnormal range once more."""
    A, B = clouds(np.random.default_rng(d), 900, 2500, d, scale)
    print(f"[case] draws d={d} scale={scale}", flush=True)
    out = ch.chamfer_estimate(dev(A), dev(B), L2, 0.2, 500, 3)
    torch.cuda.synchronize()
    assert int(out["status"].item()) == 0 and int(out["W"].item()) != 0
    idx = out["sample_idx"].cpu().numpy()
    same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, L2, rows=idx))


@pytest.mark.parametrize("d", [3, 9, 16, 64, 128, 256])
@pytest.mark.parametrize("scale", [2e18, 6e18, 3e19, 1e25, 1e37])
def test_l2_overflow(ch, orc, d, scale):
    """Some, then all of a query's distances at infinity."""
    A, B = clouds(np.random.default_rng(d), 500, 3000, d, scale)
    check(ch, orc, A, B, L2)


@pytest.mark.parametrize("d", [3, 16, 64, 128])
def test_l2_span_overflow(ch, orc, d):
    """Two clouds further apart than float32 reaches: no scale holds both, the
    distances within each are ordinary."""
    rng = np.random.default_rng(d)
    A, B = clouds(rng, 600, 2000, d, 1.0)
    A[:, 0] = np.where(rng.random(600) < 0.5, -2.5e38, 2.5e38)
    B[:, 0] = np.where(rng.random(2000) < 0.5, -2.5e38, 2.5e38)
    check(ch, orc, A, B, L2)
    for sampling in (ch.IMPORTANCE, ch.UNIFORM):
        out = ch.chamfer_estimate(dev(A), dev(B), L2, 0.2, 300, 3, sampling=sampling)
        torch.cuda.synchronize()
        assert int(out["status"].item()) == 0 and int(out["W"].item()) != 0
        idx = out["sample_idx"].cpu().numpy()
        same(out["sample_min"], out["sample_nn"], orc.nn_f32(A, B, L2, rows=idx))


@pytest.mark.parametrize("d", [9, 40, 100, 200])
@pytest.mark.parametrize("scale", [3e36, 2e37, 1e38])
def test_l1_overflow(ch, orc, d, scale):
    """Some, then all of a query's sums at infinity; at 1e38 the box's span, too."""
    rng = np.random.default_rng(d)
    A = (rng.uniform(-1, 1, (500, d)) * 3 * scale).astype(np.float32)
    B = (rng.uniform(-1, 1, (3000, d)) * 3 * scale).astype(np.float32)
    check(ch, orc, A, B, L1)
