"""Exact passes over so many (query, row) pairs that one launch of all their
workgroups would exceed the 2^32 threads that a launch may have.  A coordinate that
is not finite ends every workgroup before its work, so the call costs its launches
only; the calls are accepted and say NaN."""

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


# (l2: 256 queries by 65536 rows a workgroup at first, l1: 512 by 65536)
@pytest.mark.parametrize("metric,d,n_a,n_b", [(L2, 1, 20_000_000, 20_000_000),
                                              (L1, 9, 30_000_000, 30_000_000),
                                              (L2, 12, 30_000_000, 15_000_000)])
def test_pairs_beyond_one_launch(ch, metric, d, n_a, n_b):
    A = torch.zeros((n_a, d), device="cuda:0")
    B = torch.zeros((n_b, d), device="cuda:0")
    A[n_a // 2, 0] = float("nan")
    print(f"[case] metric={metric} d={d} n_a={n_a} n_b={n_b}", flush=True)
    total, rmin, rnn = ch.chamfer_exact(A, B, metric)
    torch.cuda.synchronize()
    assert torch.isnan(total).all() and torch.isnan(rmin).all() and (rnn == -1).all()
