"""The table build keeps every key within its region of slots, going round at the
region's end; keys of a region with more distinct keys than slots are left out and
found by a search of the keys.  Points are chosen by their hash (the bounding box
is held by points of A, so a point hashes alike in every subset): all of B in one
region of its finest table, which then has no empty slot, and all of B with home
slots in the last few of their region.  The CrudeNN bits are compared with the
oracle's."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

L1 = 1
GOLDEN = np.uint64(0x9E3779B97F4A7C15)


@pytest.fixture(scope="module")
def ch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2307_03043_amd as lib
    lib.lib()
    return lib


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda:0")


def homes(keys, log2cap):
    with np.errstate(over="ignore"):
        return (np.asarray(keys).astype(np.uint64) * GOLDEN) >> np.uint64(64 - log2cap)


# n_b, log2 of the table's slots and of a region's: the direct build's largest
# regions (2^13) and the partitioned build's (2^11)
@pytest.mark.parametrize("n_b,log2cap,region_bits", [(16384, 15, 13), (32768, 16, 11)])
@pytest.mark.parametrize("kind", ["one region", "last slots"])
def test_region(ch, orc, n_b, log2cap, region_bits, kind):
    rng = np.random.default_rng(n_b)
    L, seed, eps = 14, 5, 0.25
    box = np.array([[0, 0, 0], [1, 1, 1]], np.float32)
    A = np.concatenate([box, rng.uniform(0, 1, (400, 3)).astype(np.float32)])
    chosen = []
    have = 0
    while have < n_b:
        cand = rng.uniform(0, 1, (400_000, 3)).astype(np.float32)
        kb = ch.chamfer_hash_keys(dev(A), dev(cand), L1, eps, seed, n_scales=L)[1].cpu().numpy()
        h = homes(kb[0], log2cap)
        if kind == "one region":
            pick = (h >> np.uint64(region_bits)) == 1
        else:
            size = np.uint64(1 << region_bits)
            pick = (h & (size - np.uint64(1))) >= size - np.uint64(size // np.uint64(8))
        chosen.append(cand[pick])
        have += int(pick.sum())
    B = np.concatenate(chosen)[:n_b]
    A[2:202] = B[rng.integers(0, n_b, 200)]  # queries that meet at the finest scale
    c = orc.crude_nn(A, B, L1, eps, seed, n_scales=L)
    h = homes(c["keys_b"][0], log2cap)
    if kind == "one region":  # more distinct keys than slots
        assert len(np.unique(c["keys_b"][0])) > 1 << region_bits
        assert len(np.unique(h >> np.uint64(region_bits))) == 1
    print(f"[case] n_b={n_b} {kind}", flush=True)
    D, nn, scale = ch.crude_nn(dev(A), dev(B), L1, eps, seed, n_scales=L)
    torch.cuda.synchronize()
    assert np.array_equal(scale.cpu().numpy(), c["scale"])
    assert np.array_equal(nn.cpu().numpy(), c["nn"])
    assert np.array_equal(D.cpu().numpy().view(np.uint32), c["D"].view(np.uint32))
