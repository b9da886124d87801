"""What the operators promise beyond the plain call: selections that name a row
more than once, outputs that are also inputs, and empty inputs.  Everything is
whole numbers, compared with the CPU oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2506_09226_amd as gq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = gq.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def guarded(k, dtype, mark):
    """An output of k entries between two borders of 4096 entries that no call may touch."""
    t = torch.full((k + 8192,), mark, dtype=dtype, device="cuda")
    return t, t[4096:4096 + k]


# a selection with repeats: inside the answer, across the k-th place and over
# the whole buffer (4096 candidates); answers ranked (k <= 256) and sorted; one
# list, one merge and two merge levels
@pytest.mark.parametrize("n", [6, 5000, 70_001, 2_000_003])
@pytest.mark.parametrize("k", [1, 10, 256, 257, 1000, 2048])
@pytest.mark.parametrize("rows", ["one", "few", "pairs", "any"])
def test_topk_of_repeated_rows(ctx, n, k, rows):
    r = np.random.default_rng(n + k)
    sel = {"one": lambda: np.full(n, 3), "few": lambda: r.integers(0, 7, size=n),
           "pairs": lambda: r.permutation(np.arange(n) // 2), "any": lambda: r.integers(0, n, size=n)}[rows]()
    sel = sel.astype(np.int32)
    val = r.integers(0, 1000 if rows == "any" else 1 << 40, size=max(n, 8)).astype(np.int64)
    for desc in (True, False):
        vall, v = guarded(k, torch.int64, -77)
        rall, row = guarded(k, torch.int32, -77)
        ev, er = oracle.topk(val, k, sel=sel, descending=desc)
        _, _, cnt = gq.gq_topk(ctx, dev(val), k, sel=dev(sel), descending=desc, val_out=v, rowid_out=row)
        c = int(cnt.item())
        assert c == len(ev) == min(n, k)
        assert np.array_equal(v[:c].cpu().numpy(), ev) and np.array_equal(row[:c].cpu().numpy(), er)
        for t in (vall, rall):
            assert bool((t[:4096] == -77).all()) and bool((t[4096 + c:] == -77).all())
