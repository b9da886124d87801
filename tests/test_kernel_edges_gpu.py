"""The sizes at which a kernel changes its shape: edges of tiles and units,
remainders, and both sides of each rule that picks a variant.  Integers are
compared with the CPU oracle bit for bit, averages within 1e-12 relative."""
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


# 256-row units up to 2^17 rows; 1024-row units above, of 1..16 steps per wave
@pytest.mark.parametrize("n", [255, 257, 131_072, 131_073, 1_048_575, 2 * 1024 * 512 + 1, 17 * 1024 * 512 + 777])
@pytest.mark.parametrize("lf", [0.5, 0.9])
def test_ordered_probe_units(ctx, n, lf):
    r = np.random.default_rng(n)
    m = 57_000
    bkey = r.integers(-(1 << 62), 1 << 62, size=m)
    bpay = r.integers(-(1 << 31), 1 << 31, size=m).astype(np.int32)
    fk = np.where(r.random(n) < 0.7, bkey[r.integers(0, m, size=n)], r.integers(-(1 << 62), 1 << 62, size=n))
    fk[r.random(n) < 0.01] = np.iinfo(np.int64).min            # the empty-slot marker matches nothing
    sel = np.flatnonzero(r.random(n) < 0.6).astype(np.int32)
    table = gq.gq_join_build(ctx, dev(bkey), dev(bpay), load_factor=lf)
    fk_d, sel_d = dev(fk), dev(sel)
    half = torch.tensor([len(sel) // 2], dtype=torch.int64, device="cuda")
    for s, n_dev, used in ((None, None, None), (sel_d, None, sel), (sel_d, half, sel[:len(sel) // 2])):
        ep, ey = oracle.join(bkey, bpay, fk, used)
        prow, pay, cnt = gq.gq_join_probe(ctx, table, fk_d, sel=s, n_dev=n_dev)
        assert ctx.status() == gq.GQ_OK
        k = int(cnt.item())
        assert k == len(ep)
        assert np.array_equal(prow[:k].cpu().numpy(), ep) and np.array_equal(pay[:k].cpu().numpy(), ey)
