"""A workspace sized for n rows serves every call with fewer rows (drivers
allocate once for the largest call), so these size queries are non-decreasing
in the row count."""
import random

import pytest

import paper_2506_09226_amd as gq


def sizes():
    r = random.Random(7)
    edges = [256, 4096, 8192, 32768, 1 << 17, 1 << 19, 1 << 20, 1 << 21, 1024 * 512 * 16, 8192 * 512, 1 << 25]
    out = {0, 1, 2}
    for e in edges:
        out.update((e - 1, e, e + 1, 2 * e + 1))
    out.update(int(10 ** r.uniform(0, 9)) for _ in range(400))
    return sorted(out)


@pytest.mark.parametrize("what", ["filter", "probe", "probe_partitioned", "partition", "topk", "groupby"])
def test_workspace_grows_with_rows(what):
    L = gq.lib()
    for arg in {"partition": (0, 4, 6, 8), "topk": (1, 100, 2048),
                "groupby": ((1, 0, 0), (25, 0, 1), (64, 1, 0), (512, 0, 1), (512, 1, 1), (513, 0, 1),
                            (100_000, 0, 1), (300_000, 1, 1), (1_500_000, 0, 1), (4_000_000, 1, 1))}.get(what, (None,)):
        last = 0
        for n in sizes():
            b = {"filter": lambda: L.gq_filter_workspace_bytes(n), "probe": lambda: L.gq_join_probe_workspace_bytes(n),
                 "probe_partitioned": lambda: L.gq_join_probe_partitioned_workspace_bytes(n),
                 "partition": lambda: L.gq_radix_partition_workspace_bytes(n, arg),
                 "topk": lambda: L.gq_topk_workspace_bytes(n, arg),
                 "groupby": lambda: L.gq_groupby_workspace_bytes(n, arg[0], arg[1], arg[2])}[what]()
            assert b >= last, (what, arg, n)
            last = b


def test_topk_workspace_grows_with_k():
    """One made for k keys serves smaller answers over the same rows."""
    L = gq.lib()
    for n in sizes():
        last = 0
        for k in [1, 2, 16, 64, 100, 128, 200, 255, 256, 257, 258, 300, 511, 512, 513, 1000, 1024, 1025, 2047, 2048]:
            b = L.gq_topk_workspace_bytes(n, k)
            assert b >= last, (n, k)
            last = b


@pytest.mark.parametrize("k64,k32", [(1, 0), (0, 1), (1, 1)])
def test_groupby_workspace_grows_with_groups(k64, k32):
    """One made for a bound of max_groups serves lower bounds over the same rows."""
    L = gq.lib()
    for n in sizes():
        last = 0
        for g in [1, 2, 25, 32, 63, 64, 65, 100, 127, 128, 129, 256, 257, 511, 512, 513, 1000, 100_000, 1_500_000]:
            b = L.gq_groupby_workspace_bytes(n, g, k64, k32)
            assert b >= last, (n, g)
            last = b
